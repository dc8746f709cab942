"""The row shapes of the tree operator that only calls with many columns take (few columns run
one per wavefront above 128 buses), against the CPU oracle, and against the same columns in a
small call, bit for bit.  Bounds as for the other shapes: FP64 after three sweeps 1e-12 pu, FP32
1e-6 pu.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "c64", "start", "zip"])
@pytest.mark.parametrize("mode,n", [("tree_fp64", k) for k in (132, 155, 156, 180, 203, 204, 231, 260, 299, 315)]
                         + [("tree_fp32", k) for k in (257, 299, 315, 316, 360, 400, 411)])
def test_shapes_of_large_calls(gpu, n, mode, kind):
    T = 8 * torch.cuda.get_device_properties(gpu).multi_processor_count + 61
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    onet = oracle.build_feeder(f)
    S = W.profile_minute_year(f, steps=T, seed=n)
    Sd = torch.from_numpy(S).to(gpu).to(torch.complex64 if kind == "c64" else torch.complex128).contiguous()
    S = Sd.cpu().numpy().astype(np.complex128)
    V0, R0 = None, None
    if kind == "start":
        R0 = np.ones_like(S) * 0.97
        R0[5, n - 1] = 0.4  # refused: this column starts flat
        V0 = torch.from_numpy(R0).to(gpu)
        R0[5] = 1.0
    ai, ap = W.zip_shares(n) if kind == "zip" else (None, None)
    net = tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=ap)
    tol, cap = (0.0, 3) if mode == "tree_fp64" else (1e-6, 100)
    V, it, st = tpf.solve_timeseries(net, Sd, tol, cap, mode=mode, V0=V0)
    pick = np.r_[0:12, T // 2, T - 12:T]
    rtol, rcap = (0.0, 3) if mode == "tree_fp64" else (1e-10, 200)
    if kind == "zip":
        ref = oracle.fpi_zip(onet, S[pick], ai, ap, rtol, rcap)
    else:
        ref = oracle.fpi(onet, S[pick], rtol, rcap, None if R0 is None else R0[pick])
    assert int(st.max()) == (tpf.ST_MAX_ITER if mode == "tree_fp64" else tpf.ST_CONVERGED)
    bound = (1e-12 if mode == "tree_fp64" else 1e-6) + (2.0 ** -24 * 1.5 if kind == "c64" else 0.0)
    assert np.abs(V.cpu().numpy()[pick] - ref.V).max() <= bound
    few = tpf.solve_timeseries(net, Sd[:33].contiguous(), tol, cap, mode=mode, V0=None if V0 is None else V0[:33].contiguous())
    for x, y in zip((V, it, st), few):
        assert torch.equal(x[:33], y)
