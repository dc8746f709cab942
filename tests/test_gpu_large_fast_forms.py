"""The FP32 and mixed modes beyond 320 PQ buses (one kernel sequence per sweep): ZIP shares
with and without constant impedance, and two solves at once on two streams; and single
columns of the persistent kernels against the same column inside a larger call."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu

MODES = ["fp32", "mixed_bf16", "mixed_fp16"]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n,with_z", [(321, False), (321, True), (399, False), (399, True)])
def test_zip_shares(gpu, n, with_z, mode):
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    onet = oracle.build_feeder(f)
    az, ai, ap = W.zipz_shares(n)
    S = W.profile_minute_year(f, steps=30, seed=9)
    if with_z:
        net = tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=ap, alpha_z=az)
        ref = oracle.fpi_zip(onet, S, ai, ap, 1e-12, 200, alpha_z=az)
    else:
        net = tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=1.0 - ai)
        ref = oracle.fpi_zip(onet, S, ai, 1.0 - ai, 1e-12, 200)
    V, it, st = tpf.solve_timeseries(net, torch.from_numpy(S).to(gpu), 1e-6, 100, mode=mode)
    assert int(st.max()) == tpf.ST_CONVERGED
    assert np.abs(V.cpu().numpy() - ref.V).max() <= 1e-6  # the fast forms' contract


@pytest.mark.parametrize("mode", MODES)
def test_two_streams(gpu, mode):
    """The queued sweeps of each solve read their own active counts, and the early-stop word
    carries each solve's own number: both equal the same solve run alone, bit for bit."""
    f = W.make_feeder(400)
    net = tpf.Network.from_feeder(f)
    loads = [torch.from_numpy(W.profile_minute_year(f, steps=s, t0=t)).to(gpu) for s, t in ((700, 10), (1_100, 90_000))]
    want = [tpf.solve_timeseries(net, S, 1e-6, 100, mode=mode) for S in loads]
    outs = [tpf.alloc_outputs(net, S, mode) for S in loads]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(3):
        got = []
        for S, out, stream in zip(loads, outs, streams):
            with torch.cuda.stream(stream):
                got.append(tpf.solve_timeseries(net, S, 1e-6, 100, mode=mode, out=out))
        torch.cuda.synchronize()
        for a, b in zip(want, got):
            assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("mode,n", [(m, 150) for m in MODES] + [(m, k) for m in ("tree_fp64", "tree_fp32")
                                                               for k in (20, 99, 180, 399)])
def test_one_column_alone(gpu, mode, n):
    f = W.make_feeder(n + 1, load_scale=100.0 / max(n, 100))
    net = tpf.Network.from_feeder(f)
    S = torch.from_numpy(W.profile_minute_year(f, steps=9_000, seed=4)).to(gpu)
    V, it, st = tpf.solve_timeseries(net, S, 1e-6, 100, mode=mode)
    for c in (0, 17, 4_500, 8_999):
        one = tpf.solve_timeseries(net, S[c:c + 1].contiguous(), 1e-6, 100, mode=mode)
        assert torch.equal(one[0][0], V[c]) and one[1][0] == it[c] and one[2][0] == st[c]
        assert float((V[c] - 1.0).abs().max()) > 1e-3  # a loaded column
