"""The persistent FP32 and mixed kernel for 129 to 320 PQ buses at the edges of its tiling and
batches, against the CPU oracle (1e-6 pu, the fast forms' contract) and against itself: a
column's result must not depend on the batch it is solved in, bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu

MODES = ["fp32", "mixed_bf16", "mixed_fp16"]


def _feeder(n):
    return W.make_feeder(n + 1, load_scale=100.0 / n)


def _solve(net, S, mode, **kw):
    V, it, st = tpf.solve_timeseries(net, S, 1e-6, 100, mode=mode, **kw)
    return V.cpu().numpy(), it.cpu().numpy(), st.cpu().numpy()


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n", [129, 136, 137, 160, 192, 193, 255, 257, 300, 313, 319, 320])
def test_every_tile_remainder(gpu, n, mode):
    f = _feeder(n)
    S = W.profile_minute_year(f, steps=37, seed=n)
    ref = oracle.fpi(oracle.build_feeder(f), S, 1e-10, 200)
    V, it, st = _solve(tpf.Network.from_feeder(f), torch.from_numpy(S).to(gpu), mode)
    assert np.all(st == tpf.ST_CONVERGED)
    assert np.abs(V - ref.V).max() <= 1e-6


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("T", [1, 16, 17, 4_096, 4_097, 9_001])
def test_columns_do_not_depend_on_their_batch(gpu, T, dtype, mode):
    f = _feeder(150)
    net = tpf.Network.from_feeder(f)
    S = torch.from_numpy(W.profile_minute_year(f, steps=T, seed=4) * (np.arange(T)[:, None] % 13 / 6.0)).to(gpu)
    S = S.to(dtype).contiguous()
    V, it, st = _solve(net, S, mode)
    pick = np.unique(np.r_[0, T // 2, T - 1, np.random.default_rng(0).integers(0, T, 6)])
    for c in pick:
        one = _solve(net, S[c:c + 1].contiguous(), mode)
        assert np.array_equal(one[0][0], V[c]) and one[1][0] == it[c] and one[2][0] == st[c]
    host = S.cpu().numpy()[pick].astype(np.complex128)
    ref = oracle.fpi(oracle.build_feeder(f), host, 1e-10, 200)
    assert np.abs(V[pick] - ref.V).max() <= 1e-6


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_starts_shares_and_bad_columns(gpu, dtype, mode):
    n, T = 170, 50
    f = _feeder(n)
    onet = oracle.build_feeder(f)
    S = W.profile_minute_year(f, steps=T, seed=8)
    Sd = torch.from_numpy(S).to(gpu).to(dtype)
    Sh = Sd.cpu().numpy().astype(np.complex128)
    ref = oracle.fpi(onet, Sh, 1e-10, 200)
    # given starts: near, refused (a modulus out of range, a NaN) and exact
    V0 = ref.V + 1e-4
    V0[3, 5], V0[7, n - 1] = 1.7, np.nan
    V, it, st = _solve(tpf.Network.from_feeder(f), Sd, mode, V0=torch.from_numpy(V0).to(gpu).to(dtype).contiguous())
    assert np.all(st == tpf.ST_CONVERGED) and np.abs(V - ref.V).max() <= 1e-6
    # ZIP loads, with and without a constant-impedance share
    az, ai, ap = W.zipz_shares(n)
    for z in (None, az):
        p = ap if z is not None else 1.0 - ai
        rz = oracle.fpi_zip(onet, Sh, ai, p, 1e-10, 200) if z is None else \
            oracle._fpi_zipz(oracle._load(), onet, Sh, az, ai, ap, 1e-10, 200, None)
        V, it, st = _solve(tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=p, alpha_z=z), Sd, mode)
        assert np.all(st == tpf.ST_CONVERGED) and np.abs(V - rz.V).max() <= 1e-6
    # a NaN load ends its column alone, an infeasible one runs to the cap
    bad = Sd.clone()
    bad[9, 4], bad[20] = float("nan"), 60.0 * bad[20]
    V, it, st = _solve(tpf.Network.from_feeder(f), bad, mode)
    assert st[9] == tpf.ST_NONFINITE and st[20] == tpf.ST_MAX_ITER and it[20] == 100
    rest = np.setdiff1d(np.arange(T), [9, 20])
    assert np.all(st[rest] == tpf.ST_CONVERGED) and np.abs(V[rest] - ref.V[rest]).max() <= 1e-6


def test_in_place(gpu):
    f = _feeder(140)
    net = tpf.Network.from_feeder(f)
    S = torch.from_numpy(W.profile_minute_year(f, steps=90, seed=2)).to(gpu)
    want = _solve(net, S, "mixed_fp16")
    out = tpf.alloc_outputs(net, S, mode="mixed_fp16")
    got = _solve(net, S, "mixed_fp16", out=(S,) + out[1:])
    assert all(np.array_equal(a, b) for a, b in zip(want, got))
