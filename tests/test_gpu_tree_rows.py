"""The tree operator laid out in rows of lanes (shallow trees) at the edges of its shapes, one
and three phases, against the CPU oracle of the dense form, and against itself: a column's
result must not depend on the batch it is solved in, bit for bit.

Bounds: FP64 after a fixed number of sweeps 1e-12 pu (rounding of sums over at most 1,024
currents, drops of about 0.1 pu: 1e-14 per sweep); FP32 1e-6 pu, the fast forms' contract.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu


def _feeder(n):
    return W.make_feeder(n + 1, load_scale=100.0 / max(n, 100))


def _solve(net, S, mode, tol=1e-6, max_iter=100, **kw):
    V, it, st = tpf.solve_timeseries(net, S, tol, max_iter, mode=mode, **kw)
    return V.cpu().numpy(), it.cpu().numpy(), st.cpu().numpy()


SIZES = [1, 2, 3, 15, 16, 24, 33, 43, 44, 59, 67, 68, 79, 99, 127, 128, 159, 160, 199, 231, 256, 257, 299, 399, 400,
         499, 600, 699, 730, 731, 999, 1024]


@pytest.mark.parametrize("n", SIZES)
def test_every_shape(gpu, n):
    f = _feeder(n)
    net, onet = tpf.Network.from_feeder(f), oracle.build_feeder(f)
    S = W.profile_minute_year(f, steps=37, seed=n)
    Sd = torch.from_numpy(S).to(gpu)
    V, it, st = _solve(net, Sd, "tree_fp64", 0.0, 3)
    assert np.all(it == 3) and np.abs(V - oracle.fpi(onet, S, 0.0, 3).V).max() <= 1e-12
    V, it, st = _solve(net, Sd, "tree_fp32")
    assert np.all(st == tpf.ST_CONVERGED) and np.abs(V - oracle.fpi(onet, S, 1e-10, 200).V).max() <= 1e-6


@pytest.mark.parametrize("mode", ["tree_fp64", "tree_fp32"])
@pytest.mark.parametrize("nb", [1, 4, 15, 16, 39, 40, 79, 99, 100, 127, 128, 160, 200])
def test_every_three_phase_shape(gpu, nb, mode):
    f = W.make_feeder_3ph(nb + 1, load_scale=100.0 / max(nb, 100))
    net, onet = tpf.Network.from_feeder_3ph(f), oracle.build_feeder_3ph(f)
    S = W.profile_minute_year(f, steps=21, seed=nb)
    Sd = torch.from_numpy(S).to(gpu)
    if mode == "tree_fp64":
        V, it, st = _solve(net, Sd, mode, 0.0, 3)
        assert np.all(it == 3) and np.abs(V - oracle.fpi(onet, S, 0.0, 3).V).max() <= 1e-12
    else:
        V, it, st = _solve(net, Sd, mode)
        assert np.all(st == tpf.ST_CONVERGED) and np.abs(V - oracle.fpi(onet, S, 1e-10, 200).V).max() <= 1e-6


@pytest.mark.parametrize("mode", ["tree_fp64", "tree_fp32"])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,T", [(20, 1), (40, 33), (99, 16), (99, 40_001), (180, 9_001), (700, 3)])
def test_columns_do_not_depend_on_their_batch(gpu, n, T, dtype, mode):
    f = _feeder(n)
    net = tpf.Network.from_feeder(f)
    S = torch.from_numpy(W.profile_minute_year(f, steps=T, seed=4) * (np.arange(T)[:, None] % 13 / 6.0)).to(gpu)
    S = S.to(dtype).contiguous()
    V, it, st = _solve(net, S, mode)
    for c in np.unique(np.r_[0, T // 2, T - 1, np.random.default_rng(0).integers(0, T, 6)]):
        one = _solve(net, S[c:c + 1].contiguous(), mode)
        assert np.array_equal(one[0][0], V[c]) and one[1][0] == it[c] and one[2][0] == st[c]
    out = tpf.alloc_outputs(net, S, mode=mode)
    got = _solve(net, S, mode, out=(S,) + out[1:])  # in place
    assert all(np.array_equal(a, b) for a, b in zip((V, it, st), got))


@pytest.mark.parametrize("mode", ["tree_fp64", "tree_fp32"])
@pytest.mark.parametrize("n", [30, 59, 99, 180, 399])
def test_starts_shares_and_bad_columns(gpu, n, mode):
    T = 50
    f = _feeder(n)
    onet = oracle.build_feeder(f)
    S = W.profile_minute_year(f, steps=T, seed=8)
    Sd = torch.from_numpy(S).to(gpu)
    ref = oracle.fpi(onet, S, 1e-10, 200)
    # given starts: near, refused (a modulus out of range, a NaN) and exact
    V0 = ref.V + 1e-4
    V0[3, 5], V0[7, n - 1] = 1.7, np.nan
    net = tpf.Network.from_feeder(f)
    V, it, st = _solve(net, Sd, mode, V0=torch.from_numpy(V0).to(gpu))
    flat = _solve(net, Sd, mode)
    assert np.all(st == tpf.ST_CONVERGED) and np.abs(V - ref.V).max() <= 1e-6
    assert all(np.array_equal(a[[3, 7]], b[[3, 7]]) for a, b in zip((V, it, st), flat))
    az, ai, ap = W.zipz_shares(n)
    rz = oracle.fpi_zip(onet, S, ai, 1.0 - ai, 1e-10, 200)
    V, it, st = _solve(tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=1.0 - ai), Sd, mode)
    assert np.all(st == tpf.ST_CONVERGED) and np.abs(V - rz.V).max() <= 1e-6
    # a NaN load ends its column alone, an overloaded one (infeasible but for 30 buses) as the
    # oracle's does
    bad = Sd.clone()
    bad[9, 4], bad[20] = float("nan"), 60.0 * bad[20]
    V, it, st = _solve(net, bad, mode)
    over = oracle.fpi(onet, 60.0 * S[20:21], 1e-6, 100).status[0]
    assert st[9] == tpf.ST_NONFINITE and (st[20] == tpf.ST_CONVERGED) == (over == tpf.ST_CONVERGED)
    rest = np.setdiff1d(np.arange(T), [9, 20])
    assert np.all(st[rest] == tpf.ST_CONVERGED) and np.array_equal(V[rest], flat[0][rest])
