"""The FP64 sweep kernel at the edges of its tiling, against the CPU oracle at equal sweep
counts: 16-bus tiles and 4-bus k-steps with every remainder, one to eight waves, one to
three tiles per wave, tiles whose k-steps are shared out among waves (MT % 4 = 1, 2, 3), and
columns past the first fill.

Bound: |V| ~ 1 and Z I is three real sums of n products whose terms add up to less than 1 pu,
so (3 n + 10) 2^-52 <= 3e-13 pu for n <= 320 per sweep; the map contracts, so 1e-12.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [1, 3, 4, 5, 15, 16, 17, 31, 33, 47, 49, 63, 64, 65, 80, 81, 96, 97, 112, 113, 128, 129, 145, 161, 192, 193,
         209, 241, 256, 257, 273, 303, 320]


def _loads(f, T, seed):
    return W.profile_minute_year(f, steps=T, seed=seed)


@pytest.mark.parametrize("n", SIZES)
def test_every_tile_remainder(gpu, n):
    f = W.make_feeder(n + 1, load_scale=min(1.0, 100.0 / n))
    net, onet = tpf.Network.from_feeder(f), oracle.build_feeder(f)
    S = _loads(f, 37, n)
    V0 = np.ones_like(S) + 0.01 * (np.arange(37)[:, None] % 3 - 1)
    V0[5, n - 1] = 1.6  # refused: this column starts flat
    flat = V0.copy()
    flat[5] = 1.0
    for start, same in ((None, None), (V0, flat)):
        ref = oracle.fpi(onet, S, 0.0, 4, same)
        V, it, st = tpf.solve_timeseries(net, torch.from_numpy(S).to(gpu), 0.0, 4,
                                         V0=None if start is None else torch.from_numpy(start).to(gpu))
        assert np.array_equal(it.cpu().numpy(), ref.iters) and np.array_equal(st.cpu().numpy(), ref.status)
        assert np.abs(V.cpu().numpy() - ref.V).max() <= 1e-12


@pytest.mark.parametrize("n", [15, 65, 87, 99, 145, 300])
def test_zip_shares_at_tile_remainders(gpu, n):
    f = W.make_feeder(n + 1, load_scale=min(1.0, 100.0 / n))
    ai, ap = W.zip_shares(n)
    onet = oracle.build_feeder(f)
    S = _loads(f, 21, n)
    ref = oracle.fpi_zip(onet, S, ai, ap, 0.0, 4)
    V, it, st = tpf.solve_timeseries(tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=ap), torch.from_numpy(S).to(gpu),
                                     0.0, 4)
    assert np.array_equal(it.cpu().numpy(), ref.iters) and np.array_equal(st.cpu().numpy(), ref.status)
    assert np.abs(V.cpu().numpy() - ref.V).max() <= 1e-12


@pytest.mark.parametrize("n,T", [(5, 70_001), (70, 16_385), (99, 8_209)])
def test_columns_past_the_first_fill(gpu, n, T):
    """More columns than the resident workgroups hold: the queue deals out the rest, every
    column once, each with its own loads."""
    f = W.make_feeder(n + 1)
    net, onet = tpf.Network.from_feeder(f), oracle.build_feeder(f)
    S = _loads(f, T, 3)
    V, it, st = tpf.solve_timeseries(net, torch.from_numpy(S).to(gpu), 1e-7, 100)
    assert int(st.max()) == tpf.ST_CONVERGED and int(it.min()) >= 1
    pick = np.unique(np.r_[0:40, np.random.default_rng(1).integers(0, T, 400), T - 40:T])
    ref = oracle.fpi(onet, S[pick], 1e-7, 100)
    same = it.cpu().numpy()[pick] == ref.iters
    assert same.mean() > 0.99  # a last step on the tolerance may fall to either side
    assert np.abs(V.cpu().numpy()[pick][same] - ref.V[same]).max() <= 1e-12


@pytest.mark.parametrize("tol", [0.0, 1e-200, 1e-160, 1e-12, 1e-6, 0.3, 1e160, float("inf")])
def test_stopping_rule_over_tolerances(gpu, tol):
    """d < tol is decided on |dV|^2: the smallest and largest tolerances keep their meaning."""
    f = W.make_feeder(20)
    net, onet = tpf.Network.from_feeder(f), oracle.build_feeder(f)
    S = _loads(f, 16, 9)
    ref = oracle.fpi(onet, S, tol, 6)
    V, it, st = tpf.solve_timeseries(net, torch.from_numpy(S).to(gpu), tol, 6)
    assert np.abs(V.cpu().numpy() - ref.V).max() <= 1e-11  # 1e-12 may stop one sweep apart
    if tol == 0.0:
        assert np.all(it.cpu().numpy() == 6) and np.all(st.cpu().numpy() == tpf.ST_MAX_ITER)
    elif tol >= 1e-6:
        assert np.array_equal(it.cpu().numpy(), ref.iters) and np.array_equal(st.cpu().numpy(), ref.status)
