"""FP64 beyond 320 PQ buses: every shape of the product's tiles (single tiles, 32 x 32, 64 x 32 and
64 x 64 blocks, staged ones) gives a column the same bits, whether its complex products are
three or four real ones, and the oracle's voltages after three sweeps (1e-12 pu, as in the other
tests of these kernels).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ratio", [None, 0.3])  # x = ratio r: four products
@pytest.mark.parametrize("n", [321, 999, 1_100])
def test_every_shape(gpu, n, ratio):
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    x = f.x if ratio is None else ratio * np.asarray(f.r)
    net = tpf.Network(n + 1, f.frm, f.to, f.r, x)
    T = 6_400 * 1_000 // n  # staged at 256 compute units; the parts below: 64 x 64, 64 x 32, 32 x 32, single
    S = W.profile_minute_year(f, steps=T, seed=8)
    Sd = torch.from_numpy(S).to(gpu)
    want = tpf.solve_timeseries(net, Sd, 0.0, 3, mode="fp64")
    for m in (3_000 * 1_000 // n, 1_000, 777, 250, 101, 17, 1):
        got = tpf.solve_timeseries(net, Sd[:m].contiguous(), 0.0, 3, mode="fp64")
        for a, b in zip(want, got):
            assert torch.equal(a[:m], b), m
    pick = np.r_[0:3, T - 2:T]
    ref = oracle.fpi(oracle.build_network(n + 1, f.frm, f.to, f.r, x), S[pick], 0.0, 3).V
    assert np.abs(want[0].cpu().numpy()[pick] - ref).max() <= 1e-12


def test_operator_beyond_the_cache(gpu):
    f = W.make_feeder(3_601, load_scale=0.02)
    net = tpf.Network.from_feeder(f)
    Sd = torch.from_numpy(W.profile_minute_year(f, steps=500, seed=8)).to(gpu)
    want = tpf.solve_timeseries(net, Sd, 0.0, 2, mode="fp64")
    for m in (300, 64, 20, 1):
        for a, b in zip(want, tpf.solve_timeseries(net, Sd[:m].contiguous(), 0.0, 2, mode="fp64")):
            assert torch.equal(a[:m], b), m
