"""The FP64 sweeps of large networks over every tile shape their batch size picks (16 x 16 and
32 x 32 with the k-steps split among waves, 64 x 64), at bus counts around the tiles and
slabs, against the CPU oracle at equal sweep counts.

Bound: |V| ~ 1 and Z I is three real sums of n products whose terms add up to less than 1 pu,
so (3 n + 10) 2^-52 <= 7e-13 pu for n <= 1,000 per sweep; the map contracts, so 2e-12.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(gpu, n, T, dtype=torch.complex128, sweeps=3, start=False, in_place=False, shares=False):
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    onet = oracle.build_feeder(f)
    S = W.profile_minute_year(f, steps=T, seed=n)
    Sd = torch.from_numpy(S).to(gpu).to(dtype).contiguous()
    S = Sd.cpu().numpy().astype(np.complex128)
    V0 = None
    if start:
        V0 = np.ones_like(S) + 0.02 * (np.arange(T)[:, None] % 3 - 1)
        V0[T // 2, n - 1] = 0.4  # refused: this column starts flat
    pick = np.unique(np.r_[0:min(T, 20), T // 2, max(0, T - 20):T])
    if shares:
        ai, ap = W.zip_shares(n)
        net = tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=ap)
        ref = oracle.fpi_zip(onet, S[pick], ai, ap, 0.0, sweeps)
    else:
        net = tpf.Network.from_feeder(f)
        R0 = None
        if start:
            R0 = V0[pick].copy()
            R0[pick == T // 2] = 1.0
        ref = oracle.fpi(onet, S[pick], 0.0, sweeps, R0)
    out = tpf.alloc_outputs(net, Sd)
    if in_place:
        out = (Sd,) + out[1:]
    V, it, st = tpf.solve_timeseries(net, Sd, 0.0, sweeps, out=out,
                                     V0=None if V0 is None else torch.from_numpy(V0).to(gpu).to(dtype).contiguous())
    assert np.all(it.cpu().numpy() == sweeps) and np.all(st.cpu().numpy() == tpf.ST_MAX_ITER)
    bound = 2e-12 if dtype == torch.complex128 else 2e-12 + 2.0 ** -24 * 1.5
    assert np.abs(V.cpu().numpy()[pick] - ref.V).max() <= bound


@pytest.mark.parametrize("n,T", [(321, 1), (321, 17), (336, 33), (400, 64), (321, 500), (353, 650), (383, 1_000),
                                 (321, 11_001), (385, 10_017), (999, 5)])
def test_every_shape(gpu, n, T):
    _check(gpu, n, T)


@pytest.mark.parametrize("T", [3, 700, 11_000])
@pytest.mark.parametrize("kind", ["c64", "start", "in_place", "shares"])
def test_forms_of_a_call(gpu, T, kind):
    _check(gpu, 330, T, dtype=torch.complex64 if kind == "c64" else torch.complex128, start=kind == "start",
           in_place=kind == "in_place", shares=kind == "shares")


@pytest.mark.parametrize("T", [40, 700, 11_000])
def test_columns_retire_one_by_one(gpu, T):
    """Loads from idle to heavy retire after different sweep counts: the lists of active
    columns shrink and every column keeps its own result."""
    n = 330
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    net, onet = tpf.Network.from_feeder(f), oracle.build_feeder(f)
    S = W.profile_minute_year(f, steps=T, seed=5) * (np.arange(T)[:, None] % 41 / 20.0)
    V, it, st = tpf.solve_timeseries(net, torch.from_numpy(S).to(gpu), 1e-9, 100)
    assert int(st.max()) == tpf.ST_CONVERGED
    it = it.cpu().numpy()
    assert len(np.unique(it)) > 3
    pick = np.unique(np.r_[0:41, T - 5:T])
    pick = pick[pick < T]
    ref = oracle.fpi(onet, S[pick], 1e-9, 100)
    same = it[pick] == ref.iters
    assert same.mean() > 0.9  # a last step on the tolerance may fall to either side
    assert np.abs(V.cpu().numpy()[pick][same] - ref.V[same]).max() <= 2e-12
