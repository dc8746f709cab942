"""FP64 beyond 320 PQ buses: a column's voltages, sweep count and status do not depend on how
many other columns are in the call, bit for bit, although the batch size picks the shape of
the product's tiles.
"""
import numpy as np
import pytest
import torch

import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solve(net, S, **kw):
    return tuple(a.cpu().numpy() for a in tpf.solve_timeseries(net, S, 1e-9, 100, **kw))


@pytest.mark.parametrize("kind", ["plain", "c64", "start", "in_place", "zip"])
@pytest.mark.parametrize("n,T,parts", [(330, 11_000, [1, 40, 700, 3_000]), (999, 4_100, [3, 90, 260, 1_000])])
def test_a_part_of_the_columns_gives_the_same_bits(gpu, n, T, parts, kind):
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    ai, ap = W.zip_shares(n) if kind == "zip" else (None, None)
    net = tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=ap)
    S = W.profile_minute_year(f, steps=T, seed=6) * (0.2 + np.arange(T)[:, None] % 17 / 10.0)
    Sd = torch.from_numpy(S).to(gpu).to(torch.complex64 if kind == "c64" else torch.complex128).contiguous()
    V0 = torch.full_like(Sd, 0.98 + 0.01j) if kind == "start" else None
    if kind == "in_place":  # the state cannot live in the output then; same bits all the same
        own = Sd.clone()
        want = _solve(net, own, out=(own,) + tpf.alloc_outputs(net, own)[1:])
    else:
        want = _solve(net, Sd, V0=V0)
    assert len(np.unique(want[1])) > 1
    for m in parts:
        for a in (0, (T - m) // 2, T - m):
            got = _solve(net, Sd[a:a + m].contiguous(), V0=None if V0 is None else V0[a:a + m].contiguous())
            for x, y in zip(want, got):
                assert np.array_equal(x[a:a + m], y), (m, a)
