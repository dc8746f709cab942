"""FP64 dense sweeps on nearly resistive feeders with loads at unity power factor: the voltage
angles are small against the drops, and a product that forms Im(Z I) from terms of the size of
Re Z Re I would lose them.

Bound, componentwise: with u = 2^-53 and T = max_i sum_k |Zr||Ii| + |Zi||Ir|, a sum of 2 n
products that keeps the two parts of Im(Z I) apart from those of Re(Z I) errs by at most 2 n u T per
sweep, the injections add (relative) 10 u, and the map contracts by more than 2:
|d Im V| <= 2 (2 n + 20) u T against the same sweeps in extended precision.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu

SWEEPS = 3


def _reference(net, S):
    Z, w = net.zw()
    Z, w = Z.astype(np.clongdouble), w.astype(np.clongdouble)
    S = S.astype(np.clongdouble)
    v = np.ones_like(S)
    for _ in range(SWEEPS):
        i = np.conj(S / v)
        v = w + np.stack([(Z * row).sum(axis=1) for row in i])
    t = (np.abs(i.imag) @ np.abs(Z.real).T + np.abs(i.real) @ np.abs(Z.imag).T).max()
    return v, float(t)


@pytest.mark.parametrize("n,T", [(9, 5), (40, 5), (70, 5), (99, 40), (120, 5), (149, 5), (256, 5), (299, 5), (320, 5),
                                 (330, 1), (330, 40), (330, 700), (330, 11_000), (999, 2)])
@pytest.mark.parametrize("ratio", [2.0 ** -14, 0.0])
def test_small_angles_keep_their_digits(gpu, n, T, ratio):
    f = W.make_feeder(n + 1, load_scale=100.0 / max(n, 100))
    net = tpf.Network(n + 1, f.frm, f.to, f.r, ratio * f.r)
    S = np.ascontiguousarray(W.profile_minute_year(f, steps=T, seed=n).real.astype(np.complex128))
    V, it, _ = tpf.solve_timeseries(net, torch.from_numpy(S).to(gpu), 0.0, SWEEPS)
    assert int(it.min()) == SWEEPS
    pick = np.unique(np.r_[0:min(T, 3), T // 2, T - 1])
    ref, t = _reference(net, S[pick])
    err = np.abs(V.cpu().numpy()[pick].imag - ref.imag).max()
    assert err <= 2 * (2 * n + 20) * 2.0 ** -53 * t
    for c in pick:  # and a column's bits are its own
        one = tpf.solve_timeseries(net, torch.from_numpy(S[c:c + 1]).to(gpu), 0.0, SWEEPS)[0]
        assert torch.equal(one[0], V[c])


@pytest.mark.parametrize("n,T", [(10, 20), (33, 20), (60, 20), (70, 50), (99, 50), (128, 20), (149, 20), (256, 20),
                                 (320, 20), (330, 20), (330, 700), (330, 5_000)])
@pytest.mark.parametrize("kind", ["plain", "c64", "start", "zip"])
def test_resistive_feeders(gpu, n, T, kind):
    """x = r / 10 against the oracle at equal sweep counts: the bound of the other FP64 shapes,
    (3 n + 10) 2^-52 per sweep of a contracting map, 2e-12."""
    f = W.make_feeder(n + 1, load_scale=100.0 / max(n, 100))
    x = 0.1 * np.asarray(f.r)
    onet = oracle.build_network(n + 1, f.frm, f.to, f.r, x)
    ai, ap = W.zip_shares(n) if kind == "zip" else (None, None)
    net = tpf.Network(n + 1, f.frm, f.to, f.r, x, alpha_i=ai, alpha_p=ap)
    S = torch.from_numpy(W.profile_minute_year(f, steps=T, seed=n)).to(gpu)
    S = S.to(torch.complex64 if kind == "c64" else torch.complex128).contiguous()
    host = S.cpu().numpy().astype(np.complex128)
    V0 = torch.full_like(S, 0.97 - 0.02j) if kind == "start" else None
    V, it, st = tpf.solve_timeseries(net, S, 0.0, SWEEPS, V0=V0)
    pick = np.unique(np.r_[0:10, T // 2, T - 10:T])
    if kind == "zip":
        ref = oracle.fpi_zip(onet, host[pick], ai, ap, 0.0, SWEEPS)
    else:
        ref = oracle.fpi(onet, host[pick], 0.0, SWEEPS, None if V0 is None else V0.cpu().numpy()[pick])
    bound = 2e-12 + (2.0 ** -24 * 1.5 if kind == "c64" else 0.0)
    assert np.abs(V.cpu().numpy()[pick] - ref.V).max() <= bound
