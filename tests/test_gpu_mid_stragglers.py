"""Columns that never converge among columns that do, at 129 to 320 PQ buses in the FP32 and
mixed modes: the others neither wait for them nor change.

Time: with every 32nd column infeasible (100 sweeps against about 5.5) the columns' sweeps add
up to 1.6 times those of the feasible loads, and half of the infeasible ones' are FP32 products;
5 times the feasible time leaves room for both, and a batch of 32 that waits for its slowest
column would take 18 times.
"""
import numpy as np
import pytest
import torch

import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu

MODES = ["fp32", "mixed_bf16", "mixed_fp16"]


def _solve(net, S, mode, **kw):
    return tpf.solve_timeseries(net, S, 1e-6, 100, mode=mode, **kw)


def _ms(net, S, mode):
    out = tpf.alloc_outputs(net, S, mode=mode)
    times = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        _solve(net, S, mode, out=out)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return float(np.median(times[1:]))


@pytest.mark.parametrize("mode", MODES)
def test_infeasible_columns_do_not_hold_up_their_batch(gpu, mode):
    n, T = 200, 60_000
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    net = tpf.Network.from_feeder(f)
    S = torch.from_numpy(W.profile_minute_year(f, steps=T, seed=3)).to(gpu)
    bad = S.clone()
    bad[7::32] *= 60.0
    good_ms, bad_ms = _ms(net, S, mode), _ms(net, bad, mode)
    assert bad_ms <= 5.0 * good_ms, f"{bad_ms:.2f} ms against {good_ms:.2f} ms"


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n,T,kind", [(129, 9_000, "few"), (200, 12_345, "many"), (320, 8_200, "slow"),
                                      (299, 20_000, "few"), (160, 9_001, "start"), (170, 8_500, "zip")])
def test_same_bits_beside_slow_columns(gpu, n, T, kind, mode, dtype):
    """Against the same columns in small calls (at most 16 columns per compute unit, which hold
    a column until it ends), bit for bit, in place as well."""
    f = W.make_feeder(n + 1, load_scale=100.0 / n)
    ai, ap = W.zip_shares(n) if kind == "zip" else (None, None)
    net = tpf.Network.from_feeder(f, alpha_i=ai, alpha_p=ap)
    rng = np.random.default_rng(n)
    S = W.profile_minute_year(f, steps=T, seed=5)
    if kind == "slow":  # loads up to and past the feasible ones: every sweep count up to the cap
        S *= np.exp(rng.uniform(np.log(0.5), np.log(100.0), T))[:, None]
    else:
        S[rng.random(T) < (0.3 if kind == "many" else 0.02)] *= 60.0
    S[T // 3, n // 2] = np.nan
    Sd = torch.from_numpy(S).to(gpu).to(dtype).contiguous()
    V0 = None
    if kind == "start":
        V0 = torch.full_like(Sd, 0.97 + 0.01j)
        V0[::11, 3] = 0.3  # refused: flat
    want = _solve(net, Sd, mode, V0=V0)
    step = 16 * torch.cuda.get_device_properties(gpu).multi_processor_count
    for a in range(0, T, step):
        got = _solve(net, Sd[a:a + step].contiguous(), mode, V0=None if V0 is None else V0[a:a + step].contiguous())
        for x, y in zip(want, got):
            x = x[a:a + step].cpu().numpy()
            assert x.tobytes() == y.cpu().numpy().tobytes(), a
    it, st = want[1].cpu().numpy(), want[2].cpu().numpy()
    assert st[T // 3] == tpf.ST_NONFINITE and np.any(st == tpf.ST_MAX_ITER) and np.any(st == tpf.ST_CONVERGED)
    assert np.all(it[st == tpf.ST_MAX_ITER] == 100)
    out = tpf.alloc_outputs(net, Sd, mode=mode)
    own = _solve(net, Sd, mode, V0=V0, out=(Sd,) + out[1:])
    assert all(x.cpu().numpy().tobytes() == y.cpu().numpy().tobytes() for x, y in zip(want, own))
