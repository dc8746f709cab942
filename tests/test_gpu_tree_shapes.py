"""The tree operator on trees of other shapes than k-ary feeders: few to many levels, evenly
filled or bottom-heavy, few and many columns, so that every kernel its choice knows is taken.

Results: FP64 after three sweeps within 1e-12 pu of the oracle, FP32 within 1e-6 pu (the bounds of
the other tree tests).  The oracle iterates with the exact constants of a tree, Z as sums over the
shared path and w = 1: its own inverse of the admittance matrix leaves w off by 1.4e-12 to 2.9e-12
at 900 buses (against sums in extended precision).  Time: a sweep visits each level, and half as many again allows
for the children it visits, so L' levels instead of L take at most 1.5 L' / L times as long.
"""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2403_04578_amd as tpf

pytestmark = pytest.mark.gpu


def _tree(n, levels, heavy):
    """Parents of buses 1..n: a chain of `levels`, the others one level after another (evenly) or
    mostly at the bottom."""
    rng = np.random.default_rng(n * 100 + levels)
    depth, parent = np.zeros(n + 1, int), np.zeros(n + 1, int)
    for b in range(1, n + 1):
        if b <= levels:
            depth[b], parent[b] = b, b - 1
            continue
        d = min(levels, 1 + int(levels * rng.random() ** 0.4)) if heavy else 1 + (b - levels - 1) % levels
        parent[b] = rng.choice(np.nonzero(depth[:b] == d - 1)[0])
        depth[b] = d
    return parent[1:].astype(np.int32)


def _case(n, levels, heavy, T, phases=1, drop=1.0):
    rng = np.random.default_rng(7)
    frm, to = _tree(n, levels, heavy), np.arange(1, n + 1, dtype=np.int32)
    r = rng.uniform(0.002, 0.006, n) * drop * (20 / max(n, 20))
    x = r * rng.uniform(0.5, 2.0, n)
    s = rng.uniform(0.005, 0.02, n * phases) * np.exp(0.3j) / phases
    S = s * rng.uniform(0.5, 1.5, (T, 1))
    if phases == 1:
        onet = oracle.build_network(n + 1, frm, to, r, x)
        path = np.zeros((n, n))
        for b in range(n):
            path[b] = path[frm[b] - 1] if frm[b] else 0
            path[b, b] = 1
        Z = -(path * (r + 1j * x)) @ path.T
        return tpf.Network(n + 1, frm, to, r, x), dataclasses.replace(onet, Z=Z, w=np.ones(n, complex)), S
    z = (r + 1j * x)[:, None, None] * (0.65 * np.eye(3) + 0.35)
    return tpf.Network.three_phase(n + 1, frm, to, z), oracle.build_network_3ph(n + 1, frm, to, z), S


TREES = [(5, 2), (5, 5), (12, 4), (12, 12), (24, 3), (30, 8), (30, 15), (45, 6), (60, 5), (60, 10), (60, 14), (99, 6),
         (99, 12), (99, 18), (127, 5), (127, 13), (180, 6), (180, 14), (250, 10), (300, 6), (300, 15), (300, 20),
         (450, 10), (450, 20), (600, 12), (750, 9), (900, 8), (900, 18), (64, 40)]


@pytest.mark.parametrize("heavy", [False, True])
@pytest.mark.parametrize("T", [9, 3_001])
@pytest.mark.parametrize("n,levels", TREES)
def test_any_tree(gpu, n, levels, T, heavy):
    net, onet, S = _case(n, levels, heavy, T)
    pick = np.r_[0:5, T - 4:T]
    Sd = torch.from_numpy(S).to(gpu)
    V, it, _ = tpf.solve_timeseries(net, Sd, 0.0, 3, mode="tree_fp64")
    assert int(it.min()) == 3 and np.abs(V.cpu().numpy()[pick] - oracle.fpi(onet, S[pick], 0.0, 3).V).max() <= 1e-12
    V, _, st = tpf.solve_timeseries(net, Sd, 1e-6, 100, mode="tree_fp32")
    assert int(st.max()) == tpf.ST_CONVERGED
    assert np.abs(V.cpu().numpy()[pick] - oracle.fpi(onet, S[pick], 1e-10, 200).V).max() <= 1e-6


@pytest.mark.parametrize("zip_loads", [False, True])
@pytest.mark.parametrize("n,levels", TREES)
def test_a_column_alone_and_among_others(gpu, n, levels, zip_loads):
    """The kernel depends on the number of columns, the bits do not."""
    net, _, S = _case(n, levels, True, 3_001)
    if zip_loads:
        rng = np.random.default_rng(n)
        ai = rng.uniform(0, 0.6, n)
        frm, to = _tree(n, levels, True), np.arange(1, n + 1, dtype=np.int32)
        r = rng.uniform(0.002, 0.006, n) * (20 / max(n, 20))
        net = tpf.Network(n + 1, frm, to, r, r * rng.uniform(0.5, 2.0, n), alpha_i=ai, alpha_p=1 - ai)
    S = torch.from_numpy(S).to(gpu)
    for mode in ("tree_fp64", "tree_fp32"):
        few, it, _ = tpf.solve_timeseries(net, S[:9].contiguous(), 1e-6, 100, mode=mode)
        for X in (S, S.repeat(max(1, 6_000 // n), 1)):
            V, its, _ = tpf.solve_timeseries(net, X, 1e-6, 100, mode=mode)
            assert torch.equal(V[:9], few) and torch.equal(its[:9], it)


@pytest.mark.parametrize("T", [9, 3_001])
@pytest.mark.parametrize("n,levels", [(5, 2), (5, 5), (12, 8), (30, 5), (30, 12), (60, 6), (99, 4), (127, 7), (250, 10)])
def test_any_three_phase_tree(gpu, n, levels, T):
    net, onet, S = _case(n, levels, False, T, phases=3)
    pick = np.r_[0:3, T - 2:T]
    Sd = torch.from_numpy(S).to(gpu)
    V, it, _ = tpf.solve_timeseries(net, Sd, 0.0, 3, mode="tree_fp64")
    assert int(it.min()) == 3 and np.abs(V.cpu().numpy()[pick] - oracle.fpi(onet, S[pick], 0.0, 3).V).max() <= 1e-12
    V, _, st = tpf.solve_timeseries(net, Sd, 1e-6, 100, mode="tree_fp32")
    assert int(st.max()) == tpf.ST_CONVERGED
    assert np.abs(V.cpu().numpy()[pick] - oracle.fpi(onet, S[pick], 1e-10, 200).V).max() <= 1e-6


@pytest.mark.parametrize("n,levels,phases", [
    (12, 4, 1), (24, 3, 1), (45, 6, 1), (60, 5, 1), (60, 8, 1), (60, 10, 1), (80, 7, 1), (99, 9, 1), (127, 5, 1),
    (127, 9, 1), (12, 4, 3), (30, 5, 3), (30, 8, 3), (60, 5, 3), (60, 8, 3), (99, 6, 3)])
def test_calls_that_fill_the_chip(gpu, n, levels, phases):
    net, onet, S = _case(n, levels, False, 1_000, phases=phases)
    T = 60_001
    Sd = torch.from_numpy(S).to(gpu).repeat(61, 1)[:T].contiguous()
    pick = np.r_[0:3, 517, T - 4:T]
    V, it, _ = tpf.solve_timeseries(net, Sd, 0.0, 3, mode="tree_fp64")
    S = S[pick % 1_000]
    assert int(it.min()) == 3 and np.abs(V[pick].cpu().numpy() - oracle.fpi(onet, S, 0.0, 3).V).max() <= 1e-12
    V, _, st = tpf.solve_timeseries(net, Sd, 1e-6, 100, mode="tree_fp32")
    assert int(st.max()) == tpf.ST_CONVERGED
    assert np.abs(V[pick].cpu().numpy() - oracle.fpi(onet, S, 1e-10, 200).V).max() <= 1e-6


def _ms(gpu, n, levels, heavy, mode):
    net, _, S = _case(n, levels, heavy, 2_000)
    S = torch.from_numpy(S).to(gpu).repeat(25, 1)
    out = tpf.alloc_outputs(net, S, mode=mode)
    times = []
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        _, it, _ = tpf.solve_timeseries(net, S, 5e-7, 3, mode=mode, out=out)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return float(np.median(times[2:])) / float(it.double().mean())


@pytest.mark.parametrize("mode,n,few,many,heavy", [
    ("tree_fp32", 300, 14, 20, False), ("tree_fp32", 300, 10, 20, True), ("tree_fp32", 450, 14, 20, False),
    ("tree_fp64", 30, 8, 12, False), ("tree_fp64", 60, 8, 14, False), ("tree_fp64", 30, 8, 15, True)])
def test_more_levels_cost_what_they_add(gpu, mode, n, few, many, heavy):
    a, b = _ms(gpu, n, few, heavy, mode), _ms(gpu, n, many, heavy, mode)
    assert b <= 1.5 * many / few * a, f"{many} levels {1e3 * b:.0f} us per sweep, {few} levels {1e3 * a:.0f}"
