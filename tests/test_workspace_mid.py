"""Workspace the solves ask for at 129 to 320 PQ buses in the FP32 and mixed modes: these
networks keep their columns on chip, so it does not grow with the number of columns."""
import ctypes

import pytest

import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W


@pytest.mark.parametrize("mode", [tpf.MODE_FP32, tpf.MODE_MIXED_BF16, tpf.MODE_MIXED_FP16])
@pytest.mark.parametrize("n", [129, 200, 320])
def test_bounded_at_mid_sizes(n, mode):
    net = tpf.Network.from_feeder(W.make_feeder(n + 1))
    need = [tpf.workspace_bytes(net, tau, mode) for tau in (1, 100, 10_000, 210_240, 8_760_000)]
    assert need == sorted(need)
    # less than the per-sweep path holds per column for its state (2 n drops and 2 n injections
    # in FP32), and bounded whatever the number of columns
    assert need[2] <= 10_000 * 16 * n
    assert need[3] == need[4] <= 128 << 20


@pytest.mark.parametrize("mode", [tpf.MODE_FP32, tpf.MODE_MIXED_BF16, tpf.MODE_MIXED_FP16])
def test_per_sweep_state_beyond(mode):
    net = tpf.Network.from_feeder(W.make_feeder(322))
    assert tpf.workspace_bytes(net, 1_000, mode) >= 1_000 * 16 * 321


def test_smaller_is_refused():
    net = tpf.Network.from_feeder(W.make_feeder(200))
    o = tpf._Options(mode=tpf.MODE_FP32)
    need = tpf.workspace_bytes(net, 9_000, tpf.MODE_FP32)
    fake = ctypes.c_void_p(4096)  # never dereferenced: the size is refused first
    rc = tpf.load_library().tpf_solve_timeseries(net.handle, fake, tpf.TPF_C128, 9_000, 1e-6, 10, ctypes.byref(o), fake,
                                                 fake, fake, ctypes.c_void_p(256 * 64), need - 1, None)
    assert rc == tpf.TPF_ERR_INVALID_ARG
