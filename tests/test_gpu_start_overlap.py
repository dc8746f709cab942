"""Start voltages in the output's own array, or in one that it partly covers (the last steps'
voltages as the next ones' start, views of one buffer): the same bits as from separate arrays.
"""
import pytest
import torch

import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [("fp64", 60, 3_000), ("fp64", 330, 40), ("fp64", 330, 3_000), ("fp32", 60, 3_000), ("mixed_fp16", 99, 9_000),
         ("fp32", 150, 9_000), ("mixed_bf16", 150, 9_000), ("mixed_fp16", 299, 9_000), ("fp32", 330, 300),
         ("mixed_fp16", 330, 300), ("tree_fp64", 99, 9_000), ("tree_fp32", 300, 3_000)]


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("mode,n,T", CASES)
def test_start_and_output_share_memory(gpu, mode, n, T, dtype):
    f = W.make_feeder(n + 1, load_scale=100.0 / max(n, 100))
    net = tpf.Network.from_feeder(f)
    S = torch.from_numpy(W.profile_minute_year(f, steps=T, seed=2)).to(gpu).to(dtype).contiguous()
    V = tpf.solve_timeseries(net, S, 1e-6, 100, mode="fp64")[0]
    V0 = V + 0.01 * torch.arange(T, device=gpu)[:, None] / T  # every column its own start
    V0[T // 3, 2] = 0.3  # refused: this column starts flat
    V0 = V0.to(dtype).contiguous()
    for cap in (100, 0):
        want = tpf.solve_timeseries(net, S, 1e-6, cap, mode=mode, V0=V0)
        for shift in (-1, 0, 1, 7):
            buf = torch.zeros(T + 8, n, dtype=dtype, device=gpu)
            a, b = (1, 1 + shift)  # first rows of the start and of the output
            start, out = buf[a:a + T], buf[b:b + T]
            start.copy_(V0)
            got = tpf.solve_timeseries(net, S, 1e-6, cap, mode=mode, V0=start,
                                       out=(out,) + tpf.alloc_outputs(net, S, mode=mode)[1:])
            assert all(torch.equal(torch.view_as_real(x) if x.is_complex() else x,
                                   torch.view_as_real(y) if y.is_complex() else y) for x, y in zip(want, got)), (cap, shift)
