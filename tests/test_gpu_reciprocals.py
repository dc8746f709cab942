"""The sweeps' reciprocals are those of the division.

FP32: one Newton step on the hardware's estimate, compared over every mantissa.  FP64: the
estimate is good to 2^-23 at least, so two steps leave 2^-92 before the last rounding, which
then differs from the division's only within 2^-92 of a midpoint between two numbers: one value
in about 2^38, none expected among 2^24.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_2403_04578_amd as tpf

pytestmark = pytest.mark.gpu


def _reciprocals(gpu, x):
    lib = tpf.load_library()
    f = lib.tpf_check_reciprocals
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_void_p]
    x = torch.from_numpy(x).to(gpu)
    y = torch.empty_like(x)
    assert f(x.data_ptr(), y.data_ptr(), x.numel(), x.dtype == torch.float64,
             torch.cuda.current_stream().cuda_stream) == 0
    return y.cpu().numpy()


@pytest.mark.parametrize("exponent", [-99, -64, -2, -1, 0, 1, 63, 124])
def test_every_float_mantissa(gpu, exponent):
    x = ((np.uint32(exponent + 127) << np.uint32(23)) | np.arange(1 << 23, dtype=np.uint32)).view(np.float32)
    assert np.array_equal(_reciprocals(gpu, x), np.float32(1) / x)


def test_floats_beyond(gpu):
    y = _reciprocals(gpu, np.array([2.0**126, 3e38, np.inf, np.nan], np.float32))
    assert np.all(np.abs(y[:2]) <= 2.0**-125) and y[2] == 0 and np.isnan(y[3])


@pytest.mark.parametrize("exponent", [-600, -40, -1, 0, 1, 40, 600])
def test_doubles(gpu, exponent):
    x = (1 + np.random.default_rng(exponent + 1000).random(1 << 24)) * 2.0**exponent
    assert np.array_equal(_reciprocals(gpu, x), 1 / x)
