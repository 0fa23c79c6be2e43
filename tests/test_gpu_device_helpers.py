"""Device helpers whose error or bits the kernels' comments state: the reciprocals of block counts, bfloat16 conversion."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2208_04187_amd import _build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def checks():
    if not _build.CHECKS_LIB.exists():
        _build.build_checks()
    lib = ctypes.CDLL(str(_build.CHECKS_LIB))
    lib.check_count_reciprocals.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p]
    lib.check_bf16_conversions.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    return lib


def _reciprocals(checks, first, n, cols):
    out = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    assert checks.check_count_reciprocals(first, n, cols, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _ulps(got, counts):
    return np.abs(got.view(np.int64) - (1.0 / counts.astype(np.float64)).view(np.int64))


@pytest.mark.parametrize("first,n", [(1, 1 << 22), ((1 << 27) - 1000, 1 << 20), ((1 << 31) - (1 << 19), 1 << 20), ((1 << 32) - 65536, 65536)])
def test_reciprocal_of_a_block_count(checks, first, n):
    counts = np.arange(first, first + n, dtype=np.int64)
    off = _ulps(_reciprocals(checks, first, n, 0), counts)
    assert off.max() <= 2, (int(off.max()), int(counts[off.argmax()]))
    assert not off[(counts & (counts - 1)) == 0].any()


@pytest.mark.parametrize("cols", range(1, 9))
def test_reciprocal_of_rows_times_columns(checks, cols):
    """The strip kernels: rows of a block once per lane, times the constant 1 / columns of the segment."""
    rows = np.arange(1, 65537, dtype=np.int64)
    off = _ulps(_reciprocals(checks, 1, rows.size, cols), rows * cols)
    assert off.max() <= 4
    assert not off[(rows * cols & (rows * cols - 1)) == 0].any()


def test_bfloat16_conversion_of_every_binary32(checks):
    bad = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    assert checks.check_bf16_conversions(bad.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert int(bad) == 0
