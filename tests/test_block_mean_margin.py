"""The block-mean rule with a reciprocal that is a few units off: the kernels take 1 / count from Newton steps or as a
product of two reciprocals (at most 4 ulp off), and the rule must still pick the definition's binary32 value.  The rule and
the Newton steps are the library's own source, run on the host; tests/test_gpu_device_helpers.py measures the device's."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import paper_2208_04187_amd as pkg

COUNTS = [3, 5, 6, 7, 9, 10, 12, 21, 24, 27, 40, 56, 63, 98, 147, 196, 198, 324, 1000003, 2 ** 31 - 1]


def _off(v: np.ndarray, ulps) -> np.ndarray:
    return (np.asarray(v, dtype=np.float64).view(np.int64) + ulps).view(np.float64)


def _rule():
    f = pkg.lib().division_block_mean_rule_rcp
    f.restype = ctypes.c_float
    f.argtypes = [ctypes.c_double, ctypes.c_uint32, ctypes.c_double, ctypes.POINTER(ctypes.c_int)]
    return f


@pytest.mark.parametrize("off", [-4, -3, -1, 0, 1, 2, 4])
def test_mean_rule_with_an_inexact_reciprocal(off):
    rule, rng, divided, calls = _rule(), np.random.default_rng(4187), 0, 0
    d = ctypes.c_int(0)
    for cnt in COUNTS:
        rcp = float(_off(np.array([1.0 / cnt]), off)[0])
        m = np.concatenate([rng.standard_normal(60).astype(np.float32),
                            (rng.integers(1, 1 << 24, 10) * 2.0 ** -149).astype(np.float32)])     # subnormal means too
        up = np.nextafter(m, np.float32(np.inf), dtype=np.float32)
        mid = (m.astype(np.float64) + up.astype(np.float64)) / 2
        for base in (mid, m.astype(np.float64)):
            S = base * cnt                                   # its quotient lands on or beside base
            for delta in (-20, -12, -6, -5, -4, -3, -2, -1, 0, 1, 2, 3, 4, 5, 6, 12, 20):
                Sd = _off(S, delta)
                want = (Sd / cnt).astype(np.float32)
                for s, w in zip(Sd.tolist(), want.view(np.uint32)):
                    got = np.float32(rule(s, cnt, rcp, ctypes.byref(d)))
                    divided += d.value
                    calls += 1
                    assert got.view(np.uint32) == w, (cnt, delta, s)
    assert 0 < divided < calls


@pytest.mark.parametrize("error", [0.0, 2.0 ** -30, -2.0 ** -30, 2.0 ** -23, -2.0 ** -23, 2.0 ** -20, -2.0 ** -20])
def test_newton_steps_reach_the_reciprocal(error):
    """From an estimate that is off by `error`: within 2 ulp of 1 / count, and exact for a power of two."""
    f = pkg.lib().division_count_reciprocal
    f.restype = ctypes.c_double
    f.argtypes = [ctypes.c_uint32, ctypes.c_double]
    counts = list(range(1, 3000)) + COUNTS + [2 ** k for k in range(32)] + [2 ** k + 1 for k in range(12, 32)] + [2 ** 32 - 1]
    for cnt in counts:
        off = int(_off(np.array([f(cnt, (1.0 / cnt) * (1.0 + error))]), 0).view(np.int64)[0] - np.array([1.0 / cnt]).view(np.int64)[0])
        assert abs(off) <= 2, (cnt, off)
        assert off == 0 or cnt & (cnt - 1)
    assert f(0, 1.0) == 0.0
