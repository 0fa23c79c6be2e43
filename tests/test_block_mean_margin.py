"""The block-mean rule with a reciprocal that is a few units off: the kernels take 1 / count from Newton steps or as a
product of two reciprocals (at most 4 ulp off), and the rule must still pick the definition's binary32 value."""
from __future__ import annotations

import numpy as np
import pytest


def _rule(S, cnt, rcp):
    """mean_with_rcp: the product unless it is within 16 ulp of a binary32 midpoint, or subnormal"""
    q = S * rcp
    low = (q.view(np.uint64) & np.uint64(0x1FFFFFFF)).astype(np.int64)
    divide = (np.abs(low - 0x10000000) < 16) | ((q != 0) & (np.abs(q) < 2.0 ** -126))
    return np.where(divide, S / cnt, q).astype(np.float32)


@pytest.mark.parametrize("off", [-4, -3, -1, 0, 1, 2, 4])
def test_mean_rule_with_an_inexact_reciprocal(off):
    rng = np.random.default_rng(4187)
    for cnt in [3, 5, 6, 7, 9, 10, 12, 21, 24, 27, 40, 56, 63, 98, 147, 196, 198, 324, 1000003, 2 ** 31 - 1]:
        rcp = 1.0 / np.float64(cnt)
        rcp = (np.array([rcp]).view(np.int64) + off).view(np.float64)[0]
        m = rng.standard_normal(20000).astype(np.float32)
        up = np.nextafter(m, np.float32(np.inf), dtype=np.float32)
        mid = (m.astype(np.float64) + up.astype(np.float64)) / 2
        for base in (mid, m.astype(np.float64)):
            S = base * cnt                                   # its quotient lands on or beside base
            for d in range(-6, 7):
                Sd = (S.view(np.int64) + d).view(np.float64)
                assert np.array_equal(_rule(Sd, float(cnt), rcp), (Sd / cnt).astype(np.float32)), (cnt, d)
