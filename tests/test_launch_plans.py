"""The launches that the library plans, read on the host (tests/host_checks.hip): no device is needed."""
from __future__ import annotations

import ctypes

import pytest

from paper_2208_04187_amd import _build
from paper_2208_04187_amd.binding import _MapDesc

F32, BF16, C16 = 0, 1, 2


class _Launch(ctypes.Structure):
    _fields_ = [("what", ctypes.c_int), ("kind", ctypes.c_int), ("dt", ctypes.c_int), ("waves", ctypes.c_int), ("gx", ctypes.c_uint32),
                ("gy", ctypes.c_uint32), ("walked", ctypes.c_uint32), ("shapes", ctypes.c_uint32), ("maps", ctypes.c_uint32), ("out", ctypes.c_void_p)]


@pytest.fixture(scope="module")
def host():
    if not _build.HOST_CHECKS_LIB.exists():
        _build.build_checks()
    lib = ctypes.CDLL(str(_build.HOST_CHECKS_LIB))
    i64, ci = ctypes.c_int64, ctypes.c_int
    lib.division_packed_bytes_3d.restype = ctypes.c_size_t
    lib.division_packed_bytes_3d.argtypes = [i64] * 5 + [ci] * 3
    for name in ("division_compress_maps", "division_decompress_maps"):
        getattr(lib, name).argtypes = [ci, ctypes.c_void_p, ctypes.c_void_p]
    return lib


def _dims(shape):
    return shape if len(shape) == 5 else (shape[0], shape[1], 1, shape[2], shape[3])


def _launches(lib):
    found = (_Launch * 64)()
    n = lib.check_take_launches(found, 64)
    assert n <= 64
    return list(found[:n])


def _maps(lib, entries, compress=True):
    """entries: (shape, dt, B, b[, xhat]) per map, buffers 2^38 bytes apart where no address is named (never touched)"""
    descs = []
    for i, (shape, dt, B, b, *out) in enumerate(entries):
        need = lib.division_packed_bytes_3d(*_dims(shape), B, b, dt)
        base = (2 * i + 1) << 38
        descs.append(_MapDesc(base, base + (1 << 37), out[0] if out else base, need, *_dims(shape), dt, B, b, 0))
    descs = (_MapDesc * len(descs))(*descs)
    call = lib.division_compress_maps if compress else lib.division_decompress_maps
    assert call(len(descs), descs, None) == 0
    return _launches(lib)


@pytest.mark.parametrize("maps", range(1, 9))
@pytest.mark.parametrize("shape", [(64, 16, 224, 224), (1, 100, 16, 56, 56), (1, 257, 216, 216), (4, 58, 184, 184), (1, 37, 116, 116)])
def test_sixteen_wavefronts_take_no_more_workgroups_than_cus_where_they_walk(host, shape, maps):
    """A workgroup fills its CU: one more than there are CUs would start when the others have walked to their end."""
    planes, cus = shape[0] * shape[1], host.check_cus()
    for dt in (F32, BF16, C16):
        (launch,) = _maps(host, [(shape, dt, 8, 2)] * maps)
        assert launch.waves == 16 and (launch.walked or shape != (64, 16, 224, 224))
        if launch.walked:
            assert launch.walked == maps and launch.gy == 1 and launch.gx <= min(cus, maps * planes)
        else:
            assert (launch.gx, launch.gy) == (planes, maps)
