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
    """entries: (shape, dt, B, b[, xhat[, packed[, packed_bytes]]]) per map, buffers 2^38 bytes apart where no address is named (never touched)"""
    descs = []
    for i, (shape, dt, B, b, *at) in enumerate(entries):
        need = lib.division_packed_bytes_3d(*_dims(shape), B, b, dt)
        base = (2 * i + 1) << 38
        out, packed, size = (list(at) + [None] * 3)[:3]
        descs.append(_MapDesc(base, packed or base + (1 << 37), out or base, size or need, *_dims(shape), dt, B, b, 0))
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


@pytest.fixture(scope="module")
def pool():
    if not _build.MASK_CHECKS_LIB.exists():
        _build.build_checks()
    lib = ctypes.CDLL(str(_build.MASK_CHECKS_LIB))
    i64, ci, vp, sz = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t
    lib.division_maxpool_forward.argtypes = [vp, i64, i64, i64, i64, ci, ci, vp, vp, sz, vp]
    lib.division_maxpool_backward.argtypes = [vp, sz, vp, i64, i64, i64, i64, ci, ci, vp, vp]
    lib.check_pool_kernel.restype = ctypes.c_char_p
    lib.check_pool_kernel.argtypes = [ctypes.POINTER(ctypes.c_uint32)]
    return lib


def _pool_backward(lib, shape, dt, k, offset=0):
    es = 2 if dt == BF16 else 4
    rc = lib.division_maxpool_backward(1 << 40, 1 << 40, 1 << 41, *shape, dt, k, (1 << 42) + offset * es, None)
    groups = ctypes.c_uint32()
    return rc, lib.check_pool_kernel(ctypes.byref(groups)).decode().strip("()"), groups.value


@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("offset", [0, 4])
@pytest.mark.parametrize("H", [2, 27, 28, 100, 223])
@pytest.mark.parametrize("W", [4, 12, 28, 32, 44, 100, 224])
def test_pooling_backward_of_whole_pieces_streams(pool, dt, offset, H, W):
    """k = 2 on rows of whole four-element pieces at such a boundary: no widths, heights or offsets that miss the streaming kernel."""
    P = max(1, 12_000_000 // (H * W))
    rc, name, groups = _pool_backward(pool, (1, P, H, W), dt, 2, offset)
    assert rc == 0 and name.startswith("maxpool2_backward_fast<"), name
    pieces = P * H * W // int(name.split(",")[1])
    assert groups * 256 * (2 if name.startswith("maxpool2_backward_fast<uint16_t, 4") else 1) >= pieces
    assert name.endswith("true>" if H % 2 else "false>")


def test_pooling_backward_of_other_maps(pool):
    for shape, dt, k, offset, want in (((64, 100, 27, 27), BF16, 2, 0, "maxpool_backward_kernel<uint16_t, 1>"), ((64, 600, 27, 27), BF16, 2, 0, "maxpool_backward_kernel<uint16_t, 4>"),
                                       ((64, 100, 56, 56), BF16, 3, 2, "maxpool_backward_kernel<uint16_t, 4>"), ((64, 100, 56, 56), BF16, 3, 1, "maxpool_backward_scalar<uint16_t>"),
                                       ((4, 32, 14, 14), BF16, 3, 0, "maxpool_backward_scalar<uint16_t>"), ((4, 512, 7, 7), BF16, 3, 0, "maxpool_backward_kernel<uint16_t, 1>"),
                                       ((4, 32, 14, 14), F32, 3, 0, "maxpool_backward_kernel<float, 1>"), ((64, 100, 56, 56), F32, 3, 1, "maxpool_backward_kernel<float, 4>"),
                                       ((64, 600, 27, 28), BF16, 2, 2, "maxpool_backward_kernel<uint16_t, 4>")):
        rc, name, _ = _pool_backward(pool, shape, dt, k, offset)
        assert rc == 0 and name == want, (shape, dt, k, offset, name)


@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("H,W", [(33, 64), (223, 224), (101, 96), (15, 32), (28, 28), (27, 40)])
def test_pooling_forward_of_odd_heights_streams(pool, dt, H, W):
    """k = 2: even heights of whole eight-element pieces, and odd ones of whole mask words."""
    assert pool.division_maxpool_forward(1 << 40, 4, 64, H, W, dt, 2, 1 << 41, 1 << 42, 1 << 40, None) == 0
    name = pool.check_pool_kernel(ctypes.byref(ctypes.c_uint32())).decode()
    assert name.startswith("(maxpool2_forward_fast<") == (W % (32 if H % 2 else 8) == 0)
    assert pool.division_maxpool_forward(1 << 40, 64, 160, H, W, dt, 2, 1 << 41, 1 << 42, 1 << 40, None) == 0
    name = pool.check_pool_kernel(ctypes.byref(ctypes.c_uint32())).decode()
    assert name.startswith("(maxpool2_forward_fast<") == (W % (32 if H % 2 else 8) == 0 and not (dt == F32 and H % 2 and W <= 128))


@pytest.mark.parametrize("shape,dt,B", [((306, 1, 1, 114), BF16, 2), ((832, 1, 1, 154), F32, 4), ((1940, 1, 1, 238), BF16, 8), ((297, 1, 104, 3), F32, 12), ((800, 2, 3, 37, 2), C16, 3),
                                        ((260, 1, 1, 4099), F32, 18), ((512, 1, 19, 19), F32, 12)])
def test_units_of_many_planes_have_lanes_for_a_machine_of_wavefronts(host, shape, dt, B):
    """Eight wavefronts per CU, or a lane for every unit of four elements."""
    planes, units = shape[0] * shape[1], (shape[-1] * shape[-2] * (shape[2] if len(shape) == 5 else 1) + 3) // 4
    (launch,) = _maps(host, [(shape, dt, B, 2)])
    name = (ctypes.c_char * 128)()
    host.division_kernel_name_3d.argtypes = [ctypes.c_int, ctypes.c_void_p] + [ctypes.c_int64] * 5 + [ctypes.c_int] * 3 + [ctypes.c_char_p, ctypes.c_size_t]
    assert host.division_kernel_name_3d(0, None, *_dims(shape), dt, B, 2, name, 128) == 0 and name.value.startswith(b"compress_units<")
    assert launch.gx * max(launch.waves, 1) >= min(8 * host.check_cus(), planes * units // 64), (launch.gx, launch.waves)
    # eight maps share the machine: no more lanes per plane than that takes, of the planes of all of them
    (eight,) = _maps(host, [(shape, dt, B, 2)] * 8)
    assert eight.gy == 8 and eight.waves <= launch.waves and eight.gx * max(eight.waves, 1) <= launch.gx * max(launch.waves, 1)
    lone = _maps(host, [((8 * shape[0],) + shape[1:], dt, B, 2)])[0]
    assert eight.waves == lone.waves


def test_calls_that_the_units_kernel_does_not_gain_keep_their_own(host):
    pk = (ctypes.c_char * 128)()
    host.division_kernel_name_3d.argtypes = [ctypes.c_int, ctypes.c_void_p] + [ctypes.c_int64] * 5 + [ctypes.c_int] * 3 + [ctypes.c_char_p, ctypes.c_size_t]
    for shape, dt, B, b, want in (((1746, 1, 1, 2032), BF16, 4, 1, "compress_tile<"), ((1048, 1, 1, 7196), F32, 4, 8, "compress_tile<"), ((5340, 1, 1, 663), BF16, 64, 2, "compress_rows<"),
                                  ((5340, 1, 1, 663), BF16, 64, 1, "compress_units<"), ((5340, 1, 1, 663), F32, 64, 2, "compress_units<"), ((3760, 1, 131, 1), F32, 2, 4, "compress_rows<"),
                                  ((3760, 1, 131, 1), F32, 2, 1, "compress_units<"), ((2516, 1, 37, 5), BF16, 2, 4, "compress_rows<"), ((2516, 1, 37, 5), BF16, 12, 4, "compress_units<"),
                                  ((308, 16, 134, 12), F32, 4, 4, "compress_wave<"), ((308, 16, 134, 12), F32, 8, 4, "compress_seg<"), ((308, 16, 42, 18), F32, 4, 4, "compress_seg<"),
                                  ((80, 16, 62, 20), F32, 4, 2, "compress_seg<")):
        assert host.division_kernel_name_3d(0, None, *_dims(shape), dt, B, b, pk, 128) == 0
        assert pk.value.decode().startswith(want), (shape, dt, B, b, pk.value)
    # few planes: lanes for all B slices of a block
    assert _maps(host, [((153, 1, 2, 7, 33), BF16, 8, 2)])[0].waves == 1


A, B_, C_ = (2, 16, 28, 28), (3, 8, 33, 17), (5, 7, 14, 14)


def test_maps_of_several_shapes_are_one_launch(host):
    (launch,) = _maps(host, [(A, F32, 8, 2), (B_, F32, 8, 2), (A, F32, 8, 2), (C_, F32, 64, 2), (C_, F32, 4, 2)], compress=False)
    assert (launch.what, launch.shapes, launch.maps) == (2, 4, 5)


def test_a_shape_alone_in_its_launch_has_its_own_kernel(host):
    """One shape of a type, or what is left when a launch is full: the kernel of the single-map call."""
    found = _maps(host, [(A, F32, 8, 2), (B_, BF16, 8, 2), (B_, BF16, 8, 2), (C_, C16, 8, 2)], compress=False)
    assert [(q.what, q.dt, q.gy) for q in found] == [(1, F32, 1), (1, BF16, 2), (1, C16, 1)]
    alone = _maps(host, [(B_, BF16, 8, 2)] * 2, compress=False)
    assert alone[0].kind == found[1].kind
    found = _maps(host, [((1, k + 1, 28, 28), F32, 8, 2) for k in range(17)], compress=False)
    assert [(q.what, q.shapes) for q in found] == [(2, 16), (1, 1)]


def _order(host, entries):
    return [q.out for q in _maps(host, entries, compress=False)]


def test_maps_that_share_memory_keep_the_order_of_their_descriptors(host):
    x, y = 1 << 46, 1 << 47
    size = 4 * 2 * 16 * 28 * 28
    # B = 2 has a launch of its own and would go first: the overlapping map A before it has to be written before
    own = (B_, F32, 2, 2)
    for at in (x, x + size - 4, x - 16):
        assert _order(host, [(A, F32, 8, 2, x), (*own, at), (C_, F32, 8, 2, y)]) == [x, at, y]
    assert len(_maps(host, [(A, F32, 8, 2, x), (*own, x + size), (C_, F32, 8, 2, y)], compress=False)) == 2        # side by side: mixed
    # a map rebuilt from a buffer that another map's output covers
    assert _order(host, [(A, F32, 8, 2, x), (C_, F32, 8, 2, y, x + 256), (B_, F32, 8, 2)]) == [x, y, 5 << 38]
    # two maps read one buffer: nothing is written there
    assert len(_maps(host, [(A, F32, 8, 2, x, 1 << 48), (C_, F32, 8, 2, y, 1 << 48)], compress=False)) == 1


def test_the_size_named_for_a_packed_buffer_does_not_decide_what_overlaps(host):
    """A capacity beyond the buffer's own bytes is no memory that the call reads; the largest ones would wrap around."""
    x, y = 1 << 46, 1 << 47
    for size in (1 << 49, (1 << 64) - 1):
        assert len(_maps(host, [(A, F32, 8, 2, x, None, size), (C_, F32, 8, 2, y, None, size)], compress=False)) == 1
        assert _order(host, [(A, F32, 8, 2, x, None, size), (C_, F32, 8, 2, y, x + 256, size), (B_, F32, 8, 2, None, None, size)]) == [x, y, 5 << 38]


def test_overlaps_of_random_ranges_are_those_of_every_pair(host):
    import random
    rng = random.Random(3)
    seen = set()
    for _ in range(400):
        entries, outs, ins = [], [], []
        for k in range(rng.randint(2, 6)):
            shape, B = rng.choice([(A, 8), (B_, 8), (C_, 4)])
            n = 4 * shape[0] * shape[1] * shape[2] * shape[3]
            need = host.division_packed_bytes_3d(*_dims(shape), B, 2, F32)
            o, p = (1 << 40) + 64 * rng.randint(0, 12000), (1 << 40) + 64 * rng.randint(0, 12000)
            entries.append((shape, F32, B, 2, o, p))
            outs.append((o, o + n, k))
            ins.append((p, p + need, k))
        if len({e[:4] for e in entries}) < 2:
            continue
        want = any(a[0] < b[1] and b[0] < a[1] for i, a in enumerate(outs) for b in outs[:i] + ins)
        mixed = any(q.what == 2 for q in _maps(host, entries, compress=False))
        assert mixed != want
        seen.add(want)
    assert seen == {True, False}


MIXED, LINES, PLANES = 14, 15, 16                     # the launches of several shapes


def test_small_maps_of_several_shapes_compress_in_one_launch(host):
    entries = [(A, F32, 8, 2), (B_, F32, 8, 2), (A, F32, 8, 2), (C_, F32, 64, 2), (C_, F32, 4, 2)]
    assert [q.kind for q in _maps(host, entries)] == [MIXED]
    # another type or code width, or a shape that is left alone: launches of their own
    kinds = [q.kind for q in _maps(host, entries + [(A, BF16, 8, 2), (A, F32, 8, 4)])]
    assert kinds[0] == MIXED and len(kinds) == 3 and MIXED not in kinds[1:]
    # a large map beside them keeps its kernel, and so does what its own kernel serves far better
    large = (64, 256, 56, 56)
    assert sorted(q.kind == MIXED for q in _maps(host, [(large, F32, 8, 2)] + entries)) == [False, True]
    assert all(q.kind != MIXED for q in _maps(host, [((22, 48, 1, 384), F32, 4, 8)] * 3 + [((2, 797, 1, 768), F32, 4, 8)]))
    # ten shapes: eight in a launch; one shape: none
    many = [q.kind for q in _maps(host, [((1, k + 1, 28, 28), F32, 8, 2) for k in range(10)])]
    assert many == [MIXED, MIXED]
    assert MIXED not in [q.kind for q in _maps(host, [(A, F32, 8, 2)] * 5)]


def test_maps_that_share_memory_are_compressed_in_their_order(host):
    """A packed buffer over another's input or output: a launch per shape, in the order of the descriptors."""
    x, p = 1 << 46, 1 << 47
    for out, packed in ((None, p + 64), (None, (1 << 38) + 256)):        # over the first map's packed buffer, over its input
        found = _maps(host, [(A, F32, 8, 2, None, p), (B_, F32, 8, 2, out, packed), (C_, F32, 8, 2)])
        assert len(found) == 3 and MIXED not in [q.kind for q in found]
    assert len(_maps(host, [(A, F32, 8, 2, None, p), (B_, F32, 8, 2, None, x), (C_, F32, 8, 2)])) == 1


def test_shapes_of_one_kernel_share_a_launch(host):
    rows = [((64, 3136, 1, 384), C16, 64, 2), ((64, 784, 1, 768), C16, 64, 2), ((64, 196, 1, 1536), C16, 64, 2)]
    assert [q.kind for q in _maps(host, rows)] == [LINES]
    # other instances (groups of planes per wavefront, another way to add a block) keep launches of their own
    kinds = [q.kind for q in _maps(host, rows + [((64, 3136, 1, 96), C16, 64, 2), ((64, 784, 1, 192), C16, 64, 2)])]
    assert sorted(k == LINES for k in kinds) == [False, False, True] and MIXED not in kinds
    planes = [((128, 64, 32, 32), F32, 4, 2), ((128, 128, 16, 16), F32, 4, 2), ((128, 256, 8, 8), F32, 4, 2), ((128, 512, 4, 4), F32, 4, 2)]
    (launch,) = _maps(host, [m for m in planes for _ in range(4)])
    alone = [_maps(host, [m] * 4)[0] for m in planes]
    assert launch.kind == PLANES and launch.gx == sum(q.gx * q.gy for q in alone) and launch.gy == 1
    # types, code widths and the kernels of other shapes do not share it
    kinds = [q.kind for q in _maps(host, [planes[0], planes[1], ((128, 64, 32, 32), BF16, 4, 2), ((128, 64, 32, 32), F32, 4, 4), ((64, 256, 56, 56), F32, 8, 2)])]
    assert sorted(k == PLANES for k in kinds) == [False, False, False, True]
    # rows of odd width, items under B = 8 and lanes share it up to 64 workgroups per CU; beyond, those have launches of their own
    few = [((8, 64, 28, 28), F32, 8, 2), ((8, 256, 55, 55), F32, 8, 2), ((8, 512, 13, 13), F32, 8, 2), ((8, 960, 7, 7), F32, 8, 2), ((8, 512, 24, 24), F32, 8, 2)]
    (launch,) = _maps(host, few)
    assert launch.kind == PLANES and launch.gx == sum(q.gx * q.gy for q in (_maps(host, [m])[0] for m in few))
    kinds = [q.kind for q in _maps(host, [((64, 256, 55, 55), F32, 8, 2), planes[0], planes[1]])]
    assert len(kinds) == 2 and kinds.count(PLANES) == 1
    kinds = [q.kind for q in _maps(host, [((256, 256, 55, 55), F32, 8, 2), ((256, 512, 13, 13), F32, 8, 2), planes[0]])]
    assert len(kinds) == 3 and PLANES not in kinds
    # 25 maps are two launches, and maps over one another's memory a launch for each shape
    assert [q.kind for q in _maps(host, [planes[2]] * 13 + [planes[3]] * 12)].count(PLANES) == 0
    assert [q.kind for q in _maps(host, [planes[2]] * 12 + [planes[3]] * 12 + [planes[1]])].count(PLANES) == 1
    x = 1 << 46
    assert PLANES not in [q.kind for q in _maps(host, [(*planes[2], None, x), (*planes[3], None, x + 256), planes[1]])]


def test_the_launches_whose_planes_are_tested_for_not_a_number(host):
    """What test_shared_launches_keep_planes_apart of the kernel tests sends where."""
    for kinds, specs in (([MIXED], [((1, 40, 14, 14), 8), ((1, 41, 9, 13), 4), ((3, 14, 1, 96), 64), ((2, 21, 5, 5), 64), ((1, 39, 33, 17), 18), ((1, 15, 40, 44), 8)]),
                         ([LINES], [((1, 2101, 1, 384), 8), ((7, 301, 1, 768), 8)]), ([LINES], [((1, 2101, 1, 384), 64), ((1, 1201, 1, 768), 64)]),
                         ([PLANES], [((1, 2057, 32, 32), 4), ((1, 8209, 8, 8), 4)]),
                         ([PLANES], [((1, 8209, 13, 13), 8), ((1, 1031, 35, 35), 8), ((1, 8211, 14, 14), 8), ((3, 5741, 7, 7), 8), ((3, 2741, 10, 12), 8)])):
        assert [q.kind for q in _maps(host, [(s, F32, B, 2) for s, B in specs])] == kinds, specs


def test_chunk_kernels_of_few_planes_leave_their_launch(host):
    """One shape by itself: planes that would be a few workgroups' chain in the chunk kernels."""
    for shape, dt, B, b in (((2, 3, 64, 64), F32, 8, 1), ((1, 2, 8, 53, 53), F32, 64, 1), ((30, 1, 1, 3413), BF16, 8, 4), ((2, 20, 30, 30), F32, 4, 2), ((5, 33, 24, 24), F32, 18, 4)):
        assert [q.kind for q in _maps(host, [(shape, dt, B, b)] * 2)] == [MIXED], shape
    for shape, dt, B, b in (((64, 600, 30, 30), F32, 4, 2), ((4, 4, 147, 147), F32, 18, 2), ((2, 3, 56, 56), F32, 8, 2), ((1, 1, 300, 300), F32, 18, 2)):
        assert MIXED not in [q.kind for q in _maps(host, [(shape, dt, B, b)] * 2)], shape
    # over one another's memory: in their order, each by itself
    x = 1 << 46
    found = _maps(host, [((2, 3, 64, 64), F32, 8, 1, None, x), ((2, 20, 30, 30), F32, 4, 1, None, x + 64), ((2, 3, 56, 56), F32, 8, 1)])
    assert [q.kind == MIXED for q in found] == [True, True, False]


def test_chunk_kernels_of_one_shape_over_one_another_keep_launches_of_eight(host):
    """Nine maps of a shape and more, two of them eight or more descriptors apart over the same memory: the later one is compressed last."""
    shape, x, p = (2, 3, 64, 64), 1 << 46, 1 << 47
    apart = [(shape, F32, 8, 1)] * 16
    assert [(q.kind == MIXED, q.maps) for q in _maps(host, apart)] == [(True, 1)]
    for first, last in (((None, p), (None, p)), ((None, p), (None, p + 64)), ((None, x), (None, (2 * 0 + 1) << 38))):
        for others in ([], [(A, F32, 8, 2), (C_, F32, 64, 2)]):
            entries = [(shape, F32, 8, 1, *first)] + [(shape, F32, 8, 1)] * 14 + [(shape, F32, 8, 1, *last)] + others
            found = _maps(host, entries)
            assert [(q.kind == MIXED, q.gy) for q in found[:2]] == [(False, 8), (False, 8)], (first, last, [(q.kind, q.gy) for q in found])
    # eight of them never had an order among themselves
    assert [q.kind == MIXED for q in _maps(host, [(shape, F32, 8, 1, None, p)] * 8)] == [True]


@pytest.mark.parametrize("shape,B,dt,kind,most", [((1, 300, 27, 27), 8, BF16, 6, 8), ((1, 50, 73, 73), 8, BF16, 6, 2), ((1, 30, 103, 103), 8, BF16, 6, 1), ((1, 40, 147, 147), 8, BF16, 6, 1),
                                                  ((1, 1216, 14, 14), 8, F32, 3, 1), ((1, 600, 30, 30), 8, BF16, 3, 1), ((1, 2432, 14, 14), 8, C16, 3, 1)])
def test_decompression_shares_planes_by_all_maps_of_the_launch(host, shape, B, dt, kind, most):
    """decompress_units (6) and decompress_table (3): few planes are shared among more workgroups until a launch has `most` per CU, however many maps hold them."""
    planes, found = shape[0] * shape[1], []
    for maps in range(1, 9):
        (launch,) = _maps(host, [(shape, dt, B, 2)] * maps, compress=False)
        assert (launch.kind, launch.gy) == (kind, maps)
        found.append(launch.gx)
        assert kind != 6 or launch.gx == planes or launch.gx * maps <= most * host.check_cus()
    assert found == sorted(found, reverse=True) and found[0] > found[-1]
    if kind == 3:                                           # a workgroup per CU, or what each would be by itself in a launch of eight times the planes
        big = (8 * shape[0],) + shape[1:]
        assert found[-1] * 8 <= max(2 * host.check_cus() + 8, _maps(host, [(big, dt, B, 2)], compress=False)[0].gx + 8)


@pytest.mark.parametrize("maps", [1, 3, 8, 9, 25])
def test_a_shape_by_itself_is_launched_as_a_batch_of_it(host, maps):
    """division_compress_maps launches the plan that it has made to decide; division_compress_batch makes its own: the same launches, the same maps."""
    host.division_compress_batch.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 3 + [ctypes.c_int64] * 4 + [ctypes.c_int] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    for shape, dt, B, b in (((64, 256, 56, 56), F32, 8, 2), ((2, 3, 1, 3136), F32, 8, 2), ((2, 16, 28, 28), F32, 8, 2), ((3, 8, 33, 17), BF16, 8, 4), ((64, 768, 17, 17), F32, 8, 2),
                            ((2, 2, 1, 768), BF16, 8, 4), ((64, 2048, 7, 7), C16, 8, 2), ((8, 512, 24, 24), F32, 8, 1), ((64, 600, 30, 30), F32, 4, 2), ((64, 64, 147, 147), F32, 8, 2),
                            ((64, 256, 56, 56), BF16, 64, 2), ((1, 1, 300, 300), F32, 18, 2), ((64, 16, 224, 224), F32, 8, 2)):
        mine = [(q.kind, q.dt, q.waves, q.gx, q.gy, q.walked) for q in _maps(host, [(shape, dt, B, b)] * maps)]
        x = (ctypes.c_void_p * maps)(*[(2 * i + 1) << 38 for i in range(maps)])
        packed = (ctypes.c_void_p * maps)(*[((2 * i + 1) << 38) + (1 << 37) for i in range(maps)])
        seeds = (ctypes.c_uint64 * maps)()
        assert host.division_compress_batch(maps, x, packed, seeds, *shape, dt, B, b, 1 << 40, None) == 0
        assert mine == [(q.kind, q.dt, q.waves, q.gx, q.gy, q.walked) for q in _launches(host)], shape


@pytest.mark.parametrize("es", [2, 4])
def test_rounds_of_odd_rows_read_no_dword_beyond_the_map(host, es):
    """compress_rowstrip loads whole dwords: aligned ones, all that hold an element of the round, none behind the map's last (bfloat16 rounds that start in
    the middle of a dword would otherwise end two bytes behind a map that ends with a page)."""
    host.check_round_span.argtypes = [ctypes.c_uint32] * 4 + [ctypes.POINTER(ctypes.c_uint32)]
    host.check_round_span.restype = ctypes.c_uint32
    n = ctypes.c_uint32()
    for G in (1, 2, 3, 4):
        for HW in (2 * 13, 13 * 13, 17 * 17, 35 * 35, 36 * 55, 55 * 55):
            for P in range(1, 26):
                for p0 in range(0, P, G):
                    planes = min(G, P - p0)
                    begin = (p0 * HW - host.check_round_span(p0, planes, HW, es, ctypes.byref(n))) * es
                    assert begin % 4 == 0 and n.value % 4 == 0
                    assert begin <= p0 * HW * es < begin + 4 and (p0 + planes) * HW * es <= begin + n.value <= (P * HW * es + 3) // 4 * 4
