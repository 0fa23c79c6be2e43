"""Small maps at the edges of the kernels' tiles (remainders, halves of vectors, first and last planes), bit for bit
against the CPU oracle: packed buffers and rebuilt maps are whole numbers and single IEEE operations, so equal."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2208_04187_amd as pkg

pytestmark = pytest.mark.gpu

FORMATS = {"f32": (torch.float32, False, oracle.F32), "bf16": (torch.bfloat16, False, oracle.BF16),
           "c16": (torch.float32, True, oracle.F32_C16)}


def _host(t):
    """numpy form of a tensor: float32 as it is, bfloat16 as its 16-bit patterns"""
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def _names(shape, B, b, mode, out_ptr=0):
    """Kernel instances that compress and rebuild the map"""
    dtype, c16, _ = FORMATS[mode]
    kn = pkg.division_kernel_name_3d if len(shape) == 5 else pkg.division_kernel_name
    return kn(0, shape, B, b, dtype, c16=c16), kn(1, shape, B, b, dtype, data_ptr=out_ptr, c16=c16)


def _round_trip(shape, B, b, mode, seed=7, offset=0, relu=False, x=None):
    """Compress and rebuild a map (x, or normal values) whose rebuilt copy starts `offset` elements into its buffer."""
    dtype, c16, dt = FORMATS[mode]
    three = len(shape) == 5
    gen = torch.Generator().manual_seed(seed * 1000 + B * 10 + b)
    if x is None:
        x = torch.randn(shape, generator=gen)
    x = (x.relu() if relu else x).to(dtype)
    xh = _host(x)
    comp = pkg.division_compress_3d if three else pkg.division_compress
    dec = pkg.division_decompress_3d if three else pkg.division_decompress
    nbytes = (pkg.division_packed_bytes_3d if three else pkg.division_packed_bytes)(*shape, B, b, dtype, c16)
    packed = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda:0")
    comp(x.to("cuda:0"), B, b, seed, packed=packed, c16=c16)
    ref = oracle.compress(xh, B, b, seed, dt)
    torch.cuda.synchronize()
    assert np.array_equal(packed.cpu().numpy(), ref), "packed buffer"
    guard = 16
    buf = torch.full((offset + x.numel() + guard,), -1.0, dtype=dtype, device="cuda:0")
    dec(packed, shape, B, b, dtype, out=buf[offset:offset + x.numel()].view(shape), c16=c16)
    torch.cuda.synchronize()
    want = oracle.decompress(ref, shape, B, b, dt)
    got = _host(buf[offset:offset + x.numel()].cpu()).reshape(shape)
    assert np.array_equal(np.asarray(got).view(np.uint8), np.asarray(want).reshape(shape).view(np.uint8)), "rebuilt map"
    assert bool((buf[:offset] == -1).all()) and bool((buf[offset + x.numel():] == -1).all()), "written outside the map"


@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("shape,B,offset", [
    ((3, 5, 1, 8), 8, 0),                # a plane is one vector
    ((1, 1, 1, 4), 4, 0),                # half a vector in all
    ((3, 7, 5, 28), 8, 0),               # rows of 3.5 vectors: a vector spans two rows and two planes
    ((3, 7, 5, 12), 4, 0),
    ((5, 3, 6, 24), 12, 0),              # whole rows, blocks of a vector and a half
    ((2, 3, 16, 40), 8, 0),
    ((2, 3, 16, 40), 8, 4),              # the rebuilt map starts in the middle of a vector
    ((1, 1, 7, 1024), 64, 0),
    ((9, 57, 1, 264), 8, 0),             # chunk ends inside a plane
    ((2, 3, 3, 9, 16), 8, 0),
    ((2, 3, 3, 5, 20), 4, 0),
])
def test_two_byte_rows_of_whole_pieces(shape, B, b, offset):
    assert _names(shape, B, b, "bf16", 256 + 2 * offset)[1].startswith("decompress_rowvec<" if offset else "decompress_stream")
    _round_trip(shape, B, b, "bf16", offset=offset)


@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("shape,B,lu4,lu2", [
    # shape, B, how a block is summed in 4-byte and 2-byte maps: log2 of its vectors (DPP), through LDS (-1), two rounds of it (-2)
    ((3, 5, 1, 96), 64, -2, -1),         # a block of two rounds, the last one short; rounds past the plane
    ((1, 1, 1, 96), 64, -2, -1),         # a single plane: the other groups lie past the map
    ((7, 11, 1, 160), 128, -2, -2),
    ((5, 9, 1, 192), 64, -2, -1), ((3, 67, 1, 232), 64, -1, -1), ((2, 3, 1, 776), 64, -1, -1), ((2, 3, 1, 1536), 128, -1, -1),
    ((1, 3, 1, 1544), 256, -2, -2),      # a block is a whole wavefront of vectors, the last one two vectors
    ((3, 5, 1, 104), 32, -1, 2), ((2, 9, 1, 1000), 32, -1, 2),
    ((5, 7, 1, 72), 8, 1, 0), ((2, 3, 1, 2056), 8, None, 0), ((2, 3, 1, 1032), 16, 2, 1),      # (4-byte planes of 514 vectors: compress_regs)
    ((5, 7, 1, 72), 4, 0, None), ((3, 5, 1, 2040), 4, 0, None), ((3, 5, 1, 2040), 16, 2, 1),
])
def test_rows_of_power_of_two_blocks(shape, B, lu4, lu2, b, mode):
    name, lu = _names(shape, B, b, mode)[0], lu2 if mode == "bf16" else lu4
    assert name.startswith("compress_line<") and name.endswith(", %d>" % lu) if lu is not None else not name.startswith("compress_line<"), name
    _round_trip(shape, B, b, mode)


@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("shape,B", [
    ((1, 3, 1, 768), 8), ((1, 3, 1, 768), 4), ((1, 3, 1, 768), 16),         # every round whole
    ((2, 3, 1, 200), 8), ((2, 3, 1, 72), 8), ((2, 3, 1, 24), 4), ((1, 2, 1, 1032), 16),      # the last round partly past the plane
    ((1, 3, 1, 96), 64), ((1, 2, 1, 160), 128),                             # block sums through LDS
    ((1, 2, 29, 29), 8), ((1, 2, 17, 17), 8), ((1, 2, 56, 56), 8),
    ((2, 3, 1, 3136), 8), ((2, 3, 1, 3136), 4), ((1, 3, 1, 2052), 8),       # one row in the register kernel: a block's units are added from +0 too
])
def test_tiny_negative_sum_has_mean_minus_zero(shape, B, mode):
    """A sum of one smallest negative number: its mean underflows to -0, which is kept; only a block of -0 has mean +0."""
    tiny = -(2.0 ** -133 if mode == "bf16" else 2.0 ** -149)
    x = torch.zeros(shape)
    x.view(-1)[::B] = tiny                        # at most one in the blocks of a one-row map
    x[0, 1] = -x[0, 1].abs()                      # the same beside -0,
    x[0, 1, :B, :B] = -0.0                        # and a block of -0 alone
    _round_trip(shape, B, 2, mode, x=x)


@pytest.mark.parametrize("mode", ["f32", "c16"])
@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("shape,B,items", [
    # shape, B, items of sixteen elements per lane (0: another kernel takes the planes)
    ((1, 1, 17, 17), 8, 0), ((41, 101, 17, 17), 8, 0),    # a row per lane: one plane; several planes per workgroup, the last one short
    ((3, 7, 13, 13), 4, 0), ((5, 5, 9, 13), 8, 0), ((2, 3, 35, 35), 8, 0), ((29, 67, 35, 35), 4, 0), ((1, 3, 64, 55), 8, 0), ((2, 2, 2, 17), 4, 0),
    ((2, 3, 19, 19), 8, 0), ((3, 2, 21, 23), 4, 0), ((2, 3, 57, 41), 4, 0), ((1, 1, 163, 163), 8, 0),         # too few slots filled, too many items
    ((2, 2, 300, 5), 8, 0), ((1, 2, 200, 3), 4, 0), ((2, 2, 9, 250), 4, 0), ((3, 5, 9, 14, 14), 8, 0), ((2, 2, 3, 22, 30), 8, 0), ((1, 3, 2, 30, 35), 4, 0),
    ((2, 2, 3, 15, 21), 8, 0),                            # an odd number of elements per slice
    ((3, 5, 29, 29), 8, 1), ((3, 5, 29, 29), 4, 1), ((1, 1, 29, 29), 8, 1), ((2, 1, 3, 1001), 8, 1), ((2, 2, 100, 37), 8, 1),   # (29: 28 rows and one)
    ((2, 3, 4, 14, 14), 8, 1), ((1, 2, 5, 16, 9), 4, 1), ((5, 41, 4, 14, 14), 4, 1),
    ((3, 3, 40, 33), 8, 2), ((1, 2, 73, 73), 8, 2), ((1, 2, 101, 97), 8, 2), ((1, 1, 128, 111), 4, 2), ((1, 2, 147, 147), 8, 2),
    ((1, 2, 127, 129), 8, 2), ((3, 5, 28, 45), 8, 2), ((1, 2, 1000, 5), 4, 2), ((2, 2, 8, 18, 26), 8, 2), ((1, 2, 4, 30, 34), 8, 2), ((1, 2, 6, 22, 35), 8, 2),
])
def test_items_of_sixteen_elements(shape, B, items, b, mode):
    name = _names(shape, B, b, mode)[0]
    if b == 1 and shape[2:] == (147, 147):
        items = 0                                         # (no 1-bit instance of sixteen wavefronts in the kernel asked first)
    assert name.startswith("compress_seg<") and name.endswith(", %d>" % items) if items else not name.startswith("compress_seg<"), name
    _round_trip(shape, B, b, mode, relu=b == 2)


@pytest.mark.parametrize("mode", ["f32", "c16"])
@pytest.mark.parametrize("shape,B", [
    ((4, 6, 29, 29), 8), ((4, 6, 29, 29), 4), ((4, 6, 4, 14, 14), 8), ((4, 6, 5, 16, 9), 4),       # an item of sixteen elements per lane
    ((4, 6, 37, 37), 8), ((4, 6, 40, 33), 8), ((4, 6, 73, 73), 8), ((4, 6, 147, 147), 8), ((4, 6, 147, 147), 4),   # two items
    ((4, 6, 127, 127), 8), ((4, 6, 101, 97), 8), ((4, 6, 8, 18, 26), 8), ((4, 6, 4, 30, 34), 8), ((4, 6, 6, 22, 35), 8),
    ((4, 6, 9, 14, 14), 8), ((4, 6, 5, 22, 22), 4),                                                                 # other kernels
    ((4, 6, 56, 56), 8), ((4, 6, 28, 28), 8), ((4, 6, 17, 17), 8), ((4, 6, 57, 57), 18), ((4, 6, 1, 768), 8), ((4, 6, 1, 96), 64),
])
def test_a_value_that_is_not_finite_stays_in_its_block(shape, B, mode):
    """One NaN or infinity per plane, in the first and last columns and rows among other places: the codes of such a
    plane are unspecified, the means of its other blocks are not."""
    dtype, c16, dt = FORMATS[mode]
    three = len(shape) == 5
    dims = (1,) * (5 - len(shape)) + shape[2:]
    planes, rng = shape[0] * shape[1], np.random.default_rng(sum(shape) + B)
    x = torch.randn(shape, generator=torch.Generator().manual_seed(B))
    flat = x.view((planes,) + dims)
    hit, low = [], [-(-d // B) for d in dims]
    for p in range(planes):
        at = [int(rng.choice([0, d - 1, rng.integers(0, d), min(d - 1, 4 * int(rng.integers(0, d // 4 + 1)))])) for d in dims]
        at[2] = 0 if p % 2 == 0 else at[2]                       # what the last column's loads run into
        flat[(p, *at)] = (float("nan"), float("inf"), -float("inf"))[p % 3]
        hit.append(((at[0] // B) * low[1] + at[1] // B) * low[2] + at[2] // B)
    comp, dec = (pkg.division_compress_3d, pkg.division_decompress_3d) if three else (pkg.division_compress, pkg.division_decompress)
    packed = comp(x.to("cuda:0"), B, 2, 3, c16=c16)
    back = dec(packed, shape, B, 2, dtype, c16=c16)
    torch.cuda.synchronize()
    lay = (pkg.division_packed_layout_3d if three else pkg.division_packed_layout)(*shape, B, 2, dtype, c16)
    view = np.uint16 if c16 else np.uint32

    def means(buf):
        return np.ascontiguousarray(buf[lay["lfc_off"]:lay["lfc_off"] + lay["lfc_bytes"]]).view(view).reshape(planes, -1)

    got, want = means(packed.cpu().numpy()), means(oracle.compress(x.numpy(), B, 2, 3, dt))
    exponent = 0x7F80 if c16 else 0x7F800000
    finite_got, finite_want = (got & exponent) != exponent, (want & exponent) != exponent
    assert np.array_equal(np.nonzero(~finite_want)[1], np.array(hit))                      # one mean per plane
    assert np.array_equal(finite_got, finite_want), np.argwhere(finite_got != finite_want)[:8]
    assert np.array_equal(got[finite_want], want[finite_want])
    nan = back.cpu().view((planes,) + dims)[0::3].isnan()                                 # planes that hold a NaN
    for i, m in enumerate(nan):
        b0 = [v // B * B for v in np.argwhere(m.numpy())[0]]
        assert not bool(m.sum() > m[b0[0]:b0[0] + B, b0[1]:b0[1] + B, b0[2]:b0[2] + B].sum()), "the block's neighbours came back as NaN"


# ---------------------------------------------------------------- maps of several shapes in one launch

# rows of whole vectors (2-D, 3-D, 2-byte rows of half vectors), any width (2-D, 3-D; an odd number of elements; planes ending inside
# vectors), one-block planes, and shapes that keep a launch of their own (rows or blocks below four)
MIXED = [((2, 3, 28, 28), 8), ((3, 5, 14, 14), 8), ((5, 7, 7, 7), 8), ((1, 3, 55, 55), 8), ((2, 3, 12, 20), 12), ((1, 1, 13, 13), 8),
         ((2, 3, 3, 9, 11), 4), ((2, 2, 4, 8, 8), 4), ((3, 3, 9, 3), 4), ((2, 2, 8, 8), 2), ((1, 5, 17, 9), 64), ((1, 7, 1, 197), 8),
         ((2, 1, 1, 4100), 64), ((3, 1, 33, 65), 18), ((1, 2, 3, 35, 35), 8), ((4, 3, 5, 7), 4), ((2, 5, 9, 28), 4), ((2, 67, 2, 2), 8)]


@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("b", [1, 2, 4, 8])
def test_decompress_of_several_shapes_in_one_call(mode, b):
    dtype, c16, dt = FORMATS[mode]
    gen = torch.Generator().manual_seed(b)
    specs = [s for k, s in enumerate(MIXED) for _ in range(1 + (k * 7 + b) % 4)]         # more maps and shapes than a launch holds
    xs = [(torch.randn(s, generator=gen) * 1.5).to(dtype) for s, _ in specs]
    Bs, bs = [B for _, B in specs], [b] * len(specs)
    ref = [oracle.compress(_host(x), B, b, 50 + k, dt) for k, (x, B) in enumerate(zip(xs, Bs))]
    packed = [torch.from_numpy(r).to("cuda:0") for r in ref]
    bufs = [torch.full((x.numel() + 16,), -7.0, dtype=dtype, device="cuda:0") for x in xs]
    out = [v[:x.numel()].view(x.shape) for v, x in zip(bufs, xs)]
    pkg.division_decompress_maps(packed, [s for s, _ in specs], Bs, bs, dtype, out=out, c16=c16)
    torch.cuda.synchronize()
    for (shape, B), x, r, v in zip(specs, xs, ref, bufs):
        want = np.asarray(oracle.decompress(r, shape, B, b, dt)).reshape(-1)
        got = _host(v.cpu())
        assert np.array_equal(got[:x.numel()].view(np.uint8), want.view(np.uint8)), (shape, B)
        assert bool((v[x.numel():] == -7.0).all()), (shape, B)


# maps of several shapes compressed in one launch: one to eight units per lane, planes of less than a unit, several planes per workgroup and
# the last one short, blocks of one to many lanes, rows and blocks of one and two elements, planes that start in the middle of a dword
SMALL = [((2, 3, 28, 28), 8), ((3, 5, 14, 14), 8), ((5, 7, 7, 7), 8), ((1, 3, 55, 55), 8), ((2, 3, 12, 20), 12), ((1, 1, 13, 13), 8), ((2, 3, 3, 9, 11), 4),
         ((2, 2, 4, 8, 8), 4), ((3, 3, 9, 3), 4), ((2, 2, 8, 8), 2), ((1, 5, 17, 9), 64), ((1, 7, 1, 197), 8), ((2, 1, 1, 4100), 64), ((3, 1, 33, 65), 18),
         ((1, 2, 3, 35, 35), 8), ((4, 3, 5, 2), 4), ((2, 5, 9, 1), 4), ((2, 67, 2, 2), 8), ((3, 3, 1, 1), 8), ((1, 1, 1, 3), 1), ((7, 3, 1, 5), 3),
         ((1, 2, 147, 147), 8), ((1, 1, 180, 180), 64), ((1, 1, 16, 44, 45), 64), ((2, 1, 1, 3136), 4), ((1, 300, 4, 4), 4), ((2, 31, 6, 7), 1)]


@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("b", [1, 2, 4, 8])
def test_compress_of_several_shapes_in_one_call(mode, b):
    dtype, c16, dt = FORMATS[mode]
    gen = torch.Generator().manual_seed(b)
    for first in range(0, len(SMALL), 9):
        specs = [s for k, s in enumerate(SMALL[first:first + 9]) for _ in range(1 + (k * 5 + b) % 3)]
        xs = [(torch.randn(s, generator=gen) * 1.5).relu_().to(dtype) if k % 2 else (torch.randn(s, generator=gen) - 0.5).to(dtype) for k, (s, _) in enumerate(specs)]
        # every third map starts at an odd element of its memory
        on = []
        for k, x in enumerate(xs):
            area = torch.zeros(x.numel() + 8, dtype=dtype, device="cuda:0")
            at = 1 if k % 3 == 2 else 0
            area[at:at + x.numel()] = x.reshape(-1).to("cuda:0")
            on.append(area[at:at + x.numel()].view(x.shape))
        ref = [oracle.compress(_host(x), B, b, (7 << 32) + k, dt, threads=16) for k, (x, (_, B)) in enumerate(zip(xs, specs))]
        out = [torch.full((r.size + 16,), 0xA5, dtype=torch.uint8, device="cuda:0") for r in ref]
        pkg.division_compress_maps(on, [B for _, B in specs], b, [(7 << 32) + k for k in range(len(specs))], packed=[p[:r.size] for p, r in zip(out, ref)], c16=c16)
        torch.cuda.synchronize()
        for (shape, B), r, p in zip(specs, ref, out):
            got = p.cpu().numpy()
            assert np.array_equal(got[:r.size], r), (shape, B)
            assert bool((got[r.size:] == 0xA5).all()), (shape, B)


# values at the edges of binary32 and planes of nothing but zeros of either sign, in a launch of several shapes
@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
def test_compress_of_several_shapes_special_planes(mode):
    dtype, c16, dt = FORMATS[mode]
    shapes = [((1, 9, 14, 14), 8), ((1, 9, 9, 13), 4), ((1, 9, 3, 7, 7), 8), ((1, 9, 1, 96), 64), ((1, 9, 5, 5), 64)]
    xs = []
    for s, _ in shapes:
        x = torch.randn(s, generator=torch.Generator().manual_seed(3))
        f = x.view(9, -1)
        f[0], f[1], f[2], f[3] = 0.0, -0.0, 2.5, torch.where(torch.arange(f.shape[1]) % 2 == 0, 0.0, -0.0)
        f[4] *= 2.0 ** -140
        f[5] *= 2.0 ** -91
        f[6, 3] = 1e30
        f[7] = -(2.0 ** -133 if mode == "bf16" else 2.0 ** -149) * (torch.arange(f.shape[1]) % 8 == 0)
        xs.append(x.to(dtype))
    ref = [oracle.compress(_host(x), B, 2, 5, dt) for x, (_, B) in zip(xs, shapes)]
    packed = pkg.division_compress_maps([x.to("cuda:0") for x in xs], [B for _, B in shapes], 2, [5] * len(shapes), c16=c16)
    torch.cuda.synchronize()
    for s, r, p in zip(shapes, ref, packed):
        assert np.array_equal(p.cpu().numpy(), r), s


# the launches of several shapes (small maps; rows of one instance of compress_line; planes of few registers; all small planes), on planes at the edges of
# binary32 with planes of NaN and of infinities among them: those are unspecified, every other plane is what the oracle makes of it
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 1), ("bf16", 4), ("c16", 2), ("c16", 8)])
@pytest.mark.parametrize("specs", [
    [((1, 40, 14, 14), 8), ((1, 41, 9, 13), 4), ((3, 14, 1, 96), 64), ((2, 21, 5, 5), 64), ((1, 39, 33, 17), 18), ((1, 15, 40, 44), 8)],
    [((1, 2101, 1, 384), 8), ((7, 301, 1, 768), 8)], [((1, 2101, 1, 384), 64), ((1, 1201, 1, 768), 64)],
    [((1, 2057, 32, 32), 4), ((1, 8209, 8, 8), 4)],
    [((1, 8209, 13, 13), 8), ((1, 1031, 35, 35), 8), ((1, 8211, 14, 14), 8), ((3, 5741, 7, 7), 8), ((3, 2741, 10, 12), 8)],
])
def test_shared_launches_keep_planes_apart(specs, mode, b):
    from tests.test_gpu_parity import _special_planes
    dtype, c16, dt = FORMATS[mode]
    xs, bad = [], []
    for k, (s, _) in enumerate(specs):
        x = _special_planes(s, 5 + k).to(dtype)
        planes = s[0] * s[1]
        hit = [1, planes // 2, planes - 1]
        f = x.view(planes, -1)
        sign = torch.where(torch.arange(f.shape[1]) % 3 == 0, 1.0, -1.0).to(dtype)
        f[hit[0]], f[hit[1]], f[hit[2], ::5] = float("nan"), float("inf") * sign, float("nan")
        xs.append(x)
        bad.append(hit)
    packed = pkg.division_compress_maps([x.to("cuda:0") for x in xs], [B for _, B in specs], b, [11] * len(specs), c16=c16)
    torch.cuda.synchronize()
    for (s, B), x, hit, p in zip(specs, xs, bad, packed):
        planes = s[0] * s[1]
        got, want = oracle.split_packed(p.cpu().numpy(), s, B, b, dt), oracle.split_packed(oracle.compress(_host(x), B, b, 11, dt, threads=16), s, B, b, dt)
        good = np.setdiff1d(np.arange(planes), hit)
        for part in ("codes", "meta", "lfc"):
            g, w = np.ascontiguousarray(got[part]).reshape(planes, -1), np.ascontiguousarray(want[part]).reshape(planes, -1)
            assert np.array_equal(g[good].view(np.uint8), w[good].view(np.uint8)), (s, B, part)


def test_decompress_of_maps_that_share_memory_keeps_their_order():
    # the second map is rebuilt over the first one
    gen = torch.Generator().manual_seed(1)
    shapes = [((2, 3, 28, 28), 8), ((2, 3, 14, 14), 8), ((1, 2, 8, 8), 8)]
    ref = [oracle.compress(torch.randn(s, generator=gen).numpy(), B, 2, 9, oracle.F32) for s, B in shapes]
    area = torch.zeros(2 * 3 * 28 * 28, device="cuda:0")
    last = torch.zeros(128, device="cuda:0")
    pk = [torch.from_numpy(r).to("cuda:0") for r in ref]
    outs = [area.view(2, 3, 28, 28), area[:1176].view(2, 3, 14, 14), last.view(1, 2, 8, 8)]
    for _ in range(3):
        area.zero_()
        pkg.division_decompress_maps(pk, [s for s, _ in shapes], [B for _, B in shapes], 2, out=outs)
        torch.cuda.synchronize()
        want = np.asarray(oracle.decompress(ref[0], shapes[0][0], 8, 2, oracle.F32)).reshape(-1).copy()
        want[:1176] = np.asarray(oracle.decompress(ref[1], shapes[1][0], 8, 2, oracle.F32)).reshape(-1)
        assert np.array_equal(area.cpu().numpy(), want)
        assert np.array_equal(last.cpu().numpy(), np.asarray(oracle.decompress(ref[2], shapes[2][0], 8, 2, oracle.F32)).reshape(-1))


# a map whose kernel has a launch of its own (B = 2) after one that waits for a launch of several shapes, over the same memory
def test_decompress_of_a_map_with_a_launch_of_its_own_over_another_keeps_their_order():
    shapes = [((2, 3, 28, 28), 8), ((2, 3, 15, 11), 2), ((1, 5, 14, 14), 8)]
    gen = torch.Generator().manual_seed(9)
    xs = [torch.randn(s, generator=gen) for s, _ in shapes]
    ref = [oracle.compress(x.numpy(), B, 2, 5, oracle.F32) for x, (_, B) in zip(xs, shapes)]
    back = [np.asarray(oracle.decompress(r, s, B, 2, oracle.F32)).reshape(-1) for r, (s, B) in zip(ref, shapes)]
    packed = [torch.from_numpy(r).to("cuda:0") for r in ref]
    area, last = torch.zeros(4704, device="cuda:0"), torch.zeros(980, device="cuda:0")
    pkg.division_decompress_maps(packed, [s for s, _ in shapes], [B for _, B in shapes], 2, out=[area.view(shapes[0][0]), area[1000:1990].view(shapes[1][0]), last.view(shapes[2][0])])
    torch.cuda.synchronize()
    want = back[0].copy()
    want[1000:1990] = back[1]
    assert np.array_equal(area.cpu().numpy(), want) and np.array_equal(last.cpu().numpy(), back[2])


# planes of sixteen wavefronts: eight maps of 37 planes, more than there are workgroups, so that a workgroup takes several planes
# (some one more than others) and loads the next one's units as the codes of the present one leave
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 8), ("bf16", 4), ("bf16", 1), ("c16", 2)])
@pytest.mark.parametrize("shape,B", [((1, 37, 116, 116), 8), ((37, 1, 60, 240), 4), ((37, 1, 4, 60, 60), 8), ((1, 37, 8, 60, 100), 8)])
def test_sixteen_wavefronts_over_several_planes(shape, B, mode, b):
    dtype, c16, dt = FORMATS[mode]
    name = _names(shape, B, b, mode)[0]
    assert name.startswith("compress_regs") and name.endswith(", 16>"), name
    gen = torch.Generator().manual_seed(b)
    xs = [torch.randn(shape, generator=gen).to(dtype) for _ in range(8)]
    seeds = [900 + k for k in range(8)]
    packed = pkg.division_compress_maps([x.to("cuda:0") for x in xs], B, b, seeds, c16=c16)
    torch.cuda.synchronize()
    for x, s, p in zip(xs, seeds, packed):
        assert np.array_equal(p.cpu().numpy(), oracle.compress(_host(x), B, b, s, dt, threads=16))


# the walk over the planes of several maps: maps that begin in the middle of a workgroup's stride, more than one map between two planes
# of a workgroup, planes that do not fill the last rounds of units, pad bytes of every map
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 1), ("bf16", 2), ("bf16", 1), ("bf16", 8), ("c16", 4)])
@pytest.mark.parametrize("shape,B,maps", [((1, 87, 224, 224), 8, 3), ((1, 51, 204, 204), 4, 7), ((1, 53, 16, 56, 56), 8, 5), ((1, 150, 9, 68, 68), 8, 2), ((1, 300, 224, 224), 4, 1)])
def test_sixteen_wavefronts_walk_over_several_maps(shape, B, maps, mode, b):
    dtype, c16, dt = FORMATS[mode]
    gen = torch.Generator().manual_seed(b)
    xs = [torch.randn(shape, generator=gen).to(dtype) for _ in range(maps)]
    seeds = [77 + 3 * k for k in range(maps)]
    ref = [oracle.compress(_host(x), B, b, s, dt, threads=16) for x, s in zip(xs, seeds)]
    packed = [torch.full((r.size,), 0xA5, dtype=torch.uint8, device="cuda:0") for r in ref]
    pkg.division_compress_maps([x.to("cuda:0") for x in xs], B, b, seeds, packed=packed, c16=c16)
    torch.cuda.synchronize()
    for r, p in zip(ref, packed):
        assert np.array_equal(p.cpu().numpy(), r)


# compress_units: the lookup of four elements at a time (rows that end anywhere inside them, widths and blocks of three, the last row,
# the last slice) and of one (B = 2), one to sixteen lanes per block in the block sums, rounds of units and rows the plane does not have
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 4), ("bf16", 8), ("bf16", 1), ("c16", 2)])
@pytest.mark.parametrize("shape,B", [((3, 5, 17, 17), 64), ((3, 5, 17, 17), 2), ((3, 3, 90, 3), 3), ((2, 3, 91, 3), 12), ((3, 3, 27, 27), 64), ((3, 3, 27, 27), 18),
                                     ((2, 3, 13, 37), 5), ((2, 3, 65, 65), 64), ((2, 2, 73, 73), 3), ((3, 3, 11, 7, 7), 8), ((2, 3, 16, 14, 14), 12),
                                     ((2, 2, 16, 28, 28), 16), ((2, 3, 9, 13, 3), 4), ((2, 3, 20, 21, 2), 4), ((2, 3, 2, 14, 14), 8), ((3, 3, 5, 9, 9), 2),
                                     ((2, 2, 2, 28, 28), 12), ((3, 87, 1, 33), 8), ((3, 87, 1, 69), 4), ((2, 131, 1, 131), 18), ((1, 257, 1, 1521), 4),
                                     ((1, 256, 1, 2049), 8), ((3, 87, 13, 13), 64), ((5, 53, 9, 9), 12), ((3, 87, 2, 7, 7), 12), ((3, 87, 3, 5, 7), 4),
                                     ((2, 2, 4, 56, 56), 64)])
def test_units_block_lookup_and_block_sums(shape, B, mode, b):
    assert _names(shape, B, b, mode)[0].startswith("compress_units<")
    _round_trip(shape, B, b, mode)


# compress_any: workgroups of one, four and sixteen wavefronts, one to 64 lanes per block, lanes that share a word of codes (words that
# end past the plane), rows and blocks of one and two elements, planes of an odd element count
@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("shape,B,b", [((3, 3, 6, 2), 3, 1), ((2, 3, 9, 1), 5, 1), ((2, 3, 28, 28), 3, 1), ((2, 3, 2, 768), 12, 1), ((1, 2, 147, 147), 64, 1), ((2, 2, 147, 146), 18, 1), ((1, 2, 199, 199), 18, 2), ((1, 2, 203, 198), 64, 8),
                                       ((1, 2, 201, 199), 2, 4), ((1, 1, 8200, 5), 64, 2), ((1, 1, 20000, 2), 64, 4), ((2, 3, 3, 3, 5), 2, 1),
                                       ((1, 2, 8, 53, 53), 64, 1), ((1, 2, 33, 35, 37), 16, 2), ((1, 2, 33, 37, 33), 2, 4), ((1, 1, 150, 151, 2), 6, 8),
                                       ((1, 2, 16, 57, 57), 4, 4)])
def test_general_kernel_lanes_per_block(shape, B, b, mode):
    assert _names(shape, B, b, mode)[0].startswith("compress_any")
    _round_trip(shape, B, b, mode)


# compress_seg on planes of even widths (multiples of 4 and not, ragged block rows and columns), of 256 planes and more
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 8), ("c16", 4)])
@pytest.mark.parametrize("shape,B", [((2, 130, 42, 18), 8), ((1, 257, 26, 70), 4), ((1, 256, 19, 46), 8), ((1, 256, 57, 70), 4)])
def test_items_of_even_widths(shape, B, mode, b):
    assert _names(shape, B, b, mode)[0].startswith("compress_seg<")
    _round_trip(shape, B, b, mode)


# decompress_units: rows or blocks of one and two elements, which are looked up element by element, beside those that are not
@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("shape,B,b,each", [((3, 5, 35, 35), 2, 2, True), ((5, 3, 601, 2), 4, 1, True), ((2, 3, 1203, 1), 3, 8, True), ((3, 5, 36, 36), 1, 4, True), ((2, 3, 7, 13, 17), 2, 2, True),
                                            ((300, 3, 27, 27), 2, 2, True), ((3, 5, 37, 37), 3, 2, False), ((5, 3, 401, 3), 3, 4, False), ((2, 3, 70, 71), 2, 2, True)])
def test_decompress_units_of_narrow_rows_and_blocks(shape, B, b, each, mode):
    name = _names(shape, B, b, mode)[1]
    assert name.startswith("decompress_units<") and (name.count(",") == 3) == each, name
    _round_trip(shape, B, b, mode)


# rows of 17 and 35 elements, the rows of three planes side by side (maps of many planes): planes left over, fewer rows than columns, one row of
# blocks, elements that start in the middle of a dword; and the same widths with more rows than columns, which keep their slots
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 1), ("bf16", 4), ("bf16", 8), ("c16", 2)])
@pytest.mark.parametrize("shape,B", [((1, 4096, 17, 17), 8), ((1, 4097, 17, 17), 4), ((2, 2049, 3, 17), 8), ((1, 4099, 9, 17), 4), ((1, 4097, 21, 17), 8),
                                     ((1, 2048, 35, 35), 8), ((1, 2050, 35, 35), 4), ((1, 2051, 2, 35), 8), ((1, 2049, 33, 35), 4), ((1, 2049, 37, 35), 8)])
def test_rows_of_three_planes_side_by_side(shape, B, mode, b):
    assert _names(shape, B, b, mode)[0].startswith("compress_rowstrip<")
    _round_trip(shape, B, b, mode)


# rows long enough for the register kernel: a block is the units of one row, the last one may be short
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 8), ("c16", 4), ("f32", 1)])
@pytest.mark.parametrize("shape,B", [((2, 3, 1, 3136), 8), ((2, 3, 1, 3136), 4), ((1, 3, 1, 2052), 8), ((1, 2, 1, 3324), 8), ((1, 2, 1, 8196), 8), ((1, 2, 1, 20000), 8)])
def test_long_rows_in_registers(shape, B, mode, b):
    assert _names(shape, B, b, mode)[0].startswith("compress_regs<")
    _round_trip(shape, B, b, mode)


# decompress_units, the rounds of a plane shared among workgroups: two to eight shares, the last one short, planes that start anywhere in a unit
@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("shape,B", [((1, 1500, 27, 27), 8), ((1, 7, 27, 27), 4), ((1, 401, 73, 73), 8), ((1, 90, 73, 73), 18), ((1, 3, 147, 147), 8), ((1, 129, 147, 147), 8),
                                     ((1, 5, 8, 14, 15), 8), ((1, 300, 55, 55), 18)])
def test_decompress_units_of_few_planes(shape, B, b):
    assert _names(shape, B, b, "bf16")[1].startswith("decompress_units<")
    _round_trip(shape, B, b, "bf16")


# shapes that one kernel serves, too large for the launch of small maps: rows of one instance of compress_line, and the small planes that compress_planes
# holds; a shape that finds no other beside them, several maps of a shape, more maps than a launch holds
@pytest.mark.parametrize("mode,b", [("f32", 2), ("f32", 1), ("f32", 8), ("bf16", 4), ("bf16", 1), ("c16", 2)])
@pytest.mark.parametrize("specs", [
    [((1, 2101, 1, 384), 8), ((7, 301, 1, 768), 8), ((1, 2101, 1, 384), 8), ((2, 1100, 1, 776), 8), ((1, 1057, 1, 1000), 8)],
    [((1, 2101, 1, 384), 64), ((7, 301, 1, 760), 64), ((1, 4201, 1, 192), 64)],
    [((1, 2057, 32, 32), 4), ((3, 2741, 16, 16), 4), ((1, 8209, 8, 8), 4), ((1, 8209, 4, 4), 4), ((3, 2741, 16, 16), 4), ((1, 8203, 6, 14), 4), ((2, 4101, 20, 24), 4)],
    [((1, 2059, 28, 28), 8), ((1, 8211, 14, 14), 8), ((3, 701, 21, 32), 8), ((1, 8205, 10, 16), 8), ((1, 8211, 4, 4), 64)],
    [((1, 8209, 8, 8), 4)] * 13 + [((1, 8205, 4, 4), 4)] * 12,
    # few enough workgroups that rows of odd width, items under B = 8 and lanes share it too
    [((1, 8209, 13, 13), 8), ((3, 1801, 17, 17), 8), ((3, 1701, 20, 27), 8), ((1, 1031, 35, 35), 8), ((1, 771, 50, 55), 8), ((1, 8209, 9, 15), 8)],
    [((1, 8209, 13, 13), 4), ((3, 1801, 17, 17), 4), ((3, 1701, 20, 27), 4), ((1, 1031, 35, 35), 4), ((1, 771, 55, 55), 4), ((1, 8209, 9, 15), 4)],
    [((3, 2741, 10, 12), 8), ((3, 2741, 18, 22), 8), ((3, 5741, 7, 7), 8), ((1, 9209, 5, 7), 8), ((3, 3741, 11, 5), 16), ((1, 8211, 14, 14), 8), ((3, 2741, 8, 8), 4)],
])
def test_compress_of_shapes_that_share_a_kernel(specs, mode, b):
    dtype, c16, dt = FORMATS[mode]
    gen = torch.Generator().manual_seed(b)
    xs = [torch.randn(s, generator=gen).to(dtype) for s, _ in specs]
    ref = [oracle.compress(_host(x), B, b, (3 << 32) + k, dt, threads=16) for k, (x, (_, B)) in enumerate(zip(xs, specs))]
    packed = [torch.full((r.size,), 0xA5, dtype=torch.uint8, device="cuda:0") for r in ref]
    pkg.division_compress_maps([x.to("cuda:0") for x in xs], [B for _, B in specs], b, [(3 << 32) + k for k in range(len(specs))], packed=packed, c16=c16)
    torch.cuda.synchronize()
    for (shape, B), r, p in zip(specs, ref, packed):
        assert np.array_equal(p.cpu().numpy(), r), (shape, B)


# strips of 32 elements turn their 16-byte pieces in LDS by their place in the round and store their codes as whole words, those of 28 do neither: heights that
# leave slots empty, rounds that end early
@pytest.mark.parametrize("mode", ["f32", "bf16", "c16"])
@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("shape,B", [((3, 11, 32, 32), 8), ((1, 5, 19, 32), 4), ((7, 3, 30, 32), 18), ((2, 5, 26, 32), 12), ((3, 7, 32, 32), 16), ((3, 7, 16, 16), 4),
                                     ((1, 19, 10, 16), 8), ((1, 13, 14, 16), 12), ((5, 5, 25, 28), 8), ((1, 3, 28, 28), 18), ((3, 9, 14, 14), 8), ((1, 11, 12, 14), 12)])
def test_strips_of_all_heights(shape, B, b, mode):
    assert _names(shape, B, b, mode)[0].startswith("compress_strip<")
    _round_trip(shape, B, b, mode)


# single-block planes in few wavefronts: fewer rounds on more lanes than the thirteen of larger maps
@pytest.mark.parametrize("b", [1, 2, 8])
@pytest.mark.parametrize("shape,B,mode", [((1, 5, 28, 28), 64, "f32"), ((3, 90, 20, 20), 64, "c16"), ((1, 301, 24, 40), 64, "bf16"), ((2, 9, 32, 48), 64, "bf16"), ((7, 130, 14, 14), 18, "f32"),
                                          ((1, 3, 2, 20, 22), 64, "bf16"), ((1, 3, 8, 7, 7), 8, "f32")])
def test_single_block_planes_in_few_wavefronts(shape, B, b, mode):
    if b != 1 or shape[0] * shape[1] >= 256: assert not _names(shape, B, b, mode)[0].endswith(", 13>")
    assert _names(shape, B, b, mode)[0].startswith("compress_one<")
    _round_trip(shape, B, b, mode)


# single-block planes of 49 to 52 vectors: sixteen lanes of four rounds from a plane per CU on
@pytest.mark.parametrize("b", [1, 2, 8])
@pytest.mark.parametrize("shape,B,mode", [((4, 64, 14, 14), 64, "f32"), ((1, 257, 10, 20), 20, "f32"), ((3, 101, 16, 13), 16, "c16"), ((2, 133, 20, 20), 64, "bf16"), ((1, 301, 26, 16), 26, "bf16")])
def test_single_block_planes_of_about_fifty_vectors(shape, B, b, mode):
    assert _names(shape, B, b, mode)[0].startswith("compress_one<") and not _names(shape, B, b, mode)[0].endswith(", 13>")
    assert _names((64, 256) + shape[2:], B, b, mode)[0].endswith(", 4>")
    _round_trip(shape, B, b, mode)
