// Part of division.hip (included inside its unnamed namespace, in this order): packed layout, launch plans, launches, the implementation behind the C ABI.

// ------------------------------------------------------------------ host side

struct Layout {
    uint64_t P, HW, LD, LH, LW, nb, WPP;      // HW = elements per plane (D*H*W), nb = LD*LH*LW blocks
    size_t codes_off, codes_bytes, meta_off, meta_bytes, lfc_off, lfc_bytes, total;
};

size_t align16(size_t v) { return (v + 15u) & ~(size_t)15u; }

// A plane is D x H x W elements (Appendix D: 3-D maps); D = 1 for the 2-D maps of Sec. 4.1.
int make_layout(int64_t N, int64_t C, int64_t D, int64_t H, int64_t W, int B, int b, int dt, Layout* L) {
    if (N <= 0 || C <= 0 || D <= 0 || H <= 0 || W <= 0 || B < 1 || (b != 1 && b != 2 && b != 4 && b != 8)) return DIVISION_EINVAL;
    if (dt != DIVISION_F32 && dt != DIVISION_BF16 && dt != DIVISION_F32_C16) return DIVISION_EINVAL;
    const uint64_t lim31 = 0x7fffffffull;
    if ((uint64_t)N > lim31 || (uint64_t)C > lim31 || (uint64_t)D > lim31 || (uint64_t)H > lim31 || (uint64_t)W > lim31)
        return DIVISION_ERANGE;
    L->P = (uint64_t)N * (uint64_t)C;
    if ((uint64_t)D * (uint64_t)H > lim31) return DIVISION_ERANGE;
    L->HW = (uint64_t)D * (uint64_t)H * (uint64_t)W;
    if (L->P > lim31 || L->HW > lim31 || L->P * L->HW > (1ull << 40)) return DIVISION_ERANGE;
    L->LD = ((uint64_t)D + B - 1) / B;
    L->LH = ((uint64_t)H + B - 1) / B;
    L->LW = ((uint64_t)W + B - 1) / B;
    L->nb = L->LD * L->LH * L->LW;
    const uint64_t cpw = 32 / b;
    L->WPP = (L->HW + cpw - 1) / cpw;
    const size_t lfc_es = dt == DIVISION_F32 ? 4 : 2;          // H^L: element type of x, bfloat16 in the cached-as-bf16 mode
    const size_t meta_es = dt == DIVISION_F32_C16 ? 4 : 8;      // (delta, Delta) per plane
    L->codes_off = 0;
    L->codes_bytes = (size_t)(4 * L->P * L->WPP);
    L->meta_off = align16(L->codes_bytes);
    L->meta_bytes = (size_t)(meta_es * L->P);
    L->lfc_off = align16(L->meta_off + L->meta_bytes);
    L->lfc_bytes = (size_t)(lfc_es * L->P * L->nb);
    L->total = align16(L->lfc_off + L->lfc_bytes);
    return DIVISION_OK;
}

uint64_t gcd_u64(uint64_t a, uint64_t b) { while (b) { uint64_t t = a % b; a = b; b = t; } return a; }

Regions make_regions(const Layout& L) {
    Regions rg;
    rg.meta_off = L.meta_off;
    rg.lfc_off = L.lfc_off;
    rg.pad_off[0] = L.codes_off + L.codes_bytes; rg.pad_len[0] = (uint32_t)(L.meta_off - rg.pad_off[0]);
    rg.pad_off[1] = L.meta_off + L.meta_bytes;   rg.pad_len[1] = (uint32_t)(L.lfc_off - rg.pad_off[1]);
    rg.pad_off[2] = L.lfc_off + L.lfc_bytes;     rg.pad_len[2] = (uint32_t)(L.total - rg.pad_off[2]);
    return rg;
}

// the two keys of a 64-bit seed
uint32_t seed_key_a(uint64_t seed) { return mix32((uint32_t)(seed & 0xffffffffu) ^ 0x243F6A88u); }
uint32_t seed_key_c(uint64_t seed) { return mix32((uint32_t)(seed >> 32) ^ 0x85A308D3u); }

// Preferred LDS footprint of one wavefront's chunk in compress_wave (small chunks = many wavefronts
// per CU; 8.7 KB measured best over the ResNet-50 set); a single plane of up to kWavePlaneMax bytes is
// taken whatever the preference says.
constexpr uint32_t kWaveChunkLds = 8704u;
constexpr uint32_t kWavePlaneMax = 17u << 10;

// Compute units of the current device (sizes the grids of the kernels that walk over planes).  Asked
// once per device and kept: a table of constants of the machine, not state of a call.
int num_cus() {
    constexpr int kMaxDev = 64;
    static std::atomic<int> cus[kMaxDev];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) return 256;
    int v = cus[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cus[dev].store(v, std::memory_order_relaxed);
    return v;
}

// dynamic LDS above the default limit needs a one-time opt-in per kernel
template <typename Args>
hipError_t allow_large_lds(void (*kern)(Args), size_t lds) {
    if (lds <= 48u * 1024u) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
}

template <typename T, int BITS, int B>
hipError_t launch_tile_vec(int vec, const TileArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(TileArgs) = vec == 4 ? compress_tile<T, BITS, B, 4, 256>
                           : vec == 2 ? compress_tile<T, BITS, B, 2, 256>
                                      : compress_tile<T, BITS, B, 1, 256>;
    hipError_t e = allow_large_lds(kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, a);
    return hipGetLastError();
}

template <typename T, int BITS>
hipError_t launch_tile(int B, int vec, const TileArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    return B == 8 ? launch_tile_vec<T, BITS, 8>(vec, a, grid, lds, st)
                  : launch_tile_vec<T, BITS, 4>(vec, a, grid, lds, st);
}

template <typename T, int BITS, int B>
hipError_t launch_wave_vec(int vec, const WaveArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(WaveArgs) = vec == 4 ? compress_wave<T, BITS, B, 4>
                           : vec == 2 ? compress_wave<T, BITS, B, 2>
                                      : compress_wave<T, BITS, B, 1>;
    hipLaunchKernelGGL(kern, grid, dim3(64), lds, st, a);
    return hipGetLastError();
}

template <typename T, int BITS>
hipError_t launch_wave(int B, int vec, const WaveArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    return B == 8 ? launch_wave_vec<T, BITS, 8>(vec, a, grid, lds, st)
                  : launch_wave_vec<T, BITS, 4>(vec, a, grid, lds, st);
}

// Fills the plane-in-registers compress plan; false when the shape is not covered.
bool plan_regs(const Layout& L, int64_t D, int64_t H, int64_t W, int B, size_t es, const void* x,
               RegsArgs* a, uint32_t* grid, size_t* lds, int* nw_out) {
    if (B % 4 != 0 || W % 4 != 0) return false;
    if (D > 1 && B != 8) return false;            // 3-D maps: the B = 8 instances only
    if (((uintptr_t)x % (4 * es)) != 0) return false;
    const uint64_t q4 = L.HW / 4;
    const bool any_b = B != 4 && B != 8;          // the instance that reads B from its arguments
    int nw;
    if (any_b) {
        // a lane adds the unit sums of its block one after the other: at most 64 of them (blocks of
        // up to 16 x 16, longer ones on maps of few rows), several blocks per plane
        const uint64_t brows = (uint64_t)B < (uint64_t)H ? (uint64_t)B : (uint64_t)H;
        if (brows * ((uint64_t)B / 4) > 64 || L.nb == 1) return false;
        if (q4 >= 512 && q4 <= (uint64_t)kRegUnits * 64) nw = 1;
        else if (q4 > (uint64_t)kRegUnits * 64 && q4 <= (uint64_t)kRegUnits * 256) nw = 4;
        else return false;
    } else if (q4 >= 512 && q4 <= (uint64_t)kRegUnits * 64) nw = 1;
    else if (q4 >= (D > 1 ? (uint64_t)kRegUnits * 64 + 1 : 2048) && q4 <= (uint64_t)kRegUnits * 256) nw = 4;
    else if (q4 > (uint64_t)kRegUnits * 256 && q4 <= (uint64_t)kRegUnits * 1024) nw = 16;   // image-sized planes: 1024 threads, one workgroup per CU
    else return false;
    const uint64_t nt = 64ull * nw, w4 = (uint64_t)W / 4;
    if (!fastdiv_ok(kRegUnits * nt, w4) || !fastdiv_ok(L.nb + nt, L.LW) || L.HW * es >= (1ull << 31)) return false;
    if (!fastdiv_ok((uint64_t)H, (uint64_t)B) || !fastdiv_ok(w4, (uint64_t)B / 4)) return false;
    if (!fastdiv_ok((uint64_t)D * (uint64_t)H, (uint64_t)H) || !fastdiv_ok(L.nb + nt, L.LH * L.LW)) return false;
    *a = RegsArgs{};
    a->D = (uint32_t)D;
    a->d_H = make_fastdiv((uint32_t)H);
    a->d_slice = make_fastdiv((uint32_t)(L.LH * L.LW));
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)L.LH; a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP;
    a->q4 = (uint32_t)q4; a->w4 = (uint32_t)w4;
    a->B = (uint32_t)B;
    a->d_w4 = make_fastdiv((uint32_t)w4);
    a->d_LW = make_fastdiv((uint32_t)L.LW);
    a->d_B = make_fastdiv((uint32_t)B);
    a->d_upb = make_fastdiv((uint32_t)B / 4);
    *lds = 8ull * kRegUnits * nt + 4ull * ((L.nb + 1 + 3) & ~3ull) + 8ull * nw + 16 + (D > 1 ? 8ull * L.nb * B + 16 : 0);
    *grid = (uint32_t)L.P;
    *nw_out = nw;
    return *lds <= (nw == 16 ? (size_t)kLdsMax : (size_t)(60u * 1024u));
}

// Whether a workgroup per CU walks over the planes of all maps of a launch of sixteen-wavefront instances, loading the next
// plane as the codes of the present one leave, or each plane has a workgroup of its own.  A workgroup fills its CU, so one more
// than there are CUs would wait until others have walked to their end: the walk is over all maps together (a grid per map,
// rounded up, made 3, 5, 6 and 7 maps 1.25-1.5 times slower: 3 maps of 64 x 16 x 224 x 224 55.4 us each with a workgroup per
// plane, 69.2 so, 45.3 together).  The walk runs all thirteen rounds of units untested, so planes of fewer rounds want fewer of
// them wasted or more planes to overlap (fp32 / bfloat16, a workgroup per plane -> walk): 257 planes of 12.2 rounds 23.9 -> 21.6 / 20.9 -> 18.7,
// of 10.6 rounds 20.5 -> 19.4 / 18.5 -> 18.3, of 8.3 rounds 17.7 -> 18.0 / 16.7 -> 18.0; 1024 planes of 8.3 rounds 42.9 -> 39.5 / 34.3 -> 33.8,
// of 6.2 rounds 34.8 -> 33.2 / 28.9 -> 32.3.
bool regs_walk(uint64_t planes, uint64_t q4) {
    const uint64_t cus = (uint64_t)num_cus(), round = 1024;
    return q4 > 10 * round ? planes > cus : q4 > 8 * round && planes >= 4 * cus;
}

template <typename T, int BITS>
hipError_t launch_regs(int B, int nw, const RegsArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(RegsArgs);
    if (a.D > 1) kern = nw == 1 ? compress_regs_3d<T, BITS, 8, 1> : nw == 4 ? compress_regs_3d<T, BITS, 8, 4> : compress_regs_3d<T, BITS, 8, 16>;
    else if (nw == 1 && a.H == 1 && (B == 8 || B == 4)) kern = B == 8 ? compress_regs_row<T, BITS, 8> : compress_regs_row<T, BITS, 4>;
    else if (nw == 1) kern = B == 8 ? compress_regs<T, BITS, 8, 1> : B == 4 ? compress_regs<T, BITS, 4, 1> : compress_regs<T, BITS, 0, 1>;
    else if (nw == 4) kern = B == 8 ? compress_regs<T, BITS, 8, 4> : B == 4 ? compress_regs<T, BITS, 4, 4> : compress_regs<T, BITS, 0, 4>;
    else kern = B == 8 ? compress_regs<T, BITS, 8, 16> : compress_regs<T, BITS, 4, 16>;
    const hipError_t e = allow_large_lds(kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(64 * nw), lds, st, a);
    return hipGetLastError();
}

// Fills the plan of the register kernel for any width; false when the shape is not covered: 2-D maps
// of at most 8 x 1024 units that fit LDS beside their row sums (up to about 163 x 163 elements).
constexpr uint64_t kUnitsMin = 128;       // units per plane from which a plane gets a whole wavefront or more
constexpr uint64_t kUnitsSubMin = 64;     // units per plane from which the instance with 8, 16 or 32 lanes per plane is used under B = 4
                                          // and 8 in two dimensions (below, compress_wave is level or ahead: 14 x 5 under B = 8 11.5 us against 14.9)
constexpr uint64_t kUnitsSubMinAny = 20;  // under other block sizes and in three dimensions, where compress_rows takes what is left: 13 x 13
                                          // under B = 64 16.6 us there and 11.3 here, 2 x 7 x 7 under B = 12 17.8 and 15.1; level at 18 units (14 x 5)
constexpr uint64_t kUnitsRowMin = 8;      // for maps of one row (maps of 4 M elements, against compress_wave: rows of 335 under B = 8 28.9 us
                                          // and 11.9 here, 1521 under B = 4 30.9 and 14.1)
// planes of a map from which one row, small planes and even widths leave the chunk kernels (wave, rows, tile).  Maps of fewer would gain
// as well (700 of them, medians: one row 13.9 us in compress_wave and 5.1 here, 8.4 and 5.7 in compress_rows, 23.4 and 8.6 in compress_tile, small
// planes 6.2 and 5.1, volumes 8.4 and 5.1; 52 of the 700 slower): they keep the kernels they are known by
constexpr uint64_t kUnitsManyPlanes = 256;
bool plan_seg(const Layout& L, int64_t D, int64_t H, int64_t W, int B, size_t es, SegArgs* a, uint32_t* grid, size_t* lds,
              uint32_t* nt_out, int* K_out);
// maps: of the launch.
bool plan_units(const Layout& L, int64_t D, int64_t H, int64_t W, int B, int b, size_t es, const void* x, int maps,
                UnitsArgs* a, uint32_t* grid, size_t* lds, int* nw_out) {
    if (((uintptr_t)x % 4) != 0 || (H == 1 && L.P < kUnitsManyPlanes)) return false;
    // small planes of even width under B = 4 and 8 are the wavefront kernel's (pairs of elements per
    // lane): measured faster there
    // (one row: only those a lane of the wavefront kernel, which takes B rows, would do little of)
    bool seg = false;
    if (D == 1 && H > 1 && (B == 4 || B == 8) && W % 2 == 0 && 4ull * L.HW + 16ull <= kWavePlaneMax) {
        // (4-byte elements, a plane for every CU: compress_seg where it takes them; 4 M elements of 57 x 70 under B = 4 36.2 -> 9.3 us,
        // 19 x 46 under B = 8 14.3 -> 7.9, 42 x 18 11.1 -> 8.5, 63 x 32 9.8 -> 8.4; not the narrow rows of whole vectors under B = 4, of which the wavefront kernel's lanes have a block
        // row each: 308 x 16 x 134 x 12 13.5 -> 14.5, 116 x 8 level)
        SegArgs t{};
        uint32_t g = 0, nt = 0;
        size_t l = 0;
        int K = 0;
        seg = b != 1 && L.P >= kUnitsManyPlanes && !(B == 4 && W % 4 == 0 && W < 16) && plan_seg(L, D, H, W, B, es, &t, &g, &l, &nt, &K);
        if (!seg) return false;
    }
    const uint64_t q4 = (L.HW + 3) / 4;
    if (L.nb > 16383 || B > 4095) return false;              // LFC offsets are kept as 16-bit byte offsets
    // 2-D planes below 2048 elements with whole-vector rows: compress_rows keeps their vectors in registers
    // and is the faster one (28 x 28 under B = 12: 43 us against 49)
    // (not 1-bit codes of maps of one row, which the general kernel would get: rows of 96 under B = 12 45 us there, 15 here)
    if (D == 1 && W % 4 == 0 && q4 < 512 && !(H == 1 && b == 1) && !seg) return false;
    // calls that another kernel serves as well or better (maps of 0.01 to 8 M elements, that kernel -> this): one row of whole vectors under
    // B = 4 (compress_tile 10.2 -> 12.7 us on 1746 rows of 2032, ahead by 1 % over all; by 8 and more elsewhere); 2-byte rows of an odd
    // width of 256 to 1023 elements under larger blocks (compress_rows 12.1 -> 15.1 on 5340 rows of 663 under B = 64, 11 % ahead over
    // all); small planes of one column (compress_rows 7.1 -> 8.9 on 3760 of 131 rows), and of 2-byte elements under B = 2 and 3
    // (6.2 -> 7.2 on 2516 of 37 x 5)
    if (H == 1 && B == 4 && W % 4 == 0) return false;
    if (H == 1 && b != 1 && es == 2 && W % 2 != 0 && B > 8 && q4 >= 64 && q4 < 256) return false;
    if (H > 1 && b != 1 && q4 < kUnitsSubMin && (W == 1 || (es == 2 && B < 4))) return false;
    const uint64_t Bz = (uint64_t)std::min<int64_t>(B, D), Br = (uint64_t)std::min<int64_t>(B, H);      // depth and rows of a block
    const uint64_t nitem = L.nb * Bz * Br;
    const bool many = L.P >= kUnitsManyPlanes;
    // Lanes per plane.  Few planes: the launch is the latency of one, for which lanes are given to all B rows (slices) of a block, also of
    // those that the map does not have (153 volumes of 2 x 7 x 33 under B = 8 7.1 us so, 8.5 with lanes for its own).
    uint64_t lanes_for = L.nb * (D > 1 ? (uint64_t)B : 1) * (uint64_t)B;
    if (many || lanes_for > (uint64_t)kUnitsK * 1024) lanes_for = nitem;
    int nw = 1;
    uint64_t S = 64;                                          // lanes per plane
    if (q4 < kUnitsMin) {
        // small planes: 8, 16 or 32 lanes each, several planes per wavefront
        if (q4 < (!many ? kUnitsSubMin : H == 1 ? kUnitsRowMin : D == 1 && (B == 4 || B == 8) ? kUnitsSubMin : kUnitsSubMinAny)) return false;
        S = 8;
        while (S < 64 && (q4 > (uint64_t)kUnitsK * S || lanes_for > (uint64_t)kUnitsK * S)) S *= 2;
        nw = S < 64 ? 0 : 1;
    }
    if (nw) {
        while (nw < 16 && (q4 > (uint64_t)kUnitsK * 64 * nw || lanes_for > (uint64_t)kUnitsK * 64 * nw)) nw *= 2;
        S = 64ull * nw;
    }
    // Many planes that still leave the machine idle (those of all maps of the launch): more lanes for each, up to a unit per lane, until there are eight wavefronts per CU (four
    // and sixteen are slower: 8 lanes with eight units one after the other on 306 rows of 114 in bfloat16 under B = 2 10.0 us, 5.6 with 32; 2000
    // maps of all sizes together 1.50 times as fast as the kernels that had them before with four, 1.53 with eight, 1.50 with sixteen)
    if (many) {
        while (S < (b == 1 ? 512u : 1024u) && L.P * (uint64_t)maps * S < 8 * 64 * (uint64_t)num_cus() && q4 > S) S *= 2;
        nw = S < 64 ? 0 : (int)(S / 64);
    }
    if (q4 > (uint64_t)kUnitsK * S || nitem > (uint64_t)kUnitsK * S) return false;       // 8 units and 8 row segments per lane
    const uint64_t q4p = (q4 + S - 1) / S * S;
    if (!fastdiv_ok(4ull * kUnitsK * S + 4, (uint64_t)W) || !fastdiv_ok(4ull * kUnitsK * S + 4, (uint64_t)B) ||
        !fastdiv_ok(nitem + S, Br * Bz) || !fastdiv_ok(L.nb + S, L.LH * L.LW) ||
        !fastdiv_ok(4ull * kUnitsK * S + 4, (uint64_t)H))
        return false;
    *a = UnitsArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP; a->B = (uint32_t)B;
    a->D = (uint32_t)D; a->LH = (uint32_t)L.LH; a->Br = (uint32_t)Br; a->Bz = (uint32_t)Bz;
    a->d_H = make_fastdiv((uint32_t)H);
    a->d_Br = make_fastdiv((uint32_t)Br);
    a->d_BBz = make_fastdiv((uint32_t)(Bz * Br));
    a->d_slice = make_fastdiv((uint32_t)(L.LH * L.LW));
    a->q4 = (uint32_t)q4; a->q4p = (uint32_t)q4p; a->nitem = (uint32_t)nitem;
    a->S = (uint32_t)S;
    a->S_log2 = 0;
    while ((1ull << a->S_log2) < S) ++a->S_log2;
    a->d_W = make_fastdiv((uint32_t)W);
    a->d_B = make_fastdiv((uint32_t)B);
    a->d_LW = make_fastdiv((uint32_t)L.LW);
    // lanes per block in the block sums: as many as there are, at most 16, four rows and more for each
    a->J_log2 = 0;
    while (a->J_log2 < 4 && (L.nb << (a->J_log2 + 1)) <= S && (8ull << a->J_log2) <= Bz * Br) ++a->J_log2;
    const uint64_t G = nw ? 1 : 64 / S;                       // planes per round
    const uint64_t reg = (16ull * q4p + 8ull * nitem + 4ull * ((L.nb + 1 + 3) & ~3ull) + 8ull * (nw ? nw : 1) + 16 + 15) & ~15ull;
    a->reg_bytes = (uint32_t)reg;
    a->nrounds = (uint32_t)((L.P + G - 1) / G);
    *lds = reg * G;
    if (*lds > (size_t)kLdsMax) return false;
    // as many workgroups as the machine holds at once (LDS, and 16 wavefronts per CU), each taking every
    // grid-th round of planes
    const uint64_t wpg = nw ? (uint64_t)nw : 1;               // wavefronts per workgroup
    uint64_t per_cu = (160ull << 10) / *lds;
    if (per_cu > 16ull / wpg) per_cu = 16ull / wpg;
    if (per_cu < 1) per_cu = 1;
    uint64_t g = (uint64_t)num_cus() * per_cu;
    g += g & 1;            // even: with 2-byte elements the planes of a workgroup then start alike within a dword
    *grid = (uint32_t)(g < a->nrounds ? g : a->nrounds);
    *nw_out = nw;
    return true;
}

template <typename T, int BITS>
hipError_t launch_units(int nw, const UnitsArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(UnitsArgs) = nw == 0 ? compress_units<T, BITS, 0> : nw == 1 ? compress_units<T, BITS, 1>
                            : nw == 2 ? compress_units<T, BITS, 2> : nw == 4 ? compress_units<T, BITS, 4>
                                                                             : compress_units<T, BITS, 8>;
    // 1-bit codes have no instance of sixteen wavefronts (its lane pairing does not fit the 128 registers
    // a lane of 1024 threads has): the planner sends those planes elsewhere
    if constexpr (BITS != 1) { if (nw == 16) kern = compress_units<T, BITS, 16>; }
    else if (nw == 16) return hipErrorInvalidValue;
    const hipError_t e = allow_large_lds(kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(nw ? 64 * nw : 64), lds, st, a);
    return hipGetLastError();
}

// Fills the plan of compress_seg (4-byte elements, B = 4 or 8), for the planes of compress_units; false when the
// shape is not covered (an odd number of elements per slice in a 3-D map: rows would start anywhere in an element
// pair) or would leave too many lanes idle.  One or two items per lane, whichever takes fewer instructions per plane: about
// 216 for an item and 250 for a wavefront's share of everything else (five and seven items per lane were slower, 173 us
// against 102 on 64 x 64 x 147 x 147: 156 to 208 registers).
bool plan_seg(const Layout& L, int64_t D, int64_t H, int64_t W, int B, size_t es, SegArgs* a, uint32_t* grid, size_t* lds,
              uint32_t* nt_out, int* K_out) {
    if (es != 4 || (B != 4 && B != 8) || (D > 1 && (H * W) % 2 != 0)) return false;
    const uint64_t CW = ((uint64_t)W + 3) / 4, irows = ((uint64_t)H + 3) / 4, rows = irows * (uint64_t)D;
    if (CW > kSegThreads) return false;
    uint64_t best_nt = 0, best = ~0ull;
    int best_K = 0;
    for (const int K : {1, 2}) {
        const uint64_t RS = (rows + K - 1) / K;                       // item rows per round
        const uint64_t nt = (RS * CW + 63) / 64 * 64;
        if (nt > kSegThreads) continue;
        const uint64_t cost = nt / 64 * (216 * (uint64_t)K + 250);
        if (cost < best) { best = cost; best_nt = nt; best_K = K; }
    }
    if (best_K == 0) return false;
    // at least 60 % of the lanes' slots hold elements of the plane
    if (L.HW * 10 < 6ull * 16 * best_K * best_nt) return false;
    const size_t need = 8 * rows * CW + 64 + 8 * (best_nt / 64) + 4 * L.nb + 4 * L.WPP;
    const uint64_t top = rows + (uint64_t)best_K * best_nt;
    // a workgroup per plane: maps of about 165 GB and more stay with compress_units, whose workgroups walk over the planes
    if (!launch_ok(L.P, best_nt)) return false;
    if (need > (48u << 10) || !fastdiv_ok(top, irows) || !fastdiv_ok(kSegThreads, CW) || !fastdiv_ok(L.nb + best_nt, L.LW) || !fastdiv_ok(L.nb + best_nt, L.LH * L.LW)) return false;
    *a = SegArgs{};
    a->P = (uint32_t)L.P; a->D = (uint32_t)D; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)L.LH; a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP;
    a->CW = (uint32_t)CW; a->RS = (uint32_t)(best_nt / CW); a->irows = (uint32_t)irows; a->rows = (uint32_t)rows;
    a->cz0 = (uint32_t)(D < B ? D : B);
    a->cz1 = (uint32_t)(D - (int64_t)(L.LD - 1) * B);
    a->d_irows = make_fastdiv((uint32_t)irows); a->d_slice = make_fastdiv((uint32_t)(L.LH * L.LW)); a->d_LW = make_fastdiv((uint32_t)L.LW);
    a->d_CW = make_fastdiv((uint32_t)CW);
    *grid = (uint32_t)L.P;
    *nt_out = (uint32_t)best_nt;
    *K_out = best_K;
    *lds = need;
    return true;
}

template <typename T, int BITS, int K>
hipError_t launch_seg_K(int B, const SegArgs& a, uint32_t nt, dim3 grid, size_t lds, hipStream_t st) {
    if constexpr (sizeof(T) == 4) {
        const bool odd = a.W % 2 != 0;
        void (*kern)(SegArgs) = B == 8 ? (odd ? compress_seg<T, BITS, 8, true, K> : compress_seg<T, BITS, 8, false, K>)
                                       : (odd ? compress_seg<T, BITS, 4, true, K> : compress_seg<T, BITS, 4, false, K>);
        hipLaunchKernelGGL(kern, grid, dim3(nt), lds, st, a);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}
template <typename T, int BITS>
hipError_t launch_seg(int K, int B, const SegArgs& a, uint32_t nt, dim3 grid, size_t lds, hipStream_t st) {
    return K == 1 ? launch_seg_K<T, BITS, 1>(B, a, nt, grid, lds, st) : launch_seg_K<T, BITS, 2>(B, a, nt, grid, lds, st);
}

// one-block planes with an odd element count: the shapes the lane-per-plane kernels take
bool lane_shape(const Layout& L) { return L.nb == 1 && (L.HW & 1) == 1 && L.HW <= 64; }

// Fills the lane-per-plane compress plan; false when the shape is not covered.
bool plan_lane(const Layout& L, size_t es, const void* x, LaneArgs* a, uint32_t* grid, size_t* lds) {
    if (!lane_shape(L)) return false;
    *a = LaneArgs{};
    a->P = (uint32_t)L.P; a->HW = (uint32_t)L.HW; a->WPP = (uint32_t)L.WPP;
    a->nrounds = (uint32_t)((L.P + 63) / 64);
    a->vec_load = ((uintptr_t)x % 16) == 0;
    uint32_t rpw = 2;
    while (rpw > 1 && a->nrounds / rpw < 32u * (uint32_t)num_cus()) --rpw;
    a->rpw = rpw;
    *lds = 4ull * (64ull * L.HW + 4) + 16 * (es == 2 ? 1 : 0);
    *grid = (a->nrounds + rpw - 1) / rpw;
    return true;
}

// Fills the items-from-global compress plan (small planes); false when the shape is not covered.
bool plan_items(const Layout& L, int64_t H, int64_t W, int B, size_t es, const void* x,
                ItemsArgs* a, uint32_t* grid, size_t* lds, int* vec_out) {
    if ((B != 4 && B != 8) || W % 2 != 0) return false;
    const int vec = W % 4 == 0 ? 4 : 2;
    if (((uintptr_t)x % (vec * es)) != 0) return false;
    const uint64_t ipb = (uint64_t)B / vec;
    const uint64_t slots = (uint64_t)W / vec;
    const uint64_t ipr = (slots + ipb - 1) / ipb * ipb;
    const uint64_t ipp = L.LH * ipr;
    if (ipp > 64) return false;
    uint64_t S = 1, lg = 0;
    while (S < ipp) { S *= 2; ++lg; }
    const uint64_t ppr = 64 / S;
    if (ppr * L.WPP * 4 > 32u * 1024u || ppr * L.HW * es >= (1ull << 31)) return false;
    *a = ItemsArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP;
    a->ipr = (uint32_t)ipr; a->ipp = (uint32_t)ipp; a->S = (uint32_t)S; a->S_log2 = (uint32_t)lg;
    a->ppr = (uint32_t)ppr;
    a->nrounds = (uint32_t)((L.P + ppr - 1) / ppr);
    a->d_ipr = make_fastdiv((uint32_t)ipr);
    uint32_t rpw = 2;
    while (rpw > 1 && a->nrounds / rpw < 32u * (uint32_t)num_cus()) --rpw;
    a->rpw = rpw;
    *lds = 4ull * ppr * L.WPP + 16;
    *grid = (a->nrounds + rpw - 1) / rpw;
    *vec_out = vec;
    return true;
}

// Fills the strip kernel's plan: 2-D maps of width 28 or 32 (at most 32 rows) or 14 or 16 (an even number
// of rows, at most 16), 16-byte aligned, under a block size the kernel has an instance for: 8 on 28 / 14
// (the items kernel keeps 32 / 16 under B = 8), 12, 16 (where a plane has several blocks) and 18 of the
// block-size sweep; false when the shape is not covered.  *width = 100 * W + B names the instance.
bool plan_strip(const Layout& L, int64_t H, int64_t W, int B, size_t es, const void* x,
                StripArgs* a, uint32_t* grid, size_t* lds, int* width) {
    if (((uintptr_t)x % (4 * es)) != 0) return false;
    uint64_t G, upl;
    if ((W == 28 || W == 32) && H <= 32) { G = 2; upl = W == 28 ? 7 : 8; }
    else if ((W == 14 || W == 16) && H % 2 == 0 && H <= 16) { G = 8; upl = W == 14 ? 7 : 8; }
    else return false;
    const bool wide = W == 28 || W == 32;
    bool have;
    switch (B) {
        case 4: have = W == 32 || W == 16; break;
        case 8: have = true; break;
        case 12: have = true; break;
        case 16: have = wide; break;
        case 18: have = wide; break;
        default: have = false;
    }
    if (!have) return false;
    const uint64_t nseg = ((uint64_t)W + B - 1) / B;
    const bool dpp = B == 4 || B == 8;
    if (L.LW != nseg || (!dpp && G * L.nb > 64)) return false;
    *a = StripArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->HW = (uint32_t)L.HW; a->WPP = (uint32_t)L.WPP; a->nb = (uint32_t)L.nb;
    a->nrounds = (uint32_t)((L.P + G - 1) / G);
    *grid = a->nrounds;
    // the round; for the block sizes whose block rows are no DPP group also the strips' shares and the round's H^L
    *lds = dpp ? es * G * L.HW + 16 : upl * 256 * es + 64 * nseg * 8 + 256 + 16;
    *width = (int)(100 * W + B);
    return true;
}

template <typename T, int BITS>
hipError_t launch_strip(int width, const StripArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(StripArgs);
    switch (width) {
        case 2808: kern = compress_strip<T, BITS, 28, 8>; break;
        case 1408: kern = compress_strip<T, BITS, 14, 8>; break;
        case 3208: kern = compress_strip<T, BITS, 32, 8>; break;
        case 1608: kern = compress_strip<T, BITS, 16, 8>; break;
        case 3204: kern = compress_strip<T, BITS, 32, 4>; break;
        case 1604: kern = compress_strip<T, BITS, 16, 4>; break;
        case 2812: kern = compress_strip<T, BITS, 28, 12>; break;
        case 2816: kern = compress_strip<T, BITS, 28, 16>; break;
        case 2818: kern = compress_strip<T, BITS, 28, 18>; break;
        case 3212: kern = compress_strip<T, BITS, 32, 12>; break;
        case 3216: kern = compress_strip<T, BITS, 32, 16>; break;
        case 3218: kern = compress_strip<T, BITS, 32, 18>; break;
        case 1412: kern = compress_strip<T, BITS, 14, 12>; break;
        case 1612: kern = compress_strip<T, BITS, 16, 12>; break;
        default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64), lds, st, a);
    return hipGetLastError();
}

// Fills the plan of the row-per-lane strip kernel: 2-D maps of an odd width it has an instance for (13, 15,
// 17, 27, 35, 55) with at most 16 (13, 15), 32 (17, 27) or 64 rows, under B = 8 or 4, 16-byte aligned.
// *width = 100 * W + B names the instance.
bool plan_rowstrip(const Layout& L, int64_t H, int64_t W, int B, size_t es, const void* x,
                   StripArgs* a, uint32_t* grid, size_t* lds, int* width) {
    if (((uintptr_t)x % 16) != 0) return false;
    uint64_t S;
    if (W == 13 || W == 15) S = 16;
    else if (W == 17 || W == 27) S = 32;
    else if (W == 35 || W == 55) S = 64;
    else return false;
    if ((B != 8 && B != 4) || H < 2 || (uint64_t)H > S) return false;
    const uint64_t G = 64 / S;
    if (L.LW != ((uint64_t)W + B - 1) / B) return false;
    *a = StripArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->HW = (uint32_t)L.HW; a->WPP = (uint32_t)L.WPP; a->nb = (uint32_t)L.nb;
    a->nrounds = (uint32_t)((L.P + G - 1) / G);
    *grid = a->nrounds;
    *lds = 16ull * ((G * L.HW + 3) / 4) + 16;          // the round in whole 16-byte units, and the element in front of it
    const int pack = W == 17 ? kRowPack<17> : W == 35 ? kRowPack<35> : 0;
    if (pack && H <= W && L.P >= 8ull * num_cus() * G) {
        // the rows of three planes side by side (planes of more rows keep their slots, and so do maps of less than eight wavefronts per CU, which wait for
        // the longer chain through LDS: 72 planes of 35 x 35 4.4 us in slots, 4.8 so)
        const uint64_t nseg = L.LW;
        const size_t round = 16ull * ((kRowPackPlanes * L.HW + 3) / 4) + 16, shares = 8ull * nseg * 64 * pack;
        a->pack_off = (uint32_t)((std::max(round, shares) + 15) & ~15ull);
        a->LH = (uint32_t)L.LH;
        a->d_H = make_fastdiv((uint32_t)H);
        a->d_LH = make_fastdiv((uint32_t)L.LH);
        a->nrounds = (uint32_t)((L.P + kRowPackPlanes - 1) / kRowPackPlanes);
        *grid = a->nrounds;
        *lds = a->pack_off + 4ull * kRowPackPlanes * L.nb + 8ull * kRowPackPlanes;
    }
    *width = (int)(100 * W + B);
    return true;
}

template <typename T, int BITS>
hipError_t launch_rowstrip(int width, const StripArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(StripArgs);
    switch (width) {
        case 1308: kern = compress_rowstrip<T, BITS, 13, 8>; break;
        case 1304: kern = compress_rowstrip<T, BITS, 13, 4>; break;
        case 1508: kern = compress_rowstrip<T, BITS, 15, 8>; break;
        case 1504: kern = compress_rowstrip<T, BITS, 15, 4>; break;
        case 1708: kern = compress_rowstrip<T, BITS, 17, 8>; break;
        case 1704: kern = compress_rowstrip<T, BITS, 17, 4>; break;
        case 2708: kern = compress_rowstrip<T, BITS, 27, 8>; break;
        case 2704: kern = compress_rowstrip<T, BITS, 27, 4>; break;
        case 3508: kern = compress_rowstrip<T, BITS, 35, 8>; break;
        case 3504: kern = compress_rowstrip<T, BITS, 35, 4>; break;
        case 5508: kern = compress_rowstrip<T, BITS, 55, 8>; break;
        case 5504: kern = compress_rowstrip<T, BITS, 55, 4>; break;
        default: return hipErrorInvalidValue;
    }
    int wavefronts = 1;
    if (a.pack_off) {
        kern = width == 1708 ? compress_rowstrip_packed<T, BITS, 17, 8> : width == 1704 ? compress_rowstrip_packed<T, BITS, 17, 4>
             : width == 3508 ? compress_rowstrip_packed<T, BITS, 35, 8> : compress_rowstrip_packed<T, BITS, 35, 4>;
        wavefronts = width / 100 == 17 ? kRowPack<17> : kRowPack<35>;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * wavefronts), lds, st, a);
    return hipGetLastError();
}

// The Relu + compress instance of the strip kernel; a round's mask bits must be whole words.
bool plan_relu_strip(const Layout& L, int64_t H, int64_t W, int B, size_t es, const void* xy,
                     StripArgs* a, uint32_t* grid, size_t* lds, int* width) {
    // the instances whose block sums are DPP reductions: B = 8 on every strip width, B = 4 on 32 / 16
    if ((B != 8 && B != 4) || !plan_strip(L, H, W, B, es, xy, a, grid, lds, width)) return false;
    const uint64_t G = (W == 28 || W == 32) ? 2 : 8;
    return (G * L.HW) % 32 == 0;
}

template <typename T, int BITS>
hipError_t launch_relu_strip(int width, const StripArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(StripArgs);
    switch (width) {
        case 2808: kern = relu_compress_strip<T, BITS, 28, 8>; break;
        case 1408: kern = relu_compress_strip<T, BITS, 14, 8>; break;
        case 3208: kern = relu_compress_strip<T, BITS, 32, 8>; break;
        case 1608: kern = relu_compress_strip<T, BITS, 16, 8>; break;
        case 3204: kern = relu_compress_strip<T, BITS, 32, 4>; break;
        case 1604: kern = relu_compress_strip<T, BITS, 16, 4>; break;
        default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64), lds, st, a);
    return hipGetLastError();
}

template <typename T, int BITS>
hipError_t launch_items(int B, int vec, const ItemsArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(ItemsArgs);
    if (a.H == 1) {
        if (B == 8) kern = vec == 4 ? compress_items<T, BITS, 8, 4, 1> : compress_items<T, BITS, 8, 2, 1>;
        else kern = vec == 4 ? compress_items<T, BITS, 4, 4, 1> : compress_items<T, BITS, 4, 2, 1>;
    } else {
        if (B == 8) kern = vec == 4 ? compress_items<T, BITS, 8, 4, 8> : compress_items<T, BITS, 8, 2, 8>;
        else kern = vec == 4 ? compress_items<T, BITS, 4, 4, 4> : compress_items<T, BITS, 4, 2, 4>;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64), lds, st, a);
    return hipGetLastError();
}

// The Relu + compress instance of the items kernel (2-D maps, items of B rows).
template <typename T, int BITS>
hipError_t launch_relu_items(int B, int vec, const ItemsArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    void (*kern)(ItemsArgs);
    if (B == 8) kern = vec == 4 ? relu_compress_items<T, BITS, 8, 4> : relu_compress_items<T, BITS, 8, 2>;
    else kern = vec == 4 ? relu_compress_items<T, BITS, 4, 4> : relu_compress_items<T, BITS, 4, 2>;
    hipLaunchKernelGGL(kern, grid, dim3(64), lds, st, a);
    return hipGetLastError();
}

// Plan of the fused Relu + compress call on the shapes of the items kernel: the rounds a workgroup
// handles are rounded up until its mask bits are whole words.  False when the shape is not covered.
bool plan_relu_items(const Layout& L, int64_t H, int64_t W, int B, size_t es, const void* xy,
                     ItemsArgs* a, uint32_t* grid, size_t* lds, int* vec_out) {
    if (H == 1 || !plan_items(L, H, W, B, es, xy, a, grid, lds, vec_out)) return false;
    uint32_t m = 1;
    while (((uint64_t)m * a->ppr * L.HW) % 32 != 0) ++m;              // at most 16: H*W is even here
    a->rpw = (a->rpw + m - 1) / m * m;
    const uint64_t mbits = (uint64_t)a->rpw * a->ppr * L.HW;
    *lds = 4ull * (((uint64_t)a->ppr * L.WPP + 3) & ~3ull) + mbits / 8 + 16;
    *grid = (a->nrounds + a->rpw - 1) / a->rpw;
    return *lds <= 60u * 1024u;
}

// Fills the one-wavefront compress plan; false when the shape is not covered.
bool plan_wave(const Layout& L, int64_t H, int64_t W, int B, int b, size_t es, const void* x,
               WaveArgs* a, uint32_t* grid, size_t* lds, int* vec_out) {
    if (B != 4 && B != 8) return false;
    const uint64_t per_plane = 4ull * L.HW + 16ull;
    if (per_plane > kWavePlaneMax) return false;
    const int vec = (W % 4 == 0) ? 4 : (W % 2 == 0) ? 2 : 1;
    const uint32_t ipb = (uint32_t)B / (uint32_t)vec;
    const uint64_t slots = ((uint64_t)W + vec - 1) / vec;
    const uint64_t ipr = (slots + ipb - 1) / ipb * ipb;
    const uint64_t ipp = L.LH * ipr;
    uint64_t ippp = 1, lg = 0;
    if (ipp <= 64) { while (ippp < ipp) { ippp *= 2; ++lg; } }
    else ippp = (ipp + 63) / 64 * 64;
    uint64_t Gmax = kWaveChunkLds / per_plane;
    if (Gmax < 1) Gmax = 1;
    if (Gmax > L.P) Gmax = L.P;
    const uint64_t unit = 16 / gcd_u64(16, L.HW * es);
    uint32_t vec_load = ((uintptr_t)x % 16) == 0;
    if (vec_load && unit > 1 && Gmax < unit && Gmax < L.P) {
        if (unit * per_plane <= kWavePlaneMax) Gmax = unit; else vec_load = 0;
    }
    const uint64_t step = vec_load ? unit : 1;
    // pick the G that wastes the fewest lanes in partly filled rounds
    const uint64_t cpw = 32 / b, ppw = cpw / 2;
    const double c1 = 4.5 * B * vec, c3 = 8.5 * (double)cpw;
    uint64_t G = 0;
    double best = 0;
    for (uint64_t g = step; g <= Gmax; g += step) {
        const double r1 = ipp <= 64 ? (double)((g + 64 / ippp - 1) / (64 / ippp)) : (double)(g * (ippp / 64));
        const uint64_t nw = g * L.WPP, tw = nw % 64;
        const double r3 = (double)(nw / 64) + (tw == 0 ? 0.0 : tw * ppw <= 64 ? 0.25 : 1.0);
        const double per_elt = (r1 * c1 + r3 * c3 + 2.0) / (double)(g * L.HW);
        if (G == 0 || per_elt < best * 0.97) { G = g; best = per_elt; }
    }
    if (G == 0) G = Gmax;          // Gmax == P < unit: a single chunk, aligned at its start
    if (!fastdiv_ok(ippp, ipr) || !fastdiv_ok(G * L.WPP + 64, L.WPP)) return false;
    *a = WaveArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)L.LH; a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP;
    a->G = (uint32_t)G; a->ipr = (uint32_t)ipr; a->ipp = (uint32_t)ipp;
    a->ippp = (uint32_t)ippp; a->ippp_log2 = (uint32_t)lg;
    a->vec_load = vec_load;
    a->d_ipr = make_fastdiv((uint32_t)ipr);
    a->d_wpp = make_fastdiv((uint32_t)L.WPP);
    *lds = 16ull * G + 4ull * ((G * L.HW + 3) / 4 * 4) + 64;      // 16 floats of slack for ragged last words
    // the staging registers hold 16 x 64 vectors of 16 bytes
    if (vec_load && G * L.HW * es > 16ull * 1024ull) return false;
    *grid = (uint32_t)((L.P + G - 1) / G);
    *vec_out = vec;
    return true;
}

// Lanes per plane S (a power of two from min_log up) and rounds K of the instance (3, 4, 6 or 13) for
// planes of qv vectors: the pair that leaves the fewest of the K * S lane slots empty; among equals
// the one with more rounds (fewer, longer-lived lanes per plane measured better than many short ones).
bool pick_lanes_and_rounds(uint64_t qv, uint32_t min_log, uint32_t* S_out, uint32_t* log_out, uint32_t* K_out) {
    uint64_t best = 0;
    for (uint32_t lg = min_log; lg <= 6; ++lg) {
        const uint64_t S = 1ull << lg, R = (qv + S - 1) / S;
        if (R > 13) continue;
        const uint64_t K = R <= 3 ? 3 : R <= 4 ? 4 : R <= 6 ? 6 : 13;
        const uint64_t slots = K * S;
        if (best == 0 || slots < best || (slots == best && K > *K_out)) { best = slots; *S_out = (uint32_t)S; *log_out = lg; *K_out = (uint32_t)K; }
    }
    return best != 0;
}

// Fills the one-block plan: the block covers the plane, which is whole 16-byte vectors, at most
// kOneUnits per lane of a wavefront.
bool plan_one(const Layout& L, size_t es, const void* x, OneArgs* a, uint32_t* grid) {
    const uint64_t epv = 16 / es;
    if (L.nb != 1 || ((uintptr_t)x % 16) != 0 || L.HW % epv != 0) return false;
    const uint64_t qv = L.HW / epv;
    if (qv > (uint64_t)kOneUnits * 64) return false;
    // lanes per plane: a power of two from 4 up (a plane's lanes then read 64 contiguous bytes per round)
    uint32_t best_S = 0, best_log = 0, K = 0;
    if (!pick_lanes_and_rounds(qv, 2, &best_S, &best_log, &K)) return false;
    // Planes of 49 to 52 vectors (14 x 14): four lanes of thirteen rounds leave the fewest slots empty, but each round reads half a line.  Sixteen lanes of
    // four from a plane per CU on: 256 to 16384 planes of 14 x 14 4.1 -> 3.3 to 7.2 -> 6.0 us, 128 x 512 of them 19.0 -> 14.4; bfloat16 20 x 20 5.4 -> 3.6, 16384 of them
    // 8.3 -> 8.1.  Thirteen rounds leave no slot of 52 vectors empty: 2-byte ones (26 x 16) keep them from 128 planes per CU on, codes of four and eight bits up to
    // 256 (at 2 bits 24576 planes 9.5 us with thirteen rounds and 9.0 with four, 32768 10.6 and 10.9, 65536 17.5 and 18.7; at 4 bits 65536 19.1 and 19.4, 98304 28.2 and
    // 26.5; 4-byte ones gain at all sizes).
    const uint64_t cus = (uint64_t)num_cus();
    const bool fills = es == 2 && qv == 52 && L.P >= 128 * cus && (L.WPP * 32 <= 2 * L.HW || L.P < 256 * cus);
    if (best_S == 4 && K == 13 && L.P >= cus && !fills) { best_S = 16; best_log = 4; K = 4; }
    // Thirteen rounds are a long chain where the machine is nearly empty: as few as lanes allow that are at most eight wavefronts per CU.  150 drawn maps in
    // float / bfloat16 705 / 818 us; at limits of 1, 2, 4, 8 wavefronts 670, 666, 664, 662 / 744, 737, 729, 720, none slower (without a limit maps of 4 M elements
    // 1.10; instances of six rounds as well: 12 of 150 slower).  1-bit codes: from a plane per CU on (which instance takes fewer is pinned by name).
    if (K == 13 && (L.WPP * 32 >= 2 * L.HW || L.P >= cus))
        for (uint32_t lg = best_log + 1; lg <= 6; ++lg) {
            const uint64_t S = 1ull << lg, R = (qv + S - 1) / S;
            const uint32_t k = R <= 3 ? 3 : R <= 4 ? 4 : R <= 6 ? 6 : 13;
            if (k < K && L.P * S <= 8ull * 64 * cus) { best_S = (uint32_t)S; best_log = lg; K = k; }
        }
    *a = OneArgs{};
    a->P = (uint32_t)L.P; a->HW = (uint32_t)L.HW; a->WPP = (uint32_t)L.WPP;
    a->qv = (uint32_t)qv;
    a->S = best_S; a->S_log2 = best_log;
    a->ppw = 64u / best_S;
    a->K = K;
    a->NG = 1;
    *grid = (uint32_t)((L.P + a->ppw - 1) / a->ppw);
    return true;
}

// single-block planes of whole vectors: compress_one's, ahead of the kernels for general shapes
bool one_shape(const Layout& L, size_t es, const void* x) {
    OneArgs tmp{};
    uint32_t g = 0;
    return plan_one(L, es, x, &tmp, &g);
}

// Instance of compress_line: log2 of a block's vectors up to 2, beyond that block sums through LDS (-1), or with two
// rounds per block (-2).
int line_lu(const OneArgs& a) { return a.upb_log2 <= 2 ? (int)a.upb_log2 : a.upb > a.S ? -2 : -1; }

// Fills the plan of compress_line: a 1-D map (one row) of whole 16-byte vectors, several blocks per
// plane, a block a power-of-two number of vectors, at most kOneUnits vectors per lane.
bool plan_line(const Layout& L, int64_t D, int64_t H, int B, size_t es, const void* x, OneArgs* a, uint32_t* grid, size_t* lds) {
    const uint64_t epv = 16 / es;
    if (D != 1 || H != 1 || L.nb < 2 || ((uintptr_t)x % 16) != 0 || L.HW % epv != 0 || (uint64_t)B % epv != 0) return false;
    const uint64_t qv = L.HW / epv, upb = (uint64_t)B / epv;
    if ((upb & (upb - 1)) != 0 || upb > 64 || qv > (uint64_t)kLineUnits * 64) return false;
    uint32_t upb_log = 0;
    while ((1ull << upb_log) < upb) ++upb_log;
    // lanes per plane: a power of two that holds a block, or half of one that goes through LDS, at least 8 (a
    // plane's lanes then read 128 contiguous bytes per round)
    const uint32_t whole_log = upb_log > 3 ? upb_log : 3;
    uint32_t min_log = upb_log > 3 ? upb_log - 1 : 3;
    *a = OneArgs{};
    for (;; min_log = whole_log) {
        uint32_t best_S = 0, best_log = 0, K = 0;
        if (!pick_lanes_and_rounds(qv, min_log, &best_S, &best_log, &K)) return false;
        // planes of at most three rounds: twelve rounds of several plane groups per wavefront
        const uint32_t R = (uint32_t)((qv + best_S - 1) / best_S);
        a->NG = K == 3 ? 12u / R : 1u;
        a->K = K == 3 ? 12u : K;
        a->S = best_S; a->S_log2 = best_log;
        a->ppw = 64u / best_S;
        const uint64_t g = (L.P + (uint64_t)a->ppw * a->NG - 1) / ((uint64_t)a->ppw * a->NG);
        *grid = (uint32_t)g;
        // lanes for half a block may mean more and smaller wavefronts, too many for one launch of a map beyond 200 GB
        if (launch_ok(g, 64) || min_log == whole_log) break;
    }
    a->P = (uint32_t)L.P; a->HW = (uint32_t)L.HW; a->WPP = (uint32_t)L.WPP;
    a->qv = (uint32_t)qv;
    a->upb = (uint32_t)upb; a->upb_log2 = upb_log;
    a->nb = (uint32_t)L.nb;
    *lds = 0;
    const int lu = line_lu(*a);
    if (lu < 0) {
        // one binary64 partial sum per lane and round of blocks (a pad per block), one H^L per block
        const uint64_t Ri = a->K / a->NG, rows = a->NG * (lu == -2 ? (Ri + 1) / 2 : Ri);
        const uint64_t bpr = 64u >> (a->upb_log2 < a->S_log2 ? a->upb_log2 : a->S_log2);       // blocks per round
        *lds = (size_t)(rows * (64 + bpr) * 8 + rows * bpr * 4);
    }
    return true;
}

// 1-D maps the register kernel would take as well: compress_line is the faster one for 2-byte
// elements (it loads 16 bytes per lane, the register kernel 8); for fp32 the register kernel is (by 5-10 %)
bool line_first(const Layout& L, size_t es) { return es == 2 || L.HW / 4 < 512; }

// Fills the any-block-size compress plan; false when a plane does not fit LDS or the 32-bit index tricks.
// Hs = rows of one depth slice, D = depth slices (1 for a 2-D map).
bool plan_rows(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, int b, size_t es, const void* x,
               RowsArgs* a, uint32_t* grid, size_t* lds) {
    (void)b;
    const int64_t H = D * Hs;                       // rows of all slices
    if ((uint64_t)B > L.HW + 64) return false;      // keeps fdiv(r, B) exact; such a B is "one block" anyway: see below
    const uint64_t per_plane = 4ull * L.HW + 16ull * (uint64_t)H * L.LW + 12ull * L.nb + 16ull;
    if (per_plane + 256 > kLdsMax) return false;
    if (!fastdiv_ok(L.HW, (uint64_t)W) || !fastdiv_ok((uint64_t)(H > W ? H : W), (uint64_t)B)) return false;
    if (!fastdiv_ok((uint64_t)H, (uint64_t)Hs) || !fastdiv_ok(L.LD * L.LH, L.LH)) return false;
    uint64_t G = kRowsLdsTarget / per_plane;
    if (G < 1) G = 1;
    if (G > L.P) G = L.P;
    // chunk starts on 16-byte boundaries when G is a multiple of `unit`
    const uint64_t unit = 16 / gcd_u64(16, L.HW * es);
    uint32_t vec_load = ((uintptr_t)x % 16) == 0;
    if (vec_load && G % unit != 0) {
        if (G > unit) G -= G % unit;
        else if (unit * per_plane + 256 <= kLdsMax && unit <= L.P) G = unit;
        else if (G < L.P) vec_load = 0;
    }
    const uint64_t HLW = (uint64_t)H * L.LW;
    if (!fastdiv_ok(G * HLW + kThreads, HLW) || !fastdiv_ok(HLW, L.LW) || !fastdiv_ok(G * L.nb + kThreads, L.nb) ||
        !fastdiv_ok(L.nb, L.LW) || !fastdiv_ok(G * L.WPP + kThreads, L.WPP))
        return false;
    *a = RowsArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)(L.LD * L.LH); a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP; a->B = (uint32_t)B;
    a->D = (uint32_t)D; a->Hs = (uint32_t)Hs; a->LHs = (uint32_t)L.LH;
    a->G = (uint32_t)G;
    a->xs_floats = (uint32_t)((G * L.HW + 3) / 4 * 4);
    a->vec_load = vec_load;
    const uint64_t epv = 16 / es;
    a->keep = vec_load && (uint64_t)W % epv == 0 && G * (L.HW / epv) <= (uint64_t)kRowsKeep * kThreads;
    a->vecblk = a->keep && (uint64_t)B % epv == 0;
    a->qv = (uint32_t)(L.HW / epv);
    a->d_qv = make_fastdiv(a->qv ? a->qv : 1u);
    a->d_W = make_fastdiv((uint32_t)W);
    a->d_B = make_fastdiv((uint32_t)B);
    a->d_Hs = make_fastdiv((uint32_t)Hs);
    a->d_LHs = make_fastdiv((uint32_t)L.LH);
    a->d_LW = make_fastdiv((uint32_t)L.LW);
    a->d_HLW = make_fastdiv((uint32_t)HLW);
    a->d_nb = make_fastdiv((uint32_t)L.nb);
    a->d_wpp = make_fastdiv((uint32_t)L.WPP);
    *lds = 16ull * G + 4ull * a->xs_floats + 16ull * G * HLW + 4ull * ((G * L.nb + 1) & ~1ull) + 8ull * G * L.nb + 16;
    *grid = (uint32_t)((L.P + G - 1) / G);
    return *lds <= kLdsMax;
}

// Fills the workgroup-per-plane plan for planes beyond LDS; false when rows or blocks are not whole
// 16-byte vectors or the per-slice partial sums do not fit LDS.
bool plan_plane(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, size_t es, const void* x,
                PlaneArgs* a, uint32_t* grid, size_t* lds) {
    const uint64_t epv = 16 / es;
    if (((uintptr_t)x % 16) != 0 || (uint64_t)W % epv != 0 || (uint64_t)B % epv != 0) return false;
    const uint64_t H = (uint64_t)D * (uint64_t)Hs;
    const uint64_t slice = L.LH * L.LW;
    const uint64_t nitem = (uint64_t)D * slice;
    const uint64_t need = 16ull * nitem + 4ull * ((L.nb + 3) & ~3ull) + 8ull * (kThreads / 64) + 16 + 16;
    if (need > kLdsMax) return false;
    if (!fastdiv_ok(L.HW, (uint64_t)W) || !fastdiv_ok(H > (uint64_t)W ? H : (uint64_t)W, (uint64_t)B) ||
        !fastdiv_ok(H, (uint64_t)Hs) || !fastdiv_ok(nitem + kThreads, slice) || !fastdiv_ok(slice, L.LW))
        return false;
    *a = PlaneArgs{};
    a->P = (uint32_t)L.P; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW; a->LW = (uint32_t)L.LW;
    a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP; a->B = (uint32_t)B;
    a->D = (uint32_t)D; a->Hs = (uint32_t)Hs; a->LHs = (uint32_t)L.LH;
    a->nitem = (uint32_t)nitem;
    a->qv = (uint32_t)(L.HW / epv);
    a->d_W = make_fastdiv((uint32_t)W);
    a->d_B = make_fastdiv((uint32_t)B);
    a->d_Hs = make_fastdiv((uint32_t)Hs);
    a->d_LW = make_fastdiv((uint32_t)L.LW);
    a->d_LHs = make_fastdiv((uint32_t)L.LH);
    a->d_slice = make_fastdiv((uint32_t)slice);
    *lds = need;
    *grid = (uint32_t)L.P;
    return true;
}

// Fills the tiled-compress launch plan; false when the shape is not covered.
bool plan_tile(const Layout& L, int64_t H, int64_t W, int B, int b, size_t es, const void* x,
               TileArgs* a, uint32_t* grid, size_t* lds, int* vec_out, int* nt_out) {
    if (B != 4 && B != 8) return false;
    const int vec = (W % 4 == 0) ? 4 : (W % 2 == 0) ? 2 : 1;
    const uint32_t ipb = (uint32_t)B / (uint32_t)vec;
    const uint64_t slots = ((uint64_t)W + vec - 1) / vec;
    const uint64_t ipr = (slots + ipb - 1) / ipb * ipb;
    const uint64_t ipp = L.LH * ipr;
    const uint64_t per_plane = 4ull * L.HW + 8ull * ipp + 16ull;
    if (per_plane + 64 > kLdsMax) return false;
    const int nt = 256;
    uint64_t Gmax = kLdsTarget / per_plane;
    if (Gmax < 1) Gmax = 1;
    if (Gmax > L.P) Gmax = L.P;
    // chunk starts stay 16-byte aligned when G * (bytes per plane) is a multiple of 16
    const uint64_t unit = 16 / gcd_u64(16, L.HW * es);
    uint32_t vec_load = ((uintptr_t)x % 16) == 0;
    if (vec_load && unit > 1 && Gmax < unit && Gmax < L.P) {
        if (unit * per_plane + 64 <= kLdsMax) Gmax = unit; else vec_load = 0;
    }
    const uint64_t step = vec_load ? unit : 1;
    // pick the G whose last, partly filled wavefront pass wastes the fewest lanes
    const double c1 = 4.0 * B * vec, c3 = 7.5 * (32 / b);
    uint64_t G = 0;
    double best = 0;
    for (uint64_t g = step; g <= Gmax; g += step) {
        const double cost = (double)((g * ipp + 63) / 64) * c1 + (double)((g * L.WPP + 63) / 64) * c3;
        const double per_elt = cost / (double)(g * L.HW);
        if (G == 0 || per_elt < best * 0.98) { G = g; best = per_elt; }
    }
    if (G == 0) G = Gmax;          // Gmax == P < unit: a single chunk, aligned at its start
    const uint64_t nitems = G * ipp, nwords = G * L.WPP;
    if (!fastdiv_ok(nitems + 256, ipp) || !fastdiv_ok(ipp, ipr) || !fastdiv_ok(nwords + 256, L.WPP))
        return false;
    *a = TileArgs{};
    a->P = (uint32_t)L.P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)L.LH; a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP;
    a->G = (uint32_t)G; a->ipr = (uint32_t)ipr; a->ipp = (uint32_t)ipp;
    uint32_t S = 1;
    while (S < 64 && (uint64_t)S * 2 <= ipp) S *= 2;
    a->S = S;
    a->xs_floats = (uint32_t)((G * L.HW + 3) / 4 * 4);
    a->items_cap = (uint32_t)((nitems + 3) / 4 * 4);
    a->vec_load = vec_load;
    a->d_ipp = make_fastdiv((uint32_t)ipp);
    a->d_ipr = make_fastdiv((uint32_t)ipr);
    a->d_wpp = make_fastdiv((uint32_t)L.WPP);
    *lds = 16ull * G + 4ull * a->xs_floats + 8ull * a->items_cap;
    *grid = (uint32_t)((L.P + G - 1) / G);
    *vec_out = vec;
    *nt_out = nt;
    return *lds <= kLdsMax;
}

// LDS bytes of the streaming decompress kernels for G planes per workgroup
size_t dec_lds_bytes(const Layout& L, size_t es, uint64_t G) {
    return 4ull * ((G * L.WPP + 3) & ~(uint64_t)3) + 8ull * G + es * G * L.nb + 16;
}
constexpr size_t kDecLdsMax = 60u << 10;

// Planes per workgroup of the streaming decompress kernels: about 32 KB of output, in whole 128-byte
// lines where that is possible within twice the target, so that no line is shared by two
// workgroups.  Measured inside a whole compress + decompress step over the ResNet-50 set: 24-48 KB
// is the flat optimum (64 KB: 0.5-1 % slower, 12 KB: 4 % slower, 6 KB: 12 %).  A decompress kernel
// timed on its own, launch after launch, prefers 12 KB by 15 %, but not between other kernels.
// `mult`: G must be a multiple of it (flat kernel: whole 4-element vectors).
#ifndef DIVISION_DEC_CHUNK
#define DIVISION_DEC_CHUNK 32768
#endif
constexpr uint64_t kDecChunkBytes = DIVISION_DEC_CHUNK;
uint64_t dec_planes(const Layout& L, size_t es, uint64_t mult) {
    const uint64_t target = kDecChunkBytes / es;
    uint64_t G = (target + L.HW / 2) / L.HW;
    if (G < 1) G = 1;
    uint64_t unit = 128 / gcd_u64(128, L.HW * es);
    unit = unit / gcd_u64(unit, mult) * mult;
    if (unit * L.HW > 2 * target) unit = mult;
    G = (G + unit / 2) / unit * unit;
    if (G < unit) G = unit;
    if (G > L.P) G = L.P;
    return G;
}

// What the decompress kernels read of a shape whatever the plan.  Hs = rows of one depth slice, D = depth slices (1 for a 2-D map).
void dec_shape(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, DecShape* a) {
    a->P = (uint32_t)L.P; a->H = (uint32_t)(D * Hs); a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)(L.LD * L.LH); a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP; a->B = (uint32_t)B;
    a->Hs = (uint32_t)Hs; a->LHs = (uint32_t)L.LH;
    a->d_B = make_fastdiv((uint32_t)B);
    a->d_W = make_fastdiv((uint32_t)W);
    a->d_HW = make_fastdiv((uint32_t)L.HW);
    a->d_Hs = make_fastdiv((uint32_t)Hs);
    a->r_HW = 1.0 / (double)L.HW;
}
bool dec_small_idx(int64_t D, int64_t Hs, int64_t W, int B) {
    const uint64_t H = (uint64_t)(D * Hs);
    return fastdiv_ok(H, (uint64_t)B) && fastdiv_ok((uint64_t)W, (uint64_t)B) && fastdiv_ok(H, (uint64_t)Hs);
}

// decompress_stream: rows and blocks of whole pieces, one wavefront per 64 * kStreamK vectors, no staging; the lookups go by pieces
// of four elements, or of eight 2-byte elements where rows and blocks are whole vectors
bool plan_stream(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, size_t es, const void* xhat, DecShape* a, uint32_t* grid) {
    if (W % 4 != 0 || B % 4 != 0 || !dec_small_idx(D, Hs, W, B) || ((uintptr_t)xhat % 16) != 0) return false;
    const uint64_t pe = es == 2 && W % 8 == 0 && B % 8 == 0 ? 8 : 4;
    const uint64_t chunk = 64ull * kStreamK * (16 / es / pe);      // pieces
    const uint64_t q = L.HW / pe, npiece = L.P * q;
    // (2-byte maps of 256 GB and more: the staged kernel, whose workgroups rebuild 32 KB each)
    if (!fastdiv_ok(q + chunk, q) || !fastdiv_ok(q, (uint64_t)W / pe) || (npiece + chunk - 1) / chunk >= (1ull << 31) ||
        npiece >= (1ull << 40) || (es == 2 && !launch_ok((npiece + chunk - 1) / chunk, 64)))
        return false;
    a->whole8 = pe == 8;
    a->q4 = (uint32_t)q;
    a->r_q4 = 1.0 / (double)q;
    a->w4 = (uint32_t)((uint64_t)W / pe);
    a->d_q4 = make_fastdiv(a->q4);
    a->d_w4 = make_fastdiv(a->w4);
    *grid = (uint32_t)((npiece + chunk - 1) / chunk);
    return true;
}

// decompress_stream_any (several blocks per plane) and decompress_stream_one (one): rows, blocks or planes that are not whole
// vectors, a wavefront per chunk of aligned vectors, every element finds its own plane and block.
// (B >= 4 and W >= 4: a vector then leaves its row and its block column at most once, and no division is by 1; plane and plane
// count below 2^24 for the 24-bit multiplies; the three regions of the packed buffer within 32-bit byte offsets)
bool plan_any(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, size_t es, const void* xhat, uint32_t* grid) {
    if (L.HW < 4 || L.HW >= (1ull << 24) || L.P >= (1ull << 24) || ((uintptr_t)xhat % 16) != 0 || L.P * L.WPP * 4 >= (1ull << 31) ||
        L.P * L.nb * 4 >= (1ull << 31) || L.P * 8 >= (1ull << 31))
        return false;
    if (L.nb > 1 && (W < 4 || B < 4 || (D > 1 && Hs < 2) || !dec_small_idx(D, Hs, W, B) || !fastdiv_ok(L.HW, (uint64_t)W) ||
                     !fastdiv_ok((uint64_t)(D * Hs) + 1, (uint64_t)B)))
        return false;
    const uint64_t chunk = es == 2 ? kAnyChunk<bf16_t> : kAnyChunk<float>;     // elements
    const uint64_t ntot = L.P * L.HW;
    if (!fastdiv_ok(L.HW + chunk + 4, L.HW) || (ntot + chunk - 1) / chunk >= (1ull << 31) || ntot >= (1ull << 42)) return false;
    *grid = (uint32_t)((ntot + chunk - 1) / chunk);
    return true;
}


// the instances of decompress_units that look up per unit of four elements
bool units_wide(const DecShape& a) { return a.W >= 3 && a.B >= 3; }

// Fills the decompress launch plan; returns 7 (row vectors, a wavefront per chunk), 0 (row vectors of 2-byte elements, staged), 3 (block table),
// 8 (any width, a wavefront per chunk), 9 (the same for one-block planes), 6 (four consecutive elements
// per lane step, any width), 5 (word by word through LDS), 1 (flat), 4 (lane per plane) or 2 (scalar).
// Hs = rows of one depth slice, D = depth slices (1 for a 2-D map; the table kernel takes 2-D maps only).  maps: how many of them the launch holds.
int plan_decompress(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, size_t es, const void* xhat, uint64_t maps,
                    DecArgs* a, uint32_t* grid) {
    const int64_t H = D * Hs;
    dec_shape(L, D, Hs, W, B, a);
    const bool small_idx = dec_small_idx(D, Hs, W, B);
    const bool out_vec_aligned = ((uintptr_t)xhat % (4 * es)) == 0;
    // one-block planes with an odd element count: a lane per plane, 64 planes per round
    if (lane_shape(L)) {
        const uint32_t nrounds = (uint32_t)((L.P + 63) / 64);
        uint32_t rpw = 2;
        while (rpw > 1 && nrounds / rpw < 32u * (uint32_t)num_cus()) --rpw;
        a->G = rpw;
        *grid = (nrounds + rpw - 1) / rpw;
        return 4;
    }
    // 4-byte elements, one block per plane (not those of the lane kernel above, which measured the same on 7 x 7, nor those of
    // the row-vector stream kernel below): H^L is the plane's
    if (es == 4 && L.nb == 1 && !(W % 4 == 0 && B % 4 == 0) && plan_any(L, D, Hs, W, B, es, xhat, grid)) return 9;
    // fast path: rows are whole vectors that sit inside one block
    if (W % 4 == 0 && B % 4 == 0 && small_idx && out_vec_aligned) {
        if (plan_stream(L, D, Hs, W, B, es, xhat, a, grid)) return 7;
        // 2-byte maps that do not start on a 16-byte boundary, or are too large for one launch of the above (4-byte maps meet
        // neither: what the staged kernel's index tricks allow, the above's do)
        if (es == 2) {
            a->q4 = (uint32_t)(L.HW / 4);
            a->w4 = (uint32_t)(W / 4);
            uint64_t G = dec_planes(L, es, 1);
            while (G > 1 && !fastdiv_ok(G * a->q4 + kThreads, a->q4)) --G;
            if (fastdiv_ok(G * a->q4 + kThreads, a->q4) && fastdiv_ok(a->q4, a->w4) && dec_lds_bytes(L, es, G) <= kDecLdsMax) {
                a->G = (uint32_t)G;
                a->d_q4 = make_fastdiv(a->q4);
                a->d_w4 = make_fastdiv(a->w4);
                *grid = (uint32_t)((L.P + G - 1) / G);
                return 0;
            }
        }
    }
    // planes of whole vectors with few blocks: LFC indices from a table in LDS
    if (D == 1 && L.HW % 4 == 0 && L.nb > 1 && L.nb <= 255 && small_idx && out_vec_aligned && fastdiv_ok(L.HW, (uint64_t)W)) {
        a->q4 = (uint32_t)(L.HW / 4);
        uint64_t G = dec_planes(L, es, 1);
        // few planes in the launch: fewer of them per workgroup, down to a vector per lane, until every CU has a workgroup; where eight planes and more still share the
        // table, half as many up to six workgroups per CU, and again until there are three for two CUs (1216 planes of 14 x 14 in bfloat16 are 16 workgroups of 32 KB: 5.7 us,
        // 3.9 so; maps of up to 0.3 M elements 4.9 -> 3.7; until there are four for each CU, 14382 planes of 14 x 14 4.4 -> 4.8.  160 launches of one to eight maps 1047 us without,
        // 948 so; 955 without the halving up to six, 961 until a workgroup per CU where each map counted for itself.
        // Two of 1757 x 56 x 56 under B = 18, a few planes per workgroup, 6.9 and 7.3 when halved; one of 1040 x 1 x 3136 5.3 and 5.5)
        const uint64_t cus = (uint64_t)num_cus();
        auto halve = [&](uint64_t enough) { const bool few = G > 1 && (L.P + G - 1) / G * maps < enough && (G / 2) * a->q4 >= kThreads; if (few) G /= 2; return few; };
        if (G >= 16) halve(cus * 6);
        while (halve(G >= 16 ? cus * 3 / 2 : cus)) {}
        while (G > 1 && !fastdiv_ok(G * a->q4 + kThreads, a->q4)) --G;
        if (fastdiv_ok(G * a->q4 + kThreads, a->q4) && dec_lds_bytes(L, es, G) + 4ull * a->q4 + 16 <= kDecLdsMax) {
            a->G = (uint32_t)G;
            a->d_q4 = make_fastdiv(a->q4);
            *grid = (uint32_t)((L.P + G - 1) / G);
            return 3;
        }
    }
    // 4-byte elements, rows, blocks or planes that are not whole vectors, several blocks per plane
    if (es == 4 && L.nb > 1 && plan_any(L, D, Hs, W, B, es, xhat, grid)) return 8;
    // planes (2-D or 3-D) of 512 elements and more whose rows or blocks are not whole vectors: four consecutive
    // elements per lane step, planes starting on 4-byte boundaries
    if (Hs > 1 && small_idx && ((uintptr_t)xhat % 4) == 0 && L.nb <= 16383) {
        // units per plane, counting the one more that a plane starting 3 elements past a unit boundary takes
        const uint64_t q4 = (L.HW + (L.HW % 4 ? 6 : 0)) / 4;
        int nw = 1;
        while (nw < 16 && (q4 > (uint64_t)kUnitsK * 64 * nw || L.nb > (uint64_t)kUnitsLfc * 64 * nw)) nw *= 2;
        const uint64_t nt = 64ull * nw;
        if (q4 >= kUnitsMin && q4 <= (uint64_t)kUnitsK * nt && L.nb <= (uint64_t)kUnitsLfc * nt &&
            fastdiv_ok(4ull * kUnitsK * nt + 4, (uint64_t)W) && fastdiv_ok(4ull * kUnitsK * nt + 4, (uint64_t)B) &&
            fastdiv_ok(4ull * kUnitsK * nt + 4, (uint64_t)Hs)) {
            a->q4 = (uint32_t)q4;
            a->G = (uint32_t)nw;                  // wavefronts per workgroup
            uint64_t g = (uint64_t)num_cus() * (16ull / nw);
            g = (g + 3) & ~3ull;        // the planes of a workgroup start alike within a unit of the map
            *grid = (uint32_t)(g < L.P ? g : L.P);
            // few planes in the launch: the rounds of units of a plane shared among several workgroups, until there are half of what the machine holds; a third of workgroups of
            // one wavefront; as many as CUs of sixteen (maps of up to 0.3 M bfloat16 elements 5.5 -> 4.5 us; shared until it is full, 854 planes of 27 x 27
            // 4.8 -> 5.1, until half 576 of them 3.9 -> 4.0.  120 launches of one to eight maps 787 us, 692 so; 710 with a half for sixteen wavefronts too, 737 with a third of it
            // for each map by itself: eight of 300 x 27 x 27 6.3, 6.4, 6.4 and 8.5)
            const uint64_t rounds = (q4 + nt - 1) / nt;
            uint64_t parts = units_wide(*a) ? (nw == 16 ? g : nw == 1 ? g / 3 : g / 2) / (L.P * maps) : 1;
            if (parts > rounds) parts = rounds;
            a->rounds = (uint32_t)rounds;
            if (parts > 1) {
                a->rounds = (uint32_t)((rounds + parts - 1) / parts);
                *grid = (uint32_t)(L.P * ((rounds + a->rounds - 1) / a->rounds));
            }
            return 6;
        }
    }
    // 2-byte elements, planes below 512 elements or of one row: as 4-byte elements (64 x 768 x 17 x 17 14.0 us against 17.9 in
    // decompress_words, 64 x 1024 x 14 x 14 under B = 64 9.4 against 13.8 in decompress_flat; from 512 elements on decompress_units, which looks
    // nothing up per element, is level (35 x 35) or ahead (147 x 147: 46 us against 60); a map of one or two chunks is one or two
    // wavefronts' work there and four here)
    if (es == 2 && L.P * L.HW > 2 * kAnyChunk<bf16_t> && plan_any(L, D, Hs, W, B, es, xhat, grid)) return L.nb == 1 ? 9 : 8;
    // several blocks per plane, rows not whole vectors: rebuilt in LDS word by word
    if (L.nb > 1 && small_idx && out_vec_aligned && fastdiv_ok(L.HW, (uint64_t)W)) {
        const uint64_t unit = 4 / gcd_u64(4, L.HW);
        uint64_t G = dec_planes(L, 4, unit);          // the chunk is staged as fp32 whatever the element type
        const uint64_t staged = (dec_lds_bytes(L, es, G) + 15) & ~15ull;
        if (fastdiv_ok(G * L.WPP + kThreads, L.WPP) && staged + 4ull * ((G * L.HW + 3) & ~3ull) <= kDecLdsMax) {
            a->G = (uint32_t)G;
            a->out_off = (uint32_t)staged;
            a->d_wpp = make_fastdiv((uint32_t)L.WPP);
            *grid = (uint32_t)((L.P + G - 1) / G);
            return 5;
        }
    }
    // general path: flat run of G planes, G*HW a multiple of 4
    if (small_idx && out_vec_aligned && fastdiv_ok(L.HW, (uint64_t)W)) {
        const uint64_t unit = 4 / gcd_u64(4, L.HW);
        const uint64_t G = dec_planes(L, es, unit);
        if (fastdiv_ok(G * L.HW + 4ull * kThreads, L.HW) && dec_lds_bytes(L, es, G) <= kDecLdsMax) {
            a->G = (uint32_t)G;
            *grid = (uint32_t)((L.P + G - 1) / G);
            return 1;
        }
    }
    a->G = 1;
    *grid = (uint32_t)L.P;
    return 2;
}

// calls f(T{}, std::integral_constant<int, BITS>{}) for the element / cache type and code width of a call
// calls f(std::integral_constant<int, BITS>{}) for the code width of a call
template <typename F>
hipError_t with_bits(int b, F&& f) {
    return b == 2 ? f(std::integral_constant<int, 2>{}) : b == 4 ? f(std::integral_constant<int, 4>{})
                                                                  : f(std::integral_constant<int, 8>{});
}

// The kernel of a shape in a launch of several shapes: 7 (decompress_stream), 8 (_any), 9 (_one), or 0 where its maps have a launch
// of their own.  `maps` of the shape that another kernel serves better keep it when they are large: at 8 M elements what it gains
// (decompress_table 15 % on fp32 and 50-80 % on bfloat16 maps, decompress_units up to 30 %, decompress_lane 10 %) about equals what the
// launch costs.
int plan_mix(const Layout& L, int64_t D, int64_t Hs, int64_t W, int B, size_t es, const void* xhat, uint64_t maps, DecShape* a, uint32_t* grid) {
    DecArgs own{};
    const int kind = plan_decompress(L, D, Hs, W, B, es, xhat, maps, &own, grid);
    if (kind != 7 && kind != 8 && kind != 9) {
        if (kind == 0 || kind == 2 || maps * L.P * L.HW > (8u << 20) || !plan_any(L, D, Hs, W, B, es, xhat, grid)) return 0;
        *a = own;
        return L.nb == 1 ? 9 : 8;
    }
    *a = own;
    return kind;
}

enum CompKind { REGS, LANE, LINE, STRIP, ROWSTRIP, ITEMS, UNITS, SEG, WAVE, TILE, ONE, ROWS, PLANE, ANY, MIXED, LINES, PLANES };

// Everything a compress launch needs once the plan is made: the arguments of the kernel that was picked, which begin alike (head).  A
// plan zeroes them before it fills them in.
struct CompLaunch {
    int kind, B, vec, nt, nw, flat;
    uint32_t gx, gy;
    size_t lds;
    hipStream_t st;
    uint32_t seg_nt; int seg_K;                  // kind SEG: threads, items per lane
    union {
        CompHead head;
        TileArgs a; WaveArgs wa; RegsArgs ra; ItemsArgs ia; LaneArgs la; RowsArgs wa2; PlaneArgs pa; OneArgs oa; AnyArgs g; UnitsArgs ua; StripArgs sa; SegArgs sg;
        const MixedArgs* mixed;                  // kind MIXED (nt threads)
        struct { const LinesArgs* a; uint32_t K; int lu; } lines;      // kind LINES: the instance its shapes share
        struct { const PlanesArgs* a; bool all; } planes;              // kind PLANES
    };
};
struct MixLaunch { uint32_t grid; hipStream_t st; MixArgs a; };      // decompress_mixed
struct DecLaunch {
    int kind, flat, nw;
    uint32_t gx, gy;
    size_t lds;
    hipStream_t st;
    DecArgs a;
};

template <typename T, int BITS>
hipError_t launch_one(const OneArgs& a, dim3 gd, hipStream_t st) {
    void (*kern)(OneArgs) = a.K == 3 ? compress_one<T, BITS, 3> : a.K == 4 ? compress_one<T, BITS, 4> : a.K == 6 ? compress_one<T, BITS, 6> : compress_one<T, BITS, 13>;
    hipLaunchKernelGGL(kern, gd, dim3(64), 0, st, a);
    return hipGetLastError();
}
template <typename T, int BITS, int LU>
hipError_t launch_line_lu(const OneArgs& a, dim3 gd, size_t lds, hipStream_t st) {
    void (*kern)(OneArgs);
    if (a.K == 12) {
        if constexpr (LU == -2) kern = compress_line<T, BITS, 12, 4, LU>;              // (blocks of two rounds, several per plane: three rounds)
        else kern = a.NG == 12 ? compress_line<T, BITS, 12, 12, LU> : a.NG == 6 ? compress_line<T, BITS, 12, 6, LU> : compress_line<T, BITS, 12, 4, LU>;
    } else kern = a.K == 4 ? compress_line<T, BITS, 4, 1, LU> : a.K == 6 ? compress_line<T, BITS, 6, 1, LU> : compress_line<T, BITS, 13, 1, LU>;
    hipLaunchKernelGGL(kern, gd, dim3(64), lds, st, a);
    return hipGetLastError();
}
template <typename T, int BITS>
hipError_t launch_line(const OneArgs& a, dim3 gd, size_t lds, hipStream_t st) {
    switch (line_lu(a)) {
        case 0: return launch_line_lu<T, BITS, 0>(a, gd, lds, st);
        case 1: return launch_line_lu<T, BITS, 1>(a, gd, lds, st);
        case 2: return launch_line_lu<T, BITS, 2>(a, gd, lds, st);
        case -1: return launch_line_lu<T, BITS, -1>(a, gd, lds, st);
        default: return launch_line_lu<T, BITS, -2>(a, gd, lds, st);
    }
}

template <typename T, int BITS>
hipError_t launch_lines(const LinesArgs& a, uint32_t K, int lu, dim3 gd, size_t lds, hipStream_t st) {
    void (*kern)(LinesArgs);
    switch (lu) {
        case 0: kern = K == 4 ? compress_lines<T, BITS, 4, 0> : compress_lines<T, BITS, 6, 0>; break;
        case 1: kern = K == 4 ? compress_lines<T, BITS, 4, 1> : compress_lines<T, BITS, 6, 1>; break;
        case 2: kern = K == 4 ? compress_lines<T, BITS, 4, 2> : compress_lines<T, BITS, 6, 2>; break;
        case -1: kern = K == 4 ? compress_lines<T, BITS, 4, -1> : compress_lines<T, BITS, 6, -1>; break;
        default: kern = K == 4 ? compress_lines<T, BITS, 4, -2> : compress_lines<T, BITS, 6, -2>;
    }
    hipLaunchKernelGGL(kern, gd, dim3(64), lds, st, a);
    return hipGetLastError();
}

template <typename T, int BITS>
hipError_t launch_planes(const PlanesArgs& a, bool all, dim3 gd, size_t lds, hipStream_t st) {
    void (*kern)(PlanesArgs) = all ? compress_planes<T, BITS, true> : compress_planes<T, BITS, false>;
    hipLaunchKernelGGL(kern, gd, dim3(64), lds, st, a);
    return hipGetLastError();
}

template <typename T, int BITS>
hipError_t launch_mixed(const MixedArgs& a, dim3 gd, int nt, size_t lds, hipStream_t st) {
    void (*kern)(MixedArgs) = compress_mixed<T, BITS>;
    const hipError_t e = allow_large_lds(kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, gd, dim3(nt), lds, st, a);
    return hipGetLastError();
}

template <typename T>
hipError_t do_compress(const CompLaunch& c, int b) {
    const dim3 gd(c.gx, c.gy);
    hipStream_t st = c.st;
    const size_t lds = c.lds;
    const bool flat = c.flat != 0;
    if (b == 1) {
        // 1-bit codes: the kernels that have an instance for them (the planner picks nothing else)
        switch (c.kind) {
            case REGS: return launch_regs<T, 1>(c.B, c.nw, c.ra, gd, lds, st);
            case STRIP: return launch_strip<T, 1>(c.vec, c.sa, gd, lds, st);
            case ROWSTRIP: return launch_rowstrip<T, 1>(c.vec, c.sa, gd, lds, st);
            case LANE: hipLaunchKernelGGL((compress_lane<T, 1>), gd, dim3(64), lds, st, c.la); return hipGetLastError();
            case ITEMS: return launch_items<T, 1>(c.B, c.vec, c.ia, gd, lds, st);
            case UNITS: return launch_units<T, 1>(c.nw, c.ua, gd, lds, st);
            case SEG: return launch_seg<T, 1>(c.seg_K, c.B, c.sg, c.seg_nt, gd, lds, st);
            case ONE: return launch_one<T, 1>(c.oa, gd, st);
            case LINE: return launch_line<T, 1>(c.oa, gd, lds, st);
            case TILE: return launch_tile<T, 1>(c.B, c.vec, c.a, gd, lds, st);
            case MIXED: return launch_mixed<T, 1>(*c.mixed, gd, c.nt, lds, st);
            case LINES: return launch_lines<T, 1>(*c.lines.a, c.lines.K, c.lines.lu, gd, lds, st);
            case PLANES: return launch_planes<T, 1>(*c.planes.a, c.planes.all, gd, lds, st);
            default: {
                void (*kern)(AnyArgs) = flat ? compress_any<T, 1> : compress_any_3d<T, 1>;
                hipLaunchKernelGGL(kern, gd, dim3(c.nt), 0, st, c.g);
                return hipGetLastError();
            }
        }
    }
    return with_bits(b, [&](auto bits) -> hipError_t {
        constexpr int BITS = decltype(bits)::value;
        switch (c.kind) {
            case REGS: return launch_regs<T, BITS>(c.B, c.nw, c.ra, gd, lds, st);
            case STRIP: return launch_strip<T, BITS>(c.vec, c.sa, gd, lds, st);
            case ROWSTRIP: return launch_rowstrip<T, BITS>(c.vec, c.sa, gd, lds, st);
            case ITEMS: return launch_items<T, BITS>(c.B, c.vec, c.ia, gd, lds, st);
            case UNITS: return launch_units<T, BITS>(c.nw, c.ua, gd, lds, st);
            case SEG: return launch_seg<T, BITS>(c.seg_K, c.B, c.sg, c.seg_nt, gd, lds, st);
            case WAVE: return launch_wave<T, BITS>(c.B, c.vec, c.wa, gd, lds, st);
            case TILE: return launch_tile<T, BITS>(c.B, c.vec, c.a, gd, lds, st);
            case LANE: hipLaunchKernelGGL((compress_lane<T, BITS>), gd, dim3(64), lds, st, c.la); return hipGetLastError();
            case ONE: return launch_one<T, BITS>(c.oa, gd, st);
            case LINE: return launch_line<T, BITS>(c.oa, gd, lds, st);
            case MIXED: return launch_mixed<T, BITS>(*c.mixed, gd, c.nt, lds, st);
            case LINES: return launch_lines<T, BITS>(*c.lines.a, c.lines.K, c.lines.lu, gd, lds, st);
            case PLANES: return launch_planes<T, BITS>(*c.planes.a, c.planes.all, gd, lds, st);
            case ROWS: {
                void (*kern)(RowsArgs) = flat ? compress_rows<T, BITS> : compress_rows_3d<T, BITS>;
                const hipError_t e = allow_large_lds(kern, lds);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(kern, gd, dim3(kThreads), lds, st, c.wa2);
                return hipGetLastError();
            }
            case PLANE: {
                void (*kern)(PlaneArgs) = flat ? compress_plane<T, BITS> : compress_plane_3d<T, BITS>;
                const hipError_t e = allow_large_lds(kern, lds);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(kern, gd, dim3(kThreads), lds, st, c.pa);
                return hipGetLastError();
            }
            default: {
                void (*kern)(AnyArgs) = flat ? compress_any<T, BITS> : compress_any_3d<T, BITS>;
                hipLaunchKernelGGL(kern, gd, dim3(c.nt), 0, st, c.g);
                return hipGetLastError();
            }
        }
    });
}


template <typename T>
hipError_t do_decompress(const DecLaunch& c, int b) {
    // every decompress kernel has an instance for 1-bit codes too
    auto launch = [&](auto bits) -> hipError_t {
        constexpr int BITS = decltype(bits)::value;
        const int kind = c.kind;
        void (*kern)(DecArgs);
        if (kind == 7 || kind == 8 || kind == 9) {
            kern = c.flat ? decompress_stream<T, BITS> : decompress_stream_3d<T, BITS>;
            if (kind == 9) kern = decompress_stream_one<T, BITS>;
            else if (kind == 8) kern = c.flat ? decompress_stream_any<T, BITS> : decompress_stream_any_3d<T, BITS>;
            hipLaunchKernelGGL(kern, dim3(c.gx, c.gy), dim3(64), 0, c.st, c.a);
            return hipGetLastError();
        }
        if (kind == 6) {
            if (units_wide(c.a))
                kern = c.nw == 1 ? decompress_units<T, BITS, 1> : c.nw == 2 ? decompress_units<T, BITS, 2>
                     : c.nw == 4 ? decompress_units<T, BITS, 4> : c.nw == 8 ? decompress_units<T, BITS, 8>
                                                                            : decompress_units<T, BITS, 16>;
            else
                kern = c.nw == 1 ? decompress_units<T, BITS, 1, 1> : c.nw == 2 ? decompress_units<T, BITS, 2, 1>
                     : c.nw == 4 ? decompress_units<T, BITS, 4, 1> : c.nw == 8 ? decompress_units<T, BITS, 8, 1>
                                                                                 : decompress_units<T, BITS, 16, 1>;
            hipLaunchKernelGGL(kern, dim3(c.gx, c.gy), dim3(64 * c.nw), c.lds, c.st, c.a);
            return hipGetLastError();
        }
        if (c.flat)
            kern = kind == 3 ? decompress_table<T, BITS>
                 : kind == 5 ? decompress_words<T, BITS> : kind == 1 ? decompress_flat<T, BITS>
                 : kind == 4 ? decompress_lane<T, BITS> : decompress_scalar<T, BITS>;
        else
            kern = kind == 5 ? decompress_words_3d<T, BITS>
                 : kind == 1 ? decompress_flat_3d<T, BITS>
                 : kind == 4 ? decompress_lane<T, BITS> : decompress_scalar_3d<T, BITS>;
        if constexpr (sizeof(T) == 2) {                      // (and kind 0 to no others)
            if (kind == 0) kern = c.flat ? decompress_rowvec<T, BITS> : decompress_rowvec_3d<T, BITS>;
        }
        const hipError_t e = allow_large_lds(kern, c.lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(c.gx, c.gy), dim3(kind == 4 ? 64 : kThreads), c.lds, c.st, c.a);
        return hipGetLastError();
    };
    return b == 1 ? launch(std::integral_constant<int, 1>{}) : with_bits(b, launch);
}

template <typename T>
hipError_t do_decompress_mixed(const MixLaunch& c, int b) {
    auto launch = [&](auto bits) -> hipError_t {
        hipLaunchKernelGGL((decompress_mixed<T, decltype(bits)::value>), dim3(c.grid), dim3(64), 0, c.st, c.a);
        return hipGetLastError();
    };
    return b == 1 ? launch(std::integral_constant<int, 1>{}) : with_bits(b, launch);
}

// the Relu + compress kernels: the register kernel's planes (c.ra carries y and mask), c.kind == STRIP the
// strip kernel's (c.sa) or, c.kind == ITEMS, the items kernel's (c.ia); one map per launch
template <typename T>
hipError_t do_relu(const CompLaunch& c, int b) {
    return with_bits(b, [&](auto bits) -> hipError_t {
        constexpr int BITS = decltype(bits)::value;
        if (c.kind == ITEMS) return launch_relu_items<T, BITS>(c.B, c.vec, c.ia, dim3(c.gx, 1), c.lds, c.st);
        if (c.kind == STRIP) return launch_relu_strip<T, BITS>(c.vec, c.sa, dim3(c.gx, 1), c.lds, c.st);
        void (*kern)(RegsArgs);
        if (c.nw == 1) kern = c.B == 8 ? relu_compress_regs<T, BITS, 8, 1> : relu_compress_regs<T, BITS, 4, 1>;
        else kern = c.B == 8 ? relu_compress_regs<T, BITS, 8, 4> : relu_compress_regs<T, BITS, 4, 4>;
        hipLaunchKernelGGL(kern, dim3(c.gx, 1), dim3(64 * c.nw), c.lds, c.st, c.ra);
        return hipGetLastError();
    });
}

hipError_t bridge_compress(division_dtype dt, const CompLaunch& c, int b) {
    return dt == DIVISION_F32 ? division_bridge_compress_f32(&c, b)
         : dt == DIVISION_BF16 ? division_bridge_compress_bf16(&c, b) : division_bridge_compress_c16(&c, b);
}
hipError_t bridge_decompress(division_dtype dt, const DecLaunch& c, int b) {
    return dt == DIVISION_F32 ? division_bridge_decompress_f32(&c, b)
         : dt == DIVISION_BF16 ? division_bridge_decompress_bf16(&c, b) : division_bridge_decompress_c16(&c, b);
}
hipError_t bridge_decompress_mixed(division_dtype dt, const MixLaunch& c, int b) {
    return dt == DIVISION_F32 ? division_bridge_decompress_mixed_f32(&c, b)
         : dt == DIVISION_BF16 ? division_bridge_decompress_mixed_bf16(&c, b) : division_bridge_decompress_mixed_c16(&c, b);
}
hipError_t bridge_relu(division_dtype dt, const CompLaunch& c, int b) {
    return dt == DIVISION_F32 ? division_bridge_relu_f32(&c, b)
         : dt == DIVISION_BF16 ? division_bridge_relu_bf16(&c, b) : division_bridge_relu_c16(&c, b);
}

// A 3-D map with a dimension of extent 1 is a 2-D map with the same flat element order, the same
// blocks and the same packed buffer: D x 1 x W -> D x W, D x H x 1 -> D x H.  (1 x H x W needs nothing.)
void squeeze_dims(int64_t& D, int64_t& H, int64_t& W) {
    if (D > 1 && H == 1) { H = D; D = 1; }
    else if (D > 1 && W == 1) { W = H; H = D; D = 1; }
}

// A plane that is a single block has the same cached tuple under every block size that covers it:
// small 2-D planes are handed to the kernels specialised for B = 4 and B = 8.
int covering_block(const Layout& L, int64_t D, int64_t H, int64_t W, int B) {
    if (L.nb != 1 || D != 1) return B;
    const int64_t m = H > W ? H : W;
    return m <= 4 ? 4 : m <= 8 ? 8 : B;
}

int packed_layout_impl(int64_t N, int64_t C, int64_t D, int64_t H, int64_t W, int B, int b, division_dtype dt,
                       size_t* codes_off, size_t* codes_bytes, size_t* meta_off, size_t* meta_bytes,
                       size_t* lfc_off, size_t* lfc_bytes) {
    if (!codes_off || !codes_bytes || !meta_off || !meta_bytes || !lfc_off || !lfc_bytes) return DIVISION_EINVAL;
    Layout L;
    if (make_layout(N, C, D, H, W, B, b, (int)dt, &L) != DIVISION_OK) return DIVISION_EINVAL;
    *codes_off = L.codes_off; *codes_bytes = L.codes_bytes;
    *meta_off = L.meta_off;   *meta_bytes = L.meta_bytes;
    *lfc_off = L.lfc_off;     *lfc_bytes = L.lfc_bytes;
    return DIVISION_OK;
}

// The kernel of a map, or of `maps` maps of one shape in one launch: kind, grid, LDS and arguments, all but the maps themselves (head) and
// what the caller adds (stream).  x: the OR of the maps' addresses (their common alignment).
void plan_compress(const Layout& L, int64_t D, int64_t H, int64_t W, int B, int b, size_t es, const void* x, int maps, CompLaunch* c) {
    size_t& lds = c->lds;
    uint32_t& grid = c->gx;
    const bool flat = D == 1;               // the register, item, wavefront and tile kernels take 2-D maps
    // 1-bit codes (Q = 1) have no instance of the wave, rows and plane kernels, nor of the units kernel with
    // sixteen wavefronts: the wave kernel's shapes go to the tile kernel, the others to the general kernel
    const bool wide = b != 1;
    lds = 0;
    c->B = B; c->vec = 1; c->nt = 64; c->nw = 1; c->flat = flat;
    if (line_first(L, es) && plan_line(L, D, H, B, es, x, &c->oa, &grid, &lds)) c->kind = LINE;
    else if (plan_regs(L, D, H, W, B, es, x, &c->ra, &grid, &lds, &c->nw)) c->kind = REGS;
    else if (plan_lane(L, es, x, &c->la, &grid, &lds)) c->kind = LANE;
    else if (plan_line(L, D, H, B, es, x, &c->oa, &grid, &lds)) c->kind = LINE;
    else if (flat && plan_strip(L, H, W, B, es, x, &c->sa, &grid, &lds, &c->vec)) c->kind = STRIP;
    else if (flat && plan_rowstrip(L, H, W, B, es, x, &c->sa, &grid, &lds, &c->vec)) c->kind = ROWSTRIP;
    else if (flat && plan_items(L, H, W, B, es, x, &c->ia, &grid, &lds, &c->vec)) c->kind = ITEMS;
    else if (!one_shape(L, es, x) && plan_units(L, D, H, W, B, b, es, x, maps, &c->ua, &grid, &lds, &c->nw) && (wide || c->nw != 16)) c->kind = UNITS;
    else if (wide && flat && plan_wave(L, H, W, B, b, es, x, &c->wa, &grid, &lds, &c->vec)) c->kind = WAVE;
    else if (flat && plan_tile(L, H, W, B, b, es, x, &c->a, &grid, &lds, &c->vec, &c->nt)) c->kind = TILE;
    else if (plan_one(L, es, x, &c->oa, &grid)) { c->kind = ONE; lds = 0; }
    else if (wide && plan_rows(L, D, H, W, B, b, es, x, &c->wa2, &grid, &lds)) c->kind = ROWS;
    else if (wide && plan_plane(L, D, H, W, B, es, x, &c->pa, &grid, &lds)) c->kind = PLANE;
    else {
        c->kind = ANY;
        AnyArgs& g = c->g;
        g = AnyArgs{};
        g.P = (uint32_t)L.P; g.H = (uint32_t)H; g.W = (uint32_t)W; g.HW = (uint32_t)L.HW; g.D = (uint32_t)D;
        g.LH = (uint32_t)L.LH; g.LW = (uint32_t)L.LW; g.nb = (uint32_t)L.nb; g.WPP = (uint32_t)L.WPP; g.B = (uint32_t)B;
        grid = (uint32_t)L.P;
        // a wavefront, four or sixteen per plane: one to sixteen rounds of four elements per lane; more lanes than 256 only
        // where the launch still has fewer than 2^32
        c->nt = L.HW <= 1024 ? 64 : L.HW <= 8192 || !launch_ok(L.P, 1024) ? kThreads : 1024;
        // lanes per block: as many as there are, with a round of eight elements and more for each
        const uint64_t elements = (uint64_t)std::min<int64_t>(B, W) * (uint64_t)std::min<int64_t>(B, H) * (uint64_t)std::min<int64_t>(B, D);
        while (g.J_log2 < 6 && (L.nb << (g.J_log2 + 1)) <= (uint64_t)c->nt && (16ull << g.J_log2) <= elements) ++g.J_log2;
    }
    SegArgs sg;
    if (c->kind == UNITS && plan_seg(L, D, H, W, B, es, &sg, &grid, &lds, &c->seg_nt, &c->seg_K)) { c->kind = SEG; c->sg = sg; }
    c->gy = (uint32_t)maps;                 // of the grid: the maps, or one where the workgroups walk over all of them
    if (c->kind == REGS && c->nw == 16 && regs_walk(L.P * (uint64_t)maps, L.HW / 4)) { c->ra.maps = c->gy; c->gy = 1; grid = (uint32_t)num_cus(); }
}

// Makes the launch that is planned for `count` maps (at most kMaxBatch) of a shape.
int launch_compress(CompLaunch& c, const Regions& rg, int count, const void* const* x, void* const* packed, const uint64_t* seeds,
                    division_dtype dt, int b, hipStream_t st) {
    c.st = st;
    c.head.rg = rg;
    CompTab& tab = c.head.tab;
    for (int i = 0; i < count; ++i) {
        tab.x[i] = x[i];
        tab.pk[i] = packed[i];
        tab.seed_a[i] = seed_key_a(seeds[i]);
        tab.seed_c[i] = seed_key_c(seeds[i]);
    }
    return bridge_compress(dt, c, b) == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
}

int compress_impl(int count, const void* const* x, void* const* packed, const uint64_t* seeds,
                  int64_t N, int64_t C, int64_t D, int64_t H, int64_t W, division_dtype dt,
                  int B, int b, size_t packed_capacity, void* hip_stream) {
    if (count < 0 || (count > 0 && (!x || !packed || !seeds))) return DIVISION_EINVAL;
    squeeze_dims(D, H, W);
    Layout L;
    const int rc = make_layout(N, C, D, H, W, B, b, (int)dt, &L);
    if (rc != DIVISION_OK) return rc;
    B = covering_block(L, D, H, W, B);
    if (packed_capacity < L.total) return DIVISION_ESIZE;
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    uintptr_t all_x = 0;            // alignment of the batch = alignment of the OR of its pointers
    for (int i = 0; i < count; ++i) {
        if (!x[i] || !packed[i]) return DIVISION_EINVAL;
        if (((uintptr_t)x[i] % es) != 0 || ((uintptr_t)packed[i] % 16) != 0) return DIVISION_EALIGN;
        all_x |= (uintptr_t)x[i];
    }
    const void* xa = reinterpret_cast<const void*>(all_x ? all_x : 16);
    const Regions rg = make_regions(L);

    for (int i0 = 0; i0 < count; i0 += kMaxBatch) {
        const int cnt = count - i0 < kMaxBatch ? count - i0 : kMaxBatch;
        CompLaunch c;
        plan_compress(L, D, H, W, B, b, es, xa, cnt, &c);
        const int err = launch_compress(c, rg, cnt, x + i0, packed + i0, seeds + i0, dt, b, static_cast<hipStream_t>(hip_stream));
        if (err != DIVISION_OK) return err;
    }
    return DIVISION_OK;
}

int decompress_impl(int count, const void* const* packed, void* const* xhat, size_t packed_bytes,
                    int64_t N, int64_t C, int64_t D, int64_t H, int64_t W, division_dtype dt,
                    int B, int b, void* hip_stream) {
    if (count < 0 || (count > 0 && (!packed || !xhat))) return DIVISION_EINVAL;
    squeeze_dims(D, H, W);
    Layout L;
    const int rc = make_layout(N, C, D, H, W, B, b, (int)dt, &L);
    if (rc != DIVISION_OK) return rc;
    B = covering_block(L, D, H, W, B);
    if (packed_bytes < L.total) return DIVISION_ESIZE;
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    uintptr_t all_out = 0;
    for (int i = 0; i < count; ++i) {
        if (!xhat[i] || !packed[i]) return DIVISION_EINVAL;
        if (((uintptr_t)xhat[i] % es) != 0 || ((uintptr_t)packed[i] % 16) != 0) return DIVISION_EALIGN;
        all_out |= (uintptr_t)xhat[i];
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const Regions rg = make_regions(L);

    for (int i0 = 0; i0 < count; i0 += kMaxBatch) {
        const int cnt = count - i0 < kMaxBatch ? count - i0 : kMaxBatch;
        DecArgs a{};
        uint32_t grid = 0;
        const int kind = plan_decompress(L, D, H, W, B, es, reinterpret_cast<const void*>(all_out ? all_out : 16), (uint64_t)cnt, &a, &grid);
        for (int i = 0; i < cnt; ++i) { a.tab.pk[i] = packed[i0 + i]; a.tab.xhat[i] = xhat[i0 + i]; }
        a.rg = rg;
        // LDS of the streaming kernels: staged codes, meta and LFC of G planes (+ the block table)
        size_t lds = 0;
        if (kind == 4) lds = 4ull * (64ull * L.HW + 4);
        else if (kind == 6) lds = 8ull * ((L.nb + 3) & ~3ull);
        else if (kind == 7 || kind == 8 || kind == 9) lds = 0;
        else if (kind == 5) lds = a.out_off + 4ull * ((a.G * L.HW + 3) & ~3ull);
        else if (kind != 2) lds = dec_lds_bytes(L, es, a.G) + (kind == 3 ? 4ull * a.q4 + 16 : 0);
        DecLaunch c{};
        c.kind = kind; c.flat = D == 1; c.nw = kind == 6 ? (int)a.G : 0; c.gx = grid; c.gy = (uint32_t)cnt; c.lds = lds; c.st = st; c.a = a;
        if (bridge_decompress(dt, c, b) != hipSuccess) return DIVISION_EHIP;
    }
    return DIVISION_OK;
}

// What follows from the lanes per plane; the LDS of a workgroup of `threads`
size_t fit_mixed(MixedShape* a, uint32_t threads) {
    const uint64_t S = 1ull << a->S_log2;
    for (const uint32_t k : {1u, 2u, 3u, 4u, 6u, 8u}) { a->K = k; if (k * S >= a->q4) break; }
    const uint64_t runs = (uint64_t)std::min(a->B, a->D) * a->Br * a->nch;      // of a block
    a->J_log2 = 0;
    while (((uint64_t)a->nb << (a->J_log2 + 1)) <= S && (2ull << a->J_log2) <= runs) ++a->J_log2;
    a->reg_bytes = (uint32_t)((16 * a->K * S + 8 * (S / 16 + 1) + 4ull * (a->nb + 1) + 8 * (S / 64) + 15) & ~15ull);
    a->G = std::min(threads >> a->S_log2, a->P);
    while (a->G > 1 && (size_t)a->reg_bytes * a->G > kLdsMax / 2) a->G /= 2;
    while (((uint64_t)a->G << a->S_log2) % 64 != 0) ++a->G;      // whole wavefronts
    return (size_t)a->reg_bytes * a->G;
}

// Lanes, workgroups and LDS of a launch of several shapes.  Lanes per plane double where a lane has most units, while all of them
// are on the machine at once (sixteen wavefronts per CU).
void spread_mixed(MixedArgs& a, const uint32_t* maps, uint32_t shapes, uint32_t* grid, int* threads, size_t* lds) {
    const uint64_t most = (uint64_t)num_cus() * 1024;
    auto units = [&](const MixedShape& s) { return (s.q4 + (1u << s.S_log2) - 1) >> s.S_log2; };
    uint64_t lanes = 0;
    for (uint32_t s = 0; s < shapes; ++s) lanes += ((uint64_t)maps[s] * a.shape[s].P) << a.shape[s].S_log2;
    for (;;) {
        int at = -1;
        uint32_t worst = 1;
        for (uint32_t s = 0; s < shapes; ++s)
            if (units(a.shape[s]) > worst && (1u << a.shape[s].S_log2) < (uint32_t)kMixedThreads) { worst = units(a.shape[s]); at = (int)s; }
        if (at < 0) break;
        const uint64_t more = ((uint64_t)maps[at] * a.shape[at].P) << a.shape[at].S_log2;
        if (lanes + more > most) break;
        lanes += more;
        ++a.shape[at].S_log2;
    }
    uint32_t nt = 256;
    for (uint32_t s = 0; s < shapes; ++s) nt = std::max(nt, 1u << a.shape[s].S_log2);
    *grid = 0;
    *lds = 0;
    for (uint32_t s = 0; s < (uint32_t)kSharedShapes; ++s) a.first[s] = 0xffffffffu;
    for (uint32_t s = 0; s < shapes; ++s) {
        *lds = std::max(*lds, fit_mixed(&a.shape[s], nt));
        a.chunks[s] = (a.shape[s].P + a.shape[s].G - 1) / a.shape[s].G;
        a.first[s] = *grid;
        *grid += a.chunks[s] * maps[s];
    }
    *threads = (int)nt;
}

// log2 of the fewest lanes per plane that compress_mixed takes a plane of HW elements with (at most kMixedUnits units of four per lane)
uint32_t mixed_lanes_log2(uint64_t HW) {
    uint32_t lg = 3;
    while ((HW + 3) / 4 > (uint64_t)kMixedUnits << lg) ++lg;
    return lg;
}

// Fills what compress_mixed needs of a shape, with as few lanes per plane as take it; false when the shape is not covered.
// x: the OR of its maps' addresses.
bool plan_mixed(const Layout& L, int64_t D, int64_t H, int64_t W, int B, const void* x, MixedShape* a) {
    const uint64_t q4 = (L.HW + 3) / 4, most = (uint64_t)kMixedUnits * kMixedThreads;
    if (((uintptr_t)x % 4) != 0 || q4 > most || L.nb > 16383 || B > 32767) return false;      // H^L offsets are 16-bit byte offsets
    const uint64_t Br = (uint64_t)std::min<int64_t>(B, H), nch = ((uint64_t)std::min<int64_t>(B, W) + 7) / 8, top = 4 * most + 4;
    if (!fastdiv_ok(top, (uint64_t)W) || !fastdiv_ok(top, (uint64_t)B) || !fastdiv_ok(top, (uint64_t)H) || !fastdiv_ok(L.nb + kMixedThreads, L.LW) ||
        !fastdiv_ok(L.nb + kMixedThreads, L.LH * L.LW) || !fastdiv_ok(top, nch) || !fastdiv_ok(top, Br))
        return false;
    a->P = (uint32_t)L.P; a->D = (uint32_t)D; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)L.HW;
    a->LH = (uint32_t)L.LH; a->LW = (uint32_t)L.LW; a->nb = (uint32_t)L.nb; a->WPP = (uint32_t)L.WPP; a->B = (uint32_t)B;
    a->Br = (uint32_t)Br; a->nch = (uint32_t)nch;
    a->q4 = (uint32_t)q4;
    a->S_log2 = mixed_lanes_log2(L.HW);
    a->d_W = make_fastdiv((uint32_t)W); a->d_B = make_fastdiv((uint32_t)B); a->d_H = make_fastdiv((uint32_t)H);
    a->d_LW = make_fastdiv((uint32_t)L.LW); a->d_slice = make_fastdiv((uint32_t)(L.LH * L.LW));
    a->d_nch = make_fastdiv((uint32_t)nch); a->d_Br = make_fastdiv((uint32_t)Br);
    a->rg = make_regions(L);
    return fit_mixed(a, kMixedThreads) <= kLdsMax;
}

// Whether the maps of a shape are better off in a launch with other shapes than in one of their own (with the kernel `kind`).  lanes: what they take there, at
// the fewest per plane, in parts of what the machine holds at once (sixteen wavefronts per CU).  Beside others a shape saves the 2-4 us that a launch waits for
// the drain of the one before and then fills, and runs a kernel for any shape: about level with the kernels that stage planes in LDS (so: up to the
// whole machine), up to twice as slow per element as those that hold them in registers (a quarter of it), three times as compress_line (an eighth).
// 160 calls of two or three shapes of all sizes, sum of their times: 3281 us apart, 2630 so; with a half for the register kernels 2600, but maps of
// 192 x 112 x 112 and 11554 x 16 x 13 in bfloat16 17.2 -> 19.7 with their decompression, and with a quarter for compress_line rows of 384 and 768 under B = 4 7.7 -> 9.8
// Two: also where no other shape shares the launch.  The chunk kernels on few planes are one long chain in a few workgroups: single shapes of 0.01 to 8 M
// elements, in their own kernel and here, compress_tile / _plane / _any 18.4 and 10.1 us on average (60 shapes), compress_wave up to 0.3 M 8.6 and 4.5, above
// level, compress_rows up to 0.1 M 6.1 and 4.6, above level.
int mixed_gains(int kind, uint64_t lanes) {
    const uint64_t machine = (uint64_t)num_cus() * 1024;
    if (lanes > machine) return 0;
    switch (kind) {
        case TILE: case PLANE: case ANY: return 2;
        case WAVE: case ROWS: return lanes <= machine / 16 ? 2 : 1;
        case UNITS: return 1;
        case LINE: return lanes <= machine / 8;
        default: return lanes <= machine / 4;
    }
}

// Compression's launches of several shapes (one type and code width).  A shape that is left alone has a launch of its own, with its own kernel.
struct CompMixer {
    MixedArgs a;
    uint32_t nshape = 0, nmap = 0;
    uint32_t maps[kSharedShapes];
    uint64_t seeds[kSharedMaps];
    const division_map* first = nullptr;      // a descriptor of the first shape, and its smallest packed buffer
    size_t first_bytes = 0;
    uint64_t lanes = 0;                       // of all shapes, at the fewest per plane
    bool alone = false;                       // the first shape gains by itself
    CompLaunch own;                           // the launch of the first shape by itself (its first kMaxBatch maps)
    bool fits(const division_map& m, size_t n, uint64_t more) const {
        return nshape == 0 || (m.dt == first->dt && m.b == first->b && nshape < (uint32_t)kSharedShapes && nmap + n <= (size_t)kSharedMaps &&
                               lanes + more <= (uint64_t)num_cus() * 1536);
    }
    void add(const division_map& m, const CompLaunch& c, const MixedShape& sh, int gains, uint64_t more, size_t n, size_t bytes, const void* const* x, void* const* packed,
             const uint64_t* seed) {
        if (nshape == 0) { first = &m; first_bytes = bytes; nmap = 0; lanes = 0; alone = gains == 2; own = c; }
        lanes += more;
        a.shape[nshape] = sh;
        a.map0[nshape] = nmap;
        maps[nshape++] = (uint32_t)n;
        for (size_t i = 0; i < n; ++i, ++nmap) {
            a.x[nmap] = x[i]; a.pk[nmap] = packed[i]; seeds[nmap] = seed[i];
            a.seed_a[nmap] = seed_key_a(seed[i]); a.seed_c[nmap] = seed_key_c(seed[i]);
        }
    }
    int flush(hipStream_t st) {
        const uint32_t shapes = nshape;
        nshape = 0;
        if (shapes == 0) return DIVISION_OK;
        if (shapes == 1 && !alone && nmap <= (uint32_t)kMaxBatch) return launch_compress(own, a.shape[0].rg, (int)nmap, a.x, a.pk, seeds, first->dt, first->b, st);
        if (shapes == 1 && !alone)
            return compress_impl((int)nmap, a.x, a.pk, seeds, first->N, first->C, first->D, first->H, first->W, first->dt, first->B, first->b, first_bytes, st);
        CompLaunch c;
        c.kind = MIXED; c.st = st; c.gy = 1; c.mixed = &a;
        spread_mixed(a, maps, shapes, &c.gx, &c.nt, &c.lds);
        return bridge_compress(first->dt, c, first->b) == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
    }
};

// Launches that hold the maps of several shapes (one type and code width): shapes are added while they fit, then flushed.  A shape that
// is left alone has a launch of its own, with the kernel that serves it best (which shape a wavefront belongs to costs a launch of one
// 0.4-0.8 us: 5 maps of 64 x 79 x 13 and the 4 of two other shapes in the other format 9.2 us in three launches, 10.0 in two mixed ones).
struct Mixer {
    MixLaunch c;
    uint32_t nshape = 0, nmap = 0;
    const division_map* first = nullptr;      // a descriptor of the first shape, and its smallest packed buffer
    size_t first_bytes = 0;
    bool fits(const division_map& m, size_t maps, uint64_t workgroups) const {
        return nshape == 0 || (m.dt == first->dt && m.b == first->b && nshape < (uint32_t)kMixShapes && nmap + maps <= (size_t)kMixMaps &&
                               launch_ok(c.grid + workgroups, 64));
    }
    void add(const division_map& m, const Layout& L, bool flat, int kind, const DecShape& sh, uint32_t chunks, size_t maps, size_t bytes,
             const void* const* packed, void* const* xhat) {
        if (nshape == 0) {
            first = &m; first_bytes = bytes;
            c.grid = 0; nmap = 0;
            for (int i = 0; i < kMixShapes; ++i) c.a.first[i] = 0xffffffffu;
        }
        MixShape& s = c.a.shape[nshape];
        static_cast<DecShape&>(s) = sh;
        s.meta_off = L.meta_off; s.lfc_off = L.lfc_off;
        c.a.chunks[nshape] = chunks;
        c.a.info[nshape] = (uint32_t)kind | (flat ? 16u : 0u) | nshape << 5 | nmap << 16;
        c.a.first[nshape++] = c.grid;
        for (size_t i = 0; i < maps; ++i) { c.a.pk[nmap] = packed[i]; c.a.xhat[nmap++] = xhat[i]; }
        c.grid += chunks * (uint32_t)maps;
    }
    int flush(hipStream_t st) {
        const uint32_t shapes = nshape;
        nshape = 0;
        if (shapes == 0) return DIVISION_OK;
        if (shapes == 1)
            return decompress_impl((int)nmap, c.a.pk, c.a.xhat, first_bytes, first->N, first->C, first->D, first->H, first->W, first->dt, first->B, first->b, st);
        c.st = st;
        return bridge_decompress_mixed(first->dt, c, first->b) == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
    }
};

// Workgroups per CU up to which the small planes of all kernels share a launch (compress_planes, ALL).  Multi-shape calls of 0.5-30 M elements that hold strips,
// rows of odd width or lanes, 60 each, at limits of 0, 16, 32, 64 and 128: 897, 895, 887, 877, 877 us; 1119, 1100, 1074, 1057, 1058; 1152, 1116, 1106, 1098,
// 1100.  Beyond, each kernel at its own registers.  The same limit for all types and code widths, though ALL needs 138 and 154 registers for bfloat16 at two bits and
// one (three wavefronts per SIMD instead of four): twelve calls each of 2 to 40 M elements in launches of their own / in one, bfloat16 at 1, 2, 4 and 8 bits 260 / 222, 268 / 221,
// 307 / 263 and 248 / 196 us, fp32 245 / 201, 212 / 172, 292 / 233 and 243 / 206, none slower by more than 2 %.
constexpr uint64_t kHeavyWorkgroups = 64;
// Shapes of one type and code width that one kernel serves share a launch: those of one instance of compress_line, and those whose kernels
// compress_planes holds.  Kept until all shapes of a call are known; a shape that finds no other has a launch of its own.
struct SharedMixer {
    struct Shape {
        const division_map* m;
        size_t bytes;                             // the smallest of the packed buffers
        CompLaunch c;
        Regions rg;
        int key;                                  // shapes of equal keys share a launch: the instance of compress_line, LIGHT or HEAVY (compress_planes)
        std::vector<const void*> x;
        std::vector<void*> packed;
        std::vector<uint64_t> seeds;
        MixedShape mixed;                         // mixed_lanes != 0: a small shape, which has its place in compress_mixed where none of these launches has one for it
        uint64_t mixed_lanes;
    };
    enum { LIGHT = 0, HEAVY = -1, OWN = -2, GONE = -3 };
    std::vector<Shape> shapes;
    // takes the shape, and its maps, if its kernel (c: the launch of its first kMaxBatch maps) can be shared
    bool add(const CompLaunch& c, const MixedShape& mixed, uint64_t mixed_lanes, const division_map& m, const Layout& L, int64_t H, int B, size_t bytes,
             std::vector<const void*>& x, std::vector<void*>& packed, std::vector<uint64_t>& seeds) {
        if (x.size() > (size_t)kSharedMaps || !launch_ok((uint64_t)c.gx * x.size(), 64)) return false;
        int key = LIGHT;
        if (c.kind == LINE && c.oa.NG == 1 && (c.oa.K == 4 || c.oa.K == 6)) key = 100 * (int)c.oa.K + line_lu(c.oa);
        else if (c.kind == LANE || (c.kind == ITEMS && B == 8 && H > 1) || (c.kind == ROWSTRIP && !c.sa.pack_off)) key = HEAVY;
        else if (!(c.kind == STRIP && (B == 4 || B == 8)) && !(c.kind == ITEMS && B == 4 && H > 1)) return false;
        if (shapes.empty()) shapes.reserve(kSharedShapes);
        shapes.push_back({&m, bytes, c, make_regions(L), key, std::move(x), std::move(packed), std::move(seeds), mixed, mixed_lanes});
        return true;
    }
    static void put(LinesArgs& a, uint32_t n, const Shape& q) { a.shape[n] = q.c.oa; a.rg[n] = q.rg; }
    static void put(PlanesArgs& a, uint32_t n, const Shape& q) {
        a.shape[n].kind = q.c.kind == LANE ? 1u : q.c.kind == ITEMS ? 10u * (uint32_t)q.c.B + (uint32_t)q.c.vec : (uint32_t)q.c.vec;
        if (q.c.kind == LANE) a.shape[n].lane = q.c.la;
        else if (q.c.kind == ITEMS) a.shape[n].items = q.c.ia;
        else a.shape[n].strip = q.c.sa;
        a.rg[n] = q.rg;
    }
    // the launch of shapes[i] and of those behind it that share it
    template <typename Args>
    int launch(size_t i, std::vector<char>& done, hipStream_t st) {
        const Shape& f = shapes[i];
        Args a;
        uint32_t n = 0, maps = 0, grid = 0;
        CompLaunch c;
        c.lds = 0;
        for (int k = 0; k < kSharedShapes; ++k) a.first[k] = 0xffffffffu;
        for (size_t j = i; j < shapes.size() && n < (uint32_t)kSharedShapes; ++j) {
            const Shape& q = shapes[j];
            if (done[j] || (j > i && f.key == OWN) || q.m->dt != f.m->dt || q.m->b != f.m->b || q.key != f.key || maps + q.x.size() > (size_t)kSharedMaps ||
                !launch_ok(grid + (uint64_t)q.c.gx * q.x.size(), 64))
                continue;
            done[j] = 1;
            a.first[n] = grid; a.chunks[n] = q.c.gx; a.map0[n] = maps;
            put(a, n++, q);
            for (size_t k = 0; k < q.x.size(); ++k, ++maps) {
                a.x[maps] = q.x[k]; a.pk[maps] = q.packed[k]; a.seed_a[maps] = seed_key_a(q.seeds[k]); a.seed_c[maps] = seed_key_c(q.seeds[k]);
            }
            grid += q.c.gx * (uint32_t)q.x.size();
            c.lds = std::max(c.lds, q.c.lds);
        }
        const division_map& m = *f.m;
        if (n == 1 && f.x.size() <= (size_t)kMaxBatch) {
            c = f.c;
            return launch_compress(c, f.rg, (int)f.x.size(), f.x.data(), f.packed.data(), f.seeds.data(), m.dt, m.b, st);
        }
        if (n == 1) return compress_impl((int)f.x.size(), f.x.data(), f.packed.data(), f.seeds.data(), m.N, m.C, m.D, m.H, m.W, m.dt, m.B, m.b, f.bytes, st);
        c.st = st; c.gx = grid; c.gy = 1;
        if constexpr (std::is_same<Args, LinesArgs>::value) { c.kind = LINES; c.lines.a = &a; c.lines.K = f.c.oa.K; c.lines.lu = line_lu(f.c.oa); }
        else { c.kind = PLANES; c.planes.a = &a; c.planes.all = f.key == HEAVY; }
        return bridge_compress(m.dt, c, m.b) == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
    }
    static bool planes(const Shape& p, const Shape& q) { return p.key <= LIGHT && q.key <= LIGHT && p.key > OWN && q.key > OWN && p.m->dt == q.m->dt && p.m->b == q.m->b; }
    // The small shapes join a launch of their kernels that the call has in any case (the drawn calls above 877 -> 843, 1057 -> 1042 and 1098 -> 1069 us), or go where the small ones of
    // all kernels are.
    int settle(CompMixer& comp, hipStream_t st) {
        for (size_t i = 0; i < shapes.size(); ++i) {
            Shape& s = shapes[i];
            if (s.mixed_lanes == 0) continue;
            bool joins = false;
            uint64_t workgroups = 0;
            bool heavy = s.key == HEAVY;
            for (const Shape& q : shapes) {
                if (s.key <= LIGHT ? !planes(s, q) : !(q.key == s.key && q.m->dt == s.m->dt && q.m->b == s.m->b)) continue;
                workgroups += (uint64_t)q.c.gx * q.x.size();
                joins = joins || q.mixed_lanes == 0;
                heavy = heavy || (q.key == HEAVY && q.mixed_lanes == 0);
            }
            if (joins && (!heavy || workgroups <= kHeavyWorkgroups * (uint64_t)num_cus())) continue;
            if (!comp.fits(*s.m, s.x.size(), s.mixed_lanes)) {
                const int rc = comp.flush(st);
                if (rc != DIVISION_OK) return rc;
            }
            comp.add(*s.m, s.c, s.mixed, 1, s.mixed_lanes, s.x.size(), s.bytes, s.x.data(), s.packed.data(), s.seeds.data());
            s.key = GONE;
        }
        return DIVISION_OK;
    }
    int flush(hipStream_t st) {
        std::vector<char> done(shapes.size(), 0);
        for (size_t i = 0; i < shapes.size(); ++i) {
            done[i] = done[i] || shapes[i].key == GONE;
            // all small planes of a type together, or those of few registers together and the others alone
            if (shapes[i].key != HEAVY) continue;
            uint64_t workgroups = 0;
            for (const Shape& q : shapes)
                if (planes(q, shapes[i])) workgroups += (uint64_t)q.c.gx * q.x.size();
            const bool together = workgroups <= kHeavyWorkgroups * (uint64_t)num_cus();
            for (size_t j = shapes.size(); j-- > 0;)
                if (j != i && planes(shapes[j], shapes[i])) {
                    if (together) shapes[j].key = HEAVY;
                    else if (shapes[j].key == HEAVY) shapes[j].key = OWN;
                }
            if (!together) shapes[i].key = OWN;
        }
        for (size_t i = 0; i < shapes.size(); ++i) {
            if (done[i]) continue;
            const int rc = shapes[i].key > 0 ? launch<LinesArgs>(i, done, st) : launch<PlanesArgs>(i, done, st);
            if (rc != DIVISION_OK) return rc;
        }
        return DIVISION_OK;
    }
};

int kernel_name_impl(int direction, const void* data, int64_t N, int64_t C, int64_t D, int64_t H, int64_t W,
                     division_dtype dt, int B, int b, char* out, size_t cap) {
    if (!out || cap == 0) return DIVISION_EINVAL;
    squeeze_dims(D, H, W);
    Layout L;
    const int rc = make_layout(N, C, D, H, W, B, b, (int)dt, &L);
    if (rc != DIVISION_OK) return rc;
    B = covering_block(L, D, H, W, B);
    const bool flat = D == 1;
    const char* sfx = flat ? "" : "_3d";
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    const char* tn = dt == DIVISION_BF16 ? "bf16_t" : dt == DIVISION_F32_C16 ? "f32c16_t" : "float";
    int n;
    if (direction == 0) {
        CompLaunch c;
        plan_compress(L, D, H, W, B, b, es, data, 1, &c);
        switch (c.kind) {
            case LINE: n = snprintf(out, cap, "compress_line<%s, %d, %u, %u, %d>", tn, b, c.oa.K, c.oa.NG, line_lu(c.oa)); break;
            case REGS: n = snprintf(out, cap, "compress_regs%s<%s, %d, %d, %d>", sfx, tn, b, (B == 4 || B == 8) ? B : 0, c.nw); break;
            case LANE: n = snprintf(out, cap, "compress_lane<%s, %d>", tn, b); break;
            case STRIP: n = snprintf(out, cap, "compress_strip<%s, %d, %d, %d>", tn, b, c.vec / 100, c.vec % 100); break;
            case ROWSTRIP: n = snprintf(out, cap, "compress_rowstrip<%s, %d, %d, %d>", tn, b, c.vec / 100, c.vec % 100); break;
            case ITEMS: n = snprintf(out, cap, "compress_items<%s, %d, %d, %d, %d>", tn, b, B, c.vec, H == 1 ? 1 : B); break;
            case SEG: n = snprintf(out, cap, "compress_seg<%s, %d, %d, %s, %d>", tn, b, B, W % 2 != 0 ? "true" : "false", c.seg_K); break;
            case UNITS: n = snprintf(out, cap, "compress_units<%s, %d, %d>", tn, b, c.nw); break;
            case WAVE: n = snprintf(out, cap, "compress_wave<%s, %d, %d, %d>", tn, b, B, c.vec); break;
            case TILE: n = snprintf(out, cap, "compress_tile<%s, %d, %d, %d, %d>", tn, b, B, c.vec, c.nt); break;
            case ONE: n = snprintf(out, cap, "compress_one<%s, %d, %u>", tn, b, c.oa.K); break;
            case ROWS: n = snprintf(out, cap, "compress_rows%s<%s, %d>", sfx, tn, b); break;
            case PLANE: n = snprintf(out, cap, "compress_plane%s<%s, %d>", sfx, tn, b); break;
            default: n = snprintf(out, cap, "compress_any%s<%s, %d>", sfx, tn, b);
        }
    } else {
        DecArgs a{}; uint32_t grid = 0;
        const int kind = plan_decompress(L, D, H, W, B, es, data, 1, &a, &grid);
        if (kind == 6)
            n = snprintf(out, cap, "decompress_units<%s, %d, %d%s>", tn, b, (int)a.G, units_wide(a) ? "" : ", 1");
        else if (kind == 7)
            n = snprintf(out, cap, "decompress_stream%s<%s, %d>", sfx, tn, b);
        else if (kind == 8)
            n = snprintf(out, cap, "decompress_stream_any%s<%s, %d>", sfx, tn, b);
        else if (kind == 9)
            n = snprintf(out, cap, "decompress_stream_one<%s, %d>", tn, b);
        else
            n = snprintf(out, cap, "%s%s<%s, %d>", kind == 0 ? "decompress_rowvec" : kind == 3 ? "decompress_table" : kind == 5 ? "decompress_words" : kind == 1 ? "decompress_flat" : kind == 4 ? "decompress_lane" : "decompress_scalar",
                         kind == 4 ? "" : sfx, tn, b);
    }
    return (n < 0 || (size_t)n >= cap) ? DIVISION_ESIZE : DIVISION_OK;
}
