// Part of division.hip (included inside its unnamed namespace, after compress_strip.h): compress_rowstrip.

// ------------------------------------------------------------------ compress, a row of an odd-width plane per lane

// Geometry for planes of an odd width W (13, 15, 17, 27, 35, 55: maps of AlexNet and Inception-v3).
template <int W>
struct RowStripGeom {
    static_assert(W % 2 == 1 && W <= 64, "odd widths up to 64");
    static constexpr int S = W <= 16 ? 16 : W <= 32 ? 32 : 64;   // lane slots per plane = rows a plane may have
    static constexpr int G = 64 / S;                             // planes per round
    static constexpr int LPL = (G * S * W + 255) / 256;          // 16-byte units a lane loads: a round of G planes of S rows
    static constexpr int NP = (W + 1) / 2;                       // element pairs a row touches
};

// What a round of `planes` planes from plane p0 on reads of a map that starts on a 4-byte boundary: whole aligned dwords, from the one that holds its first
// element to the one that holds its last, so nothing beyond the map's own last dword (the bounds check of a buffer load is per dword).  Rounds of an odd number
// of elements of two bytes start in the middle of a dword every other time: `before` is the element in front of the round then, which is read with it.
struct RoundSpan { uint32_t before, bytes; };
__host__ __device__ __forceinline__ RoundSpan round_span(uint32_t p0, uint32_t planes, uint32_t HW, uint32_t es) {
    const uint32_t before = es == 2 ? (p0 * HW) & 1u : 0u;
    return RoundSpan{before, ((planes * HW + before) * es + 3u) & ~3u};
}

// The strip kernel for planes whose rows are not whole 16-byte vectors: a lane owns one ROW of W
// elements (W odd, compile-time) and keeps it in registers from the pooling to the codes; the lanes
// of a plane sit side by side (16, 32 or 64 slots), B = 4 or 8 rows of a block row are an aligned DPP
// group, so block sums and the plane's extremes are DPP reductions as in compress_strip.  The round
// (its planes are contiguous) is read with coalesced 16-byte loads into LDS in the map's own order
// (from the 4-byte boundary at or before its first element, see round_span); a lane takes
// its row out with scalar LDS reads (stride W words, odd: no bank conflicts inside a plane).
//
// Codes: the random word of Eq. (quantization)'s stochastic rounding belongs to a PAIR of elements
// (2j, 2j+1) of the plane, and with W odd every other row starts in the middle of a pair.  A lane
// therefore quantises the NP = (W+1)/2 pairs its row touches: its W elements shifted by the parity
// of its first element, the one slot that belongs to the neighbouring row filled with delta (code 0).
// Its (W+1) * BITS code bits start at an even element of the plane, anywhere in a word: they are
// built as words from bit 0, shifted as one string and OR-ed into the plane's cleared code words in
// LDS (the neighbour's bits of a shared word arrive by its own OR), which then leave as whole
// coalesced words.  One round per workgroup of one wavefront.
// Quant + packing of a lane's row (row sl of its plane, whose code words begin at word w0 of the round's): the round's code words are put
// together in LDS (xs) and leave from there.
template <int BITS, int W, int NT>
__device__ __forceinline__ void rowstrip_codes(const float (&x)[W], float* xs, uint32_t* dst, uint32_t nwords, bool valid, uint32_t sl, uint32_t w0,
                                               uint32_t lane, float delta, float invs, uint32_t k1, uint32_t k2) {
    constexpr int NP = RowStripGeom<W>::NP;
    constexpr int PPW = 16 / BITS;              // element pairs per code word
    constexpr int NWD = (NP + PPW - 1) / PPW;   // code words a row's pairs fill when they start at bit 0
    const uint32_t rscale = 1u << (16 - BITS);
    auto sync = [&]() { if (NT == 64) wave_sync(); else lds_barrier(); };
    sync();
    uint32_t* cw = reinterpret_cast<uint32_t*>(xs);
    {
        const u32x4 z{0u, 0u, 0u, 0u};
        for (uint32_t i = lane; i * 4u < nwords; i += NT) reinterpret_cast<u32x4*>(cw)[i] = z;
    }
    sync();
    {
        const uint32_t f0 = sl * (uint32_t)W;            // the row's first element in the plane
        const bool odd = (f0 & 1u) != 0;                 // it is the second element of its pair
        const uint32_t j0 = f0 >> 1;                     // first pair the row touches
        uint32_t w[NWD];
#pragma unroll
        for (int wi = 0; wi < NWD; ++wi) {
            uint32_t acc = 0;
#pragma unroll
            for (int pj = PPW - 1; pj >= 0; --pj) {
                const int jj = wi * PPW + pj;
                if (jj >= NP) continue;
                // slots 2jj and 2jj+1 of the row's pairs: elements 2jj - odd and 2jj + 1 - odd of the row
                const float e_even = 2 * jj < W ? x[2 * jj < W ? 2 * jj : 0] : delta;               // slot 2jj, row starts a pair
                const float e_odd0 = 2 * jj >= 1 ? x[2 * jj >= 1 ? 2 * jj - 1 : 0] : delta;         // slot 2jj, row starts mid-pair
                const float f_even = 2 * jj + 1 < W ? x[2 * jj + 1 < W ? 2 * jj + 1 : 0] : delta;   // slot 2jj+1
                const float f_odd0 = x[2 * jj < W ? 2 * jj : 0];                                    // slot 2jj+1, mid-pair (2jj <= W-1)
                const float h0 = odd ? e_odd0 : e_even;
                const float h1 = odd ? f_odd0 : f_even;
                acc = push_pair<BITS>(acc, h0, h1, delta, invs, k1 + (j0 + (uint32_t)jj) * kWeyl, k2, rscale);
            }
            w[wi] = acc;
        }
        if (valid) {
            const uint32_t bit = 2u * j0 * (uint32_t)BITS;           // where the row's string starts in the plane's code bits
            const uint32_t sh = bit & 31u;
            uint32_t* pw = cw + w0 + (bit >> 5);
#pragma unroll
            for (int i = 0; i <= NWD; ++i) {
                const uint64_t two = ((uint64_t)(i < NWD ? w[i < NWD ? i : 0] : 0u) << 32) | (i > 0 ? w[i > 0 ? i - 1 : 0] : 0u);
                const uint32_t v = (uint32_t)(two >> (32u - sh));
                // a word that is all zero adds nothing (the slots past the row's own elements are zero)
                if (v != 0u) __hip_atomic_fetch_or(pw + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    sync();
    for (uint32_t wd = lane; wd < nwords; wd += NT) dst[wd] = cw[wd];
}

template <typename T, int BITS, int W, int B>
__device__ __forceinline__ void compress_rowstrip_slots(const StripShape& a, const CompPtrs& pt, uint32_t round) {
    using Geo = RowStripGeom<W>;
    constexpr int S = Geo::S, G = Geo::G, LPL = Geo::LPL;
    constexpr int NSEG = (W + B - 1) / B;       // blocks per block row
    static_assert(B == 4 || B == 8, "block rows are DPP groups");
    constexpr float Lf = float((1 << BITS) - 1);
    extern __shared__ float4 smem4[];
    float* xs = reinterpret_cast<float*>(smem4);                     // the round, later its code words

    const uint32_t lane = threadIdx.x;
    const uint32_t p0 = round * G;
    const uint32_t Gc = min((uint32_t)G, a.P - p0);

    // ---- the round's loads first: coalesced, bounds-checked (units past the round read as zero)
    static_assert(LPL * 256 > G * S * W, "with the element in front of the round");
    const RoundSpan span = round_span(p0, Gc, a.HW, sizeof(T));
    u32x4 q[LPL];
    {
        const T* src = static_cast<const T*>(pt.x) + ((size_t)p0 * a.HW - span.before);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, (int)span.bytes, 0x00020000);
#pragma unroll
        for (int k = 0; k < LPL; ++k) {
            if constexpr (sizeof(T) == 4) {
                q[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16u + (uint32_t)(k * 1024), 0, kLoadAux);
            } else {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 h = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane * 8u + (uint32_t)(k * 512), 0, kLoadAux);
                q[k] = u32x4{h.x << 16, h.x & 0xffff0000u, h.y << 16, h.y & 0xffff0000u};
            }
        }
    }
    // the lane's place: plane g of the round, row sl of the plane
    const uint32_t g = lane / S, sl = lane % S;
    const bool live = g < Gc;
    const bool valid = live && sl < a.H;
    const uint32_t bi = sl / B;                                        // block row of the row
    const uint32_t rows = min((uint32_t)B, a.H - min(a.H, bi * (uint32_t)B));   // rows of that block row that exist
    const uint32_t p = p0 + g;
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    const uint32_t k2 = mix32(k1 + pt.seed_c);
    const uint32_t xv = (G * a.HW + span.before + 3u) / 4u;            // units of a whole round (the host sized LDS for them)
#pragma unroll
    for (int k = 0; k < LPL; ++k)
        if (lane + 64u * k < xv) reinterpret_cast<u32x4*>(xs)[lane + 64 * k] = q[k];
    wave_sync();

    // ---- the row; lanes without one take row 0 of the round and have their effects masked
    float x[W];
    {
        const float* sp = xs + span.before + (valid ? g * a.HW + sl * (uint32_t)W : 0u);
#pragma unroll
        for (int e = 0; e < W; ++e) x[e] = sp[e];
    }

    // ---- Sec. 4.1 AveragePooling: the row's share of each block of its block row, then the block
    // row's lanes together (binary64, fixed order)
    double Sm[NSEG];
#pragma unroll
    for (int s = 0; s < NSEG; ++s) Sm[s] = 0.0;
#pragma unroll
    for (int e = 0; e < W; ++e) Sm[e / B] += (double)x[e];
    float lfc[NSEG];
    const double rcp_rows = count_rcp(max(rows, 1u));
#pragma unroll
    for (int s = 0; s < NSEG; ++s) {
        const double Sb = group_sum<B>(valid ? Sm[s] : 0.0);
        const uint32_t cols = (uint32_t)(W - B * s < B ? W - B * s : B);     // a constant once the loop is unrolled
        lfc[s] = lfc_round<T>(mean_with_rcp(Sb, max(rows, 1u) * cols, count_rcp_times(rcp_rows, cols)), kC16<T>);
    }
    if (valid && sl % B == 0) {
#pragma unroll
        for (int s = 0; s < NSEG; ++s) lfc_store<T>(pt.lfc, (size_t)p * a.nb + bi * NSEG + s, lfc[s], kC16<T>);
    }

    // ---- residual H^H = H - UpSampling(H^L) in place, the plane's extremes
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < W; ++e) {
        x[e] = x[e] - lfc[e / B];
        mn = fminf(mn, x[e]);
        mx = fmaxf(mx, x[e]);
    }
    mn = valid ? mn : __builtin_inff();
    mx = valid ? mx : -__builtin_inff();
    group_minmax(S, mn, mx);

    // ---- scale of Eq. (quantization): every lane of the plane computes the same values
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    const float invs = inv * (float)(1u << (32 - BITS));
    if (live && sl == 0) meta_store(pt.meta, p, delta, Delta, kC16<T>);

    // ---- Quant + packing (every lane has taken its row out of LDS by now)
    rowstrip_codes<BITS, W, 64>(x, xs, pt.codes + (size_t)p0 * a.WPP, Gc * a.WPP, valid, sl, g * a.WPP, lane, delta, invs, k1, k2);
}

// Widths whose slots would leave half of the lanes without a row (17 of 32, 35 of 64): the rows of three planes side by side, 51 of the
// 64 lanes of a wavefront (W = 17) and 105 of the 128 of two (W = 35).  Neither the rows of a block nor those of a plane are an aligned group then:
// a lane parks its row's share of each block in LDS and a lane per block adds them; the extremes meet in LDS as
// integers of the same order (-0 below +0).
// What bounds it: vector instructions, so what a wavefront of half as many empty lanes saves.  64 x 768 x 17 x 17 under B = 8, three maps 61 -> 47 us (4.0 TB/s); 64 x 288 x
// 35 x 35, two 53 -> 47; 6664 planes of 35 x 35 cached as bfloat16 under B = 4 14.9 -> 13.4.
template <int W> constexpr int kRowPack = W == 17 ? 1 : W == 35 ? 2 : 0;      // wavefronts of a workgroup, 0: not packed
constexpr int kRowPackPlanes = 3;
// (A kernel of its own: as a branch of compress_rowstrip it took the slots' small calls from 3.2 to 3.3 us, 1500 x 35 x 35 from 5.6 to 5.75.)
template <typename T, int BITS, int W, int B>
__global__ void __launch_bounds__(64 * kRowPack<W>) compress_rowstrip_packed(StripArgs a) {
    constexpr int NT = 64 * kRowPack<W>, G = kRowPackPlanes;
    constexpr int LPL = (G * W * W + 4 * NT - 1) / (4 * NT);          // 16-byte units a lane loads (at most W rows)
    constexpr uint32_t NSEG = (W + B - 1) / B;                        // blocks per block row
    constexpr float Lf = float((1 << BITS) - 1);
    extern __shared__ float4 smem4[];
    float* xs = reinterpret_cast<float*>(smem4);                      // the round, then the rows' shares of the blocks, then its code words
    double* share = reinterpret_cast<double*>(smem4);                 // [NSEG][NT]
    float* lfcs = reinterpret_cast<float*>(reinterpret_cast<char*>(smem4) + a.pack_off);      // [G * nb]
    int* ext = reinterpret_cast<int*>(lfcs + G * a.nb);               // [G] minima, [G] maxima
    auto sync = [&]() { if (NT == 64) wave_sync(); else lds_barrier(); };

    const uint32_t lane = threadIdx.x;
    const CompPtrs pt = comp_ptrs(a.tab, a.rg, lane);
    const uint32_t p0 = xcd_run_index(blockIdx.x, a.nrounds) * G;
    const uint32_t Gc = min((uint32_t)G, a.P - p0);

    // ---- the round's loads first: coalesced, bounds-checked (units past the round read as zero)
    static_assert(LPL * 4 * NT > G * W * W, "with the element in front of the round");
    const RoundSpan span = round_span(p0, Gc, a.HW, sizeof(T));
    u32x4 q[LPL];
    {
        const T* src = static_cast<const T*>(pt.x) + ((size_t)p0 * a.HW - span.before);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, (int)span.bytes, 0x00020000);
#pragma unroll
        for (int k = 0; k < LPL; ++k) {
            if constexpr (sizeof(T) == 4) {
                q[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16u + (uint32_t)(k * NT * 16), 0, kLoadAux);
            } else {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 h = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane * 8u + (uint32_t)(k * NT * 8), 0, kLoadAux);
                q[k] = u32x4{h.x << 16, h.x & 0xffff0000u, h.y << 16, h.y & 0xffff0000u};
            }
        }
    }
    const uint32_t g = fdiv(lane, a.d_H), sl = lane - g * a.H;        // the lane's place: plane g of the round, row sl of the plane
    const bool valid = g < Gc;
    const uint32_t p = p0 + g;
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    const uint32_t k2 = mix32(k1 + pt.seed_c);
    if (lane < 2 * G) ext[lane] = lane < G ? 0x7fffffff : (int)0x80000000;
    const uint32_t xv = (G * a.HW + span.before + 3u) / 4u;           // units of a whole round (the host sized LDS for them)
#pragma unroll
    for (int k = 0; k < LPL; ++k)
        if (lane + (uint32_t)(NT * k) < xv) reinterpret_cast<u32x4*>(xs)[lane + NT * k] = q[k];
    sync();

    // ---- the row; lanes without one take row 0 of the round and have their effects masked
    float x[W];
    {
        const float* sp = xs + span.before + (valid ? lane * (uint32_t)W : 0u);
#pragma unroll
        for (int e = 0; e < W; ++e) x[e] = sp[e];
    }
    sync();
    // ---- Sec. 4.1 AveragePooling: the row's share of each block of its block row, then a lane per block
    {
        double Sm[NSEG];
#pragma unroll
        for (uint32_t s = 0; s < NSEG; ++s) Sm[s] = 0.0;
#pragma unroll
        for (int e = 0; e < W; ++e) Sm[e / B] += (double)x[e];
#pragma unroll
        for (uint32_t s = 0; s < NSEG; ++s) share[s * NT + lane] = Sm[s];
    }
    sync();
    for (uint32_t t = lane; t < Gc * a.nb; t += NT) {
        const uint32_t br = t / NSEG, s = t - br * NSEG;              // block row, counted over the planes
        const uint32_t tg = fdiv(br, a.d_LH), bi = br - tg * a.LH;
        const uint32_t rows = min((uint32_t)B, a.H - bi * B), cols = min((uint32_t)B, W - s * B);
        const double* sp = share + (s * NT + tg * a.H + bi * B);
        double S = 0.0;
#pragma unroll
        for (uint32_t r = 0; r < B; ++r) {
            const double v = sp[r < rows ? r : 0u];
            S += r < rows ? v : 0.0;
        }
        const float lfc = lfc_round<T>(mean_of(S, rows * cols), kC16<T>);
        lfcs[t] = lfc;
        lfc_store<T>(pt.lfc, (size_t)p0 * a.nb + t, lfc, kC16<T>);
    }
    sync();
    // ---- residual H^H = H - UpSampling(H^L) in place, the plane's extremes
    float mn = __builtin_inff(), mx = -__builtin_inff();
    {
        const float* lp = lfcs + (valid ? g * a.nb + sl / B * NSEG : 0u);
        float lfc[NSEG];
#pragma unroll
        for (uint32_t s = 0; s < NSEG; ++s) lfc[s] = lp[s];
#pragma unroll
        for (int e = 0; e < W; ++e) {
            x[e] = x[e] - lfc[e / B];
            mn = fminf(mn, x[e]);
            mx = fmaxf(mx, x[e]);
        }
    }
    auto ordered = [](int v) { return v ^ ((v >> 31) & 0x7fffffff); };
    if (valid) {
        __hip_atomic_fetch_min(ext + g, ordered(__float_as_int(mn)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_max(ext + G + g, ordered(__float_as_int(mx)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    sync();
    mn = __int_as_float(ordered(ext[valid ? g : 0u]));
    mx = __int_as_float(ordered(ext[G + (valid ? g : 0u)]));

    // ---- scale of Eq. (quantization): every lane of the plane computes the same values
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    const float invs = inv * (float)(1u << (32 - BITS));
    if (valid && sl == 0) meta_store(pt.meta, p, delta, Delta, kC16<T>);
    rowstrip_codes<BITS, W, NT>(x, xs, pt.codes + (size_t)p0 * a.WPP, Gc * a.WPP, valid, sl, g * a.WPP, lane, delta, invs, k1, k2);
}

template <typename T, int BITS, int W, int B>
__global__ void __launch_bounds__(64) compress_rowstrip(StripArgs a) {
    compress_rowstrip_slots<T, BITS, W, B>(a, comp_ptrs(a.tab, a.rg, threadIdx.x), xcd_run_index(blockIdx.x, a.nrounds));
}
