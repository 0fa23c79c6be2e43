// Part of division.hip (included inside its unnamed namespace): compress_seg, items of sixteen elements of a block in
// registers (4-byte elements, B = 4 and 8).

// ------------------------------------------------------------------ compress, sixteen elements of a block per item

struct SegArgs {
    CompTab tab;
    Regions rg;
    uint32_t P, D, H, W, HW, LH, LW, nb, WPP;     // H, LH: rows, block rows of one depth slice (D = 1: a 2-D map)
    uint32_t CW;         // items per item row
    uint32_t RS;         // item rows the workgroup takes per round
    uint32_t irows;      // item rows per slice
    uint32_t rows;       // item rows of a plane
    uint32_t cz0, cz1;   // slices of a block, of a block of the last layer
    FastDiv d_irows, d_slice, d_LW, d_CW;
};

// Planes whose rows are not whole 16-byte vectors (odd widths and the like), 2-D and 3-D, under B = 4 and 8,
// 4-byte elements; a plane per workgroup.  An ITEM is four rows of four elements, sixteen of one block, loaded straight
// from global memory (16-byte loads at 4-byte boundaries, neighbouring lanes read neighbouring vectors of a row: whole
// lines) and kept in registers from the load to the codes.  (Two rows of eight under B = 8 need fewer hashes at odd
// rows, but each line is then fetched by two loads: 103 us on 64 x 64 x 147 x 147 with loads that stay in the caches, at the
// expense of the kernels that follow, and 122 with non-temporal ones.)  A lane keeps its column and steps
// down the plane, RS item rows per round, so nothing is looked up per element: what goes through LDS is one
// binary64 sum per item (a lane per block adds them, takes the mean and hands H^L back) and the code bits.
// A lane's first row starts at an even element of the plane (the map has an even width, or an even number of
// elements per slice, or one slice), so which rows start in the middle of an element pair is known at compile
// time (ODD): such a row hashes one pair more and needs no selects.
// The last column is narrower: what its items read past their row (the next row's first elements, zero past
// the plane) gets the weight 0 in the sum (a fused multiply-add where the others' weight is 1: exact for finite
// values, see below for the others, and as fast as the addition) and NaN for H^L, which minimum and maximum skip and the quantiser turns into code 0.
// What bounds it: vector instructions, then the latency between its barriers.  Against the kernel that parks the plane in
// LDS (compress_units of compress_units.h): 64 x 64 x 147 x 147 under B = 8 136 -> 102 us (3.5 TB/s of x), 73 x 73 47 -> 35, 127 x 127
// 110 -> 62, 64 x 512 x 29 x 29 49 -> 35, the volumes 32 x 256 x 4 x 14 x 14 20 -> 12.5.
template <int BITS>
__device__ __forceinline__ uint32_t push_half(uint32_t acc, float h, bool odd, float delta, float invs, uint32_t xw, uint32_t k2, uint32_t rscale) {
    // one element of a pair: push_pair without the other
    uint32_t x = xw;
    x ^= x >> 16; x *= 0x7feb352du;
    x = xor3(x, x >> 15, k2); x *= 0x846ca68bu;
    uint32_t T = (uint32_t)((h - delta) * invs), s;
    if constexpr (BITS == 8) T = min(T, 255u << 24);
    if (odd) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(s) : "v"(x), "s"(rscale), "v"(T));
    else asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[0,0,0,0]" : "=v"(s) : "v"(x ^ (x >> 16)), "s"(rscale), "v"(T));
    return __builtin_amdgcn_alignbit(acc, s, 32 - BITS);
}

constexpr uint32_t kSegThreads = 768;
template <typename T, int BITS, int B, bool ODD, int K>
__global__ void __launch_bounds__(kSegThreads) compress_seg(SegArgs a) {
    static_assert(sizeof(T) == 4 && (B == 4 || B == 8), "4-byte elements");
    constexpr int R = 4, C = 4;                           // rows and columns of an item
    constexpr uint32_t IPB = B / 4;                       // item rows, and items per row, of a block
    constexpr float Lf = float((1 << BITS) - 1);
    constexpr uint32_t kDrop = 0x80000000u;
    const uint32_t tid = threadIdx.x, NT = blockDim.x, W = a.W;
    const CompPtrs pt = comp_ptrs(a.tab, a.rg, tid);
    const uint32_t p = xcd_run_index(blockIdx.x, a.P);
    auto sync = [&]() { if (NT == 64) wave_sync(); else lds_barrier(); };

    extern __shared__ float4 smem4[];
    double* part = reinterpret_cast<double*>(smem4);                      // [rows * CW] item sums
    double* rc = part + a.rows * a.CW;                                    // [8] reciprocals of the block counts
    float* red = reinterpret_cast<float*>(rc + 8);                        // [2 * wavefronts]
    float* lfcs = red + 2 * (NT / 64u);                                   // [nb]
    uint32_t* cw = reinterpret_cast<uint32_t*>(lfcs + a.nb);              // [WPP] code words

    // ---- the lane's items, their loads first of all
    const uint32_t row0 = fdiv(tid, a.d_CW), j = tid - row0 * a.CW;
    u32x4 q[K][R];
    uint32_t f0[K];                                       // first element in the plane
    uint32_t bl[K];                                       // block
    int nr[K];                                            // rows inside the map (none: no item)
    {
        const T* src = static_cast<const T*>(pt.x) + (size_t)p * a.HW;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, (int)(a.HW * 4u), 0x00020000);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t row = row0 + a.RS * (uint32_t)k;
            uint32_t z = 0, ir = row;
            if (a.D > 1) { z = fdiv(row, a.d_irows); ir = row - z * a.irows; }
            const uint32_t r0 = ir * R;
            f0[k] = (z * a.H + r0) * W + j * C;
            nr[k] = row0 < a.RS && row < a.rows ? min(R, max((int)(a.H - r0), 0)) : 0;
            bl[k] = nr[k] > 0 ? ((z / B) * a.LH + ir / IPB) * a.LW + j / IPB : 0u;
            // rows past the plane's end read as zero, others past the item's last row are masked below
            const uint32_t off = nr[k] > 0 ? f0[k] * 4u : kDrop;
#pragma unroll
            for (int r = 0; r < R; ++r) q[k][r] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + (uint32_t)r * W * 4u, 0, kLoadAux);
        }
    }
    // meanwhile: the reciprocals, the cleared code words, the weights of the lane's columns
    if (tid < 8) {
        const uint32_t cnt = (tid & 4u ? a.cz1 : a.cz0) * (tid & 2u ? a.H - (a.LH - 1u) * B : (uint32_t)B) * (tid & 1u ? W - (a.LW - 1u) * B : (uint32_t)B);
        rc[tid] = 1.0 / (double)cnt;
    }
    for (uint32_t i = tid; i < a.WPP; i += NT) cw[i] = 0u;
    double wt[C];
    float nn[C];
#pragma unroll
    for (int e = 0; e < C; ++e) {
        const bool in = j * C + (uint32_t)e < W;
        wt[e] = in ? 1.0 : 0.0;
        nn[e] = in ? 0.0f : __builtin_nanf("");
    }
    // ---- Sec. 4.1 AveragePooling, step 1: a binary64 sum per item
    float x[K][R][C];
    bool partial[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            x[k][r][0] = __uint_as_float(q[k][r].x); x[k][r][1] = __uint_as_float(q[k][r].y);
            x[k][r][2] = __uint_as_float(q[k][r].z); x[k][r][3] = __uint_as_float(q[k][r].w);
        }
        // the plane's last item row: rows past the map count for nothing in the sum and are NaN after it.  With one item
        // per lane they are made zeros here and NaN later (62 registers, eight wavefronts per SIMD: 64 x 512 x 29 x 29 in
        // 35 us against 38); with two items a second copy of the sum is the faster form, off the
        // main path as the hint says: 72 to 74 registers, two workgroups of eleven wavefronts per CU; without the hint 102
        // registers and one workgroup (64 x 64 x 147 x 147: 102 us against 133).
        double s = 0.0;
        partial[k] = __any(nr[k] != R && nr[k] != 0);
        if (K > 1 && __builtin_expect(partial[k], 0)) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < C; ++e) {
                    s = __builtin_fma((double)x[k][r][e], r < nr[k] ? wt[e] : 0.0, s);
                    x[k][r][e] = r < nr[k] ? x[k][r][e] : __builtin_nanf("");
                }
        } else {
            if (partial[k]) {
#pragma unroll
                for (int r = 1; r < R; ++r)
#pragma unroll
                    for (int e = 0; e < C; ++e) x[k][r][e] = r < nr[k] ? x[k][r][e] : 0.0f;
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < C; ++e) s = __builtin_fma((double)x[k][r][e], wt[e], s);
        }
        // 0 * x is NaN for an infinity or a NaN, which must not reach a block it is not in: a sum that is not finite is
        // taken again over the elements of the item alone (never on ordinary inputs: sums of binary32 values are finite)
        if (__builtin_expect(__any(!(__builtin_fabs(s) < __builtin_inf())), 0)) {
            s = 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < C; ++e) s += r < nr[k] && j * C + (uint32_t)e < W ? (double)x[k][r][e] : 0.0;
        }
        const uint32_t row = row0 + a.RS * (uint32_t)k;
        if (row0 < a.RS && row < a.rows) part[row * a.CW + j] = s;        // a row past the map was read as zeros
    }
    sync();
    // ---- step 2: a lane per block adds its items in a fixed order
    for (uint32_t t0 = 0; t0 < a.nb; t0 += NT) {
        const uint32_t t = min(t0 + tid, a.nb - 1u);       // (no lane leaves: mean_with_rcp votes across the wavefront)
        uint32_t bd = 0, b2 = t;
        if (a.D > 1) { bd = fdiv(t, a.d_slice); b2 = t - bd * (a.LH * a.LW); }
        const uint32_t bi = fdiv(b2, a.d_LW), bj = b2 - bi * a.LW;
        const bool lz = bd * B + B >= a.D, lr = bi + 1u == a.LH, lc = bj + 1u == a.LW;
        const uint32_t deps = lz ? a.cz1 : a.cz0;
        // the block's IPB x IPB items per slice; those past the map are not there
        const uint32_t row1 = bi * IPB, col1 = bj * IPB;
        const double* ps = part + (bd * B * a.irows + row1) * a.CW + col1;
        double S = 0.0;
        for (uint32_t z = 0; z < deps; ++z) {
            double v[IPB][IPB];
#pragma unroll
            for (uint32_t i = 0; i < IPB; ++i)
#pragma unroll
                for (uint32_t c = 0; c < IPB; ++c) {
                    const bool there = row1 + i < a.irows && col1 + c < a.CW;
                    v[i][c] = ps[there ? i * a.CW + c : 0u];
                    v[i][c] = there ? v[i][c] : 0.0;
                }
#pragma unroll
            for (uint32_t i = 0; i < IPB; ++i)
#pragma unroll
                for (uint32_t c = 0; c < IPB; ++c) S += v[i][c];
            ps += a.irows * a.CW;
        }
        const uint32_t cnt = deps * (lr ? a.H - bi * B : (uint32_t)B) * (lc ? W - bj * B : (uint32_t)B);
        const float m = lfc_round<T>(mean_with_rcp(S, cnt, rc[(lz ? 4u : 0u) | (lr ? 2u : 0u) | (lc ? 1u : 0u)]), kC16<T>);
        lfcs[t] = m;
        lfc_store<T>(pt.lfc, (size_t)p * a.nb + t, m, kC16<T>);
    }
    sync();
    // ---- residual H^H = H - UpSampling(H^L) in place, the plane's extremes (NaN is skipped)
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float m = nr[k] > 0 ? lfcs[bl[k]] : __builtin_nanf("");
        if (K == 1 && partial[k]) {
#pragma unroll
            for (int r = 1; r < R; ++r)
#pragma unroll
                for (int e = 0; e < C; ++e) x[k][r][e] = r < nr[k] ? x[k][r][e] : __builtin_nanf("");
        }
        float le[C];
#pragma unroll
        for (int e = 0; e < C; ++e) le[e] = m + nn[e];    // (a mean of -0 becomes +0: such a block holds a negative element, no extreme and no code depends on it)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < C; e += 2) {
                x[k][r][e] = x[k][r][e] - le[e];
                x[k][r][e + 1] = x[k][r][e + 1] - le[e + 1];
                mn = fminf(mn, fminf(x[k][r][e], x[k][r][e + 1]));
                mx = fmaxf(mx, fmaxf(x[k][r][e], x[k][r][e + 1]));
            }
    }
    group_minmax(64, mn, mx);
    if (NT > 64) {
        if ((tid & 63u) == 0) { red[2 * (tid >> 6)] = mn; red[2 * (tid >> 6) + 1] = mx; }
        lds_barrier();
        for (uint32_t w = 0; w < NT / 64u; ++w) { mn = fminf(mn, red[2 * w]); mx = fmaxf(mx, red[2 * w + 1]); }
    }
    // ---- scale of Eq. (quantization), keys, meta
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    float invs = inv * (float)(1u << (32 - BITS));
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    uint32_t k2 = mix32(k1 + pt.seed_c);
    if (tid == 0) meta_store(pt.meta, p, delta, Delta, kC16<T>);
    keep_in_vgpr(delta, invs, k2);
    // ---- Quant + packing: a row's codes as one string of bits, OR-ed into the plane's cleared words
    const uint32_t rscale = 1u << (16 - BITS);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t xk = k1 + (f0[k] >> 1) * kWeyl;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool odd = ODD && (r & 1);
            // f, the row's first element: f0 + r * W; (f0 is even) its pair: f0 / 2 + r * W / 2
            const uint32_t xw = xk + ((uint32_t)r * W >> 1) * kWeyl;
            const float* h = x[k][r];
            uint32_t c = 0;                                               // the row's C * BITS code bits
            if (odd) {
                c = push_half<BITS>(c, h[3], false, delta, invs, xw + 2u * kWeyl, k2, rscale);
                c = push_pair<BITS>(c, h[1], h[2], delta, invs, xw + kWeyl, k2, rscale);
                c = push_half<BITS>(c, h[0], true, delta, invs, xw, k2, rscale);
            } else {
                c = push_pair<BITS>(c, h[2], h[3], delta, invs, xw + kWeyl, k2, rscale);
                c = push_pair<BITS>(c, h[0], h[1], delta, invs, xw, k2, rscale);
            }
            if (r < nr[k]) {
                const uint32_t bit = (f0[k] + (uint32_t)r * W) * BITS, sh = bit & 31u;
                uint32_t* w = cw + (bit >> 5);
                const uint64_t v = (uint64_t)c << sh;
                __hip_atomic_fetch_or(w, (uint32_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                // what runs over into the next word (only elements of the plane have bits there)
                if ((uint32_t)(v >> 32) != 0u) __hip_atomic_fetch_or(w + 1, (uint32_t)(v >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    sync();
    uint32_t* dst = pt.codes + (size_t)p * a.WPP;
    for (uint32_t w = tid; w < a.WPP; w += NT) dst[w] = cw[w];
}
