// Part of division.hip (included inside its unnamed namespace, in this order): compress_mixed.

// ------------------------------------------------------------------ compress, maps of several shapes in one launch

constexpr uint32_t kMixedUnits = 8;       // units (four consecutive elements) per lane, at most
constexpr int kMixedThreads = 1024;       // lanes per plane, and threads of a workgroup, at most
// (three runs of sixteen words: wide scalar loads)
struct alignas(64) MixedShape {
    uint32_t P, D, H, W, HW, LH, LW, nb, WPP, B;      // D depth slices of H rows; LH block rows per slice
    uint32_t Br, nch;        // rows of a block, and runs of up to eight elements per row of a block: of B, or of what the map has
    uint32_t q4;             // units per plane, the last one may be partly past it
    uint32_t S_log2;         // lanes per plane
    uint32_t J_log2;         // lanes per block in the block sums
    uint32_t G;              // planes per workgroup, S lanes each
    uint32_t reg_bytes;      // LDS bytes of one plane's region (a multiple of 16)
    uint32_t K;              // units per lane: 1, 2, 3, 4, 6 or 8
    FastDiv d_W, d_B, d_H, d_LW, d_slice, d_nch, d_Br;      // d_slice divides by LH * LW
    Regions rg;
};
struct MixedArgs : SharedTab { MixedShape shape[kSharedShapes]; };

// LDS byte offsets of the H^L of the four elements from e0 on (4 * nb = the sentinel for elements past the plane), two per word
__device__ __forceinline__ void mixed_offsets(const MixedShape& a, uint32_t e0, uint32_t allrows, bool flat, uint32_t (&lo)[2]) {
    uint32_t off[4];
    // four consecutive elements enter another row, and another block of their row, at most once (W, B >= 3)
    const uint32_t ra = fdiv(e0, a.d_W), c = e0 - ra * a.W;              // row, counted over all depth slices
    uint32_t r = ra, rn = ra + 1u, zb = 0, zbn = 0;
    if (!flat) {
        const uint32_t z = fdiv(ra, a.d_H);
        r = ra - z * a.H;
        const bool wrap = r + 1u == a.H;
        rn = wrap ? 0u : r + 1u;
        zb = fdiv(z, a.d_B) * a.LH;
        zbn = fdiv(wrap ? z + 1u : z, a.d_B) * a.LH;
    }
    const uint32_t bj = fdiv(c, a.d_B);
    const bool past = ra >= allrows;
    const uint32_t here = past ? a.nb : (zb + fdiv(r, a.d_B)) * a.LW + bj;
    const uint32_t next = ra + 1u >= allrows ? a.nb : (zbn + fdiv(rn, a.d_B)) * a.LW;
    const uint32_t left = past ? 4u : bj * a.B + a.B - c;                 // elements to the block's right edge
    const uint32_t rowleft = a.W - c;
    off[0] = here;
#pragma unroll
    for (uint32_t j = 1; j < 4; ++j) off[j] = j < rowleft ? here + (j >= left ? 1u : 0u) : next;
    lo[0] = (off[0] | (off[1] << 16)) << 2;
    lo[1] = (off[2] | (off[3] << 16)) << 2;
}
// the same element by element (rows or blocks of one and two)
__device__ __forceinline__ void mixed_offsets_each(const MixedShape& a, uint32_t e0, uint32_t (&lo)[2]) {
    uint32_t off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t e = e0 + j;
        const uint32_t ra = fdiv(e, a.d_W);
        const uint32_t c = e - ra * a.W;
        const uint32_t z = fdiv(ra, a.d_H);
        const uint32_t r = ra - z * a.H;
        off[j] = e < a.HW ? (fdiv(z, a.d_B) * a.LH + fdiv(r, a.d_B)) * a.LW + fdiv(c, a.d_B) : a.nb;
    }
    lo[0] = (off[0] | (off[1] << 16)) << 2;
    lo[1] = (off[2] | (off[3] << 16)) << 2;
}

// Small maps of several shapes: any width, block size and number of dimensions.  A launch of its own costs a shape 2.4 us of the host and, on the
// device, the drain of the launch before and its own filling; and the kernels that serve a shape best when the machine is full are, on a few
// planes, one long chain in a few workgroups.  Here a plane (or G small ones) has a workgroup, with lanes enough that the launch as a whole fills
// the machine: S lanes per plane, one to eight units each (K, a copy of the body per number: no round is tested), in
// registers from the load to the codes; blocks looked up while the loads fly, no table, no second plane to make one worth it; the plane is parked in LDS once,
// for the block sums, which J lanes per block add straight from there.
// What bounds it: the chain launch arguments -> loads -> LDS -> sums -> LDS -> extremes -> codes (4.9 us for tiny maps, where compress_line takes 3.4 for
// rows of one shape), and on larger ones the vector instructions of the look-ups.
// Two or three shapes of up to 0.1 M elements in all 14.9 us in launches of their own, 6.6 here; up to 0.5 M 15.0 and 8.9; up to 2 M 13.2 and 9.7
// (160 calls; 42 planes of rows of 513 and 234 of 192 in bfloat16, which share a launch now, 42 and 4.9).
template <typename T, int BITS, int K>
__device__ __forceinline__ void compress_mixed_body(const MixedShape& a, const CompPtrs& pt, uint32_t wg, char* smem) {
    constexpr float Lf = float((1 << BITS) - 1);
    const uint32_t tid = threadIdx.x;
    const uint32_t S = 1u << a.S_log2;
    const uint32_t l = tid & (S - 1u), g = tid >> a.S_log2;
    if (g >= a.G) return;                                     // whole wavefronts: G * S is a multiple of 64
    const uint32_t pf = wg * a.G, p = pf + g;                 // the workgroup's first plane, the lane's
    const bool pv = p < a.P;
    char* region = smem + g * a.reg_bytes;
    float4* xs4 = reinterpret_cast<float4*>(region);          // [K * S] the plane
    float* xs = reinterpret_cast<float*>(region);
    double* part = reinterpret_cast<double*>(xs + ((4u * K) << a.S_log2)); // [S / 16 + 1] partial sums of blocks of more than sixteen lanes
    float* lfcs = reinterpret_cast<float*>(part + (S >> 4) + 1);      // [nb + 1], last = NaN sentinel
    float* red = lfcs + a.nb + 1;                             // [2 * S / 64] cross-wave min / max

    // ---- loads first: coalesced, bounds-checked (units past the workgroup's planes read as zero, units past a plane read the next one)
    u32x4 q[K];
    {
        const uint32_t np = min(a.G, a.P - pf);
        const uint32_t odd0 = sizeof(T) == 2 ? (pf * a.HW) & 1u : 0u;      // 2-byte elements: the first plane may start in the middle of a dword
        const T* src = static_cast<const T*>(pt.x) + ((size_t)pf * a.HW - odd0);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(src), 0, (int)((((np * a.HW + odd0) * sizeof(T)) + 3u) & ~3u), 0x00020000);
        const uint32_t e0 = g * a.HW + odd0 + 4u * l;                      // the lane's first element
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t e = e0 + ((uint32_t)k << (a.S_log2 + 2u));
            if constexpr (sizeof(T) == 4) {
                q[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, e * 4u, 0, kLoadAux);
            } else {
                typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
                const u32x3 h = __builtin_amdgcn_raw_buffer_load_b96(rsrc, (e * 2u) & ~3u, 0, kLoadAux);
                q[k].x = h.x; q[k].y = h.y; q[k].z = h.z;
            }
        }
    }
    // ---- while they fly: LDS byte offset of the H^L of each element's block (4 * nb = the sentinel for elements past the plane)
    uint32_t lo[K][2];
    const uint32_t allrows = a.D * a.H;
    auto element = [&](int k) -> uint32_t { return 4u * (l + ((uint32_t)k << a.S_log2)); };
    if (a.W < 3 || a.B < 3) {
#pragma unroll
        for (int k = 0; k < K; ++k) mixed_offsets_each(a, element(k), lo[k]);
    } else if (a.D > 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) mixed_offsets(a, element(k), allrows, false, lo[k]);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) mixed_offsets(a, element(k), allrows, true, lo[k]);
    }
    if (l == 0) lfcs[a.nb] = __builtin_nanf("");
    // ---- park the plane in LDS as fp32
    f32x4 v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if constexpr (sizeof(T) == 4) v[k] = __builtin_bit_cast(f32x4, q[k]);
        else {
            const uint32_t sh = ((g * a.HW + (pf * a.HW & 1u)) & 1u) * 16u;
            const uint32_t w0 = __builtin_amdgcn_alignbit(q[k].y, q[k].x, sh), w1 = __builtin_amdgcn_alignbit(q[k].z, q[k].y, sh);
            v[k] = f32x4{__uint_as_float(w0 << 16), __uint_as_float(w0 & 0xffff0000u), __uint_as_float(w1 << 16), __uint_as_float(w1 & 0xffff0000u)};
        }
        xs4[l + ((uint32_t)k << a.S_log2)] = __builtin_bit_cast(float4, v[k]);
    }
    lds_barrier();

    // ---- Sec. 4.1 AveragePooling: J lanes per block, each every J-th run of up to eight elements
    const uint32_t J = 1u << a.J_log2, jl = l & (J - 1u);
    for (uint32_t t = l >> a.J_log2; t < (J > 1u ? S >> a.J_log2 : a.nb); t += S >> a.J_log2) {
        const bool there = t < a.nb;
        uint32_t bd = 0, t2 = t;
        if (a.D > 1) { bd = fdiv(t, a.d_slice); t2 = t - bd * (a.LH * a.LW); }
        const uint32_t bi = fdiv(t2, a.d_LW), bj = t2 - bi * a.LW;
        const uint32_t deps = min(a.B, a.D - bd * a.B);
        const uint32_t rows = min(a.B, a.H - bi * a.B);
        const uint32_t bw = min(a.B, a.W - bj * a.B);
        const float* base = xs + ((bd * a.B * a.H + bi * a.B) * a.W + bj * a.B);
        double sum = 0.0;
        for (uint32_t i = jl; there && i < deps * a.Br * a.nch; i += J) {
            uint32_t r = i, c0 = 0, z = 0;
            if (a.nch > 1) { r = fdiv(i, a.d_nch); c0 = (i - r * a.nch) * 8u; }
            if (a.D > 1) { z = fdiv(r, a.d_Br); r -= z * a.Br; }
            const float* s = base + ((z * a.H + r) * a.W + c0);
            const uint32_t n = r < rows && c0 < bw ? min(8u, bw - c0) : 0u;
            if (n == 8u) {
                float f[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) f[j] = s[j];
                sum += (((double)f[0] + (double)f[1]) + ((double)f[2] + (double)f[3])) + (((double)f[4] + (double)f[5]) + ((double)f[6] + (double)f[7]));
            } else {
                uint32_t j = 0;
                if (n >= 4u) {
                    sum += ((double)s[0] + (double)s[1]) + ((double)s[2] + (double)s[3]);
                    j = 4;
                }
                for (; j < n; ++j) sum += (double)s[j];
            }
        }
        if (J > 1u) sum += dpp_f64<kDppXor1>(sum);
        if (J > 2u) sum += dpp_f64<kDppXor2>(sum);
        if (J > 4u) sum += dpp_f64<kDppHalfMirror>(sum);
        if (J > 8u) sum += dpp_f64<kDppMirror>(sum);
        bool mine = jl == 0;
        if (J > 16u) {                                        // (one turn of the loop: every lane comes here)
            if ((l & 15u) == 0) part[l >> 4] = sum;
            lds_barrier();
            sum = 0.0;
            if (mine) for (uint32_t i = 0; i < J >> 4; ++i) sum += part[(l >> 4) + i];
        }
        mine = mine && there;
        if (mine) {
            const float lfc = lfc_round<T>(mean_of(sum, deps * rows * bw), kC16<T>);
            lfcs[t] = lfc;
            if (pv) lfc_store<T>(pt.lfc, (size_t)p * a.nb + t, lfc, kC16<T>);
        }
    }
    lds_barrier();

    // ---- residual H^H = H - UpSampling(H^L) in place, plane min / max (NaN residuals of elements past the plane are skipped)
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const char* lb = reinterpret_cast<const char*>(lfcs);
        v[k].x -= *reinterpret_cast<const float*>(lb + (lo[k][0] & 0xffffu));
        v[k].y -= *reinterpret_cast<const float*>(lb + (lo[k][0] >> 16));
        v[k].z -= *reinterpret_cast<const float*>(lb + (lo[k][1] & 0xffffu));
        v[k].w -= *reinterpret_cast<const float*>(lb + (lo[k][1] >> 16));
        mn = fminf(fminf(mn, v[k].x), fminf(v[k].y, fminf(v[k].z, v[k].w)));
        mx = fmaxf(fmaxf(mx, v[k].x), fmaxf(v[k].y, fmaxf(v[k].z, v[k].w)));
    }
    group_minmax(min(S, 64u), mn, mx);
    if (S > 64u) {
        if ((l & 63u) == 0) { red[2 * (l >> 6)] = mn; red[2 * (l >> 6) + 1] = mx; }
        lds_barrier();
        for (uint32_t w = 0; w < S >> 6; ++w) { mn = fminf(mn, red[2 * w]); mx = fmaxf(mx, red[2 * w + 1]); }
    }

    // ---- scale of Eq. (quantization), keys, meta
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    const float invs = inv * (float)(1u << (32 - BITS));
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    const uint32_t k2 = mix32(k1 + pt.seed_c);
    if (l == 0 && pv) meta_store(pt.meta, p, delta, Delta, kC16<T>);

    // ---- Quant + packing: a unit is two element pairs = 4 codes
    const uint32_t rscale = 1u << (16 - BITS);
    constexpr uint32_t CB = BITS / 2;                         // code bytes per unit (1, 2 or 4; 1-bit codes: half a byte)
    const uint32_t cbytes = BITS == 1 ? (a.q4 + 1u) / 2u : a.q4 * CB;    // code bytes of a plane
    uint8_t* codes = reinterpret_cast<uint8_t*>(pt.codes) + (size_t)pf * a.WPP * 4;
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(codes, 0, (int)(min(a.G, a.P - pf) * a.WPP * 4u), 0x00020000);
    const uint32_t cvoff = g * a.WPP * 4u;
    const uint32_t xw0 = k1 + (2u * l) * kWeyl;
    const uint32_t tail = a.HW & 3u;                          // elements of the last unit inside the plane (0: all four)
    const uint32_t tailmask = tail ? (1u << (tail * BITS)) - 1u : 0xffffffffu;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t u = l + ((uint32_t)k << a.S_log2);
        const uint32_t xw = xw0 + ((uint32_t)(2 * k) << a.S_log2) * kWeyl;
        uint32_t c = push_pair<BITS>(0u, v[k].z, v[k].w, delta, invs, xw + kWeyl, k2, rscale);
        c = push_pair<BITS>(c, v[k].x, v[k].y, delta, invs, xw, k2, rscale);
        if (u + 1u == a.q4) c &= tailmask;                    // the last unit's elements past the plane leave zero bits
        const bool in = u < a.q4;                             // (stores past the workgroup's planes are dropped by the buffer's end)
        if constexpr (BITS == 1) {
            // the four codes of a unit are half a byte: the even lane of a pair stores the byte of both units
            c = in ? c : 0u;
            c |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xf, 0xf, true) << 4;   // quad_perm [1,0,3,2]
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, crs, in && !(l & 1u) ? cvoff + (u >> 1) : 0x80000000u, 0, 0);
        } else if constexpr (CB == 1) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, crs, in ? cvoff + u : 0x80000000u, 0, 0);
        else if constexpr (CB == 2) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)c, crs, in ? cvoff + u * 2u : 0x80000000u, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b32(c, crs, in ? cvoff + u * 4u : 0x80000000u, 0, 0);
    }
    // pad bytes of the plane's last word are zero
    if (l < a.WPP * 4 - cbytes && pv) codes[(size_t)g * a.WPP * 4 + cbytes + l] = 0;
}

template <typename T, int BITS>
__global__ void __launch_bounds__(kMixedThreads, 4) compress_mixed(MixedArgs a) {
    extern __shared__ float4 smem4[];
    char* smem = reinterpret_cast<char*>(smem4);
    const SharedPlace at = shared_place(a);
    MixedShape sh;
    {
        const u32x16* from = reinterpret_cast<const u32x16*>(&a.shape[at.shape]);
        const u32x16 w0 = from[0], w1 = from[1], w2 = from[2];
        __builtin_memcpy(reinterpret_cast<char*>(&sh), &w0, 64);
        __builtin_memcpy(reinterpret_cast<char*>(&sh) + 64, &w1, 64);
        __builtin_memcpy(reinterpret_cast<char*>(&sh) + 128, &w2, 64);
    }
    const CompPtrs pt = shared_ptrs(a, sh.rg, at.map);
    switch (sh.K) {
        case 1: compress_mixed_body<T, BITS, 1>(sh, pt, at.wg, smem); break;
        case 2: compress_mixed_body<T, BITS, 2>(sh, pt, at.wg, smem); break;
        case 3: compress_mixed_body<T, BITS, 3>(sh, pt, at.wg, smem); break;
        case 4: compress_mixed_body<T, BITS, 4>(sh, pt, at.wg, smem); break;
        case 6: compress_mixed_body<T, BITS, 6>(sh, pt, at.wg, smem); break;
        default: compress_mixed_body<T, BITS, 8>(sh, pt, at.wg, smem);
    }
    if (at.wg == 0 && threadIdx.x < 48) zero_pads(a.shape[at.shape].rg, static_cast<char*>(a.pk[at.map]), threadIdx.x);
}
