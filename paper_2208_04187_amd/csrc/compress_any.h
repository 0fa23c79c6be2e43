// Part of division.hip (included inside its unnamed namespace, in this order): compress_any (2-D and 3-D).

// ------------------------------------------------------------------ compress, any shape

struct AnyArgs {
    CompTab tab;
    Regions rg;
    uint32_t P, H, W, HW, LH, LW, nb, WPP, B;      // H, LH: rows / block rows of one depth slice
    uint32_t D;                                     // depth slices (1 for a 2-D map)
    uint32_t J_log2;                                // log2 of the lanes that share a block
};

// One workgroup per plane, of one, four or sixteen wavefronts by the plane's size; x is read twice, the second time from L2.
// Pass A: 2^J_log2 lanes per block, eight loads in flight each (a lane per block left nine lanes of the workgroup with 4096
// loads one after another on 147 x 147 under B = 64).  Pass B: four consecutive elements per lane, so that neighbouring lanes
// read neighbouring memory, whose codes neighbouring lanes put together to a word; the block is looked up per four elements.
// What bounds it: the latency of its few loads per lane, and the divisions of the lookup.  Against a lane per block, a lane per word of
// codes and 256 threads whatever the plane (maps of 4 M elements, us): 147 x 147 under B = 18, b = 1 75 -> 16, 203 x 203 in bfloat16 under B = 8,
// b = 1 84 -> 25, 183 x 183 under B = 4 78 -> 22, 16 x 56 x 56 under B = 16, b = 1 521 -> 36, rows of 96 under B = 18, b = 1 224 -> 45, 13 x 13 under
// B = 64, b = 1 337 -> 30.
// ND = 3: planes of D x H x W elements with blocks of B x B x B (Appendix D).
template <typename T, int BITS, int ND>
__device__ __forceinline__ void compress_any_body(const AnyArgs& a) {
    __shared__ float red[32];
    constexpr uint32_t UPW = 8 / BITS;      // lanes (of four elements) per word
    constexpr float Lf = float((1 << BITS) - 1);
    const uint32_t tid = threadIdx.x, NT = blockDim.x;
    const uint32_t p = blockIdx.x;
    const CompPtrs pt = comp_ptrs(a.tab, a.rg, tid);
    const T* xp = static_cast<const T*>(pt.x) + (size_t)p * a.HW;
    const size_t lfc0 = (size_t)p * a.nb;      // this plane's first LFC element

    // pass A: block means; block min/max of the residual follow from the
    // block min/max of x because x -> fl(x - m) is monotone
    float mn = __builtin_inff(), mx = -__builtin_inff();
    const uint32_t J = 1u << a.J_log2, jl = tid & (J - 1u);
    for (uint32_t blk = tid >> a.J_log2; blk < a.nb; blk += NT >> a.J_log2) {
        const uint32_t bq = blk / a.LW, bj = blk - bq * a.LW;
        uint32_t bd = 0, bi = bq;
        if constexpr (ND == 3) { bd = bq / a.LH; bi = bq - bd * a.LH; }
        const uint32_t rows = min(a.B, a.H - bi * a.B), bw = min(a.B, a.W - bj * a.B);
        const uint32_t deps = ND == 3 ? min(a.B, a.D - bd * a.B) : 1u;
        const uint32_t cnt = deps * rows * bw;
        const T* bp = xp + (((size_t)bd * a.B * a.H + bi * a.B) * a.W + bj * a.B);
        // lane jl takes the block's elements jl, jl + J, ...; their row (over all slices) and column step with them
        uint32_t row = jl / bw, col = jl - row * bw;
        const uint32_t drow = J / bw, dcol = J - drow * bw;
        double S = 0.0;
        float xmin = __builtin_inff(), xmax = -__builtin_inff();
        for (uint32_t e = jl; e < cnt; e += 8u * J) {
            float v[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) {
                size_t at;
                if constexpr (ND == 3) {
                    const uint32_t zz = row / rows;
                    at = ((size_t)zz * a.H + (row - zz * rows)) * a.W + col;
                } else {
                    at = (size_t)row * a.W + col;
                }
                v[k] = Elem<T>::load(bp, e + k * J < cnt ? at : 0);
                row += drow; col += dcol;
                if (col >= bw) { col -= bw; ++row; }
            }
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) {
                const bool in = e + k * J < cnt;
                S += in ? (double)v[k] : 0.0;
                xmin = fminf(xmin, in ? v[k] : __builtin_inff());
                xmax = fmaxf(xmax, in ? v[k] : -__builtin_inff());
            }
        }
        for (uint32_t off = 1; off < J; off <<= 1) {            // (the lanes of a block are here together)
            S += __shfl_xor(S, (int)off);
            xmin = fminf(xmin, __shfl_xor(xmin, (int)off));
            xmax = fmaxf(xmax, __shfl_xor(xmax, (int)off));
        }
        const float lfc = lfc_round<T>((float)(S / (double)cnt), kC16<T>);
        if (jl == 0) lfc_store<T>(pt.lfc, lfc0 + blk, lfc, kC16<T>);
        mn = fminf(mn, xmin - lfc);
        mx = fmaxf(mx, xmax - lfc);
    }
    group_minmax(64, mn, mx);
    if ((tid & 63u) == 0) { red[2 * (tid >> 6)] = mn; red[2 * (tid >> 6) + 1] = mx; }
    __syncthreads();
    for (uint32_t w = 0; w < NT / 64u; ++w) { mn = fminf(mn, red[2 * w]); mx = fmaxf(mx, red[2 * w + 1]); }
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    if (tid == 0) meta_store(pt.meta, p, delta, Delta, kC16<T>);
    const float inv16 = inv * 65536.0f;
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    const uint32_t k2 = mix32(k1 + pt.seed_c);

    // pass B: quantise and pack (the H^L read here were written by this workgroup before the barrier above)
    auto block_row = [&](uint32_t r) -> uint32_t {              // r counts the rows of all slices
        if constexpr (ND == 3) { const uint32_t z = r / a.H; return ((z / a.B) * a.LH + (r - z * a.H) / a.B) * a.LW; }
        else return (r / a.B) * a.LW;
    };
    const bool wide = a.W >= 3 && a.B >= 3;      // four elements then enter another row, or another block of a row, at most once
    const uint32_t lastrow = a.D * a.H - 1u;
    for (uint32_t u = tid; u < a.WPP * UPW; u += NT) {           // (the lanes of a word are here together)
        const uint32_t i0 = 4u * u;
        uint32_t word = 0;
        if (i0 < a.HW) {
            uint32_t off[4];
            if (wide) {
                const uint32_t r = i0 / a.W, c = i0 - r * a.W, bj = c / a.B;
                const uint32_t here = block_row(r) + bj, next = block_row(min(r + 1u, lastrow));
                const uint32_t left = bj * a.B + a.B - c, rowleft = a.W - c;
                off[0] = here;
#pragma unroll
                for (uint32_t j = 1; j < 4; ++j) off[j] = j < rowleft ? here + (j >= left ? 1u : 0u) : next;
            } else {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) {
                    const uint32_t i = min(i0 + j, a.HW - 1u), r = i / a.W;
                    off[j] = block_row(r) + (i - r * a.W) / a.B;
                }
            }
            float v[4], m[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) v[j] = Elem<T>::load(xp, min(i0 + j, a.HW - 1u));
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) m[j] = lfc_load<T>(pt.lfc, lfc0 + off[j], kC16<T>);
#pragma unroll
            for (uint32_t j = 0; j < 4; j += 2) {
                const uint32_t w = pair_word(k1 + ((i0 + j) >> 1) * kWeyl, k2);
                const uint32_t q0 = min(quant<0>(v[j] - m[j], delta, inv16, w), (1u << BITS) - 1u);      // t may exceed L by a few ulp
                const uint32_t q1 = min(quant<1>(v[j + 1] - m[j + 1], delta, inv16, w), (1u << BITS) - 1u);
                word |= i0 + j < a.HW ? q0 << (j * BITS) : 0u;
                word |= i0 + j + 1u < a.HW ? q1 << ((j + 1u) * BITS) : 0u;
            }
        }
        if constexpr (UPW > 1) {
            word <<= (u & (UPW - 1u)) * (4u * BITS);
#pragma unroll
            for (uint32_t off = 1; off < UPW; off <<= 1) word |= (uint32_t)__shfl_xor((int)word, (int)off);
        }
        if ((u & (UPW - 1u)) == 0) pt.codes[(size_t)p * a.WPP + u / UPW] = word;
    }
}

template <typename T, int BITS>
__global__ void __launch_bounds__(1024) compress_any(AnyArgs a) { compress_any_body<T, BITS, 2>(a); }
template <typename T, int BITS>
__global__ void __launch_bounds__(1024) compress_any_3d(AnyArgs a) { compress_any_body<T, BITS, 3>(a); }
