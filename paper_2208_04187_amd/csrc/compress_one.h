// Part of division.hip (included inside its unnamed namespace, in this order): compress_one and compress_line.

// ------------------------------------------------------------------ compress, planes that are one block

struct OneShape {
    uint32_t P, HW, WPP;
    uint32_t qv;         // 16-byte vectors per plane
    uint32_t S, S_log2;  // lanes per plane (power of two, at most 64)
    uint32_t ppw;        // planes per wavefront = 64 / S
    uint32_t upb, upb_log2;  // compress_line: vectors per block (power of two, at most S); nb = blocks per plane
    uint32_t nb;
    uint32_t K;          // rounds of the instance to launch (3, 4, 6, 12 or 13): not read by the kernels
    uint32_t NG;         // compress_line: groups of 64 / S planes per wavefront (1, or 12 / rounds per plane for tiny planes)
};
struct OneArgs : CompHead, OneShape {};

constexpr int kOneUnits = 13;     // vectors per lane: planes of up to 13 * 64 vectors

// sum over aligned groups of S lanes (S a power of two <= 64, uniform in the wave) in a fixed
// order, result in every lane of the group; all lanes must be active
__device__ __forceinline__ double group_sum_any(uint32_t S, double v) {
    if (S >= 2)  v += dpp_f64<kDppXor1>(v);
    if (S >= 4)  v += dpp_f64<kDppXor2>(v);
    if (S >= 8)  v += dpp_f64<kDppHalfMirror>(v);
    if (S >= 16) v += dpp_f64<kDppMirror>(v);
    if (S >= 32) {
        const uint64_t u = (uint64_t)__double_as_longlong(v);
        const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
        auto row = [&](int lane) -> double {
            const uint32_t l = (uint32_t)__builtin_amdgcn_readlane(lo, lane), h = (uint32_t)__builtin_amdgcn_readlane(hi, lane);
            return __longlong_as_double((long long)(((uint64_t)h << 32) | l));
        };
        const double r0 = row(0), r1 = row(16), r2 = row(32), r3 = row(48);
        if (S == 64) v = (r0 + r1) + (r2 + r3);
        else v = (threadIdx.x & 32u) ? r2 + r3 : r0 + r1;
    }
    return v;
}

// The block covers the whole plane (B at least every extent of the map: the later layers of a
// network, or a block size like 64 on maps of 56 x 56 and below): H^L is the plane's mean, rows
// and columns play no part, and the plane is a flat run of 16-byte vectors.  One wavefront per
// 64 / S planes; the S lanes of a plane keep its vectors in registers (vector u in lane u mod S),
// sums and extremes are reductions over those lanes, the codes leave as one to eight bytes per
// vector.  LDS is not used.
// K: rounds the instance runs (3, 4, 6 or 13; the host picks lanes per plane and K so that a plane has at
// most K rounds of vectors and few of the K * S lane slots stay empty).  No round is tested at run time:
// a uniform test per round splits the code into blocks that each wait for every load (measured: 50 ->
// 40 us on 64 x 256 x 56 x 56); a round past the plane loads nothing (its offsets are out of range) and
// works on zeros that are masked.
template <typename T, int BITS, int K>
__global__ void __launch_bounds__(64) compress_one(OneArgs a) {
    constexpr uint32_t EPV = 16 / sizeof(T);
    constexpr uint32_t CBV = EPV * BITS / 8;
    constexpr bool HALF = EPV * BITS == 4;                // 1-bit codes of a 4-element vector: half a byte
    constexpr float Lf = float((1 << BITS) - 1);
    constexpr uint32_t kDrop = 0x80000000u;              // an offset past every buffer here: the access is dropped
    const uint32_t tid = threadIdx.x;
    const CompPtrs pt = comp_ptrs(a.tab, a.rg, tid);
    const uint32_t sub = tid & (a.S - 1u), pl = tid >> a.S_log2;
    const uint32_t p0 = xcd_run_index(blockIdx.x, gridDim.x) * a.ppw;
    const uint32_t Gc = min(a.ppw, a.P - p0);
    const uint32_t p = p0 + pl;
    const bool live = pl < Gc;

    // the planes of a wavefront are contiguous: one bounds-checked buffer, no branch that depends on a
    // lane (a vector past its plane's end reads the neighbour's data or zero and is masked below)
    u32x4 q[K];
    {
        const T* src = static_cast<const T*>(pt.x) + (size_t)p0 * a.HW;
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, (int)(Gc * a.HW * sizeof(T)), 0x00020000);
        const uint32_t off0 = live ? (pl * a.qv + sub) * 16u : kDrop;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            // a vector past the plane's end is not fetched (offset out of range: it reads as zero)
            const uint32_t u = sub + (uint32_t)k * a.S;
            q[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, u < a.qv ? off0 + (uint32_t)k * a.S * 16u : kDrop, 0, kLoadAux);
        }
    }
    // all loads ahead of the first wait: three of thirteen came behind it (64 x 256 x 56 x 56 43.2 -> 41.8 us; 2-byte elements: level)
    if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
    // ---- Sec. 4.1 AveragePooling with one window: the mean of the plane
    double S = 0.0;
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool valid = sub + (uint32_t)k * a.S < a.qv;
        float f[EPV];
        unpack_vec<T>(q[k], f);
        double s4 = ((double)f[0] + (double)f[1]) + ((double)f[2] + (double)f[3]);
        float vmn = fminf(fminf(f[0], f[1]), fminf(f[2], f[3]));
        float vmx = fmaxf(fmaxf(f[0], f[1]), fmaxf(f[2], f[3]));
        if constexpr (EPV == 8) {
            s4 += ((double)f[4] + (double)f[5]) + ((double)f[6] + (double)f[7]);
            vmn = fminf(vmn, fminf(fminf(f[4], f[5]), fminf(f[6], f[7])));
            vmx = fmaxf(vmx, fmaxf(fmaxf(f[4], f[5]), fmaxf(f[6], f[7])));
        }
        S += valid ? s4 : 0.0;
        mn = fminf(mn, valid ? vmn : __builtin_inff());
        mx = fmaxf(mx, valid ? vmx : -__builtin_inff());
    }
    S = group_sum_any(a.S, S);
    const float lfc = lfc_round<T>(mean_of(S, a.HW), kC16<T>);
    // ---- extremes of the residual (x -> fl(x - m) is monotone), scale of Eq. (quantization), keys
    mn = mn - lfc;
    mx = mx - lfc;
    group_minmax(a.S, mn, mx);
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    const float invs = inv * (float)(1u << (32 - BITS));
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    const uint32_t k2 = mix32(k1 + pt.seed_c);
    uint8_t* cwave = reinterpret_cast<uint8_t*>(pt.codes) + (size_t)p0 * a.WPP * 4;
    if (live && sub == 0) {
        meta_store(pt.meta, p, delta, Delta, kC16<T>);
        lfc_store<T>(pt.lfc, (size_t)p, lfc, kC16<T>);
        uint8_t* cbase = cwave + (size_t)pl * a.WPP * 4;
        const uint32_t cbytes = HALF ? (a.qv + 1u) / 2u : a.qv * CBV;
        const uint32_t padb = a.WPP * 4 - cbytes;                     // pad bytes of the last word are zero
        for (uint32_t t = 0; t < padb; ++t) cbase[cbytes + t] = 0;
    }
    // ---- residual, Quant, packing
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(cwave, 0, (int)(Gc * a.WPP * 4u), 0x00020000);
    const uint32_t rscale = 1u << (16 - BITS);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t u = sub + (uint32_t)k * a.S;
        const uint32_t co = live && u < a.qv ? pl * a.WPP * 4u + u * CBV : kDrop;
        float h[EPV];
        unpack_vec<T>(q[k], h);
#pragma unroll
        for (uint32_t e = 0; e < EPV; ++e) h[e] = h[e] - lfc;
        const uint32_t xw0 = k1 + (u * (EPV / 2)) * kWeyl;
        if constexpr (CBV <= 4) {
            uint32_t c = 0;
#pragma unroll
            for (int j = EPV / 2 - 1; j >= 0; --j)
                c = push_pair<BITS>(c, h[2 * j], h[2 * j + 1], delta, invs, xw0 + (uint32_t)j * kWeyl, k2, rscale);
            if constexpr (HALF) {
                // the even lane of a pair stores the byte of both vectors (a vector past the plane gives zeros)
                c = co != kDrop ? c : 0u;
                c |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xf, 0xf, true) << 4;     // quad_perm [1,0,3,2]
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, crs, co != kDrop && (sub & 1u) == 0 ? pl * a.WPP * 4u + (u >> 1) : kDrop, 0, 0);
            } else if constexpr (CBV == 1) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, crs, co, 0, 0);
            else if constexpr (CBV == 2) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)c, crs, co, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b32(c, crs, co, 0, 0);
        } else {
            uint32_t lo = 0, hi = 0;
            hi = push_pair<BITS>(hi, h[6], h[7], delta, invs, xw0 + 3u * kWeyl, k2, rscale);
            hi = push_pair<BITS>(hi, h[4], h[5], delta, invs, xw0 + 2u * kWeyl, k2, rscale);
            lo = push_pair<BITS>(lo, h[2], h[3], delta, invs, xw0 + kWeyl, k2, rscale);
            lo = push_pair<BITS>(lo, h[0], h[1], delta, invs, xw0, k2, rscale);
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{lo, hi}, crs, co, 0, 0);
        }
    }
}

// 1-D maps (Appendix D, AveragePooling1D: Minibatch x Channel x N, the maps of linear and
// transformer layers) whose block is a power-of-two number of 16-byte vectors (B = 4, 8, 16, 32, 64
// for fp32): laid out like compress_one, vector u of a plane in lane u mod S of round u / S.  The planes of
// a wavefront are contiguous: their vectors are read through one bounds-checked buffer, codes and H^L leave
// through bounds-checked buffer stores (planes past the map are past the buffers), so no branch depends on a
// lane or on the round: loads and rounds are straight-line code that the compiler is free to interleave.
// K as in compress_one.
//
// What bounds it is the vector ALUs, so what a block costs beyond its elements is kept small:
// - LU >= 0: a block is 1 << LU = 1, 2 or 4 vectors; its sum is LU DPP steps over neighbouring lanes.
// - LU < 0: longer blocks (8 vectors and more).  A 64-bit DPP step is two moves and an addition, and every lane
//   would repeat the block's mean; instead the lanes park their partial sums in LDS, ONE lane per block of the
//   whole wavefront adds them in the same tree order, takes the mean, stores H^L and hands it out through LDS.
//   LU = -1: a block lies in one round.  LU = -2: S is half a block, so that a plane of a few hundred bytes
//   (96 tokens) leaves no lane empty, and a lane first adds its two rounds of the block.
// - Only rounds that can hold vectors past the plane (k >= first_masked) are masked; in the others every block is
//   whole, its count a power of two and the mean an exact scaling.
// Before and after (every lane repeating the 64-bit reduction and the mean, rounds tested at run time): 64 x 3136 planes
// of 384 floats cached as bfloat16, B = 64, b = 2: 72 -> 56 us (5.5 TB/s of x); of 96 floats: 32 -> 21.5 us;
// 32 x 512 planes of 3072 bfloat16, B = 8, b = 4: 36 -> 28.8 us.
constexpr int kLineUnits = 13;
// NG > 1: planes of at most R = K / NG rounds (a few hundred bytes each): a wavefront takes NG groups of
// 64 / S planes one after the other, all their loads issued first, so that it has K vectors per lane in
// flight like the instances for larger planes (two or three would not cover the memory latency).
// where(pt, wg): the wavefront's map and its place in it.  A callable, so that they are worked out in here: made by the caller and handed in, they have the
// compiler put half of the loads behind the first wait, and a scheduling barrier against that costs registers (64 x 3136 x 1 x 96 under B = 4 23.0 us, 23.3 with
// the barrier; 32 x 512 x 1 x 3072 in bfloat16 25.6 and 26.2, 26.6 without).
template <typename T, int BITS, int K, int NG, int LU, typename Where>
__device__ __forceinline__ void compress_line_body(const OneShape& a, Where where) {
    constexpr int R = K / NG;
    static_assert(R * NG == K, "whole groups");
    constexpr bool LDS = LU < 0;
    constexpr int UR = LU == -2 ? 2 : 1;                  // rounds per block
    constexpr int RB = (R + UR - 1) / UR;                 // rounds of blocks
    // the host gives an instance planes of at least this many rounds, so the earlier ones are whole
    constexpr int first_masked = NG > 1 ? R - 1 : K == 13 ? 6 : K == 6 ? 4 : K == 4 ? 3 : 0;
    constexpr uint32_t EPV = 16 / sizeof(T);
    constexpr uint32_t CBV = EPV * BITS / 8;
    constexpr bool HALF = EPV * BITS == 4;                // 1-bit codes of a 4-element vector: half a byte
    constexpr bool KEEP = sizeof(T) == 4 || R <= 6;       // residuals stay in registers between the extremes and the codes
    constexpr float Lf = float((1 << BITS) - 1);
    constexpr uint32_t kDrop = 0x80000000u;              // an offset past every buffer here (and no wrap when a round's offset is added): the access is dropped
    constexpr uint32_t LB = (sizeof(T) == 2 || kC16<T>) ? 2u : 4u;          // bytes of a cached H^L value
    const uint32_t tid = threadIdx.x;
    CompPtrs pt;
    uint32_t wg;
    where(pt, wg);
    const uint32_t S = a.S, sub = tid & (S - 1u), lp = tid >> a.S_log2;
    const uint32_t ppw = a.ppw * NG;                     // planes of the wavefront
    const uint32_t p0 = wg * ppw;
    const uint32_t Gc = min(ppw, a.P - p0);

    // Offset of round r's piece (`bytes` per vector) given that of round 0: in a whole round the step goes into the scalar
    // operand, otherwise a lane without a vector there is sent past the buffer.
    struct Place { uint32_t v, s; };
    auto place = [&](int r, uint32_t off, uint32_t bytes) -> Place {
        const uint32_t step = (uint32_t)r * S * bytes;
        if (r < first_masked) return Place{off, step};
        return Place{sub + (uint32_t)r * S < a.qv && off != kDrop ? off + step : kDrop, 0u};
    };
    u32x4 q[K];
    {
        const T* src = static_cast<const T*>(pt.x) + (size_t)p0 * a.HW;
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, (int)(Gc * a.HW * sizeof(T)), 0x00020000);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const uint32_t off0 = ((g * a.ppw + lp) * a.qv + sub) * 16u;          // a plane past the map is past the buffer
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // a vector past the plane's end is not fetched
                const Place at = place(r, off0, 16u);
                q[g * R + r] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at.v, (int)at.s, kLoadAux);
            }
        }
    }
    // (the one case that gains from it: 64 x 3136 x 1 x 96 in bfloat16 under B = 64 21.3 -> 20.8 us)
    if constexpr (sizeof(T) == 2 && NG > 1 && LDS) __builtin_amdgcn_sched_barrier(0);
    const uint32_t cnt_full = a.upb * EPV, cnt_last = (a.qv - (a.nb - 1u) * a.upb) * EPV;
    const double rcp_last = LU == 0 ? 0.0 : 1.0 / (double)cnt_last;
    const double rcp_full = __longlong_as_double((long long)(1023u - (31u - (uint32_t)__builtin_clz(cnt_full))) << 52);     // a power of two
    uint8_t* cwave = reinterpret_cast<uint8_t*>(pt.codes) + (size_t)p0 * a.WPP * 4;
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(cwave, 0, (int)(Gc * a.WPP * 4u), 0x00020000);
    const __amdgpu_buffer_rsrc_t lrs = __builtin_amdgcn_make_buffer_rsrc(
        static_cast<uint8_t*>(pt.lfc) + (size_t)p0 * a.nb * LB, 0, (int)(Gc * a.nb * LB), 0x00020000);
    auto put_lfc = [&](float v, Place at) {
        if constexpr (LB == 2) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(__float_as_uint(v) >> 16), lrs, at.v, (int)at.s, 0);     // v is a bfloat16
        else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), lrs, at.v, (int)at.s, 0);
    };
    const uint32_t rscale = 1u << (16 - BITS);
    auto vector_sum = [&](const u32x4& v) -> double {              // (a vector past the plane was read as zero)
        float f[EPV];
        unpack_vec<T>(v, f);
        double s4 = ((double)f[0] + (double)f[1]) + ((double)f[2] + (double)f[3]);
        if constexpr (EPV == 8) s4 += ((double)f[4] + (double)f[5]) + ((double)f[6] + (double)f[7]);
        return s4;
    };

    // ---- AveragePooling1D, blocks of 8 vectors and more: the sums of all groups through LDS
    extern __shared__ float4 smem4[];
    const uint32_t logM = min(a.upb_log2, a.S_log2), bpr_log = 6u - logM;        // lanes that share a block, blocks per round
    const uint32_t prow = 64u + (1u << bpr_log);                                  // doubles per round of blocks, one of padding per block
    double* part = reinterpret_cast<double*>(smem4);                              // [NG * RB][prow]
    float* lfcs = reinterpret_cast<float*>(part + NG * RB * prow);                // [NG * RB << bpr_log]
    if constexpr (LDS) {
        const uint32_t slot = tid + (tid >> logM);
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                double s = vector_sum(q[g * R + rb * UR]);
                if constexpr (UR == 2) { if (rb * UR + 1 < R) s += vector_sum(q[g * R + (rb * UR + 1 < R ? rb * UR + 1 : 0)]); }
                part[(g * RB + rb) * prow + slot] = s;
            }
        wave_sync();
        for (uint32_t t0 = 0; t0 < ((uint32_t)(NG * RB) << bpr_log); t0 += 64u) {
            const uint32_t t = min(t0 + tid, ((uint32_t)(NG * RB) << bpr_log) - 1u);
            const uint32_t row = t >> bpr_log, gl = t & ((1u << bpr_log) - 1u);
            const double* ps = part + row * prow + gl * ((1u << logM) + 1u);
            auto tree8 = [&](int i) -> double { return ((ps[i] + ps[i + 1]) + (ps[i + 2] + ps[i + 3])) + ((ps[i + 4] + ps[i + 5]) + (ps[i + 6] + ps[i + 7])); };
            double Sb = tree8(0);
            if (logM >= 4) Sb += tree8(8);
            if (logM >= 5) Sb += tree8(16) + tree8(24);
            if (logM >= 6) Sb += (tree8(32) + tree8(40)) + (tree8(48) + tree8(56));
            const uint32_t g = row / (uint32_t)RB, rb = row - g * (uint32_t)RB;
            const uint32_t l0 = gl << logM;                                       // the block's first lane
            const uint32_t pl = g * a.ppw + (l0 >> a.S_log2);
            const uint32_t blk = (rb << (a.S_log2 - logM)) + ((l0 & (S - 1u)) >> logM);
            const bool last = blk + 1u == a.nb;                                   // the last block may be short
            const float m = lfc_round<T>(mean_with_rcp(Sb + 0.0, last ? cnt_last : cnt_full, last ? rcp_last : rcp_full), kC16<T>);
            lfcs[t] = m;
            put_lfc(m, Place{blk < a.nb ? (pl * a.nb + blk) * LB : kDrop, 0u});
        }
        wave_sync();
    }

#pragma unroll
    for (int g = 0; g < NG; ++g) {
    const uint32_t pl = (uint32_t)g * a.ppw + lp;
    const uint32_t p = p0 + pl;
    const bool live = pl < Gc;
    // ---- shorter blocks: sums over the lanes of a block; residual extremes of the plane
    float lfcv[R];
    float h[KEEP ? R : 1][EPV];
    float mn = __builtin_inff(), mx = -__builtin_inff();
    auto place_block = [&](int k, uint32_t off) -> Place {
        const uint32_t step = (((uint32_t)k * S) >> a.upb_log2) * LB;
        if (k < first_masked) return Place{off, step};
        return Place{sub + (uint32_t)k * S < a.qv && off != kDrop ? off + step : kDrop, 0u};
    };
    const uint32_t lo0 = (sub & (a.upb - 1u)) == 0 ? (pl * a.nb + (sub >> a.upb_log2)) * LB : kDrop;     // H^L of the block whose first vector this is
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const bool masked = k >= first_masked;
        const bool valid = !masked || sub + (uint32_t)k * S < a.qv;
        float lfc;
        if constexpr (LDS) {
            lfc = lfcs[((uint32_t)(g * RB + k / UR) << bpr_log) + (tid >> logM)];
        } else {
            // a block of negative zeros sums to +0, as a sum from 0 does; added before the rounding to binary32, where a tiny
            // negative sum may become -0, which is then the mean
            const double Sb = group_sum<(LU < 0 ? 1 : 1 << LU)>(vector_sum(q[g * R + k])) + 0.0;
            float m;
            if (LU == 0 || !masked) m = (float)(Sb * rcp_full);                    // exact scaling by a power of two
            else {
                const uint32_t u = sub + (uint32_t)k * S;
                const bool last = (u & ~(a.upb - 1u)) + a.upb >= a.qv;             // the last block may be short
                m = mean_with_rcp(Sb, last ? cnt_last : cnt_full, last ? rcp_last : rcp_full);
            }
            lfc = lfc_round<T>(m, kC16<T>);
            // (S is a multiple of the block's 1 << LU vectors)
            put_lfc(lfc, place_block(k, lo0));
        }
        lfcv[k] = lfc;
        float f[EPV];
        unpack_vec<T>(q[g * R + k], f);
        float vmn = mn, vmx = mx;
#pragma unroll
        for (uint32_t e = 0; e < EPV; ++e) f[e] = f[e] - lfc;
#pragma unroll
        for (uint32_t e = 0; e < EPV; e += 2) {
            vmn = fminf(vmn, fminf(f[e], f[e + 1]));
            vmx = fmaxf(vmx, fmaxf(f[e], f[e + 1]));
        }
        mn = valid ? vmn : mn;
        mx = valid ? vmx : mx;
        if constexpr (KEEP) {
#pragma unroll
            for (uint32_t e = 0; e < EPV; ++e) h[k][e] = f[e];
        }
    }
    group_minmax(S, mn, mx);
    float delta, Delta, inv;
    plane_scale_any(mn, mx, Lf, kC16<T>, delta, Delta, inv);
    const float invs = inv * (float)(1u << (32 - BITS));
    const uint32_t k1 = mix32(p ^ pt.seed_a);
    const uint32_t k2 = mix32(k1 + pt.seed_c);
    if (live && sub == 0) {
        meta_store(pt.meta, p, delta, Delta, kC16<T>);
        uint8_t* cbase = cwave + (size_t)pl * a.WPP * 4;
        const uint32_t cbytes = HALF ? (a.qv + 1u) / 2u : a.qv * CBV;
        const uint32_t padb = a.WPP * 4 - cbytes;                     // pad bytes of the last word are zero
        for (uint32_t t = 0; t < padb; ++t) cbase[cbytes + t] = 0;
    }
    // ---- residual, Quant, packing
    const uint32_t co0 = HALF ? ((sub & 1u) == 0 ? pl * a.WPP * 4u + (sub >> 1) : kDrop) : pl * a.WPP * 4u + sub * CBV;
    const uint32_t xs0 = k1 + sub * (EPV / 2) * kWeyl;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const uint32_t u = sub + (uint32_t)k * S;
        const bool valid = k < first_masked || u < a.qv;
        float f[EPV];
        if constexpr (KEEP) {
#pragma unroll
            for (uint32_t e = 0; e < EPV; ++e) f[e] = h[k][e];
        } else {
            unpack_vec<T>(q[g * R + k], f);
#pragma unroll
            for (uint32_t e = 0; e < EPV; ++e) f[e] = f[e] - lfcv[k];
        }
        const uint32_t xw0 = xs0 + ((uint32_t)k * S * (EPV / 2)) * kWeyl;
        if constexpr (CBV <= 4) {
            uint32_t c = 0;
#pragma unroll
            for (int j = EPV / 2 - 1; j >= 0; --j)
                c = push_pair<BITS>(c, f[2 * j], f[2 * j + 1], delta, invs, xw0 + (uint32_t)j * kWeyl, k2, rscale);
            if constexpr (HALF) {
                // the even lane of a pair stores the byte of both vectors (a vector past the plane gives zeros)
                c = valid ? c : 0u;
                c |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xf, 0xf, true) << 4;     // quad_perm [1,0,3,2]
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, crs, valid && co0 != kDrop ? co0 + (uint32_t)k * S / 2u : kDrop, 0, 0);
            } else {
                const Place at = place(k, co0, CBV);
                if constexpr (CBV == 1) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, crs, at.v, (int)at.s, 0);
                else if constexpr (CBV == 2) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)c, crs, at.v, (int)at.s, 0);
                else __builtin_amdgcn_raw_buffer_store_b32(c, crs, at.v, (int)at.s, 0);
            }
        } else {
            uint32_t lo = 0, hi = 0;
            hi = push_pair<BITS>(hi, f[6], f[7], delta, invs, xw0 + 3u * kWeyl, k2, rscale);
            hi = push_pair<BITS>(hi, f[4], f[5], delta, invs, xw0 + 2u * kWeyl, k2, rscale);
            lo = push_pair<BITS>(lo, f[2], f[3], delta, invs, xw0 + kWeyl, k2, rscale);
            lo = push_pair<BITS>(lo, f[0], f[1], delta, invs, xw0, k2, rscale);
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{lo, hi}, crs, valid ? co0 + (uint32_t)k * S * CBV : kDrop, 0, 0);
        }
    }
    }
}

template <typename T, int BITS, int K, int NG, int LU>
__global__ void __launch_bounds__(64) compress_line(OneArgs a) {
    compress_line_body<T, BITS, K, NG, LU>(a, [&](CompPtrs& pt, uint32_t& wg) {
        pt = comp_ptrs(a.tab, a.rg, threadIdx.x);
        wg = xcd_run_index(blockIdx.x, gridDim.x);
    });
}

// The maps of several shapes that have the same instance, in one launch.  What it saves is the drain and the filling between the launches, 2-4 us
// each: the compress side of a Swin-T step in eight launches 170 us, in four 162; two widths of a T5-base step 62 and 58.
struct LinesArgs : SharedTab {
    OneShape shape[kSharedShapes];
    Regions rg[kSharedShapes];
};
template <typename T, int BITS, int K, int LU>
__global__ void __launch_bounds__(64) compress_lines(LinesArgs a) {
    const SharedPlace at = shared_place(a);
    const Regions& rg = a.rg[at.shape];
    if (at.wg == 0 && threadIdx.x < 48) zero_pads(rg, static_cast<char*>(a.pk[at.map]), threadIdx.x);
    compress_line_body<T, BITS, K, 1, LU>(a.shape[at.shape], [&](CompPtrs& pt, uint32_t& wg) {
        pt = shared_ptrs(a, rg, at.map);
        wg = xcd_run_index(at.wg, at.n);
    });
}
