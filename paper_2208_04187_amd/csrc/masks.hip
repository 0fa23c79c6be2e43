// 1-bit mask operators for AMD MI355X (gfx950): the Relu and Dropout operators of
// "DIVISION: Memory Efficient Training via Dual Activation Precision" (appendix on
// operator compression, Algorithms "Relu operator" and "Dropout operator").
//
//   forward:   V = sgn(H) (Relu) or V ~ Bernoulli(1 - p) (Dropout); out = V (.) H;
//              V is cached one bit per element (N^2/8 bytes per channel).
//   backward:  grad_in = V (.) grad_out.
//
// Pure streaming kernels: one 16-byte vector per lane and step, the lane's 4 (fp32) or
// 8 (bf16) mask bits are merged over 8 or 4 adjacent lanes with DPP and leave as whole
// 32-bit words.  Mask layout: bit i%32 of word i/32, pad bits zero.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/division.h"

namespace {
#include "fastdiv.h"

constexpr int kThreads = 256;
constexpr int kVecPerThread = 4;                  // 16-byte vectors a thread handles, kThreads apart
constexpr uint32_t kWeyl = 0x9E3779B9u;
constexpr uint64_t kDropoutStream = 0xD509A5B3C2E1F047ull;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 32-bit xorshift-multiply finaliser (shifts 16/15/16): the codec's random source
__host__ __device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352du;
    x ^= x >> 15; x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// random word of element pair j of a stream segment with keys (k1, k2)
__device__ __forceinline__ uint32_t pair_word(uint32_t k1, uint32_t k2, uint32_t j) {
    uint32_t x = k1 + j * kWeyl;
    x ^= x >> 16; x *= 0x7feb352du;
    x = x ^ (x >> 15) ^ k2; x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7-i inside each 8 lanes

// element helpers: T = float or uint16_t (bf16 bit pattern); values pass through bit for bit
template <typename T> struct Tr;
template <> struct Tr<float> {
    static constexpr int EPV = 4;
    static __device__ __forceinline__ bool positive(uint32_t bits) { return __uint_as_float(bits) > 0.0f; }
};
template <> struct Tr<uint16_t> {
    static constexpr int EPV = 8;
    static __device__ __forceinline__ bool positive(uint32_t bits) { return __uint_as_float(bits << 16) > 0.0f; }
};

// the EPV "is positive" bits of one vector (bit e = element e)
template <typename T>
__device__ __forceinline__ uint32_t positive_bits(u32x4 q) {
    uint32_t m = 0;
    if constexpr (sizeof(T) == 4) {
        m |= Tr<T>::positive(q.x) ? 1u : 0u; m |= Tr<T>::positive(q.y) ? 2u : 0u;
        m |= Tr<T>::positive(q.z) ? 4u : 0u; m |= Tr<T>::positive(q.w) ? 8u : 0u;
    } else {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            m |= Tr<T>::positive(w[k] & 0xffffu) ? (1u << (2 * k)) : 0u;
            m |= Tr<T>::positive(w[k] >> 16) ? (2u << (2 * k)) : 0u;
        }
    }
    return m;
}

// keeps the elements of a vector whose bit is set, +0 elsewhere
template <typename T>
__device__ __forceinline__ u32x4 select_bits(u32x4 q, uint32_t m) {
    u32x4 o;
    if constexpr (sizeof(T) == 4) {
        o.x = (m & 1u) ? q.x : 0u; o.y = (m & 2u) ? q.y : 0u;
        o.z = (m & 4u) ? q.z : 0u; o.w = (m & 8u) ? q.w : 0u;
    } else {
        uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t keep = ((m >> (2 * k)) & 1u ? 0x0000ffffu : 0u) | ((m >> (2 * k + 1)) & 1u ? 0xffff0000u : 0u);
            w[k] &= keep;
        }
        o.x = w[0]; o.y = w[1]; o.z = w[2]; o.w = w[3];
    }
    return o;
}

// Dropout's keep bits of the EPV elements starting at element e0 (a multiple of EPV):
// element i keeps its value iff the 16 random bits of element (i mod 2^32) of stream
// segment i >> 32 are >= T.
template <typename T>
__device__ __forceinline__ uint32_t keep_bits(uint64_t e0, uint32_t seed_a, uint32_t seed_c, uint32_t thr) {
    constexpr int EPV = Tr<T>::EPV;
    const uint32_t seg = (uint32_t)(e0 >> 32);
    const uint32_t k1 = mix32(seg ^ seed_a);
    const uint32_t k2 = mix32(k1 + seed_c);
    const uint32_t j0 = (uint32_t)e0 >> 1;
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < EPV / 2; ++k) {
        const uint32_t w = pair_word(k1, k2, j0 + (uint32_t)k);
        m |= ((w & 0xffffu) >= thr ? 1u : 0u) << (2 * k);
        m |= ((w >> 16) >= thr ? 2u : 0u) << (2 * k);
    }
    return m;
}

// merges the per-lane bit groups of 32/EPV adjacent lanes into the 32-bit mask word they
// share (every lane of the group ends up with the whole word); all lanes must be active
template <typename T>
__device__ __forceinline__ uint32_t merge_word(uint32_t m, uint32_t lane) {
    constexpr int EPV = Tr<T>::EPV;
    constexpr uint32_t LPW = 32 / EPV;               // lanes per word: 8 (fp32) or 4 (bf16)
    uint32_t v = m << (EPV * (lane & (LPW - 1)));
    v |= dpp_u32<kDppXor1>(v);
    v |= dpp_u32<kDppXor2>(v);
    if constexpr (LPW == 8) v |= dpp_u32<kDppHalfMirror>(v);
    return v;
}

struct MaskArgs {
    const void* in;        // x (forward) or grad_out (backward)
    void* out;             // y or grad_in
    uint32_t* mask;
    uint64_t n;            // elements
    uint64_t nwords;       // mask words = ceil(n / 32)
    uint32_t vec;          // in and out are 16-byte aligned: whole vectors move with 16-byte accesses
    uint32_t seed_a, seed_c, thr;      // dropout only
};

// MODE 0: Relu forward, 1: Dropout forward, 2: backward (mask is read)
template <typename T, int MODE>
__global__ void __launch_bounds__(kThreads) mask_kernel(MaskArgs a) {
    constexpr int EPV = Tr<T>::EPV;
    constexpr uint32_t LPW = 32 / EPV;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const T* in = static_cast<const T*>(a.in);
    T* out = static_cast<T*>(a.out);
    const uint64_t v0 = (uint64_t)blockIdx.x * (kThreads * kVecPerThread) + tid;
#pragma unroll
    for (int u = 0; u < kVecPerThread; ++u) {
        const uint64_t vi = v0 + (uint64_t)u * kThreads;       // the lane's vector
        const uint64_t e0 = vi * EPV;
        const bool whole = e0 + EPV <= a.n;
        const bool fast = whole && a.vec;
        u32x4 q = {0u, 0u, 0u, 0u};
        if (fast) {
            q = *reinterpret_cast<const u32x4*>(in + e0);
        } else if (e0 < a.n) {
            // ragged last vector, or unaligned buffers: element by element
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                if (e0 + e < a.n) {
                    if constexpr (sizeof(T) == 4) w[e] = __float_as_uint(in[e0 + e]);
                    else w[e / 2] |= (uint32_t)in[e0 + e] << (16 * (e & 1));
                }
            q.x = w[0]; q.y = w[1]; q.z = w[2]; q.w = w[3];
        }
        uint32_t m;
        if constexpr (MODE == 0) m = positive_bits<T>(q);
        else if constexpr (MODE == 1) m = keep_bits<T>(e0, a.seed_a, a.seed_c, a.thr);
        else {
            const uint64_t wi = vi / LPW;
            const uint32_t word = wi < a.nwords ? a.mask[wi] : 0u;
            m = (word >> (EPV * (uint32_t)(vi & (LPW - 1)))) & ((1u << EPV) - 1u);
        }
        // bits of elements past the end are zero
        if (!whole) m &= e0 < a.n ? (1u << (uint32_t)(a.n - e0)) - 1u : 0u;
        const u32x4 o = select_bits<T>(q, m);
        if (fast) {
            *reinterpret_cast<u32x4*>(out + e0) = o;
        } else if (e0 < a.n) {
            const uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                if (e0 + e < a.n) {
                    if constexpr (sizeof(T) == 4) out[e0 + e] = __uint_as_float(w[e]);
                    else out[e0 + e] = (uint16_t)(w[e / 2] >> (16 * (e & 1)));
                }
        }
        if constexpr (MODE != 2) {
            const uint32_t word = merge_word<T>(m, lane);
            const uint64_t wi = vi / LPW;
            if ((lane & (LPW - 1)) == 0 && wi < a.nwords) a.mask[wi] = word;
        }
    }
}

int launch(int mode, const void* in, int64_t n, division_dtype dt, void* out, void* mask, size_t mask_bytes,
           float p, uint64_t seed, void* hip_stream) {
    if (n < 0 || (dt != DIVISION_F32 && dt != DIVISION_BF16)) return DIVISION_EINVAL;
    if (n == 0) return DIVISION_OK;                 // nothing to do; the pointers may be null
    if (!in || !out || !mask) return DIVISION_EINVAL;
    if (n > (int64_t)1 << 40) return DIVISION_ERANGE;
    if (mask_bytes < division_mask_bytes(n)) return DIVISION_ESIZE;
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    if (((uintptr_t)in % es) != 0 || ((uintptr_t)out % es) != 0 || ((uintptr_t)mask % 4) != 0) return DIVISION_EALIGN;
    MaskArgs a{};
    a.in = in; a.out = out; a.mask = static_cast<uint32_t*>(mask);
    a.n = (uint64_t)n; a.nwords = ((uint64_t)n + 31) / 32;
    a.vec = ((uintptr_t)in % 16) == 0 && ((uintptr_t)out % 16) == 0;
    if (mode == 1) {
        const uint64_t s = seed ^ kDropoutStream;
        a.seed_a = mix32((uint32_t)(s & 0xffffffffu) ^ 0x243F6A88u);
        a.seed_c = mix32((uint32_t)(s >> 32) ^ 0x85A308D3u);
        // T = floor(p * 65536 + 0.5) in binary64, clipped to [0, 65536]; NaN drops nothing
        const double t = (double)p * 65536.0 + 0.5;
        a.thr = !(t >= 1.0) ? 0u : t >= 65537.0 ? 65536u : (uint32_t)t;
    }
    const uint64_t epv = 16 / es;
    const uint64_t nvec = ((uint64_t)n + epv - 1) / epv;
    const uint64_t per_block = (uint64_t)kThreads * kVecPerThread;
    const uint32_t grid = (uint32_t)((nvec + per_block - 1) / per_block);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    void (*kern)(MaskArgs);
    if (dt == DIVISION_F32) kern = mode == 0 ? mask_kernel<float, 0> : mode == 1 ? mask_kernel<float, 1> : mask_kernel<float, 2>;
    else kern = mode == 0 ? mask_kernel<uint16_t, 0> : mode == 1 ? mask_kernel<uint16_t, 1> : mask_kernel<uint16_t, 2>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), 0, st, a);
    return hipGetLastError() == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
}

// ------------------------------------------------------------------ Max-Pooling layer, kernel = stride = k

struct PoolArgs {
    const void* in;        // x (forward) or grad_out (backward)
    void* out;             // y or grad_in
    uint32_t* mask;
    uint32_t P, H, W, HW, OH, OW, k;
    uint32_t band;         // maxpool2_forward_fast: output rows a workgroup handles
    uint32_t chunk;        // maxpool_forward_kernel: elements a workgroup handles (a multiple of 32)
    uint32_t quick;        // every quotient inside a workgroup's elements is exact with the multiplier (fastdiv_ok)
    uint64_t n;            // elements of the map
    uint64_t rows;         // maxpool2_forward_fast: output rows of all planes
    double r_HW, r_wv;     // 1 / HW, 1 / pieces of a row
    FastDiv d_HW, d_W, d_OH, d_OW, d_k, d_wv;
    // (behind what maxpool_forward_kernel reads)
    uint32_t quick0;       // so are those of the place in the whole map
    uint32_t lines;        // maxpool_backward_kernel: grad_in starts on a cache line
    double r_hv, r_OH;     // 1 / pieces of a plane, 1 / OH
    FastDiv d_hv;
};

// quotient by the multiplier where the host found it exact for all numerators of this launch, else by the division
__device__ __forceinline__ uint32_t quot(uint32_t n, uint32_t d, FastDiv f, uint32_t quick) { return quick ? fdiv(n, f) : n / d; }

// n / d for n below 2^41 (one per workgroup): the quotient by rcp = 1.0 / d is at most one off
__device__ __forceinline__ uint64_t quot64(uint64_t n, uint32_t d, double rcp, uint32_t* rest) {
    uint64_t q = (uint64_t)((double)n * rcp);
    int64_t r = (int64_t)(n - q * d);
    if (r < 0) { --q; r += d; }
    if (r >= (int64_t)d) { ++q; r -= d; }
    *rest = __builtin_amdgcn_readfirstlane((uint32_t)r);
    return ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(q >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)q);
}

// the same for a launch all of whose numerators n the multiplier takes (quick): scalar instructions; small launches are the latency of this
__device__ __forceinline__ uint64_t quot64(uint64_t n, uint32_t d, FastDiv f, uint32_t quick, double rcp, uint32_t* rest) {
    if (!quick) return quot64(n, d, rcp, rest);
    const uint32_t q = fdiv((uint32_t)n, f);
    *rest = (uint32_t)n - q * d;
    return q;
}

__global__ void __launch_bounds__(kThreads) zero_words(uint32_t* p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kThreads) p[i] = 0u;
}

template <typename T> __device__ __forceinline__ float as_float(T v);
template <> __device__ __forceinline__ float as_float<float>(float v) { return v; }
template <> __device__ __forceinline__ float as_float<uint16_t>(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

// Forward, any size: a workgroup takes `chunk` consecutive elements of the map wherever rows and planes end, i.e. whole
// mask words, and works on every window that has elements among them: the location bits (first maximum in row-major
// order wins) are set in an LDS image of those words, which then leave with plain stores, and the maxima of the windows
// that begin in the chunk are written.  The windows on a chunk's border are worked on by both neighbours, a few per cent
// of the work; in exchange no word is shared, the mask needs no clearing, and small planes fill a workgroup like large
// ones.  A workgroup per band of one plane, a cleared mask and atomics on the shared words took 98 us on
// 22 x 2914 x 14 x 14 (k = 3, bfloat16), 39 us on 74 x 292 x 33 x 33 (k = 2, bfloat16) and 30 us on 8 x 64 x 224 x 224 (k = 3), this 9,
// 15 and 19.5 (5.9 TB/s).
// What bounds it: the load instructions (one per window row for pairs, one per element otherwise).
// K: the window's extent where it is known (2, 3), else 0.  PAIR: k = 2, rows of whole aligned element pairs.
template <typename T, int K, bool PAIR>
__global__ void __launch_bounds__(kThreads) maxpool_forward_kernel(PoolArgs a) {
    extern __shared__ uint32_t words[];
    const uint32_t tid = threadIdx.x;
    const uint32_t k = K ? (uint32_t)K : a.k;
    const uint64_t e0 = (uint64_t)blockIdx.x * a.chunk;                       // first element, at a word boundary
    const uint32_t len = (uint32_t)min((uint64_t)a.chunk, a.n - e0);
    const uint32_t nwords = (len + 31u) >> 5;
    for (uint32_t w = tid; w < nwords; w += kThreads) words[w] = 0u;
    // window rows with elements in the chunk: from row oi0 of plane p0 (oi0 == OH: row 0 of the next plane) to row
    // oi1 of plane p1 (rows past a plane's last window belong to none)
    uint32_t at0, at1;
    const uint64_t p0 = quot64(e0, a.HW, a.r_HW, &at0), p1 = quot64(e0 + len - 1u, a.HW, a.r_HW, &at1);
    const uint32_t oi0 = min(at0 / a.W / k, a.OH), oi1 = min(at1 / a.W / k, a.OH - 1u);
    const uint64_t wr0 = p0 * a.OH + oi0, wr1 = p1 * a.OH + oi1;
    const uint32_t nwin = wr1 >= wr0 ? (uint32_t)(wr1 - wr0 + 1u) * a.OW : 0u;
    // base: the first window row's first element; the chunk begins `skip` elements behind it (negative: before it)
    const uint64_t base = p0 * a.HW + (oi0 < a.OH ? (uint64_t)oi0 * k * a.W : (uint64_t)a.HW);
    const int32_t skip = (int32_t)((int64_t)e0 - (int64_t)base);
    const T* xp = static_cast<const T*>(a.in) + base;
    T* yp = static_cast<T*>(a.out) + wr0 * a.OW;
    const uint32_t of0 = oi0 < a.OH ? oi0 : 0u;                              // row inside its plane of the first window row
    const uint32_t kW = k * a.W, gap = a.HW - a.OH * kW;                     // elements of a plane below its last window
    __syncthreads();
    for (uint32_t o = tid; o < nwin; o += kThreads) {
        const uint32_t r = quot(o, a.OW, a.d_OW, a.quick);
        const uint32_t oj = o - r * a.OW;
        const uint32_t g = quot(of0 + r, a.OH, a.d_OH, a.quick);             // planes behind the first
        const uint32_t first = r * kW + g * gap + oj * k;                    // the window's first element, from base on
        const T* xw = xp + first;
        uint32_t best = 0;                                                   // place of the maximum, from `first` on
        T bt;
        if constexpr (PAIR) {
            // rows of two adjacent elements each in one load
            struct alignas(2 * sizeof(T)) Pair { T a, b; };
            const Pair r0 = *reinterpret_cast<const Pair*>(xw);
            const Pair r1 = *reinterpret_cast<const Pair*>(xw + a.W);
            bt = r0.a;
            if (as_float<T>(r0.b) > as_float<T>(bt)) { bt = r0.b; best = 1; }
            if (as_float<T>(r1.a) > as_float<T>(bt)) { bt = r1.a; best = a.W; }
            if (as_float<T>(r1.b) > as_float<T>(bt)) { bt = r1.b; best = a.W + 1; }
        } else if constexpr (K > 0) {
            T t[K * K];
#pragma unroll
            for (int i = 0; i < K * K; ++i) t[i] = xw[(uint32_t)(i / K) * a.W + (uint32_t)(i % K)];
            bt = t[0];
#pragma unroll
            for (int i = 1; i < K * K; ++i)
                if (as_float<T>(t[i]) > as_float<T>(bt)) { bt = t[i]; best = (uint32_t)(i / K) * a.W + (uint32_t)(i % K); }
        } else {
            // a window row four elements at a time (those past its end re-read its last, which is not above itself): a load per element
            // behind the comparison of the one before is k * k latencies (12 M elements, fp32: 56 x 56, k = 4 25.7 -> 16.8 us, 64 x 64, k = 8 39.8 -> 26.0)
            bt = xw[0];
            for (uint32_t wr = 0; wr < k; ++wr)
                for (uint32_t wc = 0; wc < k; wc += 4) {
                    T t[4];
                    uint32_t at[4];
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j) {
                        at[j] = wr * a.W + min(wc + j, k - 1u);
                        t[j] = xw[at[j]];
                    }
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j)
                        if (as_float<T>(t[j]) > as_float<T>(bt)) { bt = t[j]; best = at[j]; }
                }
        }
        const uint32_t at = first - (uint32_t)skip;                          // from the chunk's start on; others wrap past len
        if (at < len) yp[o] = bt;
        const uint32_t bit = at + best;
        if (bit < len) atomicOr(&words[bit >> 5], 1u << (bit & 31u));
    }
    __syncthreads();
    uint32_t* mp = a.mask + (e0 >> 5);
    for (uint32_t w = tid; w < nwords; w += kThreads) mp[w] = words[w];
}

// Forward, k = 2 on rows of whole 8-element pieces (W % 8 == 0, an even number of rows, 16-byte aligned
// x): a thread takes four adjacent windows, i.e. eight consecutive elements of two rows (two 16-byte loads
// per row for 4-byte elements, one for 2-byte ones), writes their four maxima with one store and the eight
// location bits of each row as one byte of the LDS image of the band's mask slice: bytes have one owner, so
// there is no atomic.  With an even number of rows per plane the output rows of all planes are one run, so a
// band of them is whole mask words wherever planes end, and small planes share a workgroup (a band used to end
// with its plane: 12 x 22855 x 8 x 8 163 -> 14 us); the slice leaves with plain stores and the mask needs no clearing.
// 12 M elements of odd height, the general kernel above -> this: bfloat16 33 x 64 9.8 -> 7.1 us, 223 x 224 12.1 -> 7.4, fp32 223 x 224 14.7 -> 12.7.
// NT: non-temporal loads, for rows of at least a cache line (a stem's sequence of operators 306 us against 338 without: x does
// not displace what the neighbours write); shorter rows share lines between loads (8 x 8: 23 us with them, 14 without).
// ODD: an odd number of rows of whole mask words (W % 32 == 0): the slices of a band's rows follow each other except for the last row of
// each plane, whose zero words leave with the slice of the band that holds the row before it.
template <typename T, bool NT, bool ODD>
__global__ void __launch_bounds__(kThreads) maxpool2_forward_fast(PoolArgs a) {
    extern __shared__ uint32_t words[];
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const uint32_t tid = threadIdx.x;
    const uint64_t oi0 = (uint64_t)blockIdx.x * a.band;                      // output rows, counted over all planes
    const uint32_t nrows = (uint32_t)min((uint64_t)a.band, a.rows - oi0);
    // ODD: place of the first row in its plane, planes that end with a row of the band
    uint32_t of0 = 0, ends = 0;
    uint64_t start = 2u * oi0 * a.W;                                         // first element, at a word boundary
    if constexpr (ODD) {
        const uint64_t p0 = quot64(oi0, a.OH, a.d_OH, a.quick0, a.r_OH, &of0);
        start += p0 * a.W;
        ends = quot(of0 + nrows, a.OH, a.d_OH, a.quick);
    }
    const uint32_t nwords = (2u * nrows * a.W + ends * a.W + 31u) / 32u;
    for (uint32_t w = tid; w < nwords; w += kThreads) words[w] = 0u;
    __syncthreads();
    uint8_t* bytes = reinterpret_cast<uint8_t*>(words);
    auto load = [](const T* p) -> u32x4 {
        if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
        else return *reinterpret_cast<const u32x4*>(p);
    };
    const T* xp = static_cast<const T*>(a.in) + start;
    T* yp = static_cast<T*>(a.out) + oi0 * a.OW;
    const uint32_t ow4 = a.OW / 4u;
    const uint32_t n4 = nrows * ow4;
    for (uint32_t o4 = tid; o4 < n4; o4 += kThreads) {
        const uint32_t r = quot(o4, ow4, a.d_wv, a.quick);
        const uint32_t oj4 = o4 - r * ow4;
        uint32_t base = 2u * r * a.W + oj4 * 8u;                           // first of the eight elements, upper row
        if constexpr (ODD) base += quot(of0 + r, a.OH, a.d_OH, a.quick) * a.W;
        uint32_t e0[8], e1[8];                                              // the two rows as fp32 bit patterns
        if constexpr (sizeof(T) == 4) {
            const u32x4 a0 = load(xp + base);
            const u32x4 a1 = load(xp + base + 4);
            const u32x4 b0 = load(xp + base + a.W);
            const u32x4 b1 = load(xp + base + a.W + 4);
            e0[0] = a0.x; e0[1] = a0.y; e0[2] = a0.z; e0[3] = a0.w; e0[4] = a1.x; e0[5] = a1.y; e0[6] = a1.z; e0[7] = a1.w;
            e1[0] = b0.x; e1[1] = b0.y; e1[2] = b0.z; e1[3] = b0.w; e1[4] = b1.x; e1[5] = b1.y; e1[6] = b1.z; e1[7] = b1.w;
        } else {
            const u32x4 a0 = load(xp + base);
            const u32x4 b0 = load(xp + base + a.W);
            const uint32_t wa[4] = {a0.x, a0.y, a0.z, a0.w}, wb[4] = {b0.x, b0.y, b0.z, b0.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                e0[2 * j] = wa[j] << 16; e0[2 * j + 1] = wa[j] & 0xffff0000u;
                e1[2 * j] = wb[j] << 16; e1[2 * j + 1] = wb[j] & 0xffff0000u;
            }
        }
        uint32_t m[4], byte0 = 0, byte1 = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // first maximum in row-major order: a later element wins only if it compares greater
            uint32_t best = e0[2 * j], loc = 0;
            if (__uint_as_float(e0[2 * j + 1]) > __uint_as_float(best)) { best = e0[2 * j + 1]; loc = 1; }
            if (__uint_as_float(e1[2 * j]) > __uint_as_float(best)) { best = e1[2 * j]; loc = 2; }
            if (__uint_as_float(e1[2 * j + 1]) > __uint_as_float(best)) { best = e1[2 * j + 1]; loc = 3; }
            m[j] = best;
            byte0 |= (loc < 2 ? 1u << loc : 0u) << (2 * j);
            byte1 |= (loc >= 2 ? 1u << (loc - 2) : 0u) << (2 * j);
        }
        if constexpr (sizeof(T) == 4) {
            __builtin_nontemporal_store(u32x4{m[0], m[1], m[2], m[3]}, reinterpret_cast<u32x4*>(yp + (size_t)o4 * 4u));
        } else {
            __builtin_nontemporal_store(u32x2{(m[0] >> 16) | (m[1] & 0xffff0000u), (m[2] >> 16) | (m[3] & 0xffff0000u)},
                                        reinterpret_cast<u32x2*>(yp + (size_t)o4 * 4u));
        }
        const uint32_t b0i = base >> 3;                                     // byte of the slice that holds the upper row's eight bits
        bytes[b0i] = (uint8_t)byte0;
        bytes[b0i + (a.W >> 3)] = (uint8_t)byte1;
    }
    __syncthreads();
    uint32_t* mp = a.mask + (start >> 5);
    for (uint32_t w = tid; w < nwords; w += kThreads) mp[w] = words[w];
}

// Backward, element by element: grad_in = V (.) (1_{k x k} (x) grad_out).  For 2-byte maps that start in the middle of a dword
// or are small, and planes of 2^28 output gradients and more; the others take the two kernels below.
template <typename T>
__global__ void __launch_bounds__(kThreads) maxpool_backward_scalar(PoolArgs a) {
    const uint32_t p = blockIdx.y;
    const T* gp = static_cast<const T*>(a.in) + (size_t)p * a.OH * a.OW;
    T* op = static_cast<T*>(a.out) + (size_t)p * a.HW;
    const uint64_t bit0 = (uint64_t)p * a.HW;
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < a.HW; i += gridDim.x * kThreads) {
        const uint64_t bit = bit0 + i;
        const uint32_t set = (a.mask[bit >> 5] >> (uint32_t)(bit & 31u)) & 1u;
        const uint32_t r = i / a.W;
        const uint32_t c = i - r * a.W;
        const uint32_t oi = r / a.k, oj = c / a.k;
        op[i] = set && oi < a.OH && oj < a.OW ? gp[oi * a.OW + oj] : (T)0;
    }
}

// Backward, any size on a dword boundary: a wavefront rebuilds 64 K consecutive 16-byte vectors of grad_in (4 KB at K = 4) wherever
// rows and planes end (the write stream of decompress_stream).  A vector's mask bits lie in one word; an element's place is
// found from its vector's by counting on; the gradients of the elements whose bit is set come through a bounds-checked
// buffer, the others' loads are out of its range, read as +0 and fetch nothing.  A workgroup per 512 elements of one plane and a
// branch per element took 60 us on 74 x 292 x 33 x 33
// (bfloat16) and 30 us on 2 x 716 x 42 x 207, this 22 and 12.5.  What bounds it: vector instructions (the steps from element to element).
template <typename T, int K>
__global__ void __launch_bounds__(64) maxpool_backward_kernel(PoolArgs a) {
    constexpr int EPV = Tr<T>::EPV;
    constexpr uint32_t kDrop = 0x80000000u;
    const uint32_t lane = threadIdx.x;
    const uint64_t e0 = (uint64_t)blockIdx.x * (64u * K * EPV);
    uint32_t at0;
    const uint64_t p0 = quot64(e0, a.HW, a.d_HW, a.quick0, a.r_HW, &at0);
    const uint32_t OHW = a.OH * a.OW;
    const T* gp = static_cast<const T*>(a.in) + p0 * OHW;
    // gradients of plane p0 and those behind it that the chunk can reach
    const uint64_t gbytes = min(((uint64_t)a.P - p0) * OHW * sizeof(T), (uint64_t)0x7ffffff0u);
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(gp), 0, (int)gbytes, 0x00020000);
    const uint64_t left = a.n - e0;
    const uint64_t nwords = (a.n + 31u) >> 5;
    uint32_t v[K][EPV];
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const uint32_t ev = EPV * (64u * u + lane);                          // the vector's first element, from e0 on
        const uint64_t w = (e0 + ev) >> 5;
        const uint32_t bits = (w < nwords ? a.mask[w] : 0u) >> ((uint32_t)(e0 + ev) & 31u);
        const uint32_t t = at0 + ev;
        // (planes of more elements than a chunk: the vector lies in the first or the second one)
        uint32_t g = a.HW >= 64u * K * EPV ? (t >= a.HW ? 1u : 0u) : quot(t, a.HW, a.d_HW, a.quick);
        const uint32_t i = t - g * a.HW;
        uint32_t r = quot(i, a.W, a.d_W, a.quick);
        uint32_t c = i - r * a.W;
        uint32_t oi = quot(r, a.k, a.d_k, a.quick), oj = quot(c, a.k, a.d_k, a.quick);
        uint32_t cr = c - oj * a.k, rr = r - oi * a.k;                       // place inside the window
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const bool set = ((bits >> e) & 1u) && oi < a.OH && oj < a.OW;
            const uint32_t off = set ? (g * OHW + oi * a.OW + oj) * (uint32_t)sizeof(T) : kDrop;
            if constexpr (sizeof(T) == 4) v[u][e] = __builtin_amdgcn_raw_buffer_load_b32(grs, off, 0, 0);
            else v[u][e] = __builtin_amdgcn_raw_buffer_load_b16(grs, off, 0, 0);
            // the next element: one column, and where they end one row, one plane on
            ++c; ++cr;
            const bool nw = cr == a.k;
            oj += nw ? 1u : 0u; cr = nw ? 0u : cr;
            const bool nr = c == a.W;
            c = nr ? 0u : c; oj = nr ? 0u : oj; cr = nr ? 0u : cr;
            r += nr ? 1u : 0u; rr += nr ? 1u : 0u;
            const bool nv = rr == a.k;
            oi += nv ? 1u : 0u; rr = nv ? 0u : rr;
            const bool np = r == a.H;
            r = np ? 0u : r; oi = np ? 0u : oi; rr = np ? 0u : rr;
            g += np ? 1u : 0u;
        }
    }
    T* out = static_cast<T*>(a.out) + e0;
    const uint32_t obytes = left < 64u * K * EPV ? ((uint32_t)left * (uint32_t)sizeof(T)) & ~3u : 64u * K * 16u;
    const __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)obytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < K; ++u) {
        u32x4 o;
        if constexpr (sizeof(T) == 4) o = u32x4{v[u][0], v[u][1], v[u][2], v[u][3]};
        else o = u32x4{v[u][0] | (v[u][1] << 16), v[u][2] | (v[u][3] << 16), v[u][EPV - 4] | (v[u][EPV - 3] << 16), v[u][EPV - 2] | (v[u][EPV - 1] << 16)};
        // stores past the map are dropped by the bound, dword by dword; the whole offset in the vector operand (the
        // compiler counts the wait states behind a wide store only without a scalar offset register)
        // (not non-temporal where they cut cache lines, whose halves would then leave one by one: fp32 maps of 0.5 M elements 8 bytes past
        // a line 3.4 against 3.1 us)
        if (a.lines) __builtin_amdgcn_raw_buffer_store_b128(o, ors, (64u * u + lane) * 16u, 0, 2);
        else __builtin_amdgcn_raw_buffer_store_b128(o, ors, (64u * u + lane) * 16u, 0, 0);
    }
    // a map of an odd number of 2-byte elements ends in the middle of a dword, which lies behind the bound
    if constexpr (sizeof(T) == 2) {
        if ((left & 1u) && left < 64u * K * EPV) {
#pragma unroll
            for (int u = 0; u < K; ++u)
#pragma unroll
                for (int e = 0; e < EPV; e += 2)
                    if (EPV * (64u * u + lane) + (uint32_t)e + 1u == (uint32_t)left) out[left - 1u] = (T)v[u][e];
        }
    }
}

// Backward, k = 2 on rows of whole pieces of PE elements (grad_in aligned to a piece, grad_out to its PE / 2 gradients): a thread
// rebuilds one piece, which lies under PE / 2 adjacent windows: one mask word, one load of their gradients, one non-temporal
// store; a workgroup of four wavefronts writes 4 KB (2 KB) and ends (what a write stream wants here).  The rows of all planes are
// one run, so planes end anywhere in a workgroup (one that ended with its plane: 12 x 22855 x 8 x 8 130 -> 12 us); the last row of a
// plane of odd height (ODD) has no bits set, so any window row's gradients will do for its address.
// PE: whole 16-byte vectors where the rows allow it; four 2-byte elements (widths such as 28 or 100, half the bytes per store)
// otherwise.  Maps of 12 M elements, the general kernel above -> this: bfloat16 28 x 28 13.0 -> 6.6 us, 100 x 100 12.5 -> 6.6, 111 x 100
// 12.6 -> 7.0, 223 x 224 13.2 -> 6.5; fp32 111 x 112 12.8 -> 11.1.
template <typename T, int PE> constexpr int kPieces = PE * sizeof(T) == 8 ? 2 : 1;      // a thread's, kThreads apart: 4 KB per workgroup
template <typename T, int PE, bool ODD>
__global__ void __launch_bounds__(kThreads) maxpool2_backward_fast(PoolArgs a) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr int U = kPieces<T, PE>;
    const uint32_t wv = a.W / (uint32_t)PE, hv = a.HW / (uint32_t)PE;       // pieces of a row, of a plane
    const uint64_t v0 = (uint64_t)blockIdx.x * (kThreads * U);
    uint32_t at0;                                                           // place of the block's first piece in its plane (ODD) or row
    const uint64_t first = ODD ? quot64(v0, hv, a.d_hv, a.quick0, a.r_hv, &at0) : quot64(v0, wv, a.d_wv, a.quick0, a.r_wv, &at0);
    uint32_t bits[U];
    u32x2 q[U];                                                             // the gradients (of a piece of 8 bytes: in x)
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t bit = (v0 + kThreads * u + threadIdx.x) * PE;
        if (bit >= a.n) break;
        const uint32_t t = at0 + kThreads * u + threadIdx.x;
        uint32_t c;
        uint64_t wr;                                                        // window row, counted over all planes
        if constexpr (ODD) {
            // planes behind the block's first
            const uint32_t g = hv >= (uint32_t)(kThreads * U) ? (t >= hv ? 1u : 0u) : fdiv(t, a.d_hv);
            const uint32_t i = t - g * hv, r = quot(i, wv, a.d_wv, a.quick);
            c = i - r * wv;
            wr = (first + g) * a.OH + min(r >> 1, a.OH - 1u);
        } else {
            const uint32_t dr = quot(t, wv, a.d_wv, a.quick);
            c = t - dr * wv;
            wr = (first + dr) >> 1;
        }
        bits[u] = a.mask[bit >> 5] >> (uint32_t)(bit & 31u);
        const T* g = static_cast<const T*>(a.in) + wr * a.OW + c * (PE / 2u);
        if constexpr (U == 2) q[u].x = *reinterpret_cast<const uint32_t*>(g);
        else q[u] = *reinterpret_cast<const u32x2*>(g);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t bit = (v0 + kThreads * u + threadIdx.x) * PE;
        if (bit >= a.n) break;
        T* out = static_cast<T*>(a.out) + bit;
        const uint32_t m = bits[u], x = q[u].x, y = q[u].y;
        // two 2-byte elements under window j of the piece
        auto pair = [&](uint32_t w, int j) -> uint32_t { return (m & (1u << (2 * j)) ? w : 0u) | (m & (2u << (2 * j)) ? w << 16 : 0u); };
        if constexpr (sizeof(T) == 4)
            __builtin_nontemporal_store(u32x4{m & 1u ? x : 0u, m & 2u ? x : 0u, m & 4u ? y : 0u, m & 8u ? y : 0u}, reinterpret_cast<u32x4*>(out));
        else if constexpr (PE == 8)
            __builtin_nontemporal_store(u32x4{pair(x & 0xffffu, 0), pair(x >> 16, 1), pair(y & 0xffffu, 2), pair(y >> 16, 3)}, reinterpret_cast<u32x4*>(out));
        else
            __builtin_nontemporal_store(u32x2{pair(x & 0xffffu, 0), pair(x >> 16, 1)}, reinterpret_cast<u32x2*>(out));
    }
}

int pool_args(bool forward, const void* in, void* out, const void* mask, int64_t N, int64_t C, int64_t H, int64_t W,
              division_dtype dt, int k, size_t mask_bytes, PoolArgs* a) {
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || k < 1 || (dt != DIVISION_F32 && dt != DIVISION_BF16)) return DIVISION_EINVAL;
    // the pooled-size buffer (y / grad_out) may be null when there is no whole window
    const bool no_window = H / k == 0 || W / k == 0;
    if (!mask || (!in && !(no_window && !forward)) || (!out && !(no_window && forward))) return DIVISION_EINVAL;
    const uint64_t P = (uint64_t)N * (uint64_t)C, HW = (uint64_t)H * (uint64_t)W;
    if (N > 0x7fffffff || C > 0x7fffffff || H > 0x7fffffff || W > 0x7fffffff || P > 0x7fffffffull || HW > 0x7fffffffull ||
        P * HW > (1ull << 40) || k > 0x7fff)
        return DIVISION_ERANGE;
    if (mask_bytes < division_mask_bytes((int64_t)(P * HW))) return DIVISION_ESIZE;
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    if (((uintptr_t)in % es) != 0 || ((uintptr_t)out % es) != 0 || ((uintptr_t)mask % 4) != 0) return DIVISION_EALIGN;
    a->in = in; a->out = out; a->mask = static_cast<uint32_t*>(const_cast<void*>(mask));
    a->P = (uint32_t)P; a->H = (uint32_t)H; a->W = (uint32_t)W; a->HW = (uint32_t)HW;
    a->OH = (uint32_t)(H / k); a->OW = (uint32_t)(W / k); a->k = (uint32_t)k;
    a->n = P * HW;
    a->r_HW = 1.0 / (double)HW;
    return DIVISION_OK;
}

}  // namespace

extern "C" {

size_t division_mask_bytes(int64_t n) { return n < 0 ? 0 : (size_t)((n + 31) / 32) * 4u; }

int division_relu_forward(const void* x, int64_t n, division_dtype dt, void* y, void* mask, size_t mask_capacity,
                          void* hip_stream) {
    return launch(0, x, n, dt, y, mask, mask_capacity, 0.0f, 0, hip_stream);
}

int division_dropout_forward(const void* x, int64_t n, division_dtype dt, float p, uint64_t seed, void* y, void* mask,
                             size_t mask_capacity, void* hip_stream) {
    return launch(1, x, n, dt, y, mask, mask_capacity, p, seed, hip_stream);
}

int division_mask_backward(const void* mask, size_t mask_bytes, const void* grad_out, int64_t n, division_dtype dt,
                           void* grad_in, void* hip_stream) {
    return launch(2, grad_out, n, dt, grad_in, const_cast<void*>(mask), mask_bytes, 0.0f, 0, hip_stream);
}

int division_maxpool_forward(const void* x, int64_t N, int64_t C, int64_t H, int64_t W, division_dtype dt, int k,
                             void* y, void* mask, size_t mask_capacity, void* hip_stream) {
    PoolArgs a{};
    const int rc = pool_args(true, x, y, mask, N, C, H, W, dt, k, mask_capacity, &a);
    if (rc != DIVISION_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    // rows of whole 8-element pieces, an even number of them per plane or each of whole mask words: the output rows of all planes are one run
    // (not large fp32 maps of odd height and rows of up to 512 bytes, of which the general kernel has 12 M elements of 33 x 64 in 11.5 us, this
    // one in 12.2; 33 x 160 12.4 and 12.2; 1 M elements of 33 x 64 3.8 and 3.3)
    const bool odd = a.H % 2 != 0, pairs = odd && dt == DIVISION_F32 && a.W <= 128 && a.n > (4u << 20);
    if (k == 2 && a.OH > 0 && !pairs && a.W % (odd ? 32 : 8) == 0 && a.W <= 16384 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)y % (4 * es)) == 0) {
        // about 8 KB of x per workgroup (short-lived workgroups, many of them), an even number of output rows (whole mask
        // words), at most 64 Ki mask bits
        uint32_t band = (uint32_t)(8192 / (2ull * a.W * es)) & ~1u;
        if (band < 2) band = 2;
        a.band = band;
        a.rows = (uint64_t)a.P * a.OH;
        const uint64_t grid = (a.rows + band - 1) / band;
        a.d_wv = make_fastdiv(a.OW / 4);
        a.d_OH = make_fastdiv(a.OH);
        a.r_OH = 1.0 / (double)a.OH;
        a.quick = fastdiv_ok((uint64_t)band * (a.OW / 4), a.OW / 4) && (!odd || fastdiv_ok((uint64_t)a.OH + band, a.OH));
        a.quick0 = fastdiv_ok(a.rows, a.OH);
        if (launch_ok(grid, kThreads)) {
            // rows shorter than a cache line: several loads touch each line, which then has to stay in the caches
            const bool nt = a.W * es >= 128;
            void (*kern)(PoolArgs);
            if (dt == DIVISION_F32) kern = odd ? (nt ? maxpool2_forward_fast<float, true, true> : maxpool2_forward_fast<float, false, true>)
                                               : (nt ? maxpool2_forward_fast<float, true, false> : maxpool2_forward_fast<float, false, false>);
            else kern = odd ? (nt ? maxpool2_forward_fast<uint16_t, true, true> : maxpool2_forward_fast<uint16_t, false, true>)
                            : (nt ? maxpool2_forward_fast<uint16_t, true, false> : maxpool2_forward_fast<uint16_t, false, false>);
            // the band's rows and, of an odd height, the last rows of the planes that end in it
            const size_t bits = (size_t)band * 2 * a.W + (odd ? ((size_t)band / a.OH + 1) * a.W : 0);
            hipLaunchKernelGGL(kern, dim3((uint32_t)grid), dim3(kThreads), bits / 8 + 16, st, a);
            return hipGetLastError() == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
        }
    }
    if (a.OH == 0 || a.OW == 0) {                            // no whole window: empty output, all-zero mask
        const uint64_t nwords = (a.n + 31) / 32;
        const uint32_t zgrid = (uint32_t)((nwords + kThreads * 8ull - 1) / (kThreads * 8ull));
        hipLaunchKernelGGL(zero_words, dim3(zgrid < 1 ? 1 : zgrid), dim3(kThreads), 0, st, a.mask, nwords);
        return hipGetLastError() == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
    }
    // A chunk has at least four window rows (at most a quarter of the windows are then worked on twice) and 1024
    // elements (a workgroup's fixed work), at most 64 Ki window-row bits; beyond that the longer the better for the borders' sake, as
    // long as there are eight workgroups per CU: 8192 elements (1 KB of mask words)
    const uint64_t row_bits = (uint64_t)a.k * a.W;
    if (row_bits > 65536) return DIVISION_ERANGE;
    uint64_t chunk = 8192;
    while (chunk > 1024 && a.n / chunk < 2048) chunk /= 2;
    while (chunk < 4 * row_bits) chunk *= 2;
    while (!launch_ok((a.n + chunk - 1) / chunk, kThreads)) chunk *= 2;       // maps of 2^37 elements and more: up to 2^40 in 2^24 workgroups
    a.chunk = (uint32_t)chunk;
    const uint64_t wrows = chunk / a.W + 2 + 2 * (chunk / a.HW + 2);          // at least the window rows of a chunk
    a.d_OW = make_fastdiv(a.OW);
    a.d_OH = make_fastdiv(a.OH);
    a.quick = fastdiv_ok(wrows * a.OW + kThreads, a.OW) && fastdiv_ok(a.OH + wrows, a.OH);
    const bool pair = k == 2 && a.W % 2 == 0 && ((uintptr_t)x % (2 * es)) == 0;
    void (*kern)(PoolArgs);
    if (dt == DIVISION_F32) kern = pair ? maxpool_forward_kernel<float, 2, true> : k == 2 ? maxpool_forward_kernel<float, 2, false>
                                 : k == 3 ? maxpool_forward_kernel<float, 3, false> : maxpool_forward_kernel<float, 0, false>;
    else kern = pair ? maxpool_forward_kernel<uint16_t, 2, true> : k == 2 ? maxpool_forward_kernel<uint16_t, 2, false>
              : k == 3 ? maxpool_forward_kernel<uint16_t, 3, false> : maxpool_forward_kernel<uint16_t, 0, false>;
    hipLaunchKernelGGL(kern, dim3((uint32_t)((a.n + chunk - 1) / chunk)), dim3(kThreads), (size_t)chunk / 8, st, a);
    return hipGetLastError() == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
}

int division_maxpool_backward(const void* mask, size_t mask_bytes, const void* grad_out, int64_t N, int64_t C,
                              int64_t H, int64_t W, division_dtype dt, int k, void* grad_in, void* hip_stream) {
    PoolArgs a{};
    const int rc = pool_args(false, grad_out, grad_in, mask, N, C, H, W, dt, k, mask_bytes, &a);
    if (rc != DIVISION_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const size_t es = dt == DIVISION_BF16 ? 2 : 4;
    const uint64_t epv = 16 / es;
    // rows of whole pieces: 16 bytes, or four 2-byte elements
    const uint64_t pe = a.W % epv == 0 && ((uintptr_t)grad_in % 16) == 0 ? epv : 4;
    const uint64_t per_block = kThreads * (pe * es == 8 ? 2 : 1), nblock = (a.n / pe + per_block - 1) / per_block;      // as kPieces
    if (k == 2 && a.OH > 0 && a.W % pe == 0 && ((uintptr_t)grad_in % (pe * es)) == 0 && ((uintptr_t)grad_out % (pe / 2 * es)) == 0 &&
        launch_ok(nblock, kThreads)) {
        const uint64_t wv = a.W / pe;
        const bool odd = a.H % 2 != 0;
        a.d_wv = make_fastdiv((uint32_t)wv);
        a.r_wv = 1.0 / (double)wv;
        a.d_hv = make_fastdiv((uint32_t)(a.HW / pe));
        a.r_hv = 1.0 / (double)(a.HW / pe);
        a.quick = odd ? fastdiv_ok(a.HW / pe, wv) : fastdiv_ok(wv + per_block, wv);
        a.quick0 = fastdiv_ok(a.n / pe + per_block, odd ? a.HW / pe : wv);
        void (*fast)(PoolArgs) = dt == DIVISION_F32 ? (odd ? maxpool2_backward_fast<float, 4, true> : maxpool2_backward_fast<float, 4, false>)
                               : pe == 8 ? (odd ? maxpool2_backward_fast<uint16_t, 8, true> : maxpool2_backward_fast<uint16_t, 8, false>)
                                         : (odd ? maxpool2_backward_fast<uint16_t, 4, true> : maxpool2_backward_fast<uint16_t, 4, false>);
        hipLaunchKernelGGL(fast, dim3((uint32_t)nblock), dim3(kThreads), 0, st, a);
        return hipGetLastError() == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
    }
    const uint64_t nvec = (a.n + epv - 1) / epv;
    // Vectors a lane: one where the launch is short, whose time is the chain of a wavefront's elements (maps of 1 M elements fp32 4.4 -> 3.9 us,
    // bfloat16 5.6 -> 3.6), four beyond (16 M: fp32 18.0 -> 14.0; bfloat16 level at 20 M).  2-byte maps of a few planes and chunks have
    // half the chain again with an element a lane (32 K: 2.8 -> 2.5; level at 256 K).
    const bool f32 = dt == DIVISION_F32;
    const uint64_t vecs = a.n <= ((f32 ? 4u : 12u) << 20) ? 1 : 4;
    const bool few = !f32 && a.n <= (1u << 17) && a.P <= 1024;
    const uint64_t per_wave = 64 * vecs, grid = (nvec + per_wave - 1) / per_wave, chunk = per_wave * epv;
    const uint64_t reach = chunk / a.HW + 2;                                  // planes a chunk can reach
    if (!few && ((uintptr_t)grad_in % 4) == 0 && launch_ok(grid, 64) && reach * a.OH * a.OW * es < (1ull << 31) && (uint64_t)a.HW + chunk < (1ull << 32)) {
        a.quick0 = fastdiv_ok(a.n, a.HW);
        a.lines = ((uintptr_t)grad_in % 128) == 0;
        a.d_HW = make_fastdiv(a.HW);
        a.d_W = make_fastdiv(a.W);
        a.d_k = make_fastdiv(a.k);
        a.quick = (a.HW >= chunk || fastdiv_ok(a.HW + chunk, a.HW)) && fastdiv_ok(a.HW, a.W) && fastdiv_ok(a.H, a.k) && fastdiv_ok(a.W, a.k);
        void (*kern)(PoolArgs) = f32 ? (vecs == 4 ? maxpool_backward_kernel<float, 4> : maxpool_backward_kernel<float, 1>)
                                     : (vecs == 4 ? maxpool_backward_kernel<uint16_t, 4> : maxpool_backward_kernel<uint16_t, 1>);
        hipLaunchKernelGGL(kern, dim3((uint32_t)grid), dim3(64), 0, st, a);
        return hipGetLastError() == hipSuccess ? DIVISION_OK : DIVISION_EHIP;
    }
    void (*kern)(PoolArgs) = dt == DIVISION_F32 ? maxpool_backward_scalar<float> : maxpool_backward_scalar<uint16_t>;
    uint32_t gx = (a.HW + kThreads * 2u - 1) / (kThreads * 2u);
    if (gx < 1) gx = 1;
    if (gx > 4096) gx = 4096;
    // grid.y takes a slice of planes per launch; a multiple of 32 planes, so that every slice's
    // first mask bit starts a word
    constexpr uint32_t kSlice = 65504;
    for (uint32_t p0 = 0; p0 < a.P; p0 += kSlice) {
        PoolArgs b = a;
        const uint32_t np = a.P - p0 < kSlice ? a.P - p0 : kSlice;
        b.in = static_cast<const char*>(a.in) + (size_t)p0 * a.OH * a.OW * es;
        b.out = static_cast<char*>(a.out) + (size_t)p0 * a.HW * es;
        b.mask = a.mask + ((uint64_t)p0 * a.HW) / 32;
        hipLaunchKernelGGL(kern, dim3(gx, np), dim3(kThreads), 0, st, b);
        if (hipGetLastError() != hipSuccess) return DIVISION_EHIP;
    }
    return DIVISION_OK;
}

}  // extern "C"
