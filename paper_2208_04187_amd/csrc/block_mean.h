// Part of division.hip (included inside its unnamed namespace, after helpers.h): the mean of a block from its sum.

// (float)(S / cnt) for a positive integer cnt, the way the reference definition rounds it
// (binary64 quotient, then one rounding to binary32), without a binary64 division in the common
// case.  q = fl(S * fl(1/cnt)) carries two roundings of relative size 2^-53 each, so it lies within
// 2^-52 |S/cnt| <= 2 ulp of the exact quotient, i.e. within 3 ulp of the binary64 quotient
// d = fl(S/cnt) (half an ulp from the exact one, plus q's own grid).  q and d round to the same
// binary32 unless a rounding boundary of binary32 lies between them.  For a normal binary32 result
// those boundaries are the binary64 numbers whose low 29 bits read 1000...0 (and, for d itself to
// land on the other side, nothing closer than that): if the low 29 bits of q are at least 16 ulp
// from that pattern, no boundary is within 16 ulp of q, d is within 3, so both round alike.
// (The kernels' reciprocals may be up to 4 ulp off 1/cnt, see count_rcp: that is at most 8 ulp of q, so q and d are then
// within 10 ulp, still inside the 16.)
// A nonzero q below 2^-126 rounds to a subnormal binary32, which drops more than 29 bits, so the
// pattern test does not see its boundaries: it takes the division.  (q >= 2^-126 > d cannot
// disagree: d is then within 3 ulp below 2^-126, q's low bits are near zero, both round to 2^-126.)
// S is a sum of binary32 values, at least 2^-149 in magnitude when nonzero, so neither q nor d is
// a subnormal binary64; cnt < 2^32 is exact in binary64.  mean_rule_divides says whether q may
// stand in for d; it is host code too, so that a test can run the rule without a GPU.
__host__ __device__ __forceinline__ bool mean_rule_divides(double q) {
    uint64_t bits;
    __builtin_memcpy(&bits, &q, sizeof bits);
    const uint32_t low = (uint32_t)bits & 0x1fffffffu;
    const uint32_t dist = low > 0x10000000u ? low - 0x10000000u : 0x10000000u - low;
    const bool subnormal = q != 0.0 && __builtin_fabs(q) < 0x1p-126;
    return dist < 16u || subnormal;
}
__host__ __device__ __forceinline__ bool mean_count_is_power_of_two(uint32_t cnt) { return (cnt & (cnt - 1)) == 0; }

// The rule on the device: when any lane of the wavefront needs the division, all take it.
// rcp is 1 / cnt to within 4 ulp, exact for a power of two (a kernel that needs the mean of many blocks of one
// size takes it once and passes it in).
__device__ __forceinline__ float mean_with_rcp(double S, uint32_t cnt, double rcp) {
    if (mean_count_is_power_of_two(cnt)) return (float)(S * rcp);     // exact scaling
    const double q = S * rcp;
    if (__builtin_expect(__any(mean_rule_divides(q)), 0)) return (float)(S / (double)cnt);
    return (float)q;
}
// 1 / cnt without the division's scaling and fix-up steps (half its instructions): the hardware's estimate and two Newton
// steps, at most 2 ulp off (cnt < 2^32 and its reciprocal are far from the ends of binary64; an estimate with an error of e
// leaves e^4, so 2^-20 would do), exact for a power of two.  Then q = fl(S * rcp) lies within 5 ulp of the exact quotient
// and 6 of d, still well inside the rule's 16.
__host__ __device__ __forceinline__ double count_rcp_from(uint32_t cnt, double estimate) {
    const double c = (double)cnt;
    double r = estimate;
    r = __builtin_fma(__builtin_fma(-c, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-c, r, 1.0), r, r);
}
__device__ __forceinline__ double count_rcp(uint32_t cnt) { return count_rcp_from(cnt, __builtin_amdgcn_rcp((double)cnt)); }
// 1 / (rows * cols) from the lane's 1 / rows, cols a constant: a product of two reciprocals, at most 4 ulp off, exact for powers of two
__device__ __forceinline__ double count_rcp_times(double rcp_rows, uint32_t cols) { return rcp_rows * (1.0 / (double)cols); }
__device__ __forceinline__ float mean_of(double S, uint32_t cnt) { return mean_with_rcp(S, cnt, count_rcp(cnt)); }

// The rule for one value on the host (what a lane whose neighbours do not ask for the division computes).
inline float mean_of_host(double S, uint32_t cnt, double rcp, int* divided) {
    *divided = 0;
    if (mean_count_is_power_of_two(cnt)) return (float)(S * rcp);
    const double q = S * rcp;
    if (mean_rule_divides(q)) { *divided = 1; return (float)(S / (double)cnt); }
    return (float)q;
}
