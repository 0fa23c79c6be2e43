// Included inside the unnamed namespaces of division.hip (through helpers.h) and masks.hip: quotients by run-time divisors.

// Quotient by a runtime divisor d through one multiply-high with m = floor(2^32 / d) + 1: exact while numerator * d < 2^32 (the
// host checks it with fastdiv_ok).  The divisor 1 has no 32-bit multiplier: its m is 0 and `one` is all ones, so that the quotient
// needs no test (a test on m, uniform as it is, became a scalar branch per division: 13 in decompress_stream, 228
// in compress_units, each ending a basic block in the middle of the loads; without them decompress_stream runs
// 1.5-2.5 % faster).
struct FastDiv { uint32_t one, m; };
__device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv f) { return __umulhi(n, f.m) | (n & f.one); }
static FastDiv make_fastdiv(uint32_t d) {
    FastDiv f; f.one = d <= 1 ? 0xffffffffu : 0u; f.m = d <= 1 ? 0u : (uint32_t)((1ull << 32) / d) + 1u; return f;
}
// whether fdiv is exact for every numerator up to n_max
inline bool fastdiv_ok(uint64_t n_max, uint64_t d) { return n_max * d < (1ull << 32); }

// A launch may have at most 2^32 - 1 threads along x
inline bool launch_ok(uint64_t workgroups, uint64_t threads) { return workgroups * threads < (1ull << 32); }
