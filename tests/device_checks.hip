// Device helpers of the codec run on their own for tests/test_gpu_device_helpers.py (a library of its own: nothing of it is
// in libdivision.so).
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <type_traits>

namespace {
constexpr uint32_t kWeyl = 0x9E3779B9u;
#include "../paper_2208_04187_amd/csrc/helpers.h"
#include "../paper_2208_04187_amd/csrc/block_mean.h"

__global__ void count_reciprocals(uint32_t first, uint32_t n, uint32_t cols, double* out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double r = count_rcp(first + i);
    out[i] = cols ? count_rcp_times(r, cols) : r;
}

// every binary32 pattern: workgroup w takes the 65536 patterns with the high half w
__global__ void bf16_conversions(unsigned long long* mismatches) {
    uint32_t bad = 0;
    for (uint32_t lo = threadIdx.x; lo < 65536u; lo += blockDim.x) {
        const uint32_t u = (blockIdx.x << 16) | lo;
        const uint32_t want = (u & 0x7fffffffu) > 0x7f800000u ? (u >> 16) | 0x40u : (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
        const float f = __uint_as_float(u);
        bad += float_to_bf16_bits(f) != want || bf16_pack2(f, 0.0f) != want || bf16_pack2(0.0f, f) != want << 16;
    }
    if (bad) atomicAdd(mismatches, (unsigned long long)bad);
}
}  // namespace

extern "C" {
// out[i] = the kernels' reciprocal of first + i (cols = 0), or of (first + i) * cols as a product; out holds n doubles
int check_count_reciprocals(uint32_t first, uint32_t n, uint32_t cols, double* out, void* stream) {
    if (n == 0 || !out || (uint64_t)first + n > (1ull << 32) || first == 0) return 1;
    hipLaunchKernelGGL(count_reciprocals, dim3((n + 255u) / 256u), dim3(256), 0, static_cast<hipStream_t>(stream), first, n, cols, out);
    return hipGetLastError() == hipSuccess ? 0 : 5;
}

// *mismatches += the binary32 patterns whose bfloat16 is not the integer rule's
int check_bf16_conversions(unsigned long long* mismatches, void* stream) {
    if (!mismatches) return 1;
    hipLaunchKernelGGL(bf16_conversions, dim3(65536), dim3(256), 0, static_cast<hipStream_t>(stream), mismatches);
    return hipGetLastError() == hipSuccess ? 0 : 5;
}
}
