// The mask operators with the launches recorded instead of made, for tests/test_launch_plans.py (a library of its own; needs no
// device): the host side of masks.hip, its launches written down.
#include <hip/hip_runtime.h>

static const void* last_kernel;
static dim3 last_grid;
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) (last_kernel = reinterpret_cast<const void*>(kernel), last_grid = (grid))
#define hipGetLastError() hipSuccess
#include "../paper_2208_04187_amd/csrc/masks.hip"

#define NAMED(kernel) if (last_kernel == reinterpret_cast<const void*>(static_cast<void (*)(PoolArgs)>(kernel))) return #kernel
static const char* pool_kernel() {
    NAMED((maxpool_backward_scalar<float>));
    NAMED((maxpool_backward_scalar<uint16_t>));
    NAMED((maxpool_backward_kernel<float, 1>));
    NAMED((maxpool_backward_kernel<float, 4>));
    NAMED((maxpool_backward_kernel<uint16_t, 1>));
    NAMED((maxpool_backward_kernel<uint16_t, 4>));
    NAMED((maxpool2_backward_fast<float, 4, false>));
    NAMED((maxpool2_backward_fast<float, 4, true>));
    NAMED((maxpool2_backward_fast<uint16_t, 4, false>));
    NAMED((maxpool2_backward_fast<uint16_t, 4, true>));
    NAMED((maxpool2_backward_fast<uint16_t, 8, false>));
    NAMED((maxpool2_backward_fast<uint16_t, 8, true>));
    NAMED((maxpool2_forward_fast<float, false, false>));
    NAMED((maxpool2_forward_fast<float, true, false>));
    NAMED((maxpool2_forward_fast<float, true, true>));
    NAMED((maxpool2_forward_fast<uint16_t, false, false>));
    NAMED((maxpool2_forward_fast<uint16_t, true, false>));
    NAMED((maxpool2_forward_fast<uint16_t, false, true>));
    NAMED((maxpool2_forward_fast<uint16_t, true, true>));
    return "";
}

extern "C" {
// the pooling kernel last launched (empty: another one), and its workgroups
const char* check_pool_kernel(uint32_t* workgroups) { *workgroups = last_grid.x * last_grid.y; return pool_kernel(); }
}
