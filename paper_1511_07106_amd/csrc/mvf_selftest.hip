// Self-tests of device code that no entry point shows alone (not part of the
// libmvf ABI; built as libmvf_selftest.so for the GPU tests): the hardware
// square-root estimate that the integration kernel's square-root filter relies
// on, and the raycast's launch order.
//
// The estimate: for every binary32 x with bit pattern in [first, first + count) (positive
// values), compares the estimate (v_sqrt_f32) with the correctly rounded
// root: the largest distance in units in the last place for x >= 2^-96, and
// the largest absolute difference for x < 2^-96.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "mvf_tile_order.h"

namespace {

__global__ __launch_bounds__(256) void sqrt_check_kernel(uint32_t first, uint32_t count, unsigned int* out)
{
    unsigned int max_ulp = 0;
    float max_abs = 0.0f;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < count; j += stride) {
        const float x = __uint_as_float(first + j);
        const float e = __builtin_amdgcn_sqrtf(x);
        const float r = sqrtf(x);
        if (x >= 0x1p-96f) {
            const int d = (int)__float_as_uint(e) - (int)__float_as_uint(r);
            max_ulp = max(max_ulp, (unsigned int)(d < 0 ? -d : d));
        } else {
            max_abs = fmaxf(max_abs, fabsf(e - r));
        }
    }
    for (int o = 32; o >= 1; o >>= 1) {
        max_ulp = max(max_ulp, (unsigned int)__shfl_xor((int)max_ulp, o));
        max_abs = fmaxf(max_abs, __shfl_xor(max_abs, o));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&out[0], max_ulp);
        atomicMax(&out[1], __float_as_uint(max_abs));  // non-negative floats order like their bits
    }
}

__global__ __launch_bounds__(1024) void tile_order_kernel(mvf::TileOrder O)
{
    __shared__ int hist[mvf::kOrderBins];
    mvf::tile_order_block(O, hist);
}

}  // namespace

// The launch order of `tiles` tiles from their durations (zeroed on return), by
// a block of `threads` threads: the plan's kRayPlanInts words, then the tiles.
// Returns 0 on success.  Synchronous.
extern "C" int mvf_selftest_tile_order(uint32_t* cost, int32_t* order, int tiles, int level, int max_blocks, int slots,
                                       int fresh, int threads)
{
    if (!cost || !order || tiles <= 0 || tiles > (1 << 22) || level < 0 || level >= mvf::kRayLevels || max_blocks <= 0 ||
        slots <= 0 || (threads != 256 && threads != 1024))
        return 1;
    const size_t nc = (size_t)tiles * sizeof(uint32_t), no = ((size_t)tiles + mvf::kRayPlanInts) * sizeof(int32_t);
    uint8_t* d = nullptr;
    if (hipMalloc((void**)&d, nc + no) != hipSuccess) return 2;
    mvf::TileOrder O{reinterpret_cast<uint32_t*>(d), reinterpret_cast<int32_t*>(d + nc), tiles, level, max_blocks, slots,
                     fresh};
    int rc = 0;
    if (hipMemcpy(d, cost, nc, hipMemcpyHostToDevice) != hipSuccess) rc = 3;
    if (!rc) {
        hipLaunchKernelGGL(tile_order_kernel, dim3(1), dim3(threads), 0, nullptr, O);
        if (hipGetLastError() != hipSuccess) rc = 4;
    }
    if (!rc && (hipMemcpy(cost, d, nc, hipMemcpyDeviceToHost) != hipSuccess ||
                hipMemcpy(order, d + nc, no, hipMemcpyDeviceToHost) != hipSuccess))
        rc = 5;
    (void)hipFree(d);
    return rc;
}

// Returns 0 on success.  max_ulp: largest ulp distance for x >= 2^-96;
// max_abs: largest absolute difference for x < 2^-96.  Synchronous.
extern "C" int mvf_selftest_sqrt(uint32_t first, uint32_t count, uint32_t* max_ulp, float* max_abs)
{
    if (!max_ulp || !max_abs || first >= 0x7f800000u || count > 0x7f800000u - first) return 1;
    unsigned int* d = nullptr;
    if (hipMalloc((void**)&d, 2 * sizeof(unsigned int)) != hipSuccess) return 2;
    unsigned int h[2] = {0, 0};
    int rc = 0;
    if (hipMemcpy(d, h, sizeof(h), hipMemcpyHostToDevice) != hipSuccess) rc = 3;
    if (!rc && count) {
        hipLaunchKernelGGL(sqrt_check_kernel, dim3(4096), dim3(256), 0, nullptr, first, count, d);
        if (hipGetLastError() != hipSuccess) rc = 4;
    }
    if (!rc && hipMemcpy(h, d, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess) rc = 5;
    (void)hipFree(d);
    *max_ulp = h[0];
    memcpy(max_abs, &h[1], sizeof(float));
    return rc;
}
