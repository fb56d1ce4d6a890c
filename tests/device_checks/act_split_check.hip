// Test library: the two forms of the activation split that encoder and decoder use (csrc/pcc_device.h), side by side on
// given values, from the same header and with the same compiler flags as the kernels.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "pcc_device.h"

using namespace pcc;

// values[groups][4] -> out[groups][2 forms][hi01, hi23, lo01, lo23]: act_split4_bf16, then act_split_bf16
template <bool LEAKY>
__global__ void __launch_bounds__(64)
split_both_kernel(const float* __restrict__ values, size_t groups, uint32_t* __restrict__ out) {
    const bf16x4_bits_t minus_one = minus_identity(threadIdx.x);
    const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x, at = i < groups ? i : groups - 1;    // whole waves: MFMA takes all lanes
    const f32x4_t a = reinterpret_cast<const f32x4_t*>(values)[at];
    u32x2_t hi, lo;
    act_split4_bf16<LEAKY>(a, minus_one, hi, lo);
    uint32_t l0, l1;
    const uint32_t h0 = act_split_bf16<LEAKY>(a.x, a.y, l0), h1 = act_split_bf16<LEAKY>(a.z, a.w, l1);
    if (i < groups) {
        uint32_t* o = out + 8 * i;
        o[0] = hi.x; o[1] = hi.y; o[2] = lo.x; o[3] = lo.y;
        o[4] = h0; o[5] = h1; o[6] = l0; o[7] = l1;
    }
}

extern "C" int act_split_check(const float* d_values, size_t groups, int leaky, uint32_t* d_out, void* hip_stream) {
    if (!d_values || !d_out || groups == 0 || groups > (1u << 28) || ((uintptr_t)d_values & 15u) != 0) return -1;
    const dim3 grid((uint32_t)((groups + 63) / 64));
    if (leaky) hipLaunchKernelGGL(split_both_kernel<true>, grid, dim3(64), 0, (hipStream_t)hip_stream, d_values, groups, d_out);
    else hipLaunchKernelGGL(split_both_kernel<false>, grid, dim3(64), 0, (hipStream_t)hip_stream, d_values, groups, d_out);
    return hipGetLastError() == hipSuccess ? 0 : -2;
}
