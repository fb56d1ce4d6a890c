// Test library: the forms of the activation split that encoder and decoder use (csrc/pcc_device.h), side by side on
// given values, from the same header and with the same compiler flags as the kernels.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "pcc_device.h"

using namespace pcc;

constexpr int kForms = 6;

// The encoder's split of a pair of out-blocks and both tiles, as its layers place it behind NM MFMAs.
template <class Net, int NM>
__device__ __forceinline__ void encoder_split(f32x4_t (&v)[2][2], bf16x4_bits_t minus_one, u32x4_t (&to)[2][2]) {
    const EncoderNet<Net, Net::kLayers> net{nullptr, nullptr, (int)(threadIdx.x & 63), minus_one};
    static_for<0, NM>([&](auto m) __attribute__((always_inline)) { net.template split_piece<decltype(m)::value, NM>(v, to); });
}

// values[group][4], four groups a lane -> out[group][form][hi01, hi23, lo01, lo23]: act_split4_bf16, act_split_bf16, then
// the encoder's behind 4, 8, 16 and 40 MFMAs (each of its four schedules)
template <class Net>
__global__ void __launch_bounds__(64)
split_forms_kernel(const float* __restrict__ values, size_t quads, uint32_t* __restrict__ out) {
    const bf16x4_bits_t minus_one = minus_identity(threadIdx.x);
    const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x, quad = i < quads ? i : quads - 1;    // whole waves: MFMA takes all lanes
    f32x4_t a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = reinterpret_cast<const f32x4_t*>(values)[4 * quad + q];
    auto put = [&](int q, int form, uint32_t h0, uint32_t h1, uint32_t l0, uint32_t l1) {
        const u32x4_t w = {h0, h1, l0, l1};
        if (i < quads) reinterpret_cast<u32x4_t*>(out)[(4 * i + q) * kForms + form] = w;
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        u32x2_t hi, lo;
        act_split4_bf16<Net::kLeaky>(a[q], minus_one, hi, lo);
        put(q, 0, hi.x, hi.y, lo.x, lo.y);
        uint32_t l0, l1;
        const uint32_t h0 = act_split_bf16<Net::kLeaky>(a[q].x, a[q].y, l0), h1 = act_split_bf16<Net::kLeaky>(a[q].z, a[q].w, l1);
        put(q, 1, h0, h1, l0, l1);
    }
    auto encoder = [&](int form, auto nm) __attribute__((always_inline)) {
        f32x4_t v[2][2] = {{a[0], a[1]}, {a[2], a[3]}};            // [block][tile]
        u32x4_t to[2][2];                                          // [tile][hi, lo], a block's two words behind the other's
        encoder_split<Net, decltype(nm)::value>(v, minus_one, to);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = q >> 1, t = q & 1;
            put(q, form, to[t][0][2 * j], to[t][0][2 * j + 1], to[t][1][2 * j], to[t][1][2 * j + 1]);
        }
    };
    encoder(2, std::integral_constant<int, 4>());
    encoder(3, std::integral_constant<int, 8>());
    encoder(4, std::integral_constant<int, 16>());
    encoder(5, std::integral_constant<int, 40>());
}

// `groups` (of four values) is a multiple of four.
extern "C" int act_split_check(const float* d_values, size_t groups, int leaky, uint32_t* d_out, void* hip_stream) {
    if (!d_values || !d_out || groups == 0 || groups % 4 != 0 || groups > (1u << 24) || (((uintptr_t)d_values | (uintptr_t)d_out) & 15u) != 0) return -1;
    const size_t quads = groups / 4;
    const dim3 grid((uint32_t)((quads + 63) / 64));
    static_assert(NetPaper::kLeaky && !NetWorkload::kLeaky, "one network of each activation");
    if (leaky) hipLaunchKernelGGL(split_forms_kernel<NetPaper>, grid, dim3(64), 0, (hipStream_t)hip_stream, d_values, quads, d_out);
    else hipLaunchKernelGGL(split_forms_kernel<NetWorkload>, grid, dim3(64), 0, (hipStream_t)hip_stream, d_values, quads, d_out);
    return hipGetLastError() == hipSuccess ? 0 : -2;
}
