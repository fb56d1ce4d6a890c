// libpcc: kernels and C ABI (see include/pcc.h for the contract).
//
// Kernels (templated on the network description, see pcc_device.h)
//   encode_kernel      gather + network (MFMA) + mixture -> (start,freq) of the
//                      true sub-pixels, all pixels in parallel, the rows' right
//                      ends first
//   rans_rows_kernel   two lanes per image row, one per coder state: push the row's
//                      symbols last to first into a per-row slab, written backwards; for a small
//                      job it runs beside encode_kernel, taking the symbols as
//                      they appear, and with narrow images takes the rows to their places in the stream itself
//   compact_kernel     otherwise: slabs -> contiguous stream, with header and offsets
//   scan_kernel        exclusive prefix sum of row payload sizes in front of it, for jobs of very many rows
//   decode_kernel      persistent wavefront decoder: one workgroup (4 waves) per
//                      band of 16 rows, step t handles pixel (r, t - delay*r) of each row
//   decode_narrow_kernel  the same with bands of eight rows
//   cdf_tables_kernel  test hook: full integer CDF tables from given parameters
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "pcc.h"
#include "pcc_device.h"
#include "rans_arith.h"

namespace pcc {

constexpr uint32_t kBlobMagic = 0x57434350u;    // "PCCW"
constexpr uint32_t kStreamMagic = 0x31434350u;  // "PCC1"
constexpr int kStreamHeader = 32;
constexpr uint32_t kStreamVersion = 2;          // two coder states per row (1: one)
constexpr int kBandRows = 16, kNarrowRows = 8;      // rows of a band (decode_kernel, decode_narrow_kernel)
constexpr uint32_t kMailTag = 0x80000000u;

template <class Net>
constexpr uint32_t model_tag() { return (uint32_t)Net::K | ((uint32_t)Net::kNbhd << 8) | ((uint32_t)Net::kDelay << 16) | (16u << 24); }

// The pixel kernel's work item: a strip of 32 pixels of one row (two tiles of the network) for a wave.
constexpr int kStripPixels = 32;
constexpr int kLdsBytes = 160 * 1024;
constexpr int kTakenBytes = 16;          // LDS of the counter that a workgroup's waves take their items from
// What the pixel kernel keeps in LDS: the weights of as many leading layers as fit together with all biases,
// the biases behind them, and behind those the CDF table if there is room left (the whole image when
// everything fits).  The other layers' weights, and the table when it is not there, are read from global memory.
template <class Net>
constexpr int encode_resident_layers() {
    using Lay = Layout<Net>;
    int r = Net::kLayers;
    while (r > 0 && Lay::w_off(r) + (Lay::kLutOff - Lay::kWeightBytes) + kTakenBytes > kLdsBytes) --r;
    return r;
}
template <class Net>
constexpr int encode_table_lds_off() {      // = Layout::kLutOff when all layers are resident
    return Layout<Net>::w_off(encode_resident_layers<Net>()) + (Layout<Net>::kLutOff - Layout<Net>::kWeightBytes);
}
template <class Net>
constexpr bool encode_table_in_lds() { return encode_table_lds_off<Net>() + (Layout<Net>::kModelBytes - Layout<Net>::kLutOff) + kTakenBytes <= kLdsBytes; }
template <class Net>
constexpr int encode_model_lds_bytes() {
    return encode_table_lds_off<Net>() + (encode_table_in_lds<Net>() ? Layout<Net>::kModelBytes - Layout<Net>::kLutOff : 0);
}
// pcc_encode_probs: pixels whose head outputs a wave stages in LDS at a time, where there is room for that beside the model image.
// 0: a lane stores its outputs from its registers, runs of 3 K floats.  Smaller stages cost more than they save, in passes of one LDS
// round trip each: 1403x1021, us, with one pixel at a time, two and from the registers: six layers 462, 411, 405; two, four and from the
// registers: seven mixtures 446, 388, 375.  With eight, staged and from the registers: 30-160-160-128-60 284 and 293, four layers 247 and 257,
// five mixtures 356 and 361, the paper's network 330 and 338.
template <class Net>
constexpr int params_stage_pixels() {
    return encode_model_lds_bytes<Net>() + kTakenBytes + (Net::kEncodeThreads / 64) * 8 * Net::dim(Net::kLayers) * 4 <= kLdsBytes ? 8 : 0;
}
template <class Net>
constexpr int params_stage_bytes() { return (Net::kEncodeThreads / 64) * params_stage_pixels<Net>() * Net::dim(Net::kLayers) * 4; }

// Status words in device memory, one block for the decoder, one for the encoder, one that nobody reads (pcc_encode_probs,
// which does not wait for its kernel).  The decoder's is cleared on its stream before each call.
// The encoder's is zero whenever a call begins: the last workgroup of the compaction leaves what the call has to say in pinned
// host memory (EncodeResult) and clears it for the next call, so that a call needs no clearing, no copy and no second clearing
// around its kernels (64x64 59.7 -> 45.7 us a call, 768x512 124 -> 113); a call that fails clears it from the host.
enum { kStErr = 0, kStAbort = 1, kStTicket = 2, kStDefer = 3, kStWords = 4 };
enum { kStDone = kStTicket };                 // encoder: workgroups of the compaction that have ended
enum { kBlockDecode = 0, kBlockEncode = 1, kBlockProbs = 2, kStBlocks = 3 };
constexpr size_t kStBytes = kStWords * sizeof(int);
struct EncodeResult {                         // of a call, in pinned host memory
    uint64_t total_bytes;
    int err, defer;
};

// Most 32-bit words a row's payload can have: four of the two final coder states, and one per two symbols plus two.
__host__ __device__ inline size_t slab_words(int W) { return (6 * (size_t)W + 24) / 4 + 1; }

// ---------------------------------------------------------------------------
// shared device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ void set_error(int* status, int code) { atomicCAS(&status[kStErr], 0, code); }

// An offset of zero the optimiser cannot see through.  Added to the LDS base
// inside a loop it keeps the (loop-invariant) weight reads from being hoisted
// out of the loop and parked in registers or scratch.
__device__ __forceinline__ uint32_t opaque_zero() {
    uint32_t z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

// 16 bytes a thread at a time, kUnroll of them in flight.
__device__ __forceinline__ void copy_to_lds(uint8_t* lds, const uint8_t* __restrict__ src, int bytes) {
    constexpr int kUnroll = 17;
    const u32x4_t* s = reinterpret_cast<const u32x4_t*>(src);
    u32x4_t* d = reinterpret_cast<u32x4_t*>(lds);
    const int n = bytes / 16, step = (int)blockDim.x;
    for (int i = threadIdx.x; i < n; i += kUnroll * step) {
        u32x4_t v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) v[u] = s[min(i + u * step, n - 1)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) if (i + u * step < n) d[i + u * step] = v[u];
    }
}

// Lane group and register (g * kHeadSlots + s) that hold canonical head output c, in the order of Head.
template <class Net, class Head = Net>
__host__ __device__ constexpr int head_slot(int c) {
    for (int g = 0; g < 4; ++g)
        for (int s = 0; s < Layout<Net>::kHeadSlots; ++s)
            if (Head::head_index(g, s) == c) return g * Layout<Net>::kHeadSlots + s;
    return -1;
}

// A value of each of a pixel's two lanes (lane and lane + 32), in both of them.
__device__ __forceinline__ void both_halves(uint32_t v, uint32_t& of_half0, uint32_t& of_half1) {
    const u32x2_t r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane32_swap(v, v, false, false));
    of_half0 = r.x;
    of_half1 = r.y;
}

// ---------------------------------------------------------------------------
// encode: all pixels in parallel
//
// A work item is a strip of 32 consecutive pixels of one image row, two tiles of the network; strips are
// numbered from the right edge of the image, item = strip * rows + row, and the
// workgroups take the items in turn, one at a time.  The rows' right
// ends are therefore finished first, which is where the row coder starts (it
// pushes the symbols last to first).  The row coder may run beside this kernel:
// then the results go to sf_tagged instead of sf, one 64-bit word per symbol with
// this launch's epoch in the high half, written through to device scope.  A
// reader that finds the epoch has the symbol; nothing else is published and
// nothing has to be cleared between launches (epochs only grow).
//
// What bounds it: with weights that are dense numbers the chip's power.  A loop of these MFMAs on random operands in
// registers runs at 1.94 of 2.4 GHz (2,028 TFLOP/s); this kernel executes 1,490 TFLOP/s of them beside its LDS reads and vector
// instructions (4096x2160; 227,000 matrix operations per pixel with hi + lo, 117,120 of them the network's).
// With weights that are mostly zero (the plane predictor) it runs at 2.38 GHz and is bound by its
// SIMDs: 9,700 cycles a strip against 7,104 of the MFMAs, some 560 of the split's small ones, and 870 vector instructions of
// 4.1 that the issue port takes between them (an MFMA holds the port for 8 of its 16 cycles).
// v_mfma_f32_32x32x16_bf16, two of which give the same bits as one 16x16x32, holds it for half as long, but takes 15 % more
// power for the same numbers (1,764 TFLOP/s): 24 images with the predictor's weights 1,288 us a call against 1,334, but the
// paper's network 1,910 against 1,800 and 4096x2160 1,475 against 1,437.
// Two waves per SIMD: one does not hide its own gather and mixtures (1,562 us against 1,246).
// Pixel kernel, 24 images of 768x512, predictor: 1,455 -> 1,180 us; paper's network 1,854 -> 1,624; 4096x2160 1,578 -> 1,348.
// ---------------------------------------------------------------------------
template <class Net>
__global__ void __launch_bounds__(Net::kEncodeThreads)
encode_kernel(const uint8_t* __restrict__ model, const uint8_t* __restrict__ img, int n, int H, int W,
              uint32_t* __restrict__ sf, float* __restrict__ params, float* __restrict__ bits, int* status,
              uint64_t* sf_tagged, uint32_t epoch, uint32_t strip_begin, uint32_t strip_count) {
    using Lay = Layout<Net>;
    using Head = EncHead<Net>;
    constexpr int K = Net::K, KB0 = Net::kb(0), HEAD = Net::dim(Net::kLayers);
    extern __shared__ __align__(16) uint8_t lds[];
    uint32_t* taken = reinterpret_cast<uint32_t*>(lds + encode_model_lds_bytes<Net>());     // items of the workgroup that have been taken
    constexpr int RESIDENT = encode_resident_layers<Net>();
    constexpr uint32_t nwaves = Net::kEncodeThreads / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar: the item's row and strip are scalars too
    const int g = lane >> 4, nl = lane & 15;      // the network's lane: inputs of k-slot group g of pixel nl of a tile
    const int h = lane >> 5, px = lane & 31;      // the mixtures' lane: pixel px of the strip; its channel R (half 0) or G (half 1), and half of B
    const bf16x4_bits_t minus_one = minus_identity(lane);
    const uint32_t rows = (uint32_t)n * (uint32_t)H;
    const uint32_t P = rows * (uint32_t)W;
    const uint32_t items = strip_count * rows;              // this launch's strips: strip_begin .. strip_begin + strip_count - 1
    // This lane's first-layer inputs are runs of four consecutive image bytes.  Byte offset of a run from the strip's first pixel,
    // for the first tile.
    uint32_t run_at[KB0][2];
    bool run_used[KB0][2];
#pragma unroll
    for (int kb = 0; kb < KB0; ++kb) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            int dr = 0, off = 0;
            run_used[kb][half] = Net::run_desc(kb, g, half, dr, off);
            run_at[kb][half] = run_used[kb][half] ? (uint32_t)((dr * W + nl - 2) * 3 + off) : 3u * (uint32_t)nl;
        }
    }
    // The workgroup's waves take the next of its items as they get free, from a counter in LDS: of the two waves of a SIMD the
    // older one goes first wherever both can issue and is through its work faster.  (Dealt out beforehand, the older waves
    // ended after four fifths of the kernel's time, and the younger ones had a SIMD each for the rest.)
    auto take = [&]() __attribute__((always_inline)) {
        uint32_t k = 0;
        if (lane == 0) k = atomicAdd(taken, 1u);
        k = (uint32_t)__builtin_amdgcn_readfirstlane((int)k);
        return k * gridDim.x + blockIdx.x;      // dealt out one by one (by eights a job of few strips left most of the chip idle: 64x64 45.7 -> 42.7 us)
    };
    // An item's bytes: the lane's runs of both tiles and its pixel's own bytes r | g<<8 | b<<16.
    auto gather = [&](uint32_t item, uint32_t& rowg, int& c0, uint32_t (&runs)[KB0][2][2], uint32_t& pix) __attribute__((always_inline)) {
        const uint32_t local = item / rows, strip = strip_begin + local;
        rowg = item - local * rows;
        const uint32_t im = rowg / (uint32_t)H;
        const int r = (int)(rowg - im * (uint32_t)H);
        c0 = W - kStripPixels * (int)(strip + 1);               // negative in the leftmost strip of a ragged width
        const uint8_t* base = img + (size_t)im * H * W * 3;
        if (r >= 2 && c0 >= 2 && c0 + kStripPixels + 3 <= W) {
            // everything the strip's pixels look at lies in the image (their runs end at column c + 3 at most)
            const uint8_t* first = base + ((size_t)r * W + c0) * 3;
            __builtin_memcpy(&pix, first + 3u * (uint32_t)px, 4);     // unaligned dword; the fourth byte is the next pixel's
#pragma unroll
            for (int kb = 0; kb < KB0; ++kb) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const uint8_t* run = first + (int)run_at[kb][half];
                    __builtin_memcpy(&runs[kb][0][half], run, 4);
                    __builtin_memcpy(&runs[kb][1][half], run + 3 * 16, 4);
                }
            }
            return;
        }
        pix = 0;
        if (c0 + px >= 0) {
            const uint32_t p = rowg * (uint32_t)W + (uint32_t)(c0 + px);
            const int me = (r * W + c0 + px) * 3;
            if (p + 1 < P) __builtin_memcpy(&pix, base + me, 4);
            else pix = (uint32_t)base[me] | ((uint32_t)base[me + 1] << 8) | ((uint32_t)base[me + 2] << 16);
        }
        // a run is read with one load when all its bytes lie in the image, byte by byte at the borders
#pragma unroll
        for (int kb = 0; kb < KB0; ++kb) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    uint32_t v = 0;
                    const int c = c0 + 16 * t + nl;
                    int dr = 0, off = 0;
                    if (Net::run_desc(kb, g, half, dr, off) && c >= 0) {
                        const int rr = r + dr;
                        const int at = (rr * W + (c - 2)) * 3 + off;
                        const int col_first = c - 2 + ((off * 11) >> 5), col_last = c - 2 + (((off + 3) * 11) >> 5);
                        if (rr >= 0 && col_first >= 0 && col_last < W) {
                            __builtin_memcpy(&v, base + at, 4);
                        } else if (rr >= 0) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int col = c - 2 + (((off + i) * 11) >> 5);
                                if (col >= 0 && col < W) v |= (uint32_t)base[at + i] << (8 * i);
                            }
                        }
                    }
                    runs[kb][t][half] = v;
                }
            }
        }
    };
    // The next item's bytes are asked for before the network runs on this one's.
    // (A wave's first item is dealt by its number, and its bytes are asked for before the model is.)
    uint32_t item = wave * gridDim.x + blockIdx.x, next_row = 0, runs[KB0][2][2], next_pix = 0;
    int next_c0 = 0;
    if (item < items) gather(item, next_row, next_c0, runs, next_pix);
    if (threadIdx.x == 0) *taken = nwaves;
    if constexpr (RESIDENT == Net::kLayers) {
        copy_to_lds(lds, model, encode_model_lds_bytes<Net>());
    } else {
        copy_to_lds(lds, model, Lay::w_off(RESIDENT));
        copy_to_lds(lds + Lay::w_off(RESIDENT), model + Lay::kWeightBytes, encode_model_lds_bytes<Net>() - Lay::w_off(RESIDENT));
    }
    __syncthreads();
    const uint8_t* table_at = encode_table_in_lds<Net>() ? lds + (encode_table_lds_off<Net>() - Lay::kLutOff) : model;
    const float2* lut = reinterpret_cast<const float2*>(table_at + Lay::kLutOff);
    const float lut_scale = *reinterpret_cast<const float*>(table_at + Lay::kLutScaleOff);
    while (item < items) {
        const uint32_t rowg = next_row, pix = next_pix & 0xFFFFFFu;
        const int c0 = next_c0, c = c0 + px;
        const bool live = c >= 0;
        u32x4_t in[KB0][2][2];
#pragma unroll
        for (int kb = 0; kb < KB0; ++kb) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                uint32_t a, b, c2, d;
                run_to_bf16(run_used[kb][0] ? runs[kb][t][0] : 0u, a, b);
                run_to_bf16(run_used[kb][1] ? runs[kb][t][1] : 0u, c2, d);
                in[kb][t][0].x = a; in[kb][t][0].y = b; in[kb][t][0].z = c2; in[kb][t][0].w = d;
                in[kb][t][1] = in[kb][t][0];   // unused (layer-1 inputs are exact)
            }
        }
        item = take();
        if (item < items) gather(item, next_row, next_c0, runs, next_pix);
        f32x4_t out[Lay::kHeadOB][2];
        // the wave that feeds the matrix cores goes first (2048x1365 head outputs 524 -> 494 us, 24 images of the paper's network 1,647 -> 1,624)
        __builtin_amdgcn_s_setprio(2);
        EncoderNet<Net, RESIDENT>{lds + opaque_zero(), model + opaque_zero(), lane, minus_one}.run(in, out);
        __builtin_amdgcn_s_setprio(0);
        // The head's results are first read behind branches (which outputs are wanted, border tiles).  The wait
        // states an MFMA's result needs are counted along the instruction stream as laid out, not along a taken
        // branch, so the accumulators are made to settle here, in straight-line code.
#pragma unroll
        for (int ob = 0; ob < Lay::kHeadOB; ++ob) asm volatile("" : "+v"(out[ob][0]), "+v"(out[ob][1]));
        asm volatile("s_nop 7" ::: "memory");

        // from two tiles of four lane groups to one strip of two halves (EncHead)
        float head[Head::kSlots];
#pragma unroll
        for (int s = 0; s < Head::kGroupSlots; ++s) {
            const u32x2_t r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane16_swap(
                __float_as_uint(out[s >> 2][0][s & 3]), __float_as_uint(out[s >> 2][1][s & 3]), false, false));
            head[s] = __uint_as_float(r.x);
            head[s + Head::kGroupSlots] = __uint_as_float(r.y);
        }
        // B's values, which the two lanes of a pixel hold in turn, in both
        float item_b[Head::kBItems];
        static_for<0, (Head::kBItems + 1) / 2>([&](auto pc) {
            constexpr int b = 2 * decltype(pc)::value;
            uint32_t v0, v1;
            both_halves(__float_as_uint(head[Head::b_slot(b)]), v0, v1);
            item_b[b] = __uint_as_float(v0);
            if constexpr (b + 1 < Head::kBItems) {
                static_assert(Head::b_half(b) == 0 && Head::b_half(b + 1) == 1 && Head::b_slot(b) == Head::b_slot(b + 1), "pairs share a register");
                item_b[b + 1] = __uint_as_float(v1);
            }
        });
        const uint32_t p = rowg * (uint32_t)W + (uint32_t)c;
        if (params != nullptr) {
            // A pixel's outputs are R's, G's, B's parameters (3 K each), alphas, betas, gammas (K each): half 0 holds the first
            // and third group of 3 K, half 1 the second and fourth.
            constexpr int PX = params_stage_pixels<Net>() > 0 ? params_stage_pixels<Net>() : 1;
            float second[3 * K];
#pragma unroll
            for (int i = 0; i < 3 * K; ++i) second[i] = h == 0 ? item_b[i] : i < K ? head[3 * K + i] : item_b[2 * K + i];
            if (params_stage_pixels<Net>() > 0 && ((uintptr_t)params & 15u) == 0) {
                // The tile's head outputs are HEAD consecutive floats per pixel, 32 consecutive pixels: they go
                // through a staging area of this wave in LDS, PX pixels at a time, and leave as
                // 16-byte stores of consecutive lanes (stored straight from the registers, a lane's values are
                // two runs of 3 K floats, HEAD floats apart from its neighbour's).  LDS takes a wave's
                // instructions in order, so the reads see the writes of the same pass.  All reads of a pass before its
                // stores, whose addresses are one base and constants: 2048x1365 490 -> 470 us (432 without any outputs; they
                // are 670 MB).
                float* stage = reinterpret_cast<float*>(lds + encode_model_lds_bytes<Net>() + kTakenBytes) + wave * (PX * HEAD);
#pragma unroll
                for (int pass = 0; pass < kStripPixels / PX; ++pass) {
                    if (px / PX == pass) {
                        float* mine = stage + (px % PX) * HEAD + 3 * K * h;
#pragma unroll
                        for (int i = 0; i < 3 * K; ++i) { mine[i] = head[i]; mine[6 * K + i] = second[i]; }
                    }
                    __builtin_amdgcn_wave_barrier();
                    constexpr int CHUNKS = PX * HEAD / 4, ROUNDS = (CHUNKS + 63) / 64;
                    f32x4_t v[ROUNDS];
#pragma unroll
                    for (int i = 0; i < ROUNDS; ++i) v[i] = *reinterpret_cast<const f32x4_t*>(stage + 4 * min(lane + 64 * i, CHUNKS - 1));
                    // the strip's first column may lie before the row: chunks of columns below 0 are not stored
                    float* at = params + ((int64_t)rowg * W + c0 + pass * PX) * HEAD;
                    const int first = c0 + pass * PX < 0 ? -(c0 + pass * PX) * (HEAD / 4) : 0;
#pragma unroll
                    for (int i = 0; i < ROUNDS; ++i) {
                        const int j = lane + 64 * i;
                        if (j >= first && j < CHUNKS) *reinterpret_cast<f32x4_t*>(at + 4 * j) = v[i];
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            } else if (live) {
                float* mine = params + (size_t)p * HEAD + 3 * K * h;
#pragma unroll
                for (int i = 0; i < 3 * K; ++i) { mine[i] = head[i]; mine[6 * K + i] = second[i]; }
            }
        }
        const float rhat = (float)(pix & 0xFF) * (1.0f / 256.0f);
        const float ghat = (float)((pix >> 8) & 0xFF) * (1.0f / 256.0f);
        // the lane's own channel: R, or G given R
        uint32_t lo, freq;
        {
            float raw[3 * K];
#pragma unroll
            for (int s = 0; s < 3 * K; ++s) raw[s] = head[s];
            ChanParams<K> cp;
            channel_setup<K>(raw, lut_scale, cp);
            if (h == 1) {
                float alpha[K];
#pragma unroll
                for (int k = 0; k < K; ++k) alpha[k] = head[3 * K + k];
                couple_green<K>(cp, alpha, rhat);
            }
            const int x = (int)((pix >> (8 * h)) & 0xFF);
            lo = cq_full<K>(cp, x, lut);
            freq = cq_full<K>(cp, x + 1, lut) - lo;
        }
        // B given R and G: half 0 evaluates the lower edge, half 1 the upper one
        uint32_t lo_b, freq_b;
        {
            float raw[3 * K], beta[K], gamma[K];
#pragma unroll
            for (int i = 0; i < 3 * K; ++i) raw[i] = item_b[i];
#pragma unroll
            for (int k = 0; k < K; ++k) { beta[k] = item_b[3 * K + k]; gamma[k] = item_b[4 * K + k]; }
            ChanParams<K> cp;
            channel_setup<K>(raw, lut_scale, cp);
            couple_blue<K>(cp, beta, gamma, rhat, ghat);
            uint32_t hi_b;
            both_halves(cq_full<K>(cp, (int)(pix >> 16) + h, lut), lo_b, hi_b);
            freq_b = hi_b - lo_b;
        }
        // Cq increases strictly from 0 to 65536: a frequency outside 1 .. 65536 (also: lo not below hi) is an error
        if (live && (freq - 1u > 65535u || freq_b - 1u > 65535u)) {
            set_error(status, PCC_E_INTERNAL);
            __threadfence();                 // known before the symbols are: whoever has those reads the status
            if (freq - 1u > 65535u) freq = 1;
            if (freq_b - 1u > 65535u) freq_b = 1;
        }
        const uint32_t word = lo | ((freq - 1u) << 16), word_b = lo_b | ((freq_b - 1u) << 16);
        if (sf_tagged != nullptr) {
            if (live) {
                uint64_t* at = sf_tagged + (size_t)p * 3;
                __hip_atomic_store(at + h, ((uint64_t)epoch << 32) | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (h == 0) __hip_atomic_store(at + 2, ((uint64_t)epoch << 32) | word_b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else if (sf != nullptr) {
            uint32_t word_r, word_g;
            both_halves(word, word_r, word_g);
            if (live && h == 0) {
                const uint32_t three[3] = {word_r, word_g, word_b};
                __builtin_memcpy(sf + (size_t)p * 3, three, sizeof three);
            }
        }
        if (bits != nullptr) {
            uint32_t bits_r, bits_g;
            both_halves(__float_as_uint(16.0f - __builtin_amdgcn_logf((float)freq)), bits_r, bits_g);
            const float tot = (__uint_as_float(bits_r) + __uint_as_float(bits_g)) + (16.0f - __builtin_amdgcn_logf((float)freq_b));
            if (h == 0 && live) bits[p] = tot;
        }
    }
}

// ---------------------------------------------------------------------------
// rANS encode, two lanes per row: one per coder state.  A row's stream carries
// two interleaved states (symbol i on state i mod 2) that meet only in the order
// of the words they emit, so each state's serial chain runs in a lane of its
// own and the order is restored afterwards.  A workgroup owns 32 rows: the 64
// lanes of wave 0 each run one state's chain; waves 2 and 3 fetch the rows'
// (start, freq) words chunk by chunk (coalesced, two chunks ahead), compute the
// fp64 reciprocal of every frequency and stage both in LDS; wave 1 merges the
// words the two lanes of a row produced, in the order of the symbols that
// caused them, and copies them from LDS to the rows' slabs.  The coding wave's
// instruction stream, which bounds the kernel (it is limited by instruction
// issue, not by the latency of the chain), then holds only the chain itself.
// ---------------------------------------------------------------------------
constexpr int kRansRows = 32;
constexpr int kRansChunk = 64;                      // symbols of a row per round: 32 for each of its two lanes
constexpr int kRansThreads = 256;
constexpr uint32_t kRansBesideMaxGroups = 96;      // row-coder workgroups that may run beside the pixel kernel
constexpr uint32_t kXcds = 8;
constexpr uint32_t kRansPatience = 2048;            // polls for one symbol before a row coder beside the pixel kernel stands down (a few ms)
// Decides how much of a tall image the pixel kernel does before the row coder joins it: the share of its strips that is left for
// that is 1.1 times this over the rows.  (Alone, the row coder takes as long as the pixel kernel with the whole chip at
// some 390 rows: 56 us at any number of rows of 768 pixels against 73 at 512 rows.  Beside each other both are slower.)  Whole calls, us, with
// 300, 400, 500, 600 and 700: 2048x1365 524, 501, 488, 491, 491; 4096x2160 1,475, 1,437, 1,401, 1,422, 1,430; 800x640 154, 142,
// 141, 143, 129 (no split any more); nine shapes from 800x640 on, with the paper's network too, take 4.5, 1.8, 1.2, 2.3 and 1.7 % longer
// than with the best of the five on average.
constexpr uint32_t kRansBalanceRows = 600;
// Widest image whose rows the row coder takes to their places in the stream itself where it runs beside the pixel kernel.  A
// workgroup does so with one compute unit, the compaction with the whole chip.  Whole calls, us, with the compaction and
// without: 256x256 58.3, 57.0; three of 768x512 228.7, 224.4; 1000x3000 510.2, 505.4; 1024x1024 204.4, 203.6; 1536x800 236.4,
// 236.8; 2048x640 249.0, 250.8; 4096x512 366, 372; 6000x300 490, 502.
constexpr int kRansAssembleWidth = 1024;
// Padding symbol (start 0, frequency 2^16): pushing it leaves the state unchanged
// and never renormalises, so every chunk can be coded as a full one.
constexpr uint32_t kRansNop = 0xFFFF0000u;

// The coding wave rounds its fp64 arithmetic toward zero (MODE.FP_ROUND bits 3:2 = 3).  Written as
// assembly: the compiler would put the default mode back in front of the wave's fp64 instructions.
// rans_push (rans_arith.h) relies on it.
__device__ __forceinline__ void rans_round_toward_zero() {
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3" ::: "memory");
}

// Keeps a wave's SIMD from falling idle while the wave waits for LDS.  Where all four SIMDs of a compute unit have been without a vector or
// matrix instruction, as behind every barrier, the first ten or so vector instructions of each wave take 14 cycles instead of 4, as if the SIMDs
// shared one issue slot for some 140 cycles.  (Measured, not documented: a loop of a read, a barrier and K vector instructions takes four waves 145, 281, 321 and 401
// cycles for K = 0, 10, 20 and 40, one wave at work 140, 180, 220 and 300, two 140, 213, 299 and 372.)  Matrix instructions are not slowed and prevent it: with four 4x4x4
// MFMAs (8 cycles each) in the read's wait the loop takes four waves 165, 245, 285 and 365, with six, which outlast the wait, 215, 282, 322 and 402.  So a wait that
// vector instructions follow is filled with MFMAs of zeros, as long as the wait at least takes anyway.  (Not in the searches, whose own
// instructions fill the look-ups' waits: one MFMA each 4,076 -> 4,155 us; in the gather, behind a layer's reads, which MFMAs follow, or
// at the step's end 4,102 to 4,142.)  768x512 4,187 -> 4,076 us, with bands of 16 rows 4,733 -> 4,586; the paper's network in 512x512
// 4,909 -> 4,722.  Why some networks lose by it (kKeepAwake, kKeepAwakeWide) is not known.
template <bool ON>
struct Awake {
    static constexpr int kBehindWrite = 4, kBehindHeadReads = 6, kBehindMixtureReads = 10;      // MFMAs, of 2 to 14 tried each
    f32x4_t sink;
    bf16x4_bits_t zero;
    __device__ __forceinline__ Awake() {
        u32x2_t z = {0, 0};
        asm volatile("" : "+v"(z));
        zero = __builtin_bit_cast(bf16x4_bits_t, z);
        sink = f32x4_t{0, 0, 0, 0};
    }
    template <int N>
    __device__ __forceinline__ void keep() {
        if constexpr (ON) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                sink = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(zero, zero, sink, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    __device__ __forceinline__ void used() {              // (not to be left out as unused)
        if constexpr (ON) asm volatile("" :: "v"(sink));
    }
};

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for
// every outstanding global access (stores, polls, prefetches), which would put
// memory latency on the critical path of every round of the row coder and several
// times on every step of the decoder; neither hands global data from thread to
// thread across such a barrier.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// (v << 1) | bit, in one instruction: the bit is the carry into v + v.  The carry may be read only two wait states after
// the compare that made it, and the compiler, which sees to that in its own instructions, does not look into this one.
// So it takes `selected`, which has to be a value that a select on the same bit has made: the compiler puts the select
// two wait states behind the compare, and this behind the select.
// (Of the compiler's own making this takes two instructions, a select of 0 or 1 and a shift with an or.)
__device__ __forceinline__ uint32_t shift_in(uint32_t v, bool bit, uint32_t selected) {
    const uint64_t carry = __ballot(bit);
    uint64_t out;
    asm("v_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(v), "=s"(out) : "s"(carry), "v"(selected));
    return v;
}

// Where a call's stream goes, and what describes it.
struct StreamOut {
    uint8_t* stream;
    uint64_t cap_bytes;
    int n, H;
    uint32_t tag, dist;
    uint64_t* total_bytes;
    EncodeResult* result;
    uint64_t* sums;            // of the row coder's groups: epoch << 32 | words (kSumStoodDown: none)
    uint32_t sums_patience;    // polls of a group for the sums of those before it
};
constexpr uint32_t kSumStoodDown = 0xFFFFFFFFu;

__device__ __forceinline__ void write_header(const StreamOut& out, int W) {
    uint32_t* hdr = reinterpret_cast<uint32_t*>(out.stream);
    hdr[0] = kStreamMagic; hdr[1] = kStreamVersion; hdr[2] = (uint32_t)out.n; hdr[3] = (uint32_t)out.H; hdr[4] = (uint32_t)W;
    hdr[5] = out.tag; hdr[6] = out.dist; hdr[7] = 0;
}

// The last of a kernel's workgroups to end leaves the call's result in host memory and the status block clear.
// This workgroup's errors, and the total if it is here, before its count: all are atomic accesses at device scope, so that
// they have been made when the wave's counter of outstanding ones is zero.  (A fence would write the die's L2 back, in every
// workgroup: 254 us for 24 images of 768x512.)
__device__ __forceinline__ void leave_result(const StreamOut& out, int* status) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0 && (uint32_t)atomicAdd(&status[kStDone], 1) + 1u == gridDim.x) {
        out.result->total_bytes = __hip_atomic_load(out.total_bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        out.result->err = atomicExch(&status[kStErr], 0);
        out.result->defer = atomicExch(&status[kStDefer], 0);
        atomicExch(&status[kStDone], 0);
    }
}

// BESIDE: the pixel kernel is running; the symbols are read from sf_tagged, past the caches that are not
// coherent with the pixel kernel's stores, and each is waited for until it carries this launch's epoch.
// ASSEMBLES: the workgroups (at most kRansBesideMaxGroups) take their rows to their places in the stream themselves and there is
// no compaction behind them: each publishes its words and waits for those of the groups before it.
template <bool BESIDE, bool ASSEMBLES>
__global__ void __launch_bounds__(kRansThreads, 2 /* waves per SIMD: two workgroups per compute unit */)
rans_rows_kernel(const uint32_t* __restrict__ sf, const uint64_t* sf_tagged, uint32_t epoch, int W, uint32_t rows,
                 uint32_t* __restrict__ slabs, uint32_t* __restrict__ row_words, uint32_t* __restrict__ group_words, int* status,
                 uint32_t patience, StreamOut out) {
    static_assert(BESIDE || !ASSEMBLES, "the sums carry the epoch of the symbols");
    constexpr int kPerState = kRansChunk / 2;   // symbols of a chunk that one state (one coding lane) takes
    static_assert(kPerState == 32, "a coding lane's emission flags of a round fill one 32-bit word");
    // [buffer][row][symbol of the chunk]; the odd row strides keep the coding wave's column accesses off shared banks
    __shared__ uint32_t sym[2][kRansRows][kRansChunk + 1];
    __shared__ double rcp[2][kRansRows][kRansChunk + 1];
    // [buffer][state][row][step]: the low state word before each of the lane's symbols of the chunk, in the order
    // coded; it is one of the stream's words where the lane's flag for that step is set
    __shared__ uint32_t outw[2][2][kRansRows][kPerState + 1];
    // [buffer][row][state]: the flags, the first step's in bit 31, and [2 + state] the words the state emitted in all rounds
    // before: whoever stores the round's words has their places from these alone
    __shared__ __align__(16) uint32_t outflags[2][kRansRows][4];
    __shared__ uint32_t final_state[kRansRows][4];   // xl, xh of state 0, xl, xh of state 1 after the row's first symbol
    __shared__ uint32_t abandon;                // set by a loader whose wait ran out: every wave leaves after the round
    const int tid = threadIdx.x, lane = tid & 63;
    const bool coder = tid < 64;
    const uint32_t row0 = blockIdx.x * kRansRows;
    const uint32_t nsym = 3u * (uint32_t)W;
    const int nchunks = (int)((nsym + kRansChunk - 1) / kRansChunk);
    const uint32_t live_rows = min((uint32_t)kRansRows, rows - row0);
    const size_t sw = slab_words(W);
    // coding lane: row of the workgroup lane & 31, state lane >> 5 (symbol i of the row is coded on state i mod 2)
    const int crow = lane & (kRansRows - 1), cstate = lane >> 5;
    uint32_t xl = (uint32_t)kRansL, xh = (uint32_t)(kRansL >> 32);     // the lane's state x = xh 2^32 + xl
    uint32_t emitted = 0;            // coding lane: words of the rounds so far

    // Wave 0 codes; waves 2 and 3 load (symbols from global memory, reciprocals, both to LDS); wave 1 stores (the
    // words the coding wave produced, from LDS to the rows' slabs).  Loads and stores are kept in different waves
    // because a wave's loads and stores complete out of order with each other under one counter: a wave that
    // has stores in flight can only wait for a load by waiting for everything.
    const bool storer = tid >= 64 && tid < 128, loader = tid >= 128;
    constexpr int kLoaders = kRansThreads - 128;
    constexpr int kPerLoader = (kRansRows * kRansChunk + kLoaders - 1) / kLoaders;
    static_assert(kRansRows * kRansChunk % kLoaders == 0 && kRansRows == 32, "whole elements per thread; a row per lane pair");
    static_assert(kRansChunk % 2 == 0, "a chunk starts at an even symbol index: the state of a symbol follows from its place in the chunk");
    // The pipeline, one stage per round (a round = the coding wave codes a chunk; rounds end in a workgroup
    // barrier), so that no wave waits for memory inside a round:
    //   round k + 3  the chunk's symbols are requested from global memory into registers (two sets, by round parity)
    //   round k + 1  (beside the pixel kernel: symbols it has not written yet are waited for,) reciprocals are
    //                computed, symbols and reciprocals go to LDS buffer k & 1
    //   round k      the coding wave codes the chunk
    //   round k - 1  the words it produced are copied to the rows' slabs
    using Staged = std::conditional_t<BESIDE, uint64_t, uint32_t>;
    Staged staged[2][kPerLoader];
    auto request = [&](int k, Staged (&staged)[kPerLoader]) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kPerLoader; ++it) {
            const int e = tid - 128 + it * kLoaders;
            const uint32_t r = (uint32_t)e / kRansChunk, i = (uint32_t)e % kRansChunk;
            const uint32_t idx = (uint32_t)k * kRansChunk + i;
            // every lane loads (a padding element loads the buffer's first word): with no branch round the loads
            // the compiler can count them, and waits for one register set while the other's loads are in flight
            const bool real = r < live_rows && idx < nsym;
            const size_t at = real ? (size_t)(row0 + r) * nsym + idx : 0;
            if constexpr (BESIDE) staged[it] = __hip_atomic_load(&sf_tagged[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else staged[it] = sf[at];
        }
    };
    auto deposit = [&](int k, Staged (&staged)[kPerLoader]) __attribute__((always_inline)) {
        const int b = k & 1;
        if constexpr (BESIDE) {
            // Symbols the pixel kernel has not written yet (seldom once the pixel kernel, the faster of the two, is
            // ahead): the lane polls one of them, sleeping in between so that the polls of a coder that has
            // caught up do not load the memory system, and then loads its whole set again, all loads at once.
            // The first time it loads its set again without a poll: behind a chunk that was waited for, the next two have mostly
            // been written since they were asked for, and a poll is another way to memory and back (us a call: 64x64 40.2 -> 38.7,
            // 333x100 62.4 -> 60.7, 768x512 101.2 -> 100.4; jobs that the row coder bounds as before).
            // A running pixel kernel delivers a row's next strip within tens of microseconds.  A wait of
            // `patience` polls (milliseconds) therefore means that it is held up (other work is in front of it, the chip is
            // taken, a profiler runs the kernels one at a time): the row coder stands down, and the host launches it again after the pixel kernel.
            uint32_t spins = 0;
            for (bool again = false;; again = true) {
                size_t stale_at = 0;
                bool stale = false;
#pragma unroll
                for (int it = 0; it < kPerLoader; ++it) {
                    const int e = tid - 128 + it * kLoaders;
                    const uint32_t r = (uint32_t)e / kRansChunk, i = (uint32_t)e % kRansChunk;
                    const uint32_t idx = (uint32_t)k * kRansChunk + i;
                    if (r < live_rows && idx < nsym && (uint32_t)(staged[it] >> 32) != epoch) {
                        stale = true;
                        stale_at = (size_t)(row0 + r) * nsym + idx;
                    }
                }
                if (!stale) break;
                bool gave_up = false;
                while (again && (uint32_t)(__hip_atomic_load(&sf_tagged[stale_at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32) != epoch) {
                    if (++spins > patience) { gave_up = true; break; }
                    __builtin_amdgcn_s_sleep(32);
                }
                if (gave_up) {
                    __hip_atomic_store(&status[kStDefer], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if constexpr (ASSEMBLES) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // before this workgroup counts as ended
                    abandon = 1;
                    break;
                }
                request(k, staged);
            }
        }
#pragma unroll
        for (int it = 0; it < kPerLoader; ++it) {
            const int e = tid - 128 + it * kLoaders;
            const uint32_t r = (uint32_t)e / kRansChunk, i = (uint32_t)e % kRansChunk;
            const bool real = r < live_rows && (uint32_t)k * kRansChunk + i < nsym;
            const uint32_t v = real ? (uint32_t)staged[it] : kRansNop;
            sym[b][r][i] = v;
            rcp[b][r][i] = rans_recip_below((v >> 16) + 1u);
        }
    };
    // Wave 1: the words of a finished chunk from buffer b to the rows' slabs, one row per iteration.  Slabs fill from the end:
    // the decoder reads the words in reverse order of production.  Lane p stands
    // for the p-th symbol coded in the round (symbol kRansChunk - 1 - p of the chunk: state 1 when p is even, the
    // state's step p / 2).  Where that symbol's flag is set, its word goes behind the words of the symbols coded
    // before it, from either state: those of the rounds before, the flags set among the first ceil(p / 2) steps of state 1 and
    // the first floor(p / 2) steps of state 0.  Lanes without a word store beyond the slabs' end, which the hardware drops:
    // with a branch around each row's store, positions read from other lanes and 64-bit addresses this wave took 3,900
    // cycles a round where the coding wave takes 3,200.  All LDS reads are issued before the first store.
    const auto slab_rows = __builtin_amdgcn_make_buffer_rsrc(slabs + (size_t)row0 * sw, 0, (int)(uint32_t)(live_rows * sw * 4),
                                                             0x00020000 /* untyped dwords */);
    auto flush = [&](int b) __attribute__((always_inline)) {
        const uint32_t p = (uint32_t)lane, step = p >> 1, state = 1u - (p & 1u);
        auto first_steps = [](uint32_t nsteps) { return nsteps == 0 ? 0u : 0xFFFFFFFFu << (32u - nsteps); };   // their flag bits
        const uint32_t before1 = first_steps((p + 1) >> 1), before0 = first_steps(p >> 1);
        // in batches of rows; the next batch's LDS reads are issued before this one's stores
        constexpr int kBatch = 8;
        uint32_t word[2][kBatch], own[2][kBatch];
        u32x4_t f[2][kBatch];
        auto read = [&](int n) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const int r = n * kBatch + i;
                word[n & 1][i] = outw[b][state][r][step];
                own[n & 1][i] = outflags[b][r][state];
                f[n & 1][i] = *reinterpret_cast<const u32x4_t*>(outflags[b][r]);
            }
        };
        read(0);
        uint32_t row_at = 0;                                        // the row's slab, from the first one's
#pragma unroll
        for (int n = 0; n < kRansRows / kBatch; ++n) {
            if (n + 1 < kRansRows / kBatch) read(n + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const u32x4_t v = f[n & 1][i];
                const uint32_t ahead = (uint32_t)__popc(v.y & before1) + v.w + ((uint32_t)__popc(v.x & before0) + v.z);
                uint32_t at = 4u * ((uint32_t)sw - 1u - ahead);
                asm volatile("" : "+v"(at));                        // no branch round its computation
                at = (int)(own[n & 1][i] << step) < 0 ? at : 0xFFFFFFF0u;
                __builtin_amdgcn_raw_buffer_store_b32(word[n & 1][i], slab_rows, (int)at, (int)row_at, 0);
                row_at += 4u * (uint32_t)sw;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (tid == 0) abandon = 0;
    lds_barrier();
    if (coder) rans_round_toward_zero();
    // one round; P = the round's parity, which picks the loaders' register set
    auto round = [&](int k, auto parity) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value;
        const int b = k & 1;
        if (loader) {
            if (k >= 1 && k - 1 < nchunks) deposit(k - 1, staged[P]);
            request(min(max(k - 3, 0), nchunks - 1), staged[P]);     // outside the chunks: loads nobody uses
        } else if (storer) {
            if (k >= -1 && k + 1 < nchunks) flush(b ^ 1);
        } else if (k >= 0 && k < nchunks) {
            // The lane's symbols of the chunk, last first: kRansChunk - 2 + cstate, then every second one down to
            // cstate.  Symbols and reciprocals come from LDS in batches of kU; the next batch is requested before
            // the serial chain of the current one starts, so that only the round's first read waits for LDS.
            constexpr int kU = 8, kBatches = kPerState / kU;
            uint32_t v[2][kU];
            double rf[2][kU];
            const uint32_t* my_sym = &sym[b][crow][cstate];
            const double* my_rcp = &rcp[b][crow][cstate];
            uint32_t* my_out = &outw[b][cstate][crow][0];
            auto fetch = [&](int n) {
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    v[n & 1][u] = my_sym[kRansChunk - 2 - 2 * (n * kU + u)];
                    rf[n & 1][u] = my_rcp[kRansChunk - 2 - 2 * (n * kU + u)];
                }
            };
            uint32_t flags = 0;
            fetch(0);
#pragma unroll
            for (int n = 0; n < kBatches; ++n) {
                if (n + 1 < kBatches) fetch(n + 1);
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const uint32_t start = v[n & 1][u] & 0xFFFFu, f = (v[n & 1][u] >> 16) + 1u;
                    // renormalise when x >= f * 2^47; the low word is stored either way, at the step's own place,
                    // and only counts where the flag says it was due: no branch and no address arithmetic on the
                    // serial chain
                    const bool emit = (xh >> 15) >= f;
                    my_out[n * kU + u] = xl;
                    xl = emit ? xh : xl;
                    xh = emit ? 0u : xh;
                    flags = shift_in(flags, emit, xl);
                    rans_push(xl, xh, f, start, rf[n & 1][u]);
                }
            }
            outflags[b][crow][cstate] = flags;
            outflags[b][crow][2 + cstate] = emitted;
            emitted += (uint32_t)__popc(flags);
        }
        lds_barrier();   // all that crosses threads here is in LDS; the loaders' global loads stay in flight
        return !BESIDE || abandon == 0;
    };
    // rounds nchunks + 2 (or + 3, for an even number of rounds) down to -1, where chunk 0's words are stored
    for (int k = nchunks + 2 + (nchunks & 1); k >= 0; k -= 2) {
        if (!round(k, std::integral_constant<int, 0>()) || !round(k - 1, std::integral_constant<int, 1>())) {
            if constexpr (ASSEMBLES) {
                if (tid == 0)
                    __hip_atomic_store(&out.sums[blockIdx.x], (uint64_t)epoch << 32 | kSumStoodDown, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                leave_result(out, status);
            } else {
                if (tid < kRansRows && row0 + tid < rows) row_words[row0 + tid] = 0;    // stood down: nothing for the compaction to copy
                if (tid == 0) group_words[blockIdx.x] = 0;
            }
            return;
        }
    }
    if (coder) {
        final_state[crow][2 * cstate] = xl;
        final_state[crow][2 * cstate + 1] = xh;
        outflags[0][crow][cstate] = emitted;                        // (the last words have been stored)
    }
    lds_barrier();
    uint32_t words = 0;
    if (storer && lane < kRansRows && row0 + lane < rows) {
        const uint32_t wp = (uint32_t)sw - (outflags[0][lane][0] + outflags[0][lane][1]);
        words = (uint32_t)sw - (wp - 4u);
        // the four state words end the slab's data: the decoder reads them first
        uint32_t* slab = slabs + (size_t)(row0 + lane) * sw;
        slab[wp - 1] = final_state[lane][3];
        slab[wp - 2] = final_state[lane][2];
        slab[wp - 3] = final_state[lane][1];
        slab[wp - 4] = final_state[lane][0];
        if constexpr (!ASSEMBLES) row_words[row0 + lane] = words;
    }
    if constexpr (!ASSEMBLES) {
        if (storer) {                            // the group's sum (at most 32 times 100 MB in words)
            for (int d = 32; d >= 1; d >>= 1) words += __shfl_xor(words, d);
            if (lane == 0) group_words[blockIdx.x] = words;
        }
    } else {
        // The compaction's work in the row coder: a launch, its gap and the way from one die's L2 to another's less (us a call,
        // before and after: 64x64 41.5, 39.7; 768x512 102.5, 101.2; five of 333x217 with seven mixtures 132.8, 129.8).  What bounds
        // it is latency: the sums' way between the dies, one batch of loads and stores for rows of up to 256 words, the count.
        __shared__ uint32_t row_at[kRansRows], row_len[kRansRows], group_len, good;    // words in front of a row within the group, and in it
        __shared__ uint64_t words_before;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        if (storer) {
            uint32_t upto = words;               // lanes beyond the rows have none
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t v = __shfl_up(upto, d);
                upto += lane >= d ? v : 0u;
            }
            if (lane == 63)
                __hip_atomic_store(&out.sums[blockIdx.x], (uint64_t)epoch << 32 | upto, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool over = __any(words > (uint32_t)sw) != 0;           // not a coder's count: never read outside the slab
            if (over && lane == 0) set_error(status, PCC_E_INTERNAL);
            if (lane < kRansRows) { row_at[lane] = upto - words; row_len[lane] = words; }
            if (lane == 63) { group_len = upto; good = over ? 0u : 1u; }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // the slabs are written: all waves read them next
        } else if (wave == 2) {
            // The sums of the groups before, two to a lane.  On a chip with room for all groups they end within a few us of each
            // other.  Where other work holds a die's units, a group of that die may still wait for its start when later ones, on other
            // dies, are here: they hold their units until it has ended, or stand down when their patience is over (some 10 ms), as
            // from a missing symbol, and the call codes its rows once more.
            static_assert(kRansBesideMaxGroups <= 128, "two sums to a lane");
            uint64_t before = 0;
            uint32_t polls = 0;
            bool down = blockIdx.x != 0 && out.sums_patience == 0, waiting = !down;
            while (waiting) {
                waiting = false;
                before = 0;
#pragma unroll
                for (uint32_t i = 0; i < 2; ++i) {
                    const uint32_t k = (uint32_t)lane + 64 * i;
                    if (k >= blockIdx.x) continue;
                    const uint64_t v = __hip_atomic_load(&out.sums[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((uint32_t)(v >> 32) != epoch) waiting = true;
                    else if ((uint32_t)v == kSumStoodDown) down = true;
                    else before += (uint32_t)v;
                }
                down = __any(down) != 0;
                waiting = __any(waiting) != 0 && !down;
                if (waiting) {
                    if (++polls == out.sums_patience) { down = true; break; }
                    __builtin_amdgcn_s_sleep(2);
                }
            }
            for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor((unsigned long long)before, d);
            if (lane == 0) {
                words_before = before;
                if (down) {
                    __hip_atomic_store(&status[kStDefer], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    abandon = 1;
                }
            }
        }
        lds_barrier();
        if (abandon == 0) {
            const uint64_t table = (uint64_t)kStreamHeader + 8ull * ((uint64_t)rows + 1), first = words_before;
            uint64_t* offsets = reinterpret_cast<uint64_t*>(out.stream + kStreamHeader);
            // header, offsets and, from the last group, the end offset and the total: all inside the table, which the host has
            // checked against the capacity
            if (storer && (uint32_t)lane < live_rows) offsets[row0 + lane] = 4ull * (first + row_at[lane]);
            const uint64_t end = table + 4ull * (first + group_len);
            if (tid == 0) {
                if (row0 == 0) write_header(out, W);
                if (blockIdx.x + 1 == gridDim.x) {
                    offsets[rows] = end - table;
                    __hip_atomic_store(out.total_bytes, end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (end > out.cap_bytes) set_error(status, PCC_E_CAP);
            }
            if (end <= out.cap_bytes && good != 0 && (uint32_t)wave < live_rows) {
                // A wave per four rows apart, eight of them at a time, 16 bytes a lane and row (words lie at multiples of four
                // bytes, which such loads and stores allow).  A row has four words at least; lanes beyond its end take its last
                // four again, and places beyond the group's rows the wave's first: no branch between the loads.
                typedef uint32_t words4_t __attribute__((ext_vector_type(4), aligned(4)));
                constexpr int kRowsOfWave = kRansRows / (kRansThreads / 64);
                const uint32_t* src[kRowsOfWave];
                uint32_t* dst[kRowsOfWave];
                uint32_t last[kRowsOfWave], most = 0;
#pragma unroll
                for (int k = 0; k < kRowsOfWave; ++k) {
                    const uint32_t r = (uint32_t)(wave + 4 * k) < live_rows ? (uint32_t)(wave + 4 * k) : (uint32_t)wave;
                    const uint32_t len = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_len[r]);
                    const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_at[r]);
                    src[k] = slabs + (size_t)(row0 + r) * sw + (sw - len);
                    dst[k] = reinterpret_cast<uint32_t*>(out.stream + table) + first + at;
                    last[k] = len - 4u;
                    most = max(most, len);
                }
                for (uint32_t i = 4u * (uint32_t)lane; i - 4u * (uint32_t)lane < most; i += 256) {
                    words4_t v[kRowsOfWave];
#pragma unroll
                    for (int k = 0; k < kRowsOfWave; ++k) v[k] = *reinterpret_cast<const words4_t*>(src[k] + min(i, last[k]));
#pragma unroll
                    for (int k = 0; k < kRowsOfWave; ++k) *reinterpret_cast<words4_t*>(dst[k] + min(i, last[k])) = v[k];
                }
            }
        }
        leave_result(out, status);
    }
}

// Single workgroup: before[k] = sum_{j<k} group_words[j], for jobs of so many groups that the compaction's workgroups cannot
// each add up those before their own.
constexpr uint32_t kSumGroupsMax = 4096;
__global__ void __launch_bounds__(1024)
scan_kernel(const uint32_t* __restrict__ group_words, uint32_t groups, uint64_t* __restrict__ before) {
    __shared__ uint64_t part[1024];
    __shared__ uint64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < groups; base += 1024) {
        const uint32_t k = base + threadIdx.x;
        const uint64_t mine = k < groups ? (uint64_t)group_words[k] : 0ull;
        part[threadIdx.x] = mine;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const uint64_t add = threadIdx.x >= (uint32_t)d ? part[threadIdx.x - d] : 0ull;
            __syncthreads();
            part[threadIdx.x] += add;
            __syncthreads();
        }
        if (k < groups) before[k] = carry + part[threadIdx.x] - mine;
        __syncthreads();
        if (threadIdx.x == 1023) carry += part[1023];
        __syncthreads();
    }
}

// Header, offsets and the rows' payloads to their places in the stream.  A workgroup takes `chunk` consecutive rows (a multiple
// of four), four at a time, a wave per row.  The words before its first row are those
// of the row coder's groups before (added up by every workgroup, from L2: no launch for a scan; or from scan_kernel)
// and of the group's rows before it.  The last workgroup to end leaves the call's result in host memory and the status block
// clear: the workgroups count in one word, some 10 ns each, so there are at most kCompactBlocks of them.
// (With an offset per row from a scan by one workgroup, 24 images of 768x512 took 25 us for the scan and 9 for the copy.)
constexpr int kCompactRows = 4, kCompactThreads = 64 * kCompactRows;
constexpr uint32_t kCompactBlocks = 512;

__global__ void __launch_bounds__(kCompactThreads)
compact_kernel(const uint32_t* __restrict__ slabs, const uint32_t* __restrict__ row_words, const uint32_t* __restrict__ group_words,
               const uint64_t* __restrict__ before, int W, uint32_t rows, uint32_t chunk, int* status, StreamOut out) {
    uint8_t* const __restrict__ stream = out.stream;
    __shared__ unsigned long long part[kCompactRows];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t first = blockIdx.x * chunk, end = min(first + chunk, rows), group = first / kRansRows;      // first < rows
    const size_t sw = slab_words(W);
    const uint64_t table = (uint64_t)kStreamHeader + 8ull * ((uint64_t)rows + 1);
    uint32_t nw[kCompactRows];                 // the words of the next four rows
    auto sizes = [&](uint32_t row0) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t w = 0; w < kCompactRows; ++w) nw[w] = row0 + w < end ? row_words[row0 + w] : 0u;
    };
    sizes(first);
    unsigned long long words_before = 0;
    if (before != nullptr) {
        if (threadIdx.x == 0) words_before = before[group];
    } else {
        for (uint32_t j = threadIdx.x; j < group; j += kCompactThreads) words_before += group_words[j];
    }
    if (threadIdx.x < first - group * kRansRows) words_before += row_words[group * kRansRows + threadIdx.x];
    for (int d = 32; d >= 1; d >>= 1) words_before += __shfl_xor(words_before, d);
    if (lane == 0) part[wave] = words_before;
    __syncthreads();
    words_before = 0;
    for (int w = 0; w < kCompactRows; ++w) words_before += part[w];

    uint64_t* offsets = reinterpret_cast<uint64_t*>(stream + kStreamHeader);
    for (uint32_t row0 = first; row0 < end; row0 += kCompactRows) {
        unsigned long long mine = words_before;
        uint32_t words = nw[0];
#pragma unroll
        for (int w = 0; w < kCompactRows; ++w) {
            if (w < wave) mine += nw[w];
            if (w == wave) words = nw[w];
            words_before += nw[w];
        }
        const uint32_t row = row0 + wave;
        if (row0 + kCompactRows < end) sizes(row0 + kCompactRows);
        if (row >= rows) break;
        const uint64_t off = 4ull * mine;
        // header, this row's offset and, from the last row, the end offset and the total: all inside the table,
        // which the host has checked against the capacity
        if (lane == 0) {
            offsets[row] = off;
            if (row == 0) write_header(out, W);
            if (row + 1 == rows) {
                offsets[rows] = off + 4ull * words;
                __hip_atomic_store(out.total_bytes, table + off + 4ull * words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (words > sw) {                             // not a row coder's count: never read outside the slab
            if (lane == 0) set_error(status, PCC_E_INTERNAL);
        } else if (table + off + 4ull * words > out.cap_bytes) {
            if (lane == 0) set_error(status, PCC_E_CAP);
        } else {
            const uint32_t* src = slabs + (size_t)row * sw + (sw - words);
            uint32_t* dst = reinterpret_cast<uint32_t*>(stream + table + off);
            constexpr uint32_t kUnroll = 8;           // loads in flight
            for (uint32_t i = lane; i < words; i += 64 * kUnroll) {
                uint32_t v[kUnroll];
#pragma unroll
                for (uint32_t u = 0; u < kUnroll; ++u) if (i + 64 * u < words) v[u] = src[i + 64 * u];
#pragma unroll
                for (uint32_t u = 0; u < kUnroll; ++u) if (i + 64 * u < words) dst[i + 64 * u] = v[u];
            }
        }
    }
    leave_result(out, status);
}

// test hook: the symbols of a tagged buffer without their epochs
__global__ void __launch_bounds__(256)
untag_kernel(const uint64_t* __restrict__ tagged, size_t count, uint32_t* __restrict__ out) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) out[i] = (uint32_t)tagged[i];
}

// ---------------------------------------------------------------------------
// wavefront decode
//
// One workgroup of 4 waves owns a band of 16 image rows (or eight, with twice as
// many lanes to a pixel, see decode_narrow_kernel); step t decodes pixel
// (r, t - delay * r) of each row (delay = right reach of the neighbourhood + 1).
// Per step:
//   network   the pixels form one MFMA tile of 16; each wave computes a quarter
//             of every layer's out-blocks with its weight slices held in
//             registers for the whole kernel, and the layers meet in LDS
//   search    16 lanes per pixel find the symbol with two 16-way sweeps of
//             Cq evaluations per channel (R, then G given R, then B given R,G)
//   publish   the pixel goes to the LDS ring (next steps' neighbourhoods), to
//             the output image and, for the band's last two rows, to a mailbox
//             in global memory that the band below polls
// ---------------------------------------------------------------------------
constexpr int kDecThreads = 256;

// Where a decode step spends its cycles: built only with -DPCC_PHASE_TIMING (a measurement build; the product has
// an empty struct here and no code).  Every wave reads the shader clock at the marks of the step and sums the
// differences per phase; the workgroup that decodes ticket kPhaseTicket leaves the sums in phase_cycles.
enum { kPhGather = 0, kPhLayer0 = 1 /* + layer */, kPhMixture = 8, kPhR = 9, kPhG = 10, kPhB = 11, kPhPublish = 12,
       kPhFetch = 13, kPhBarrier = 14, kPhTop = 15, kPhCount = 16 };
#ifdef PCC_PHASE_TIMING
constexpr int kPhaseTicket = 8;
__device__ unsigned long long phase_cycles[4][kPhCount + 1];
struct PhaseClock {
    uint64_t t, acc[kPhCount];
    __device__ __forceinline__ void reset() {
        for (int i = 0; i < kPhCount; ++i) acc[i] = 0;
        t = __builtin_readcyclecounter();
    }
    __device__ __forceinline__ void mark(int i) {
        __builtin_amdgcn_sched_barrier(0);      // no instruction of one phase is moved into another
        const uint64_t now = __builtin_readcyclecounter();
        acc[i] += now - t;
        t = now;
        __builtin_amdgcn_sched_barrier(0);
    }
};
#else
struct PhaseClock {
    __device__ __forceinline__ void reset() {}
    __device__ __forceinline__ void mark(int) {}
};
#endif

// Does any first-layer run start at an odd byte of its window (NetDiagonal's copies do)?
template <class Net>
constexpr bool has_odd_runs() {
    for (int kbi = 0; kbi < Net::kb(0); ++kbi)
        for (int g = 0; g < 4; ++g)
            for (int half = 0; half < 2; ++half) {
                int dr = 0, off = 0;
                if (Net::run_desc(kbi, g, half, dr, off) && (off & 1) != 0) return true;
            }
    return false;
}

// decode LDS: the CDF table, two activation buffers, head outputs, mixtures, ring
template <class Net, int ROWS = kBandRows>
struct DecLds {
    static constexpr int kLanes = kDecThreads / ROWS;                  // lanes of a pixel
    static constexpr int kParts = kLanes / 16;                         // ... in rows of 16, which take a part of the components each
    static constexpr int kPartK = (Net::K + kParts - 1) / kParts;      // components of a part (the last part may have fewer)
    static constexpr int max_kb() {
        int m = 0;
        for (int l = 1; l < Net::kLayers; ++l) m = Net::kb(l) > m ? Net::kb(l) : m;
        return m;
    }
    static constexpr int kHS = Layout<Net>::kHeadSlots;
    static constexpr int kActBytes = max_kb() * 2 * 64 * 16;           // one layer's activations: [k-block][hi,lo][lane][16 B]
    static constexpr int kLutOff = 0;
    static constexpr Table kTable = kParts > 1 ? Table::kCopies : Table::kSpread;
    static constexpr int kLutEnd = ((kTable == Table::kCopies ? kLutCopies * kLutCopyBytes : kSpreadLutBytes) + 15) / 16 * 16;
    static constexpr bool kMiscFirst = kTable == Table::kCopies;       // (the 64 KB that an instruction's offset reaches end in front of the ring then)
    static constexpr int kAct0Off = kLutEnd + (kMiscFirst ? 16 : 0);
    static constexpr int kAct1Off = kAct0Off + kActBytes;
    // Strides in floats, padded by one 16-byte vector: consecutive pixels (and channels) then start
    // four LDS banks apart instead of on the same bank.
    static constexpr int kHeadStride = 4 * kHS + 4;                    // head outputs of one pixel: [4 groups][kHS]
    // mixture of one (pixel, channel): for each part of the components pi[kPartK], mu[kPartK], a[kPartK]
    static constexpr int kPartStride = kParts > 1 ? (3 * kPartK + 3) / 4 * 4 : 3 * Net::K <= 16 ? 20 : 24;
    static constexpr int kCpStride = kParts * kPartStride;
    static constexpr int kHeadOff = kAct1Off + kActBytes;              // [16 pixels][kHeadStride] fp32, (group, register) layout
    static constexpr int kCpOff = kHeadOff + 16 * kHeadStride * 4;     // [16 pixels][3 channels][kCpStride] fp32
    // Ring of recently decoded pixels as first-layer inputs, bf16: [ROWS + 2 rows][2 copies][2 * kRingCols columns][3].
    // Rows 0,1 are the two rows above the band.  Column c lives at slots c mod kRingCols and that + kRingCols, so the
    // values of a run of neighbour columns are always contiguous.  The second copy is one element further on, so
    // that a run of four values, which may start at any element, is two aligned dwords in one of the copies: LDS takes
    // 512 cycles over two 8-byte reads of four waves that are not 8-byte aligned, and 64 over two pairs of dwords.
    static constexpr int kRingCopyElems = 2 * Net::kRingCols * 3 + 1;  // from an element to the same one in the second copy
    static constexpr int kRingRowElems = 2 * kRingCopyElems + Net::kRingPad;
    static constexpr int kRingOff = kCpOff + 16 * 3 * kCpStride * 4;
    static constexpr int kRingEnd = kRingOff + (ROWS + 2) * kRingRowElems * 2;
    static constexpr int kMiscOff = kMiscFirst ? kLutEnd : kRingEnd;   // ticket, abort flag
    static constexpr int kSinkOff = kRingEnd + (kMiscFirst ? 0 : 16);  // where lanes with no ring element to write write
    static constexpr int kBytes = (kSinkOff + 64 * 4 + 8 * Net::K + 15) / 16 * 16;
    // Two workgroups per CU have 256 registers per lane each, too few for the whole of a wave's weight slices: there
    // the biases, and the weights of the first layer and of the head where two workgroups' LDS then still fits a CU,
    // are kept in LDS behind the above and read when used.
    static constexpr int kBiasBytes = Layout<Net>::kLutOff - Layout<Net>::kWeightBytes;
    static constexpr int kFirstBytes = Net::ob(0) * Net::kb(0) * kBlockBytes;
    static constexpr int kHeadBytes = Net::ob(Net::kLayers - 1) * Net::kb(Net::kLayers - 1) * kBlockBytes;
    static constexpr bool kBiasInLds = (Net::kSharedCuLds & 1) != 0;
    static constexpr int kBiasLds = kBiasInLds ? kBiasBytes : 0;
    static constexpr bool kFirstInLds = (Net::kSharedCuLds & 2) != 0 && 2 * (kBytes + kBiasLds + kFirstBytes) <= kLdsBytes;
    static constexpr int kFirstLds = kFirstInLds ? kFirstBytes : 0;
    static constexpr bool kHeadInLds = (Net::kSharedCuLds & 4) != 0 && 2 * (kBytes + kBiasLds + kFirstLds + kHeadBytes) <= kLdsBytes;
    static constexpr int kBiasOff = kBytes;
    static constexpr int kFirstOff = kBiasOff + kBiasLds;
    static constexpr int kHeadWOff = kFirstOff + kFirstLds;
    static constexpr int kBytesShared = kHeadWOff + (kHeadInLds ? kHeadBytes : 0);
    static constexpr bool kTwoFit = 2 * kBytesShared <= kLdsBytes;      // else a CU holds one workgroup whatever the launch asks
    static_assert(kBytes % 16 == 0 && kBiasBytes % 16 == 0, "vector alignment");
    static_assert(kAct0Off % 16 == 0 && kHeadOff % 16 == 0 && kCpOff % 16 == 0, "vector alignment");
    static_assert((16 * kHS) % 16 == 0 && (kRingRowElems * 2) % 4 == 0, "vector alignment");
    // A ring row is read by the two rows below it, which trail by delay and 2 * delay columns and
    // reach two columns further back, while the column being written and the zero columns right
    // of the image are stored: all of these must be distinct slots.
    static constexpr int kMaxReach = Net::kReach1 > Net::kReach2 ? Net::kReach1 : Net::kReach2;
    // Wave w computes out-blocks w, w + 4, ... of a layer.  Where a layer's block count is not a multiple of four,
    // the last wave has a round without a block; its spare time there, in MFMAs of the other waves' chains, is
    // kIdleSlack in layer kIdleLayer (the layer where it is largest; 0: no layer has any).  The spare rounds are used to
    // fetch the pixels of the rows above the band and to write decoded pixels to the image (decode_kernel).
    static constexpr int kLastWave = kDecThreads / 64 - 1;
    static constexpr int idle_slack(int l) {
        const int nob = Net::ob(l), slots = (nob + 3) / 4;
        return kLastWave + 4 * (slots - 1) >= nob ? Net::kb(l) * (l > 0 ? 2 : 1) : 0;
    }
    static constexpr int idle_layer() {
        int best = Net::kLayers - 1;
        for (int l = 0; l < Net::kLayers; ++l) if (idle_slack(l) > idle_slack(best)) best = l;
        return best;
    }
    static constexpr int kIdleLayer = idle_layer();
    static constexpr int kIdleSlack = idle_slack(kIdleLayer);
    // Waves that idle in that round (the last ones).  With two of them the last wave, whose lanes also publish the
    // band's last two rows to the mailbox, writes the decoded pixels to the image, and the wave before it fetches:
    // the fetching wave then has loads in flight and no stores (a wave's loads and stores complete out of order with
    // each other under one counter, so a wave that has both can only wait for a load by waiting for everything).
    // With one idle wave it does both.
    static constexpr int kIdleWaves = kIdleSlack > 0 ? 4 * ((Net::ob(kIdleLayer) + 3) / 4) - Net::ob(kIdleLayer) : 0;
    static constexpr int kStoreWave = kLastWave;
    // Waves from this one on have no block in those rounds (the last wave alone, which fetches and stores, if there are none).
    static constexpr int kFirstIdleWave = kIdleWaves > 0 ? kLastWave + 1 - kIdleWaves : kLastWave + 1;
    static constexpr int kFetchWave = kIdleWaves >= 2 ? kLastWave - 1 : kLastWave;
    // Does wave w have a round without an out-block in layer l?
    static constexpr bool wave_idles(int l, int w) { return w + 4 * ((Net::ob(l) + 3) / 4 - 1) >= Net::ob(l); }
    // The idle waves also have a (short) round to spare in the first layer where that is not the layer above: the storing
    // wave reads the pixels there that it stores in layer kIdleLayer.  (The fetch wave has then time enough for its whole job
    // in that layer, and its request moves to the step's end: decode_kernel, fetch_request.)
    static constexpr bool kIdleInFirstLayer =
        kIdleSlack > 0 && kIdleLayer != 0 && wave_idles(0, kStoreWave) && wave_idles(0, kFetchWave);
    // StepRole::kOwnsLast is one answer for all layers: the waves without a block in a layer's last round must be the same in
    // every layer that has such a round, and each must have a role of its own (a third one would compute a block too many).
    static constexpr bool same_waves_idle() {
        for (int l = 0; l < Net::kLayers; ++l)
            for (int w = 0; w <= kLastWave; ++w)
                if (Net::ob(l) % 4 != 0 && wave_idles(l, w) != (w >= kFirstIdleWave)) return false;
        return true;
    }
    static_assert(same_waves_idle() && kIdleWaves <= 2, "the roles of the decoder's waves do not fit the network's block counts");
    static_assert(kIdleLayer > 0 || kIdleSlack == 0, "the fetch must lie behind the barrier that follows the step's gather");
    static_assert(2 * Net::kDelay + 3 + kMaxReach <= Net::kRingCols, "ring too small for the neighbourhood");
    // what a row reads of the rows above must have been decoded in an earlier pass
    static_assert(Net::kReach1 <= Net::kDelay - 1 && Net::kReach2 <= 2 * Net::kDelay - 1, "schedule is not causal");
};

// rANS reader of one row, replicated in the pixel's lanes (16, or 32 with bands of eight rows).  A pixel consumes at most three of the
// row's 32-bit words; the next three, w[0..2], are requested at the end of a step's bookkeeping (settle, in
// decode_kernel) and wanted a third of a step later, so a renormalisation never waits for memory.
struct RowReader {
    uint64_t x, y;            // the two coder states: x is the next symbol's, y the one after's
    uint32_t w[3];            // words pos, pos + 1, pos + 2
    uint32_t at;              // offset of word 0 (the one after the states) from the wave's stream window, bytes
    uint32_t nwords, pos;     // words after the states; words consumed so far
    bool bad;
};

// All ones where `c` holds.  The selects of a pop are made with masks: two or more v_cndmask in a row on one condition in
// VCC take 16 cycles each while four waves of a compute unit do the same (one alone, or apart from each other, 4).
__device__ __forceinline__ uint32_t mask_of(bool c) {
    uint32_t m = c ? 0xFFFFFFFFu : 0u;
    asm volatile("" : "+v"(m));            // (not to be turned into selects again)
    return m;
}
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

// D(x) for the symbol found at (start, freq) and the renormalisation read.  No branches.  An inactive pixel (active: a
// mask) pops the whole range, which leaves the state as it is and reads nothing.  The state has at most 63 bits and freq
// 17, so the product's upper part fits a 24-bit multiplication.  A damaged stream may run past the row's words: what it
// reads there are words of another row or zeros, and the position check at the band's end reports it.
__device__ __forceinline__ void reader_pop(RowReader& rd, uint64_t& state, uint32_t start, uint32_t freq, uint32_t active) {
    const uint32_t slot = (uint32_t)state & 0xFFFFu, f = pick(active, freq, 65536u);
    uint64_t x1 = (uint64_t)(uint32_t)(state >> 16) * f + (uint64_t)(slot - (start & active));
    const uint32_t lo = (uint32_t)x1, hi = (uint32_t)(x1 >> 32) + __umul24(f, (uint32_t)(state >> 48));
    const uint32_t renorm = mask_of((((uint64_t)hi << 32) | lo) < kRansL);
    state = (uint64_t)pick(renorm, rd.w[0], lo) | ((uint64_t)pick(renorm, lo, hi) << 32);
    rd.w[0] = pick(renorm, rd.w[1], rd.w[0]);
    rd.w[1] = pick(renorm, rd.w[2], rd.w[1]);
    rd.pos -= renorm;
}

// This wave's weight slices of one layer: out-blocks ob = wave + 4 s.  Where the
// wave has no such block (ob >= NOB) it holds a copy of the layer's last block
// and its results are discarded.
// W_LDS / B_LDS: the weights / biases stay where w / b point (a copy in LDS) and are read when used.
template <int NOB, int NKB, int SLOTS, bool W_LDS, bool B_LDS>
struct WaveLayer {
    u32x4_t a[W_LDS ? 1 : SLOTS][W_LDS ? 1 : NKB];
    f32x4_t bias[B_LDS ? 1 : SLOTS];
    const uint8_t* w_at;     // + this lane's 16 bytes
    const float* b_at;       // + this lane group's four floats
    __device__ __forceinline__ void load(const uint8_t* __restrict__ w, const float* __restrict__ b, int lane, int wave) {
        if constexpr (W_LDS) w_at = w + lane * 16;
        if constexpr (B_LDS) b_at = b + 4 * (lane >> 4);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int ob = min(wave + 4 * s, NOB - 1);
            if constexpr (!B_LDS) {
                f32x4_t t = *reinterpret_cast<const f32x4_t*>(b + 16 * ob + 4 * (lane >> 4));
                asm volatile("" : "+v"(t));      // the biases start the accumulators: in the same register file as those
                bias[s] = t;
            }
            if constexpr (!W_LDS) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    u32x4_t t = *reinterpret_cast<const u32x4_t*>(w + ((ob * NKB + kb) * 64 + lane) * 16);
                    // Register allocation only: the weights, read-only MFMA operands for the whole kernel, are
                    // placed in accumulation registers, which leaves the vector registers proper to the
                    // accumulators that the vector ALU reads (no copies between the two files per block).
                    asm volatile("" : "+a"(t));
                    a[s][kb] = t;
                }
            }
        }
    }
    __device__ __forceinline__ u32x4_t A(int s, int kb, int wave) const {
        if constexpr (W_LDS) return *reinterpret_cast<const u32x4_t*>(w_at + (min(wave + 4 * s, NOB - 1) * NKB + kb) * (64 * 16));
        else return a[s][kb];
    }
    __device__ __forceinline__ f32x4_t B(int s, int wave) const {
        if constexpr (B_LDS) return *reinterpret_cast<const f32x4_t*>(b_at + 16 * min(wave + 4 * s, NOB - 1));
        else return bias[s];
    }
};

// A layer's activations in LDS: [k-block][hi, lo] in MFMA's B layout.  With bands of eight rows a tile's columns 8 to 15 are copies of
// columns 0 to 7, which are stored once, and of a block's four values in a lane the column's lane splits and stores the first
// two, its copy's lane the others.  A hand-over between layers is a chain of its own (the last block's split, its way through LDS and
// a barrier, the first read), and this halves the split (16 vector instructions to 10) and the bytes written (two 8-byte writes of
// four waves and a barrier take 136 cycles, two 4-byte ones some 85): 768x512 4,530 -> 4,317 us, and bands of eight rows pay for
// networks of three mixtures too (the paper's in 512x512 5,272 -> 4,988, 16 rows before).
template <int ROWS>
struct ActLds {
    static constexpr bool kHalved = ROWS == 8;
    static constexpr int kPartBytes = kHalved ? 32 * 16 : 64 * 16;
    __device__ __forceinline__ static int read_at(int lane) { return kHalved ? ((lane >> 4) * 8 + (lane & 7)) * 16 : lane * 16; }
    // registers i and i + 2 of a column and its copy become one register with a value each (no condition: bank_mask names the lanes)
    __device__ __forceinline__ static float share(float mine, float copys) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp((int)__float_as_uint(mine), (int)__float_as_uint(copys), 0xE4 /* quad_perm 0 1 2 3 */,
                                                                     0xF, 0xC /* lanes 8 to 15 of a row */, false));
    }
    template <bool LEAKY>
    __device__ __forceinline__ static void finish(const f32x4_t& acc, uint8_t* __restrict__ act, int ob, int lane) {
        uint32_t lo;
        const uint32_t hi = act_split_bf16<LEAKY>(share(acc.x, acc.z), share(acc.y, acc.w), lo);
        uint8_t* dst = act + (ob >> 1) * 2 * kPartBytes + read_at(lane) + 8 * (ob & 1) + ((lane & 8) >> 1);
        *reinterpret_cast<uint32_t*>(dst) = hi;
        *reinterpret_cast<uint32_t*>(dst + kPartBytes) = lo;
    }
};

// One hidden layer on this wave's out-blocks.  Same arithmetic per output element
// as EncoderNet::layers in pcc_device.h: bias, then k-blocks in order, each hi then
// lo; activation; split into hi + lo.  The out-blocks are taken one after the
// other (an accumulation chain of MFMAs issues back to back at full rate).
// In a layer's last round some waves may have no block (OWNS_LAST is false): such a wave skips the round and calls
// idle() instead, if RUN_IDLE.
template <class Act, int NOB, int NKB, int SLOTS, bool W_LDS, bool B_LDS, bool SPLIT_IN, bool LEAKY, bool ONE_BY_ONE, bool OWNS_LAST, bool RUN_IDLE,
          class Idle>
__device__ __forceinline__ void dec_hidden_layer(const WaveLayer<NOB, NKB, SLOTS, W_LDS, B_LDS>& wl, int lane, int wave,
                                                 bf16x4_bits_t minus_one, const u32x4_t (&in)[NKB][2], uint8_t* __restrict__ act_out, Idle& idle) {
    auto finish = [&](int s, const f32x4_t& acc) {
        const int ob = wave + 4 * s;
        if constexpr (Act::kHalved) {
            Act::template finish<LEAKY>(acc, act_out, ob, lane);
            return;
        }
        u32x2_t hi, lo;
        // The matrix core's subtraction saves issue slots and adds its latency to the step.  It is the faster one where two
        // workgroups share the slots (24 images of 768x512 6.30 -> 6.23 ms) and with LeakyReLU (512x512 of the paper's shape
        // 5.39 -> 5.31), the slower one for a workgroup alone with ReLU (768x512 4.69 -> 4.75).
        if constexpr (ONE_BY_ONE || LEAKY) {
            act_split4_bf16<LEAKY>(acc, minus_one, hi, lo);
        } else {
            uint32_t l0, l1;
            hi.x = act_split_bf16<LEAKY>(acc.x, acc.y, l0);
            hi.y = act_split_bf16<LEAKY>(acc.z, acc.w, l1);
            lo.x = l0; lo.y = l1;
        }
        // out-block ob is half (ob & 1) of k-block ob/2 of the next layer's operand
        uint8_t* dst = act_out + (ob >> 1) * 2 * Act::kPartBytes + lane * 16 + 8 * (ob & 1);
        *reinterpret_cast<u32x2_t*>(dst) = hi;
        *reinterpret_cast<u32x2_t*>(dst + Act::kPartBytes) = lo;
    };
    auto chain = [&](int s, f32x4_t& acc) {
        acc = wl.B(s, wave);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            const u32x4_t a = wl.A(s, kb, wave);
            acc = mfma16(a, in[kb][0], acc);
            if (SPLIT_IN) acc = mfma16(a, in[kb][1], acc);
        }
        asm volatile("" : "+v"(acc));            // register allocation only: the result where the vector ALU reads it
    };
    constexpr bool kLastShared = 4 * (SLOTS - 1) + 3 >= NOB;      // not every wave has a block in the last round
    constexpr int kBlocks = !kLastShared || OWNS_LAST ? SLOTS : SLOTS - 1;
    f32x4_t acc[SLOTS];
    if constexpr (ONE_BY_ONE) {
        // Two workgroups per CU share the matrix cores: block after block, each finished before the next begins.
#pragma unroll
        for (int s = 0; s < kBlocks; ++s) {
            chain(s, acc[s]);
            finish(s, acc[s]);
            __builtin_amdgcn_sched_barrier(0);      // the next block's instructions stay behind this one's
        }
    } else {
        // One workgroup per CU: block after block, too, but a block is finished (activation, split, store) among the MFMAs
        // of the next one: two VALU instructions issue for free beside an MFMA (16 cycles; alone it would leave 8 idle).
        // Only the last block's split is left at the end.  The first block's chain takes a k-block's input in 32 cycles,
        // the pace at which LDS delivers it to four waves.
#pragma unroll
        for (int s = 0; s < kBlocks; ++s) chain(s, acc[s]);
#pragma unroll
        for (int s = 0; s < kBlocks; ++s) finish(s, acc[s]);
        // scheduling only
#pragma unroll
        for (int i = 0; i < kBlocks * (NKB * (SPLIT_IN ? 2 : 1) + (LEAKY ? 1 : 0)); ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        }
    }
    if constexpr (kBlocks < SLOTS && RUN_IDLE) idle();
}

// ORDERED (scheduling only): the reads are issued in the order in which the MFMAs take them.  Left to itself the compiler issues
// them in another, and the first MFMA waits for the last read.  us in 512x512, before and after: the paper's network 5,320 and
// 5,265, diagonal 2,722 and 2,696, six layers 5,984 and 5,912, seven mixtures 6,222 and 6,180; 768x512 4,558 and 4,527.  With five
// k-blocks as well 768x512 takes 4,565: those are left to the compiler.  With two workgroups per CU fewer registers are live at a time:
// the paper's network spills 2 instead of 16 and 24 images of 768x512 take 7,360 us instead of 7,485, diagonal 6 for 25 and 5,050 for 5,140.
template <class Act, int NKB, bool ORDERED>
__device__ __forceinline__ void dec_load_act(const uint8_t* __restrict__ act, int lane, u32x4_t (&in)[NKB][2]) {
    act += Act::read_at(lane);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        in[kb][0] = *reinterpret_cast<const u32x4_t*>(act + (kb * 2 + 0) * Act::kPartBytes);
        if constexpr (ORDERED) __builtin_amdgcn_sched_barrier(0);
        in[kb][1] = *reinterpret_cast<const u32x4_t*>(act + (kb * 2 + 1) * Act::kPartBytes);
        if constexpr (ORDERED) __builtin_amdgcn_sched_barrier(0);
    }
}

// The whole network as seen by one wave: its weight slices of layers L .. last, and
// the per-step evaluation that hands activations from layer to layer through LDS
// (hidden layer l writes activation buffer l & 1).  Ends behind a barrier with the
// raw head outputs in `headout`.
// SHARED: the workgroup shares its CU with another (see DecLds): `lds` then holds the pieces kept there.
template <class Net, bool SHARED, int L, bool END = (L == Net::kLayers)>
struct WaveNet {
    static constexpr int NOB = Net::ob(L), NKB = Net::kb(L), SLOTS = (NOB + 3) / 4;
    static constexpr bool kHead = L == Net::kLayers - 1;
    static constexpr bool kWLds = SHARED && ((L == 0 && DecLds<Net>::kFirstInLds) || (kHead && DecLds<Net>::kHeadInLds));
    static constexpr bool kBLds = SHARED && DecLds<Net>::kBiasInLds;
    WaveLayer<NOB, NKB, SLOTS, kWLds, kBLds> wl;
    WaveNet<Net, SHARED, L + 1> rest;

    __device__ __forceinline__ void load(const uint8_t* __restrict__ model, const uint8_t* __restrict__ lds, int lane, int wave) {
        using Lay = Layout<Net>;
        using D = DecLds<Net>;
        const uint8_t* w = kWLds ? lds + (L == 0 ? D::kFirstOff : D::kHeadWOff) : model + Lay::w_off(L);
        const uint8_t* b = kBLds ? lds + D::kBiasOff + (Lay::b_off(L) - Lay::kWeightBytes) : model + Lay::b_off(L);
        wl.load(w, reinterpret_cast<const float*>(b), lane, wave);
        rest.load(model, lds, lane, wave);
    }
    // OWNS_LAST: has this wave a block in the last round of the layers whose block count is no multiple of four?  (The
    // same waves have in all of them: DecLds::same_waves_idle.)  idle: what a wave that has none does in its place.
    // settle: work of every wave that nothing waits for before the searches, in parts for the layers; it goes between the
    // MFMAs.
    template <class Act, bool OWNS_LAST, class Idle, class Settle, class Awake>
    __device__ __forceinline__ void run(const u32x4_t (&in)[NKB][2], int lane, int wave, bf16x4_bits_t minus_one, uint8_t* __restrict__ act0, uint8_t* __restrict__ act1,
                                        float* __restrict__ headout, Idle& idle, Settle& settle, Awake& awake, PhaseClock& clk) const {
        // what waves without an out-block in this layer's last round do instead (decode_kernel says what)
        constexpr bool kRunIdle = DecLds<Net>::kIdleSlack > 0 &&
                                  (L == DecLds<Net>::kIdleLayer || (L == 0 && DecLds<Net>::kIdleInFirstLayer));
        auto idle_here = [&]() __attribute__((always_inline)) { idle(std::integral_constant<int, L>()); };
        if constexpr (kHead) {
            // registers s = 4 ob + i of group g, kept in (group, register) order; out-blocks ob = wave + 4 slot
            constexpr int HS = Layout<Net>::kHeadSlots;
            constexpr int kBlocks = 4 * (SLOTS - 1) + 3 < NOB || OWNS_LAST ? SLOTS : SLOTS - 1;
#pragma unroll
            for (int slot = 0; slot < kBlocks; ++slot) {
                f32x4_t acc = wl.B(slot, wave);
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    const u32x4_t a = wl.A(slot, kb, wave);
                    acc = mfma16(a, in[kb][0], acc);
                    acc = mfma16(a, in[kb][1], acc);
                }
                const int ob = wave + 4 * slot;
                if constexpr (Act::kHalved) {
                    const f32x2_t half = {Act::share(acc.x, acc.z), Act::share(acc.y, acc.w)};
                    *reinterpret_cast<f32x2_t*>(headout + (lane & 7) * DecLds<Net>::kHeadStride + (lane >> 4) * HS + 4 * ob + ((lane & 8) >> 2)) = half;
                } else {
                    *reinterpret_cast<f32x4_t*>(headout + (lane & 15) * DecLds<Net>::kHeadStride + (lane >> 4) * HS + 4 * ob) = acc;
                }
                if constexpr (SHARED) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (kBlocks < SLOTS && kRunIdle) idle_here();
            settle(std::integral_constant<int, L>());
            lds_barrier();
            clk.mark(kPhLayer0 + L);
        } else {
            uint8_t* out = (L & 1) ? act1 : act0;
            settle(std::integral_constant<int, L>());
            dec_hidden_layer<Act, NOB, NKB, SLOTS, kWLds, kBLds, (L > 0), Net::kLeaky, SHARED, OWNS_LAST, kRunIdle>(wl, lane, wave, minus_one, in, out,
                                                                                                               idle_here);
            awake.template keep<Awake::kBehindWrite>();
            lds_barrier();
            clk.mark(kPhLayer0 + L);
            u32x4_t nxt[Net::kb(L + 1)][2];
            dec_load_act<Act, Net::kb(L + 1), Net::kb(L + 1) <= 4>(out, lane, nxt);
            // scheduling only: every read of the layer's input is issued before its first MFMA, so
            // the LDS latency is paid once per layer and not once per k-block.  With two workgroups per CU the other one
            // hides the latency, and the registers of 40 values are better spent otherwise (24 images 7.23 -> 7.06 ms).
            if constexpr (!SHARED) __builtin_amdgcn_sched_barrier(0);
            rest.template run<Act, OWNS_LAST>(nxt, lane, wave, minus_one, act0, act1, headout, idle, settle, awake, clk);
        }
    }
};
template <class Net, bool SHARED, int L>
struct WaveNet<Net, SHARED, L, true> {
    __device__ __forceinline__ void load(const uint8_t* __restrict__, const uint8_t* __restrict__, int, int) {}
};

// Symbol search by the lanes of one pixel: two sweeps of 16 evaluations, Cq(16 e) and, in the
// block b found, Cq(16 b + e), e = 0..15.  The search compares 65280 F(edge) with slot + 1 - e in floating point, both exact:
// floor(v) + e <= slot exactly when v < slot + 1 - e.  Edge 0 always passes (Cq(0) = 0; in the second sweep Cq(16 b)
// is known to pass): its lanes' constants are minus infinity.  What the symbol's interval needs is left in `found`, for
// group_interval, which is off the path from symbol to symbol.
// With 32 lanes to a pixel two rows of 16 lanes share an edge's components: the first row looks up the first kPartK of them and
// sums them, the second row looks up the others meanwhile and goes on with the first row's sum, so that the sum is made in
// the order of the components as everywhere; what a sweep finds is in the second row.  A vector instruction in a search costs more
// than its 4 cycles: behind a look-up's wait the first ten of each wave take 14 (Awake).  So the forms with fewest of them: plain copies of the table instead of spread entries (one a look-up),
// no copy of the sum before the lane swap, and rows without sums that never pass instead of a mask on the ballot: 768x512 4,318 -> 4,210 us,
// the paper's network in 512x512 4,987 -> 4,899.
struct SearchLane {            // a lane's constants
    float edge1, edge2;        // (2 (16 e) - 1) / 512 and (2 e - 1) / 512
    float e1, e2;              // 16 e and e; minus infinity for e = 0; infinity in lanes that have no sums
    int e, shift;              // the lane's edge; position in a ballot of the pixel's lanes
    int base4;                 // 4 x first lane of that row
    uint32_t table;            // LDS address of the table's copy that the lane reads (Table::kCopies)
};
struct Found {
    uint32_t next1;            // Cq(16 e + 16), 65536 for e = 15
    uint32_t c2;               // Cq(16 b + e), but for b = e = 0
    int b, count, x;           // block, edges that passed in the second sweep, the symbol 16 b + count - 1
};

// Scheduling only: the fractions are computed here.
template <int K>
__device__ __forceinline__ void pin(CqLookup<K>& q) {
#pragma unroll
    for (int k = 0; k < K; ++k) asm volatile("" : "+v"(q.t[k]));
}

// cq_scaled for components that two rows share: K in all, the lane's are PK (the first row's) or the K - PK behind them.
template <int K, int PK>
__device__ __forceinline__ float cq_scaled_shared(const ChanParams<PK>& cp, CqLookup<PK>& q) {
    float2 (&td)[PK] = q.td;
    // Scheduling only: all table reads are in flight before the first is used.
    if constexpr (PK == 4) {
        asm volatile("" : "+v"(td[0].x), "+v"(td[0].y), "+v"(td[1].x), "+v"(td[1].y), "+v"(td[2].x), "+v"(td[2].y), "+v"(td[3].x), "+v"(td[3].y));
    } else if constexpr (PK == 3) {
        asm volatile("" : "+v"(td[0].x), "+v"(td[0].y), "+v"(td[1].x), "+v"(td[1].y), "+v"(td[2].x), "+v"(td[2].y));
    } else {
        static_assert(PK == 2, "three, five or seven components");
        asm volatile("" : "+v"(td[0].x), "+v"(td[0].y), "+v"(td[1].x), "+v"(td[1].y));
    }
    float acc = 0.0f, phi[PK];
#pragma unroll
    for (int k = 0; k < PK; ++k) {
        phi[k] = __builtin_fmaf(q.t[k], td[k].y, td[k].x);
        acc = __builtin_fmaf(cp.pi[k], phi[k], acc);
    }
    // the first row's sum in the second row (the first row goes on with anything: its lanes never pass, SearchLane::e1)
    uint32_t any;
    asm("" : "=v"(any));
    const u32x2_t swapped = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane16_swap(any, __float_as_uint(acc), false, false));
    acc = __uint_as_float(swapped.x);
#pragma unroll
    for (int k = 0; k < K - PK; ++k) acc = __builtin_fmaf(cp.pi[k], phi[k], acc);
    return fminf(acc, 1.0f) * 65280.0f;
}

// during1(), during2(): called when a sweep's table reads are issued; memory requests made there queue behind them.
// K components in all, PK of them (or the rest) the lane's own.
template <int K, int PK, class During1, class During2>
__device__ __forceinline__ int group_search(const ChanParams<PK>& cp, float slot1, const float2* __restrict__ lut, const SearchLane& sl,
                                            Found& found, During1&& during1, During2&& during2) {
    auto scaled = [&](CqLookup<PK>& q) __attribute__((always_inline)) {
        if constexpr (PK < K) return cq_scaled_shared<K, PK>(cp, q);
        else return cq_scaled<K>(cp, q);
    };
    constexpr bool kShared = PK < K;            // two rows share an edge's components
    constexpr Table kTable = kShared ? Table::kCopies : Table::kSpread;
    // the edges of the pixel that have passed
    auto passed = [&](bool pass) __attribute__((always_inline)) {
        const uint64_t all = __ballot(pass) >> sl.shift;
        return kShared ? __popc((uint32_t)all) : __popcll(all & 0xFFFFull);
    };
    CqLookup<PK> q1, q2;
    cq_lookup<PK, kTable>(cp, sl.edge1, lut, q1, sl.table);
    __builtin_amdgcn_sched_barrier(0);       // scheduling only: the table reads first, then what they leave time for
    during1();
    cq_fractions<PK>(q1);
    float limit1 = slot1 - sl.e1;
    asm volatile("" : "+v"(limit1) :: "memory");
    pin<PK>(q1);
    const float v1 = scaled(q1);
    const int b = passed(v1 < limit1) - 1;
    const float bf = (float)b;
    cq_lookup<PK, kTable>(cp, __builtin_fmaf(bf, 1.0f / 16.0f, sl.edge2), lut, q2, sl.table);
    __builtin_amdgcn_sched_barrier(0);
    during2();
    cq_fractions<PK>(q2);
    float limit2 = __builtin_fmaf(bf, -16.0f, slot1 - sl.e2);
    found.next1 = (uint32_t)__builtin_amdgcn_update_dpp(65536, (int)((uint32_t)v1 + 16u * (uint32_t)sl.e), 0x101 /* row_shl:1 */,
                                                        0xF, 0xF, false);
    int first = 16 * b - 1;
    asm volatile("" : "+v"(limit2), "+v"(found.next1), "+v"(first) :: "memory");
    pin<PK>(q2);
    const float v2 = scaled(q2);
    found.count = passed(v2 < limit2);
    found.b = b;
    found.x = first + found.count;
    found.c2 = (uint32_t)v2 + (uint32_t)(first + 1 + sl.e);
    return found.x;
}

// Cq(x) and Cq(x + 1) - Cq(x), picked from the lanes that evaluated them, in three parts that can stand apart: two
// lane picks, one that needs the first's result, and the interval.
struct Interval { uint32_t up, lower, upper; };
__device__ __forceinline__ void interval_pick(const Found& f, const SearchLane& sl, Interval& v) {
    v.up = (uint32_t)__builtin_amdgcn_ds_bpermute(sl.base4 + 4 * f.b, (int)f.next1);                   // Cq(16 b + 16)
    v.lower = (uint32_t)__builtin_amdgcn_ds_bpermute(sl.base4 + 4 * f.count - 4, (int)f.c2);
}
__device__ __forceinline__ void interval_pick_upper(const Found& f, const SearchLane& sl, Interval& v) {
    // edge 0 is nobody's upper end: it stands in for the block's end
    v.upper = (uint32_t)__builtin_amdgcn_ds_bpermute(sl.base4 + 4 * (f.count & 15), (int)(sl.e == 0 ? v.up : f.c2));
}
__device__ __forceinline__ void interval_of(const Found& f, const Interval& v, uint32_t& start, uint32_t& freq) {
    start = f.x == 0 ? 0u : v.lower;
    freq = v.upper - start;
}

// N consecutive floats (N <= 16) from a 16-byte aligned LDS address, as whole vector reads.
template <int N>
__device__ __forceinline__ void lds_read_floats(const float* __restrict__ src, float (&dst)[N]) {
    constexpr int NV = (N + 3) / 4;
    f32x4_t v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = reinterpret_cast<const f32x4_t*>(src)[i];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const f32x4_t q = v[i >> 2];
        dst[i] = (i & 3) == 0 ? q.x : (i & 3) == 1 ? q.y : (i & 3) == 2 ? q.z : q.w;
    }
}

// What a wave of the decoder does besides its blocks: fetch the rows above the band, store decoded pixels (to the image
// and for the band below); and whether it has a block in the last round of layers that do not fill it.
template <bool FETCHES, bool STORES, bool OWNS_LAST>
struct StepRole {
    static constexpr bool kFetches = FETCHES, kStores = STORES, kOwnsLast = OWNS_LAST;
};

// MINBLOCKS = 1: all registers to one workgroup per CU (lowest latency per step).  MINBLOCKS = 2: two
// workgroups share a CU (some spills; a step takes Net::kSharedAlonePercent to Net::kSharedStepPercent of the time, so
// this only pays for jobs of so many bands that the work per CU, not an image's chain of steps, sets the time: choose_decode).
// ROWS = 16: 16 lanes to a pixel.  ROWS = 8 (half of a tile's columns are copies): 32 lanes, which share the mixture components
// in two halves, and half the pixels to a wave, so that the searches, more than half of a step's instructions, have a fifth
// fewer of them (437 -> 349 vector instructions with five components); and a column and its copy share the activation split (ActLds).
template <class Net, int MINBLOCKS>
__global__ void __launch_bounds__(kDecThreads, MINBLOCKS)
decode_kernel(const uint8_t* __restrict__ model, const uint8_t* __restrict__ stream, uint64_t nbytes, int n, int H,
              int W, int nbands, uint32_t dist, uint8_t* __restrict__ img_out, uint32_t* mailbox, int* status,
              uint32_t spin_limit) {
    constexpr int ROWS = kBandRows;
#include "decode_bands.h"
}
template <class Net>
__global__ void __launch_bounds__(kDecThreads, 1)
decode_narrow_kernel(const uint8_t* __restrict__ model, const uint8_t* __restrict__ stream, uint64_t nbytes, int n, int H,
                     int W, int nbands, uint32_t dist, uint8_t* __restrict__ img_out, uint32_t* mailbox, int* status,
                     uint32_t spin_limit) {
    constexpr int MINBLOCKS = 1, ROWS = kNarrowRows;
#include "decode_bands.h"
}

// ---------------------------------------------------------------------------
// test hook: full tables from given head outputs
// ---------------------------------------------------------------------------
template <class Net>
__global__ void __launch_bounds__(256)
cdf_tables_kernel(const uint8_t* __restrict__ model, const float* __restrict__ params, const uint8_t* __restrict__ rg,
                  size_t count, uint32_t* __restrict__ cq) {
    constexpr int K = Net::K, HEAD = Net::dim(Net::kLayers);
    extern __shared__ __align__(16) uint8_t lds[];
    float2* lut = reinterpret_cast<float2*>(lds);
    const float2* src = reinterpret_cast<const float2*>(model + Layout<Net>::kLutOff);
    for (int i = threadIdx.x; i < kLutEntries + 1; i += blockDim.x) lut[i] = src[i];
    __syncthreads();
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= count * 3) return;
    const size_t p = idx / 3;
    const int ch = (int)(idx - p * 3);
    const float* o = params + p * HEAD;
    float raw[3 * K];
    for (int s = 0; s < 3 * K; ++s) raw[s] = s < 2 * K ? o[3 * K * ch + s] : __builtin_canonicalizef(o[3 * K * ch + s]);     // clamp_log_sigma
    ChanParams<K> cp;
    channel_setup<K>(raw, *reinterpret_cast<const float*>(model + Layout<Net>::kLutScaleOff), cp);
    const float rhat = (float)rg[2 * p] * (1.0f / 256.0f), ghat = (float)rg[2 * p + 1] * (1.0f / 256.0f);
    float c1[K], c2[K];
    for (int k = 0; k < K; ++k) { c1[k] = ch == 1 ? o[9 * K + k] : o[10 * K + k]; c2[k] = o[11 * K + k]; }
    if (ch == 1) couple_green<K>(cp, c1, rhat);
    if (ch == 2) couple_blue<K>(cp, c1, c2, rhat, ghat);
    uint32_t* dst = cq + idx * 257;
    for (int e = 0; e <= 256; ++e) dst[e] = cq_full<K>(cp, e, lut);
}

// ---------------------------------------------------------------------------
// pcc_decode_static: the decoder's mailbox in an array that is part of the loaded code object, so that the call
// allocates nothing.  Each GPU the library runs on holds its own copy at its own address (resolved once per device,
// see static_scratch()); host code never uses the array's name for anything but that resolution.
// ---------------------------------------------------------------------------
constexpr size_t kStaticScratchBytes = PCC_STATIC_SCRATCH_BYTES;

// Zero `count` 32-bit words (a kernel rather than a memset node: a caller may be capturing the stream).
__global__ void __launch_bounds__(256)
clear_words_kernel(uint32_t* __restrict__ dst, size_t count) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) dst[i] = 0u;
}

}  // namespace pcc

static __device__ __align__(256) uint32_t scratch[pcc::kStaticScratchBytes / 4];

// ===========================================================================
// host side
// ===========================================================================
using namespace pcc;

enum { kNetWorkload = 0, kNetPaper = 1, kNetDiagonal = 2, kNetFewerLayers = 3, kNetFewerFilters = 4, kNetMoreMixtures = 5, kNetMostMixtures = 6, kNetMoreLayers = 7, kNetMoreFilters = 8 };

struct pcc_ctx {
    int device = 0;
    int net = kNetWorkload;        // which network description the blob matched
    uint8_t* d_model = nullptr;
    // workspace (grown on demand)
    uint8_t* d_ws = nullptr;
    size_t ws_bytes = 0;
    int* d_status = nullptr;       // the status blocks, and the encoder's stream size behind them
    uint64_t* d_total = nullptr;
    uint64_t* d_sums = nullptr;    // behind it: words of the row coder's groups, tagged with the epoch
    int* h_status = nullptr;       // pinned: the decoder's block after a call, the encoder's result behind it
    EncodeResult* h_result = nullptr;
    EncodeResult* d_result = nullptr;         // the same, as kernels see it
    int* status(int block) const { return d_status + block * kStWords; }
    // layout of the last encode inside the workspace
    uint32_t* d_sf = nullptr;
    size_t sf_count = 0;
    int num_cus = 0;
    uint32_t* d_static_scratch = nullptr;   // this device's copy of the static scratch array (pcc_decode_static)
    uint32_t dist = 0;             // written to / checked against stream header word 6
    uint32_t spin_limit = 1u << 22;      // polls of a band for one pixel of the band above (seconds) before the call fails (PCC_DECODE_SPIN_LIMIT, for tests)
    int decode_variant = 0;              // 0: chosen per job; 1: one workgroup per CU; 2: two; 3: one, bands of eight rows (PCC_DECODE_VARIANT, for measurements)
    // the row coder of a small job runs beside the pixel kernel, on a stream of its own
    bool overlap = true;
    uint32_t patience = kRansPatience;        // polls for a symbol before a row coder beside the pixel kernel stands down
    uint32_t sums_patience = 4 * kRansPatience;      // ... and for the words of its groups before (shorter polls: some 10 ms)
    hipStream_t side = nullptr;
    hipEvent_t ev_joined = nullptr;           // the pixel kernel's first part is done: the row coder may join
    // symbols handed from the pixel kernel to a row coder running beside it: epoch << 32 | start | (freq - 1) << 16.
    // Zero when allocated and written by nothing else, so a word carries an epoch only if that launch wrote it.
    uint64_t* d_tagged = nullptr;
    size_t tagged_count = 0;
    uint32_t epoch = 0;               // of the last launch that wrote d_tagged
    bool last_tagged = false;         // the last encode left its symbols in d_tagged, not in d_sf
    // optional per-kernel timing
    bool profiling = false;
    hipEvent_t ev[2 * PCC_N_TIMINGS] = {};
    bool ev_used[PCC_N_TIMINGS] = {};
    float last_ms[PCC_N_TIMINGS] = {};
};

namespace {

inline uint32_t rd32(const uint8_t* p) {
    return (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16) | ((uint32_t)p[3] << 24);
}
inline float rdf(const uint8_t* p) { uint32_t u = rd32(p); float f; memcpy(&f, &u, 4); return f; }

// fp32 -> bf16 bits, exact values only (caller has checked representability)
inline bool bf16_exact(float f, uint16_t* out) {
    uint32_t u; memcpy(&u, &f, 4);
    *out = (uint16_t)(u >> 16);
    return (u & 0xFFFFu) == 0u;
}

struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) return;
        ok = hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard() { if (prev >= 0) (void)hipSetDevice(prev); }
};

int ensure_workspace(pcc_ctx* ctx, size_t bytes) {
    if (bytes <= ctx->ws_bytes) return PCC_OK;
    if (ctx->d_ws) { (void)hipFree(ctx->d_ws); ctx->d_ws = nullptr; ctx->ws_bytes = 0; }
    ctx->d_sf = nullptr; ctx->sf_count = 0;
    const size_t want = bytes + bytes / 8 + 4096;
    if (hipMalloc((void**)&ctx->d_ws, want) != hipSuccess) { (void)hipGetLastError(); return PCC_E_HIP; }
    ctx->ws_bytes = want;
    return PCC_OK;
}

// Zeros in all of d_tagged, waited for: neither the caller's stream, where the pixel kernel writes it, nor the context's, where the
// row coder reads it, is ordered after the null stream, whose hipMemset returns before it has begun.  A late one wiped
// symbols that had been written, and until then a row coder could find those of a freed context with its own epoch.  (A context's
// first encode takes 10 us longer for the wait, with an event for the second stream in its place or a kernel that clears as well.)
int clear_tagged(pcc_ctx* ctx, hipStream_t st) {
    if (hipMemsetAsync(ctx->d_tagged, 0, ctx->tagged_count * sizeof(uint64_t), st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess) {
        (void)hipGetLastError();
        return PCC_E_HIP;
    }
    return PCC_OK;
}

// `st` is idle.
int ensure_tagged(pcc_ctx* ctx, size_t count, hipStream_t st) {
    if (count <= ctx->tagged_count) return PCC_OK;
    if (ctx->d_tagged) { (void)hipFree(ctx->d_tagged); ctx->d_tagged = nullptr; ctx->tagged_count = 0; }
    const size_t want = count + count / 8 + 512;
    if (hipMalloc((void**)&ctx->d_tagged, want * sizeof(uint64_t)) != hipSuccess) { (void)hipGetLastError(); return PCC_E_HIP; }
    ctx->tagged_count = want;
    const int rc = clear_tagged(ctx, st);
    if (rc != PCC_OK) ctx->tagged_count = 0;
    return rc;
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Device address of this GPU's copy of `scratch`, resolved once per device with that device current (the caller
// holds a DeviceGuard).  nullptr if the runtime cannot resolve it.
constexpr int kMaxDevices = 64;
uint32_t* static_scratch(int device) {
    static std::mutex mu;
    static uint32_t* ptr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        ptr[device] = static_cast<uint32_t*>(p);
    }
    return ptr[device];
}

inline void prof_reset(pcc_ctx* ctx) {
    for (int i = 0; i < PCC_N_TIMINGS; ++i) { ctx->ev_used[i] = false; ctx->last_ms[i] = 0.0f; }
}
inline void prof_begin(pcc_ctx* ctx, int which, hipStream_t st) {
    if (ctx->profiling) (void)hipEventRecord(ctx->ev[2 * which], st);
}
inline void prof_end(pcc_ctx* ctx, int which, hipStream_t st) {
    if (ctx->profiling) { (void)hipEventRecord(ctx->ev[2 * which + 1], st); ctx->ev_used[which] = true; }
}
// after the stream has been synchronised
inline void prof_collect(pcc_ctx* ctx) {
    if (!ctx->profiling) return;
    for (int i = 0; i < PCC_N_TIMINGS; ++i)
        if (ctx->ev_used[i] && hipEventElapsedTime(&ctx->last_ms[i], ctx->ev[2 * i], ctx->ev[2 * i + 1]) != hipSuccess) {
            (void)hipGetLastError();
            ctx->last_ms[i] = 0.0f;
        }
}

bool dims_ok(int n, int H, int W) {
    if (n < 1 || H < 1 || W < 1) return false;
    const uint64_t P = (uint64_t)n * H * W;
    return P < (1ull << 31) && (uint64_t)W < (1u << 24) && (uint64_t)n * H < (1ull << 31) &&
           (uint64_t)H * W * 3 < (1ull << 31);   // byte offsets within one image are 32-bit
}

// Calls f with a value of the network description type that `net` names.
template <class F>
auto with_net(int net, F&& f) {
    switch (net) {
        case kNetPaper: return f(NetPaper{});
        case kNetDiagonal: return f(NetDiagonal{});
        case kNetFewerLayers: return f(NetFewerLayers{});
        case kNetFewerFilters: return f(NetFewerFilters{});
        case kNetMoreMixtures: return f(NetMoreMixtures{});
        case kNetMostMixtures: return f(NetMostMixtures{});
        case kNetMoreLayers: return f(NetMoreLayers{});
        case kNetMoreFilters: return f(NetMoreFilters{});
        default: return f(NetWorkload{});
    }
}

// Does the blob header describe network Net?  (activation id 0 = ReLU, 1 = LeakyReLU 0.01)
template <class Net>
bool header_matches(const uint8_t* p) {
    if (rd32(p + 8) != (uint32_t)Net::kLayers) return false;
    for (int i = 0; i < 8; ++i)
        if (rd32(p + 12 + 4 * i) != (i <= Net::kLayers ? (uint32_t)Net::dim(i) : 0u)) return false;
    return rd32(p + 44) == (uint32_t)Net::K && rd32(p + 48) == (uint32_t)Net::kNbhd &&
           rd32(p + 52) == (uint32_t)Net::kDelay && rd32(p + 56) == (Net::kLeaky ? 1u : 0u);
}

// Weights and biases of the blob -> MFMA operand tiles in the order the kernels read them.
template <class Net>
int pack_model(const uint8_t* p, size_t blob_bytes, uint32_t dist, std::vector<uint8_t>& image) {
    using Lay = Layout<Net>;
    constexpr int NL = Net::kLayers;
    size_t need = 64;
    for (int l = 0; l < NL; ++l) need += 4 * ((size_t)Net::dim(l) * Net::dim(l + 1) + Net::dim(l + 1));
    if (blob_bytes != need) return PCC_E_BLOB;
    const uint8_t* wsrc[NL];
    const uint8_t* bsrc[NL];
    const uint8_t* q = p + 64;
    for (int l = 0; l < NL; ++l) {
        wsrc[l] = q; q += 4 * (size_t)Net::dim(l) * Net::dim(l + 1);
        bsrc[l] = q; q += 4 * (size_t)Net::dim(l + 1);
    }
    auto Wat = [&](int l, int o, int i) { return rdf(wsrc[l] + 4 * ((size_t)o * Net::dim(l) + i)); };
    auto Bat = [&](int l, int o) { return rdf(bsrc[l] + 4 * (size_t)o); };

    // the decoder's image; behind it, with the head's rows in other orders, the encoder's and, where it has its own, that of the decoder
    // with two workgroups per unit
    image.assign((Net::kSharedByCoefficient ? 3 : 2) * Lay::kModelBytes, 0);
    uint16_t* w16 = reinterpret_cast<uint16_t*>(image.data());
    for (int l = 0; l < NL; ++l) {
        const int nob = Net::ob(l), nkb = Net::kb(l);
        const bool head = l == NL - 1;
        for (int ob = 0; ob < nob; ++ob)
            for (int kb = 0; kb < nkb; ++kb)
                for (int lane = 0; lane < 64; ++lane)
                    for (int i = 0; i < 8; ++i) {
                        const int m = lane & 15, g = lane >> 4;
                        // output feature of A row m of this out-block
                        const int o = head ? Net::head_index(m >> 2, 4 * ob + (m & 3)) : 16 * ob + m;
                        // input feature of k-slot (g, i) of this k-block
                        const int in = l == 0 ? Net::in_index(kb, g, i) : 32 * kb + kslot_feature(g, i);
                        float v = 0.0f;
                        if (o >= 0 && o < Net::dim(l + 1) && in >= 0 && in < Net::dim(l)) v = Wat(l, o, in);
                        uint16_t h;
                        if (!bf16_exact(v, &h)) return PCC_E_BLOB;
                        if (l == 0 && v != 0.0f) {
                            // fold the 1/256 input scaling into the first layer: exact unless it underflows
                            const float s = v * (1.0f / 256.0f);
                            if (!bf16_exact(s, &h) || s * 256.0f != v) return PCC_E_BLOB;
                        }
                        w16[(Lay::w_off(l) + (((ob * nkb + kb) * 64 + lane) * 16)) / 2 + i] = h;
                    }
        float* b = reinterpret_cast<float*>(image.data() + Lay::b_off(l));
        for (int s = 0; s < 16 * nob; ++s) {
            const int ob = s >> 4, m = s & 15;
            const int o = head ? Net::head_index(m >> 2, 4 * ob + (m & 3)) : s;
            b[s] = (o >= 0 && o < Net::dim(l + 1)) ? Bat(l, o) : 0.0f;
        }
    }
    // Component CDF table in units of 2^-24 so that forward differences are exact in fp32.
    float* lut = reinterpret_cast<float*>(image.data() + Lay::kLutOff);
    const double lut_scale = dist == 0 ? (double)kLutScaleGaussian : (double)kLutScaleLogistic;
    *reinterpret_cast<float*>(image.data() + Lay::kLutScaleOff) = (float)lut_scale;
    std::vector<double> tq(kLutEntries + 1);
    for (int i = 0; i < kLutEntries; ++i) {
        const double z = (i - 768) / lut_scale;
        const double F = dist == 0 ? 0.5 * erfc(-z / sqrt(2.0)) : 1.0 / (1.0 + exp(-z));
        tq[i] = nearbyint(F * 16777216.0);
    }
    tq[0] = 0.0;
    tq[kLutEntries - 1] = 16777216.0;
    tq[kLutEntries] = tq[kLutEntries - 1];
    for (int i = 0; i < kLutEntries; ++i) {
        lut[2 * i] = (float)(tq[i] / 16777216.0);
        lut[2 * i + 1] = (float)((tq[i + 1] - tq[i]) / 16777216.0);
    }
    lut[2 * kLutEntries] = 1.0f;
    lut[2 * kLutEntries + 1] = 0.0f;

    // head_index(g, s): canonical output in register s of lane group g, or -1
    constexpr int kHead = NL - 1;
    auto reordered = [&](uint8_t* copy, auto head_index) {
        memcpy(copy, image.data(), Lay::kModelBytes);
        for (int s = 0; s < 16 * Net::ob(kHead); ++s) {
            const int ob = s >> 4, m = s & 15, c = head_index(m >> 2, 4 * ob + (m & 3));
            // the row of the first image's head that holds this output, or one that holds none
            int from = -1;
            for (int k = 0; k < 16 * Net::ob(kHead); ++k) if (Net::head_index((k & 15) >> 2, 4 * (k >> 4) + (k & 3)) == c) from = k;
            for (int kb = 0; kb < Net::kb(kHead); ++kb)
                for (int g = 0; g < 4; ++g) {
                    uint8_t* to = copy + Lay::w_off(kHead) + ((ob * Net::kb(kHead) + kb) * 64 + 16 * g + m) * 16;
                    if (c < 0) memset(to, 0, 16);
                    else memcpy(to, image.data() + Lay::w_off(kHead) + (((from >> 4) * Net::kb(kHead) + kb) * 64 + 16 * g + (from & 15)) * 16, 16);
                }
            if (c < 0) memset(copy + Lay::b_off(kHead) + 4 * s, 0, 4);
            else memcpy(copy + Lay::b_off(kHead) + 4 * s, image.data() + Lay::b_off(kHead) + 4 * from, 4);
        }
    };
    reordered(image.data() + Lay::kModelBytes, [](int g, int s) { return EncHead<Net>::head_index(g, s); });
    if constexpr (Net::kSharedByCoefficient)
        reordered(image.data() + 2 * Lay::kModelBytes, [](int g, int s) { return SharedHead<Net>::head_index(g, s); });
    return PCC_OK;
}

template <class Net>
bool set_kernel_attributes() {
    constexpr int enc = encode_model_lds_bytes<Net>() + kTakenBytes + params_stage_bytes<Net>(), dec = DecLds<Net>::kBytes,
                  narrow = DecLds<Net, kNarrowRows>::kBytes;
    static_assert(enc <= kLdsBytes && dec <= kLdsBytes && narrow <= kLdsBytes && DecLds<Net>::kBytesShared <= kLdsBytes,
                  "the network does not fit a compute unit's LDS");
    bool ok = true;
    ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(&encode_kernel<Net>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, enc) == hipSuccess;
    ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_kernel<Net, 1>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, dec) == hipSuccess;
    ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_kernel<Net, 2>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, DecLds<Net>::kBytesShared) == hipSuccess;
    ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_narrow_kernel<Net>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, narrow) == hipSuccess;
    // The decoders read the CDF table, or its copies, from LDS address 0 on (cq_lookup, Table::kSpread and kCopies): their dynamic
    // array must begin there, that is, they must have no static one in front of it.
    static_assert(DecLds<Net>::kLutOff == 0 && DecLds<Net, kNarrowRows>::kLutOff == 0, "the table's LDS address is a literal in cq_lookup");
    const void* const decoders[] = {reinterpret_cast<const void*>(&decode_kernel<Net, 1>), reinterpret_cast<const void*>(&decode_kernel<Net, 2>),
                                    reinterpret_cast<const void*>(&decode_narrow_kernel<Net>)};
    for (const void* decoder : decoders) {
        hipFuncAttributes attr;
        ok = ok && hipFuncGetAttributes(&attr, decoder) == hipSuccess && attr.sharedSizeBytes == 0;
    }
    return ok;
}

uint32_t encode_strips(int W) { return ((uint32_t)W + kStripPixels - 1) / kStripPixels; }

// Workgroups of the pixel kernel.  reserve_cus: compute units left free for a kernel that runs beside it.
uint32_t encode_blocks(const pcc_ctx* ctx, int n, int H, uint32_t strips, uint32_t reserve_cus) {
    const uint64_t items = (uint64_t)strips * (uint64_t)n * H;          // dims_ok: below 2^31
    const uint32_t cus = (ctx->num_cus > 0 ? (uint32_t)ctx->num_cus : 256u) - reserve_cus;
    return items > cus ? cus : (uint32_t)items;     // persistent: one workgroup per CU, whose waves take its items
}

// sf_tagged: see encode_kernel
template <class Net>
int launch_encode(pcc_ctx* ctx, const uint8_t* d_img, int n, int H, int W, uint32_t* sf, float* params, float* bits,
                  uint64_t* sf_tagged, uint32_t reserve_cus, uint32_t strip_begin, uint32_t strip_count, hipStream_t st) {
    const int lds = encode_model_lds_bytes<Net>() + kTakenBytes + (params != nullptr ? params_stage_bytes<Net>() : 0);
    const uint32_t blocks = encode_blocks(ctx, n, H, strip_count, reserve_cus);
    const uint8_t* model = ctx->d_model + Layout<Net>::kModelBytes;
    hipLaunchKernelGGL((encode_kernel<Net>), dim3(blocks), dim3(Net::kEncodeThreads), lds, st, model, d_img, n, H, W,
                       sf, params, bits, ctx->status(params != nullptr ? kBlockProbs : kBlockEncode), sf_tagged, ctx->epoch, strip_begin, strip_count);
    return hipGetLastError() == hipSuccess ? PCC_OK : PCC_E_HIP;
}

int launch_encode_any(pcc_ctx* ctx, const uint8_t* d_img, int n, int H, int W, uint32_t* sf, float* params, float* bits,
                      uint64_t* sf_tagged, uint32_t reserve_cus, uint32_t strip_begin, uint32_t strip_count, hipStream_t st) {
    return with_net(ctx->net, [&](auto net) {
        return launch_encode<decltype(net)>(ctx, d_img, n, H, W, sf, params, bits, sf_tagged, reserve_cus, strip_begin,
                                            strip_count, st);
    });
}

// A decode that is running, in any context of the process; both entry points return when theirs is done.
struct RunningDecode {
    std::atomic<int>& running;
    const int sharers;                            // that run on this GPU at this one's begin, itself included
    static std::atomic<int>& on(int device) {     // (pcc_create takes no other devices: static_scratch)
        static std::atomic<int> count[kMaxDevices];
        return count[device];
    }
    explicit RunningDecode(int device) : running(on(device)), sharers(running.fetch_add(1, std::memory_order_relaxed) + 1) {}
    ~RunningDecode() { running.fetch_sub(1, std::memory_order_relaxed); }
    RunningDecode(const RunningDecode&) = delete;
};

// How a job is decoded: the kernel, its bands to an image and its workgroups.
struct DecodeLaunch {
    enum { kOne = 1, kTwo = 2, kNarrow = 3 } kernel;       // one or two workgroups per compute unit; one, bands of eight rows
    int nbands;
    uint32_t grid;
};

size_t mailbox_bytes(int n, int nbands, int W) { return align_up((size_t)n * nbands * 2 * (size_t)W * 4, 256); }

// most_bytes: what there is for the mailbox, if that is limited (bands of eight rows need twice as much of it)
// sharers: decodes that run on the GPU, this one included
template <class Net>
DecodeLaunch choose_decode(const pcc_ctx* ctx, int n, int H, int W, size_t most_bytes, int sharers) {
    const int nbands = (H + kBandRows - 1) / kBandRows, narrow_bands = (H + kNarrowRows - 1) / kNarrowRows;
    const uint64_t bands = (uint64_t)n * nbands;                      // dims_ok: below 2^31
    const uint64_t cus = ctx->num_cus > 0 ? (uint64_t)ctx->num_cus : 256u;
    // One workgroup per CU decodes a step in the shortest time; two per CU decode twice as many bands at once, at
    // Net::kSharedAlonePercent of that time per step while a unit's other workgroup waits and Net::kSharedStepPercent
    // while both are busy.  The steps on a job's longest path follow from the order of the tickets (band-major): a band
    // holds its place for `hold` steps and begins `stride` steps behind the band above, ticket k begins where ticket
    // k - places ended, so the last ticket begins behind stride steps per band above it (the chain of an image), or
    // behind whole rounds of the places and the bands of the last, partial one.  times alone / per step: within 3 % of the
    // measured time with one workgroup per CU.  With two the time per step goes from one figure to the other with the
    // share of the places that are busy on average, from a fifth of them to four fifths.
    // Fitted per network to 57 jobs of 192 to 2,000 bands (6 to 48 images of 768x512, 65 to 500 of 64x64, 2 to 4 of
    // 4096x2160, images of a few rows and of a few columns).  768x512, ms with one and with two per CU: 16 images 5.38 and 5.84, 18 images
    // 6.31 and 5.91, 48 images 12.4 and 10.0; the paper's shape, 8 images 6.08 and 6.44, 24 images 7.38 and 7.35.  Of 170 jobs with ten models
    // (one to 300 images, 64x64 to 4096x2160) the launch chosen of the three takes as long as the best one on average and 2.4 % longer at most.
    // Bands of eight rows take Net::kNarrowPercent of the time of a step, and are twice as many: they are for jobs whose chain of
    // steps, not whose work per CU, sets the time.  768x512, ms with bands of 16 and of 8 rows: 1 image 4.60 and 4.08, 4 images 4.69
    // and 4.25, 8 images 4.82 and 4.85 (the hand-overs of 500 bands), 10 images 4.81 and 5.84; 4096x2160 21.8 and 19.6; 768x512 with seven
    // mixtures, 8 images 8.00 and 6.60, 12 images 8.06 and 8.02.
    // They hold twice the places for it, which other decodes then wait for: beside another decode (threads with a context and a stream
    // each) they are for jobs of which four, the hardware queues of a process, keep three quarters of the chip busy at most.  ms until each
    // thread has decoded an image, with 16 rows and with 8: 4096x2160, two threads 22.2 and 22.5, three 24.8 and 31.6, four 25.9
    // and 41.1; 2048x1365, two 12.5 and 11.3, three 12.6 and 12.7, four 13.3 and 14.0; 1024x1024, four 8.14 and 7.67.
    auto steps = [&](uint64_t places, int rows, int per_image) {
        const uint64_t hold = (uint64_t)W + (uint64_t)Net::kDelay * ((H < rows ? H : rows) - 1), stride = (uint64_t)Net::kDelay * rows;
        const uint64_t last = (uint64_t)n * per_image - 1;
        return hold + std::max(stride * (last / n), hold * (last / places) + stride * (last % places / n));
    };
    const uint64_t hold = (uint64_t)W + (uint64_t)Net::kDelay * ((H < kBandRows ? H : kBandRows) - 1);
    const double steps_two = (double)steps(2 * cus, kBandRows, nbands), busy = (double)(bands * hold) / (steps_two * (double)(2 * cus));
    const double pace = Net::kSharedAlonePercent +
                        ((double)Net::kSharedStepPercent - Net::kSharedAlonePercent) * std::min(std::max((busy - 0.2) / 0.6, 0.0), 1.0);
    double best = 100.0 * (double)steps(cus, kBandRows, nbands);
    auto kernel = DecodeLaunch::kOne;
    if (DecLds<Net>::kTwoFit && bands > cus && steps_two * pace < best) { kernel = DecodeLaunch::kTwo; best = steps_two * pace; }
    const bool narrow_fits = mailbox_bytes(n, narrow_bands, W) <= most_bytes;
    const double steps_narrow = (double)steps(cus, kNarrowRows, narrow_bands);
    const double narrow_busy = (double)n * narrow_bands * (W + (double)Net::kDelay * ((H < kNarrowRows ? H : kNarrowRows) - 1)) / steps_narrow;    // places, on average
    const bool narrow_room = narrow_busy <= (sharers <= 1 ? Net::kNarrowAlonePercent / 100.0 : 0.75 / 4.0) * (double)cus;
    if (narrow_fits && narrow_room && (double)Net::kNarrowPercent * steps_narrow < best) kernel = DecodeLaunch::kNarrow;
    if (ctx->decode_variant == 1) kernel = DecodeLaunch::kOne;
    if (ctx->decode_variant == 2) kernel = DecodeLaunch::kTwo;
    if (ctx->decode_variant == 3) kernel = narrow_fits ? DecodeLaunch::kNarrow : DecodeLaunch::kOne;
    const int per_image = kernel == DecodeLaunch::kNarrow ? narrow_bands : nbands;
    if (kernel == DecodeLaunch::kTwo) return {kernel, per_image, (uint32_t)std::min((uint64_t)n * per_image, 2 * cus)};
    // Workgroups: one for each band that can run at a time, and two for the turn from one band to the next.  One for every band held units
    // for bands that were not to begin for a long time, and polled there: with bands of eight rows a decode that started alone then left none
    // for one that came behind it.  ms a decode where each thread decodes four times, with bands of 16 rows alone, with a workgroup a band and now:
    // the paper's network, two threads with four images of 768x512 6.24, 6.74, 6.08, with one of 4096x2160 27.6, 30.0, 27.3, three with one of
    // 2048x1365 16.2, 17.1, 15.8; six layers, two with four of 768x512 6.97, 7.45, 6.77.  A decode by itself is not slower for it (33 jobs with
    // three networks): four images of 768x512 4.38 and 4.28, the paper's network 5.66 and 5.47, 4096x2160 19.98 and 19.65.
    const int rows = kernel == DecodeLaunch::kNarrow ? kNarrowRows : kBandRows;
    const uint64_t stride = (uint64_t)Net::kDelay * rows;
    const uint64_t at_once = std::min((uint64_t)per_image, ((uint64_t)W + (uint64_t)Net::kDelay * ((H < rows ? H : rows) - 1) + stride - 1) / stride + 2);
    return {kernel, per_image, (uint32_t)std::min((uint64_t)n * at_once, cus)};
}

template <class Net>
void launch_decode(pcc_ctx* ctx, const DecodeLaunch& how, const uint8_t* d_stream, size_t nbytes, int n, int H, int W,
                   uint8_t* d_img_out, uint32_t* d_mail, uint32_t spin_limit, hipStream_t st) {
    constexpr int kLds = DecLds<Net>::kBytes, kLdsShared = DecLds<Net>::kBytesShared;
    int* status = ctx->status(kBlockDecode);
    if (how.kernel == DecodeLaunch::kOne)
        hipLaunchKernelGGL((decode_kernel<Net, 1>), dim3(how.grid), dim3(kDecThreads), kLds, st, ctx->d_model, d_stream,
                           (uint64_t)nbytes, n, H, W, how.nbands, ctx->dist, d_img_out, d_mail, status, spin_limit);
    else if (how.kernel == DecodeLaunch::kTwo)
        hipLaunchKernelGGL((decode_kernel<Net, 2>), dim3(how.grid), dim3(kDecThreads), kLdsShared, st,
                           ctx->d_model + (Net::kSharedByCoefficient ? 2 * Layout<Net>::kModelBytes : 0), d_stream,
                           (uint64_t)nbytes, n, H, W, how.nbands, ctx->dist, d_img_out, d_mail, status, spin_limit);
    else {
        constexpr int kLdsNarrow = DecLds<Net, kNarrowRows>::kBytes;
        hipLaunchKernelGGL((decode_narrow_kernel<Net>), dim3(how.grid), dim3(kDecThreads), kLdsNarrow, st, ctx->d_model, d_stream,
                           (uint64_t)nbytes, n, H, W, how.nbands, ctx->dist, d_img_out, d_mail, status, spin_limit);
    }
}

DecodeLaunch choose_decode_any(const pcc_ctx* ctx, int n, int H, int W, size_t most_bytes, int sharers) {
    return with_net(ctx->net, [&](auto net) { return choose_decode<decltype(net)>(ctx, n, H, W, most_bytes, sharers); });
}

inline int head_outputs(const pcc_ctx* ctx) {
    return with_net(ctx->net, [](auto net) { using Net = decltype(net); return Net::dim(Net::kLayers); });
}

}  // namespace

extern "C" {

const char* pcc_strerror(int code) {
    switch (code) {
        case PCC_OK: return "ok";
        case PCC_E_ARG: return "invalid argument";
        case PCC_E_BLOB: return "unsupported or malformed weight blob";
        case PCC_E_CAP: return "output capacity too small";
        case PCC_E_STREAM: return "malformed stream";
        case PCC_E_HIP: return "HIP runtime error";
        case PCC_E_INTERNAL: return "internal error (zero frequency or device wait expired)";
        case PCC_E_UNIMPL: return "not implemented";
        case PCC_E_SCRATCH: return "job needs more scratch memory than the library's static array holds";
        default: return "unknown error";
    }
}

size_t pcc_stream_bound(int n, int H, int W) {
    if (n < 1 || H < 1 || W < 1) return 0;
    const size_t rows = (size_t)n * H;
    return (size_t)kStreamHeader + 8 * (rows + 1) + rows * 4 * slab_words(W);
}

long pcc_wavefront_steps(int H, int W, int delay) {
    if (H < 1 || W < 1 || delay < 1) return 0;
    return (long)W + (long)delay * (H - 1);
}

int pcc_create(pcc_ctx** out, const void* h_blob, size_t blob_bytes, int hip_device) {
    if (!out || !h_blob) return PCC_E_ARG;
    *out = nullptr;
    const uint8_t* p = (const uint8_t*)h_blob;
    if (blob_bytes < 64 || rd32(p) != kBlobMagic || rd32(p + 4) != 1u) return PCC_E_BLOB;
    const uint32_t dist = rd32(p + 60);   // 0 = Gaussian mixture (Eq. (1)), 1 = logistic mixture (Eq. (8))
    if (dist > 1u) return PCC_E_BLOB;
    int net;
    if (header_matches<NetWorkload>(p)) net = kNetWorkload;
    else if (header_matches<NetPaper>(p)) net = kNetPaper;
    else if (header_matches<NetDiagonal>(p)) net = kNetDiagonal;
    else if (header_matches<NetFewerLayers>(p)) net = kNetFewerLayers;
    else if (header_matches<NetFewerFilters>(p)) net = kNetFewerFilters;
    else if (header_matches<NetMoreMixtures>(p)) net = kNetMoreMixtures;
    else if (header_matches<NetMostMixtures>(p)) net = kNetMostMixtures;
    else if (header_matches<NetMoreLayers>(p)) net = kNetMoreLayers;
    else if (header_matches<NetMoreFilters>(p)) net = kNetMoreFilters;
    else return PCC_E_BLOB;

    std::vector<uint8_t> image;
    const int prc = with_net(net, [&](auto tag) { return pack_model<decltype(tag)>(p, blob_bytes, dist, image); });
    if (prc != PCC_OK) return prc;

    DeviceGuard guard(hip_device);
    if (!guard.ok) { (void)hipGetLastError(); return PCC_E_HIP; }
    pcc_ctx* ctx = new (std::nothrow) pcc_ctx();
    if (!ctx) return PCC_E_INTERNAL;
    ctx->device = hip_device;
    ctx->net = net;
    ctx->dist = dist;
    hipDeviceProp_t prop;
    bool ok = hipGetDeviceProperties(&prop, hip_device) == hipSuccess;
    if (ok) ctx->num_cus = prop.multiProcessorCount;
    ctx->d_static_scratch = static_scratch(hip_device);
    ok = ok && ctx->d_static_scratch != nullptr;
    ok = ok && hipMalloc((void**)&ctx->d_model, image.size()) == hipSuccess;
    constexpr size_t kBlocksBytes = kStBlocks * kStBytes, kStatusBytes = kBlocksBytes + (1 + kRansBesideMaxGroups) * sizeof(uint64_t);
    static_assert(kBlocksBytes % sizeof(uint64_t) == 0 && kStBytes % alignof(EncodeResult) == 0, "alignment");
    ok = ok && hipMalloc((void**)&ctx->d_status, kStatusBytes) == hipSuccess;
    ok = ok && hipMemset(ctx->d_status, 0, kStatusBytes) == hipSuccess;
    ok = ok && hipHostMalloc((void**)&ctx->h_status, kStBytes + sizeof(EncodeResult), hipHostMallocDefault) == hipSuccess;
    if (ok) {
        ctx->h_result = reinterpret_cast<EncodeResult*>(ctx->h_status + kStWords);
        ok = hipHostGetDevicePointer((void**)&ctx->d_result, ctx->h_result, 0) == hipSuccess;
    }
    ok = ok && hipMemcpy(ctx->d_model, image.data(), image.size(), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && with_net(net, [](auto tag) { return set_kernel_attributes<decltype(tag)>(); });
    // limits from the environment: negative values are taken as zero (no patience), never as huge unsigned ones
    auto env_limit = [](const char* e) { const long v = atol(e); return (uint32_t)std::min<long>(std::max<long>(v, 0), 0x7FFFFFFFl); };
    if (const char* e = getenv("PCC_DECODE_SPIN_LIMIT")) ctx->spin_limit = env_limit(e);
    if (const char* e = getenv("PCC_DECODE_VARIANT")) {
        const int v = atoi(e);
        if (v >= 0 && v <= 3) ctx->decode_variant = v;
    }
    if (const char* e = getenv("PCC_ENCODE_OVERLAP")) ctx->overlap = atoi(e) != 0;
    if (const char* e = getenv("PCC_RANS_PATIENCE")) {
        ctx->patience = env_limit(e);
        ctx->sums_patience = (uint32_t)std::min<uint64_t>(4ull * ctx->patience, 0xFFFFFFFFull);
    }
    if (const char* e = getenv("PCC_RANS_SUMS_PATIENCE")) ctx->sums_patience = env_limit(e);
    ok = ok && hipStreamCreateWithFlags(&ctx->side, hipStreamNonBlocking) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&ctx->ev_joined, hipEventDisableTiming) == hipSuccess;
    if (!ok) { (void)hipGetLastError(); pcc_destroy(ctx); return PCC_E_HIP; }
    ctx->d_total = reinterpret_cast<uint64_t*>(ctx->d_status + kStBlocks * kStWords);
    ctx->d_sums = ctx->d_total + 1;
    *out = ctx;
    return PCC_OK;
}

void pcc_destroy(pcc_ctx* ctx) {
    if (!ctx) return;
    DeviceGuard guard(ctx->device);
    if (ctx->d_model) (void)hipFree(ctx->d_model);
    if (ctx->d_ws) (void)hipFree(ctx->d_ws);
    if (ctx->d_status) (void)hipFree(ctx->d_status);
    if (ctx->h_status) (void)hipHostFree(ctx->h_status);
    for (hipEvent_t e : ctx->ev) if (e) (void)hipEventDestroy(e);
    if (ctx->d_tagged) (void)hipFree(ctx->d_tagged);
    if (ctx->ev_joined) (void)hipEventDestroy(ctx->ev_joined);
    if (ctx->side) (void)hipStreamDestroy(ctx->side);
    delete ctx;
}

int pcc_model_info(const pcc_ctx* ctx, int* h_info) {
    if (!ctx || !h_info) return PCC_E_ARG;
    with_net(ctx->net, [&](auto tag) {
        using Net = decltype(tag);
        h_info[0] = Net::dim(Net::kLayers);
        h_info[1] = Net::K;
        h_info[2] = Net::kNbhd;
        h_info[3] = Net::kDelay;
        h_info[4] = (int)ctx->dist;
        h_info[5] = Net::kLayers;
        return 0;
    });
    return PCC_OK;
}

int pcc_encode_probs(pcc_ctx* ctx, const uint8_t* d_img, int n, int H, int W, float* d_params, float* d_bits,
                     void* hip_stream) {
    if (!ctx || !d_img || !d_params || !dims_ok(n, H, W)) return PCC_E_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    return launch_encode_any(ctx, d_img, n, H, W, nullptr, d_params, d_bits, nullptr, 0, 0, encode_strips(W),
                             (hipStream_t)hip_stream);
}

int pcc_encode(pcc_ctx* ctx, const uint8_t* d_img, int n, int H, int W, uint8_t* d_stream, size_t cap_bytes,
               size_t* h_nbytes_out, void* hip_stream) {
    if (!ctx || !d_img || !d_stream || !h_nbytes_out || !dims_ok(n, H, W)) return PCC_E_ARG;
    if (((uintptr_t)d_stream & 7u) != 0) return PCC_E_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    const uint64_t P = (uint64_t)n * H * W;
    const uint32_t rows = (uint32_t)((uint64_t)n * H);
    const size_t table = (size_t)kStreamHeader + 8 * ((size_t)rows + 1);
    if (cap_bytes < table) return PCC_E_CAP;

    const size_t sf_bytes = align_up(P * 3 * sizeof(uint32_t), 256);
    const size_t slab_bytes = align_up((size_t)rows * slab_words(W) * 4, 256);
    const uint32_t groups = (rows + kRansRows - 1) / kRansRows;
    const bool scan = groups > kSumGroupsMax;
    const size_t rw_bytes = align_up((size_t)rows * 4, 256), gw_bytes = align_up((size_t)groups * 4, 256);
    int rc = ensure_workspace(ctx, sf_bytes + slab_bytes + rw_bytes + gw_bytes + (scan ? (size_t)groups * 8 : 0));
    if (rc != PCC_OK) return rc;
    uint32_t* d_sf = reinterpret_cast<uint32_t*>(ctx->d_ws);
    uint32_t* d_slabs = reinterpret_cast<uint32_t*>(ctx->d_ws + sf_bytes);
    uint32_t* d_rw = reinterpret_cast<uint32_t*>(ctx->d_ws + sf_bytes + slab_bytes);
    uint32_t* d_gw = reinterpret_cast<uint32_t*>(ctx->d_ws + sf_bytes + slab_bytes + rw_bytes);
    uint64_t* d_before = scan ? reinterpret_cast<uint64_t*>(ctx->d_ws + sf_bytes + slab_bytes + rw_bytes + gw_bytes) : nullptr;
    ctx->d_sf = d_sf;
    ctx->sf_count = (size_t)P * 3;

    // A small job's row coder is a handful of workgroups, each bound by the instruction stream of its one coding wave.  It runs
    // beside the pixel kernel, on compute units the pixel kernel's grid leaves free (a pixel workgroup fills a
    // unit's LDS, so the workgroups of both kernels are resident whatever order the dispatcher takes them in),
    // and takes each symbol when it finds it written.  The row coder and what comes after it go to a stream of
    // the context's own; nothing orders that stream after the caller's, so this is only done when the caller's
    // stream is idle and the pixel kernel starts at once.  A large job's row coder needs the whole chip and
    // runs after the pixel kernel, on the caller's stream.
    // Beside the pixel kernel the stream's first rows are written while pixels are still being read.  A stream buffer that shares bytes
    // with the images therefore gets the kernels one after the other: the compaction, the last, is the only one that writes it.
    const uintptr_t img_at = (uintptr_t)d_img, stream_at = (uintptr_t)d_stream;
    const bool apart = img_at + P * 3 <= stream_at || stream_at + std::min<size_t>(cap_bytes, pcc_stream_bound(n, H, W)) <= img_at;
    const uint32_t cus = ctx->num_cus > 0 ? (uint32_t)ctx->num_cus : 256u;
    bool beside = ctx->overlap && apart && groups <= kRansBesideMaxGroups && cus >= 2 * kRansBesideMaxGroups;
    if (beside) {
        const hipError_t busy = hipStreamQuery(st);
        if (busy != hipSuccess) { (void)hipGetLastError(); beside = false; }
    }
    if (beside) {
        rc = ensure_tagged(ctx, (size_t)P * 3, st);
        if (rc != PCC_OK) return rc;
        if (++ctx->epoch == 0) {      // wrapped: the words of old launches would pass for new ones
            rc = clear_tagged(ctx, st);
            if (rc == PCC_OK && hipMemsetAsync(ctx->d_sums, 0, kRansBesideMaxGroups * sizeof(uint64_t), st) != hipSuccess) rc = PCC_E_HIP;
            if (rc == PCC_OK && hipStreamSynchronize(st) != hipSuccess) rc = PCC_E_HIP;
            if (rc != PCC_OK) { (void)hipGetLastError(); --ctx->epoch; return rc; }
            ctx->epoch = 1;
        }
    }
    ctx->last_tagged = beside;
    uint64_t* d_tagged = beside ? ctx->d_tagged : nullptr;
    // Workgroups go to the chip's eight dies in turn and stay there: a die must have room for its share of both
    // kernels, or a pixel workgroup waits for a compute unit until others of its die have ended and then works
    // through its share of the items alone.
    const uint32_t reserve = beside ? kXcds * ((groups + kXcds - 1) / kXcds) : 0u;

    prof_reset(ctx);
    int* d_status = ctx->status(kBlockEncode);
    const uint32_t tag = with_net(ctx->net, [](auto net) { return model_tag<decltype(net)>(); });
    const StreamOut out = {d_stream, (uint64_t)cap_bytes, n, H, tag, ctx->dist, ctx->d_total, ctx->d_result, ctx->d_sums, ctx->sums_patience};
    bool assembles = beside && W <= kRansAssembleWidth;
    auto launch_rans = [&](hipStream_t s) {
        prof_begin(ctx, PCC_T_ENCODE_RANS, s);
        const auto kernel = !beside ? rans_rows_kernel<false, false> : assembles ? rans_rows_kernel<true, true> : rans_rows_kernel<true, false>;
        hipLaunchKernelGGL(kernel, dim3(groups), dim3(kRansThreads), 0, s, d_sf, d_tagged, ctx->epoch, W,
                           rows, d_slabs, d_rw, d_gw, d_status, beside ? ctx->patience : 0u, out);
        prof_end(ctx, PCC_T_ENCODE_RANS, s);
    };
    // what follows the row coder, and the wait for it
    auto finish = [&](hipStream_t s) -> int {
        if (!assembles) {
            if (scan) {
                prof_begin(ctx, PCC_T_ENCODE_SCAN, s);
                hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, d_gw, groups, d_before);
                prof_end(ctx, PCC_T_ENCODE_SCAN, s);
            }
            prof_begin(ctx, PCC_T_ENCODE_COMPACT, s);
            const uint32_t chunk = kCompactRows * (uint32_t)(((uint64_t)rows + kCompactRows * kCompactBlocks - 1) / (kCompactRows * kCompactBlocks));
            hipLaunchKernelGGL(compact_kernel, dim3((rows + chunk - 1) / chunk), dim3(kCompactThreads), 0, s, d_slabs, d_rw,
                               d_gw, d_before, W, rows, chunk, d_status, out);
            prof_end(ctx, PCC_T_ENCODE_COMPACT, s);
        }
        if (hipGetLastError() != hipSuccess) return PCC_E_HIP;
        // The pixel kernel, on the caller's stream, ends before the row coder: waiting for it first costs nothing, waiting for it
        // after the compaction 8.6 us, and an event for the compaction to wait for holds the host up for 20.
        if (s != st && hipStreamSynchronize(st) != hipSuccess) { (void)hipGetLastError(); return PCC_E_HIP; }
        if (hipStreamSynchronize(s) != hipSuccess) { (void)hipGetLastError(); return PCC_E_HIP; }
        return PCC_OK;
    };
    // Whatever fails, the call leaves through `drain`: its streams are waited for (a row coder without its pixel kernel stands
    // down when its patience is over), so nothing still writes the caller's stream buffer or the workspace after the return, and
    // the status block is clear again for the next call.
    auto drain = [&](int code) -> int {
        if (beside) (void)hipStreamSynchronize(ctx->side);
        (void)hipStreamSynchronize(st);
        (void)hipMemsetAsync(d_status, 0, kStBytes, st);
        (void)hipStreamSynchronize(st);
        (void)hipGetLastError();
        return code;
    };
    const uint32_t strips = encode_strips(W);
    if (!beside) {
        prof_begin(ctx, PCC_T_ENCODE_PIXELS, st);
        rc = launch_encode_any(ctx, d_img, n, H, W, d_sf, nullptr, nullptr, nullptr, 0, 0, strips, st);
        if (rc != PCC_OK) return drain(rc);
        prof_end(ctx, PCC_T_ENCODE_PIXELS, st);
        launch_rans(st);
        rc = finish(st);
        if (rc != PCC_OK) return drain(rc);
    } else {
        // An image of few rows: the row coder follows the pixel kernel through the whole image.  A tall image: the
        // pixel kernel is the longer one; it does the first strips with the whole chip, and the row coder joins it
        // (an event; the launch gap does not matter at this size) for a last part sized so that both end together.
        // Both times are in proportion to the width, the pixel kernel's to the rows as well.
        //
        // The pixel kernel is queued first.  Two streams may share one of the process's few hardware queues and then run
        // their kernels in the order in which they were queued: a row coder in front of the pixel kernel that it waits
        // for would hold it up until its patience is over (768x512: 2,250 us a call instead of 154, for about one pair
        // of a codec and a caller's stream in six), behind it the call merely runs in sequence (201 us).  With queues of
        // their own the order costs nothing (64x64 65.2 -> 62.9 us, 768x512 142.7 -> 139.6): the pixel kernel, the longer
        // one, starts a launch earlier.  Since each call queues the kernel that waits for nothing first, calls of several
        // threads cannot wait for each other in a circle either.
        const double share = 1.1 * kRansBalanceRows / rows * (double)(cus - reserve) / cus;   // of the strips, beside
        const uint32_t strips_alone = share >= 1.0 ? 0u : (uint32_t)((1.0 - share) * strips);
        prof_begin(ctx, PCC_T_ENCODE_PIXELS, st);
        if (strips_alone != 0) {
            rc = launch_encode_any(ctx, d_img, n, H, W, nullptr, nullptr, nullptr, d_tagged, 0, 0, strips_alone, st);
            if (rc != PCC_OK) return drain(rc);
            if (hipEventRecord(ctx->ev_joined, st) != hipSuccess) return drain(PCC_E_HIP);
            if (hipStreamWaitEvent(ctx->side, ctx->ev_joined, 0) != hipSuccess) return drain(PCC_E_HIP);
        }
        rc = launch_encode_any(ctx, d_img, n, H, W, nullptr, nullptr, nullptr, d_tagged, reserve, strips_alone,
                               strips - strips_alone, st);
        if (rc != PCC_OK) return drain(rc);
        prof_end(ctx, PCC_T_ENCODE_PIXELS, st);
        launch_rans(ctx->side);
        rc = finish(ctx->side);
        if (rc != PCC_OK) return drain(rc);
        if (ctx->h_result->err == 0 && ctx->h_result->defer != 0) {
            // A group of the row coder saw nothing of the pixel kernel, or of a group before it, for a long time and stood down.  The
            // symbols are all there now; code them on the caller's stream.
            assembles = false;           // (the groups that stood down have said so in this epoch's sums)
            launch_rans(st);
            rc = finish(st);
            if (rc != PCC_OK) return drain(rc);
            if (ctx->h_result->defer != 0) return drain(PCC_E_INTERNAL);   // a symbol was never written
        }
    }
    prof_collect(ctx);
    if (ctx->h_result->err != 0) return drain(ctx->h_result->err);
    const uint64_t total = ctx->h_result->total_bytes;
    if (total > cap_bytes) return PCC_E_CAP;
    *h_nbytes_out = (size_t)total;
    return PCC_OK;
}

// Both decoders: `d_mail` is the mailbox (zeroed here), big enough for the job.
static int decode_with_mailbox(pcc_ctx* ctx, const DecodeLaunch& how, const uint8_t* d_stream, size_t nbytes, int n, int H, int W,
                               uint8_t* d_img_out, uint32_t* d_mail, size_t mail_bytes, bool clear_by_kernel, hipStream_t st) {
    if (clear_by_kernel) {
        const size_t words = mail_bytes / 4;
        hipLaunchKernelGGL(clear_words_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<uint32_t*>(ctx->status(kBlockDecode)),
                           (size_t)kStWords);
        hipLaunchKernelGGL(clear_words_kernel, dim3((uint32_t)std::min<size_t>((words + 255) / 256, 1024)), dim3(256), 0, st,
                           d_mail, words);
        if (hipGetLastError() != hipSuccess) return PCC_E_HIP;
    } else {
        if (hipMemsetAsync(ctx->status(kBlockDecode), 0, kStBytes, st) != hipSuccess) return PCC_E_HIP;
        if (hipMemsetAsync(d_mail, 0, mail_bytes, st) != hipSuccess) return PCC_E_HIP;
    }
    const uint32_t spin_limit = ctx->spin_limit;
    prof_reset(ctx);
    prof_begin(ctx, PCC_T_DECODE, st);
    with_net(ctx->net, [&](auto net) {
        launch_decode<decltype(net)>(ctx, how, d_stream, nbytes, n, H, W, d_img_out, d_mail, spin_limit, st);
        return 0;
    });
    prof_end(ctx, PCC_T_DECODE, st);
    if (hipGetLastError() != hipSuccess) return PCC_E_HIP;
    if (hipMemcpyAsync(ctx->h_status, ctx->status(kBlockDecode), kStBytes, hipMemcpyDeviceToHost, st) != hipSuccess)
        return PCC_E_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) { (void)hipGetLastError(); return PCC_E_HIP; }
    prof_collect(ctx);
    return ctx->h_status[kStErr];
}

int pcc_decode(pcc_ctx* ctx, const uint8_t* d_stream, size_t nbytes, int n, int H, int W, uint8_t* d_img_out,
               void* hip_stream) {
    if (!ctx || !d_stream || !d_img_out || !dims_ok(n, H, W)) return PCC_E_ARG;
    if (((uintptr_t)d_stream & 7u) != 0) return PCC_E_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    const uint64_t rows = (uint64_t)n * H;
    const uint64_t table = (uint64_t)kStreamHeader + 8 * (rows + 1);
    if (nbytes < table + 16 * rows) return PCC_E_STREAM;   // every row payload holds at least its two 8-byte states
    const RunningDecode self(ctx->device);
    DecodeLaunch how = choose_decode_any(ctx, n, H, W, SIZE_MAX, self.sharers);
    size_t mail_bytes = mailbox_bytes(n, how.nbands, W);
    int rc = ensure_workspace(ctx, mail_bytes);
    if (rc != PCC_OK && how.kernel == DecodeLaunch::kNarrow) {        // no memory for twice as many bands
        how = choose_decode_any(ctx, n, H, W, mail_bytes - 1, self.sharers);
        mail_bytes = mailbox_bytes(n, how.nbands, W);
        rc = ensure_workspace(ctx, mail_bytes);
    }
    if (rc != PCC_OK) return rc;
    ctx->d_sf = nullptr; ctx->sf_count = 0;
    return decode_with_mailbox(ctx, how, d_stream, nbytes, n, H, W, d_img_out, reinterpret_cast<uint32_t*>(ctx->d_ws),
                               mail_bytes, false, (hipStream_t)hip_stream);
}

size_t pcc_decode_static_scratch_bytes(int n, int H, int W) {
    if (!dims_ok(n, H, W)) return 0;
    return mailbox_bytes(n, (H + kBandRows - 1) / kBandRows, W);
}

int pcc_decode_static(pcc_ctx* ctx, const uint8_t* d_stream, size_t nbytes, int n, int H, int W, uint8_t* d_img_out,
                      void* hip_stream) {
    if (!ctx || !d_stream || !d_img_out || !dims_ok(n, H, W)) return PCC_E_ARG;
    if (((uintptr_t)d_stream & 7u) != 0) return PCC_E_ARG;
    if (pcc_decode_static_scratch_bytes(n, H, W) > kStaticScratchBytes) return PCC_E_SCRATCH;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    const uint64_t rows = (uint64_t)n * H;
    const uint64_t table = (uint64_t)kStreamHeader + 8 * (rows + 1);
    if (nbytes < table + 16 * rows) return PCC_E_STREAM;
    // bands of eight rows where the array is large enough for them
    const RunningDecode self(ctx->device);
    const DecodeLaunch how = choose_decode_any(ctx, n, H, W, kStaticScratchBytes, self.sharers);
    const size_t mail_bytes = mailbox_bytes(n, how.nbands, W);
    // the array keeps the last call's words (tagged pixels of another image): the part this job uses is cleared
    return decode_with_mailbox(ctx, how, d_stream, nbytes, n, H, W, d_img_out, ctx->d_static_scratch, mail_bytes, true,
                               (hipStream_t)hip_stream);
}

int pcc_cdf_tables(pcc_ctx* ctx, const float* d_params, const uint8_t* d_rg, size_t count, uint32_t* d_cq,
                   void* hip_stream) {
    if (!ctx || !d_params || !d_rg || !d_cq || count == 0 || count > (1u << 26)) return PCC_E_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    const size_t threads = count * 3;
    const dim3 grid((uint32_t)((threads + 255) / 256));
    with_net(ctx->net, [&](auto net) {
        hipLaunchKernelGGL(cdf_tables_kernel<decltype(net)>, grid, dim3(256), (kLutEntries + 1) * 8, (hipStream_t)hip_stream,
                           ctx->d_model, d_params, d_rg, count, d_cq);
        return 0;
    });
    return hipGetLastError() == hipSuccess ? PCC_OK : PCC_E_HIP;
}

int pcc_set_profiling(pcc_ctx* ctx, int enabled) {
    if (!ctx) return PCC_E_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    if (enabled && !ctx->ev[0]) {
        for (hipEvent_t& e : ctx->ev)
            if (hipEventCreate(&e) != hipSuccess) { (void)hipGetLastError(); return PCC_E_HIP; }
    }
    ctx->profiling = enabled != 0;
    prof_reset(ctx);
    return PCC_OK;
}

int pcc_last_timings(pcc_ctx* ctx, float* h_ms) {
    if (!ctx || !h_ms) return PCC_E_ARG;
    for (int i = 0; i < PCC_N_TIMINGS; ++i) h_ms[i] = ctx->last_ms[i];
    return PCC_OK;
}

int pcc_copy_intervals(pcc_ctx* ctx, uint32_t* d_out, size_t count, void* hip_stream) {
    if (!ctx || !d_out) return PCC_E_ARG;
    if (!ctx->d_sf || count != ctx->sf_count) return PCC_E_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return PCC_E_HIP;
    if (ctx->last_tagged) {
        const uint32_t blocks = (uint32_t)((count + 255) / 256 < 4096 ? (count + 255) / 256 : 4096);
        hipLaunchKernelGGL(untag_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream, ctx->d_tagged, count, d_out);
        return hipGetLastError() == hipSuccess ? PCC_OK : PCC_E_HIP;
    }
    if (hipMemcpyAsync(d_out, ctx->d_sf, count * sizeof(uint32_t), hipMemcpyDeviceToDevice, (hipStream_t)hip_stream) !=
        hipSuccess) return PCC_E_HIP;
    return PCC_OK;
}

#ifdef PCC_PHASE_TIMING
// measurement build only: cycles per phase and wave of the last decode's workgroup of ticket kPhaseTicket,
// h_out[4][kPhCount + 1] (the last value is the number of steps)
int pcc_debug_phase_cycles(unsigned long long* h_out) {
    return hipMemcpyFromSymbol(h_out, HIP_SYMBOL(pcc::phase_cycles), sizeof(unsigned long long) * 4 * (kPhCount + 1)) == hipSuccess
               ? PCC_OK : PCC_E_HIP;
}
#endif

}  // extern "C"
