// Device-side building blocks shared by the encode and decode kernels.
//
// Encoder and decoder must derive bit-identical integer CDF values for every
// pixel, otherwise decoding desynchronises.  Everything between "bytes of the
// neighbourhood" and "Cq(e)" is therefore written once, here, and compiled
// with floating-point contraction off: the same inputs give the same bits in
// both kernels.  They do so by the same instructions but for the split of an
// activation into hi + lo, which has three forms: act_split_bf16 on the vector
// ALU and act_split4_bf16 with the subtraction on the matrix core, of which the
// decoder has one per network and launch, and EncoderNet's, which is the second
// in pieces.  All are exact, and a test compares their bits.
// Where an activation rounds to infinity their lo parts differ, but the pixel
// is NaN from the next layer on in each form, and MFMA has one NaN
// (0xFFC00000) for every product with a NaN, 0 x inf or inf - inf in it.
// An MFMA output element depends only on its A row, its B column and the
// order of the k blocks, all of which are fixed below, so it does not matter
// which other pixels share a tile.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace pcc {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Network descriptions.  Tiles are v_mfma_f32_16x16x32_bf16: out-blocks of 16
// features, k-blocks of 32 inputs; ob(l) / kb(l) are the padded block counts of
// layer l.  Two consecutive out-blocks of a hidden layer form one k-block of the
// next layer, so ob(l) = 2 kb(l+1).
// ---------------------------------------------------------------------------

// Canonical input index 3*j + ch (neighbour j in raster order, channel ch) of slot i
// (0..7) of lane group g in first-layer k-block kbi, or -1 for a padding slot, for a
// network whose byte runs carry the neighbours in place.
template <class Net>
__host__ __device__ constexpr int run_in_index(int kbi, int g, int i) {
    int dr = 0, off = 0;
    if (!Net::run_desc(kbi, g, i >> 2, dr, off)) return -1;
    const int b = off + (i & 3);
    const int len = dr == 0 ? 6 : Net::kUpBytes;
    if (b >= len) return -1;
    return (dr == -2 ? 0 : dr == -1 ? Net::kUpBytes : 2 * Net::kUpBytes) + b;
}

// The decoder's head: canonical output in register s of lane group g after the last layer, or -1.  Groups 0..2 hold their
// channel's 3 K parameters, group 3 the coupling coefficients component by component (alpha, beta, gamma), so that two parts of the
// components are read at one distance from each other, whichever the coefficient.
template <int K>
__host__ __device__ constexpr int decoder_head_index(int g, int s) {
    return s >= 3 * K ? -1 : g < 3 ? 3 * K * g + s : 9 * K + K * (s % 3) + s / 3;
}

// The measured workloads' network: 30 -> 160 -> 160 -> 128 -> 60, ReLU, K = 5,
// neighbourhood {rows r-2, r-1 at columns c-2..c+1; row r at c-2, c-1}, wavefront delay 2.
struct NetWorkload {
    static constexpr int kLayers = 4;
    static constexpr int K = 5;
    static constexpr int kNbhd = 10, kDelay = 2;
    static constexpr int kReach1 = 1, kReach2 = 1;   // columns right of c that rows r-1 and r-2 are read at
    static constexpr int kUpBytes = 12;       // bytes of one upper row's neighbours (columns c-2..c+1)
    static constexpr int kRingCols = 8;       // decoder ring columns (power of two)
    static constexpr int kRingPad = 2;        // extra 16-bit elements per ring row
    static constexpr bool kLeaky = false;
    // Decoder with two workgroups per CU (256 registers per lane each): what of a wave's weight slices is then read
    // from a copy in LDS instead of held in registers, chosen by measurement (1: the biases, 2: the first layer's
    // weights, 4: the head's).  LDS copies cost time too, so a few spilled registers can be the better deal.  24 images of
    // 768x512 with two per CU, ms (spilled registers):
    //   copies             none         first layer   head         first and head   all
    //   this network       7.85 (61)    7.15 (47)     6.98 (45)    6.38 (29)        6.49 (0)
    //   the paper's        9.44 (42)    8.09 (27)     8.00 (29)    7.58 (16)        7.80 (0)
    //   diagonal           6.84 (45)    6.31 (47)     6.21 (40)    5.24 (25)        5.41 (0)
    //   five mixtures      10.85 (49)   9.47 (30)     9.87 (34)    8.57 (19)        8.95 (0)
    //   seven mixtures     13.61 (104)  13.12 (87)    12.77 (80)   13.15 (87)       11.22 (44)
    //   six layers         12.14 (93)   11.19 (75)    11.27 (62)   10.39 (47)       8.86 (8)
    //   four layers        6.38 (11)    6.60 (0)      6.43 (0)     6.64 (0)         6.83 (0)
    //   64 filters         5.65 (0)     5.69 (0)      5.63 (0)     5.73 (0)         5.89 (0)
    // (The paper's and diagonal before a layer's input was read in order, dec_load_act; since then first layer 7.41 and 5.18, head
    // 7.37 and 5.40, first and head 7.37 (2) and 5.05 (6).)
    // (Seven mixtures: the first layer and the head do not fit a CU twice, `all` is the biases and the first layer.)
    static constexpr int kEncodeThreads = 512;    // pixel kernel: threads of a workgroup
    static constexpr int kSharedCuLds = 6;
    // Two workgroups per unit: does that kernel read a head whose coupling coefficients stand coefficient by coefficient (SharedHead)?
    // 20 images of 768x512, us with the other order and with this one: this network 6,096 and 6,072, with the predictor's weights 6,066
    // and 6,011, 64 filters 5,501 and 5,449, five mixtures of the ablation 8,262 and 8,386; the others within 0.2 %.  (One workgroup per unit:
    // this network 6,594 and 6,717, 64 filters 5,767 and 5,809.)
    static constexpr bool kSharedByCoefficient = true;
    // Time of a decode step with two workgroups per CU, in percent of a step with one, while the other workgroup waits and
    // while both are busy (fitted to whole jobs; the host chooses between the launches with them: choose_decode).
    static constexpr unsigned kSharedAlonePercent = 112, kSharedStepPercent = 138;
    // Bands of eight rows with 32 lanes to a pixel (decode_narrow_kernel): the time for a single image in percent of the time with
    // bands of 16 rows, the hand-overs of twice as many bands included.  512x512, us with 16 and with eight: this network 3,946 and 3,520,
    // the paper's 5,181 and 4,730, diagonal 2,734 and 2,587, five mixtures 6,003 and 5,313, seven 6,814 and 5,560, four layers 4,688 and
    // 4,281, six 5,773 and 5,261, 64 filters 4,383 and 3,989, 192 6,738 and 6,132.
    static constexpr unsigned kNarrowPercent = 89;
    // And the percentage of the chip that they may keep busy, on average, in a decode that is alone when it starts: less than all in diagonal order,
    // where all bands of an image run at a time and eight rows gain little.  With 16 and with eight rows, us of a decode alone, and ms a decode where two
    // threads decode four times each and the first one starts so: one of 768x512 (15 %) 3,340 and 3,158, 3.40 and 3.24; one of 2048x1365 (40 %) 8,873 and
    // 8,537, 9.13 and 9.40; four of 512x512 (51 %) 2,709 and 2,670, 2.85 and 3.15; two of 1024x1024 (50 %) 5,462 and 5,372, 5.70 and 6.27; four of 768x512
    // (61 %) 3,363 and 3,297, 3.51 and 3.96.
    static constexpr unsigned kNarrowAlonePercent = 100;
    // Decoder with one workgroup per unit: are the waits for LDS filled with MFMAs (Awake)?  512x512 with bands of eight rows, us without and
    // with: this network 3,600 and 3,500, the paper's 4,905 and 4,734, six layers (256x256) 2,643 and 2,621, four 2,155 and 2,140, 192 filters
    // 3,094 and 3,060, five mixtures 2,672 and 2,650, seven 2,770 and 2,772 (but 8,257 and 8,118 for twelve of 768x512, with bands of 16); not
    // with 64 filters 3,980 and 4,005 and in diagonal order (768x512) 3,168 and 3,238.
    static constexpr bool kKeepAwake = true;
    // And with bands of 16 rows?  768x512, 8 to 20 images, us without and with: this network 4,977 and 4,847, 6,698 and 6,558, the paper's 6,070 and
    // 6,043, 6,882 and 6,861; four layers 5,452 and 5,516, 6,202 and 6,304.
    static constexpr bool kKeepAwakeWide = true;
    __host__ __device__ static constexpr int dim(int l) { return l == 0 ? 30 : l == 1 ? 160 : l == 2 ? 160 : l == 3 ? 128 : 60; }
    __host__ __device__ static constexpr int ob(int l) { return l == 0 ? 10 : l == 1 ? 10 : l == 2 ? 8 : 4; }
    __host__ __device__ static constexpr int kb(int l) { return l == 0 ? 1 : l == 1 ? 5 : l == 2 ? 5 : 4; }
    // Head output held by lane group g in register s = 4*out_block + i after the
    // last layer: groups 0..2 hold their channel's 15 parameters, group 3 the coupling coefficients.
    __host__ __device__ static constexpr int head_index(int g, int s) { return decoder_head_index<K>(g, s); }
    // First-layer operand: slots 0-3 (half 0) and 4-7 (half 1) of lane group g in k-block
    // kbi are four consecutive neighbour bytes of one row: row offset dr, first byte off
    // within the row's run that starts at column c-2.  Returns false for an unused half.
    __host__ __device__ static constexpr bool run_desc(int kbi, int g, int half, int& dr, int& off) {
        (void)kbi;
        if (half == 0) { dr = g < 2 ? -2 : -1; off = (g & 1) ? 8 : 0; }
        else { dr = g == 0 ? -2 : (g == 2 ? -1 : 0); off = g == 1 ? 0 : 4; }
        return true;
    }
    __host__ __device__ static constexpr int in_index(int kbi, int g, int i) { return run_in_index<NetWorkload>(kbi, g, i); }
};

// The paper's own network (Sec. III-B; hyper-parameter table of Sec. IV-E): the 12
// unmasked taps of a 5x5 first layer {rows r-2, r-1 at columns c-2..c+2; row r at c-2,
// c-1} -> 128 -> 128 -> 128 -> 128 -> 36, LeakyReLU (slope 0.01), K = 3, delay 3.
struct NetPaper {
    static constexpr int kLayers = 5;
    static constexpr int K = 3;
    static constexpr int kNbhd = 12, kDelay = 3;
    static constexpr int kReach1 = 2, kReach2 = 2;
    static constexpr int kUpBytes = 15;
    static constexpr int kRingCols = 16;
    static constexpr int kRingPad = 4;
    static constexpr bool kLeaky = true;
    static constexpr int kEncodeThreads = 512;
    static constexpr int kSharedCuLds = 6;
    static constexpr bool kSharedByCoefficient = false;
    static constexpr unsigned kSharedAlonePercent = 108, kSharedStepPercent = 137;
    static constexpr unsigned kNarrowPercent = 91, kNarrowAlonePercent = 100;
    static constexpr bool kKeepAwake = true, kKeepAwakeWide = true;
    __host__ __device__ static constexpr int dim(int l) { return l == 0 ? 36 : l == 5 ? 36 : 128; }
    __host__ __device__ static constexpr int ob(int l) { return l == 4 ? 3 : 8; }
    __host__ __device__ static constexpr int kb(int l) { return l == 0 ? 2 : 4; }
    __host__ __device__ static constexpr int head_index(int g, int s) { return decoder_head_index<K>(g, s); }
    __host__ __device__ static constexpr bool run_desc(int kbi, int g, int half, int& dr, int& off) {
        if (kbi == 0) { dr = g < 2 ? -2 : -1; off = ((g & 1) ? 8 : 0) + 4 * half; return true; }
        dr = 0; off = 4 * half;
        return g == 0;
    }
    __host__ __device__ static constexpr int in_index(int kbi, int g, int i) { return run_in_index<NetPaper>(kbi, g, i); }
};

// The same network in the diagonal decoding order (Sec. III-C, Eq. (7)): a pass decodes the
// anti-diagonal r + c = t (delay 1), so the neighbours (r-2,c+2), (r-1,c+1), (r-1,c+2) are not yet
// decoded; their nine inputs carry copies of pixel (r-1,c) instead.  The copies are made by
// reading that pixel's bytes again: extra runs that start at byte 5, 6 or 8 of row r-1.
struct NetDiagonal : NetPaper {
    static constexpr int kDelay = 1;
    static constexpr int kReach1 = 0, kReach2 = 1;   // row r-1 is read up to column c, row r-2 up to c+1
    static constexpr int kRingCols = 8;
    static constexpr int kRingPad = 4;
    static constexpr unsigned kSharedAlonePercent = 118, kSharedStepPercent = 138;
    static constexpr unsigned kNarrowPercent = 95, kNarrowAlonePercent = 48;
    static constexpr bool kKeepAwake = false, kKeepAwakeWide = false;
    __host__ __device__ static constexpr bool run_desc(int kbi, int g, int half, int& dr, int& off) {
        if (kbi == 0) {
            if (g == 0) { dr = -2; off = 4 * half; }                          // row r-2, bytes 0..7
            else if (g == 1) { dr = half ? -1 : -2; off = half ? 6 : 8; }     // row r-2 bytes 8..11 | copy for (r-2,c+2)
            else if (g == 2) { dr = -1; off = 4 * half; }                     // row r-1, bytes 0..7
            else { dr = -1; off = half ? 6 : 5; }                             // copies for (r-1,c+1) | (r-1,c+2)
            return true;
        }
        if (g == 0) { dr = 0; off = 4 * half; return true; }                  // row r, bytes 0..5
        dr = -1; off = 8;                                                     // row r-1 byte 8: pixel (r-1,c), blue
        return g == 1 && half == 0;
    }
    __host__ __device__ static constexpr int in_index(int kbi, int g, int i) {
        if (kbi == 0) {
            if (g == 0) return i;
            if (g == 1) return i < 4 ? 8 + i : (i < 7 ? 12 + (i - 4) : -1);
            if (g == 2) return 15 + i;
            return i == 0 ? -1 : (i < 4 ? 24 + (i - 1) : (i < 7 ? 27 + (i - 4) : -1));
        }
        if (g == 0) return i < 6 ? 30 + i : -1;
        return (g == 1 && i == 0) ? 23 : -1;
    }
};

// The paper's network with another number of mixture components, filters or layers (the ablations of
// Sec. IV-E; wavefront order): 36 -> C -> ... -> C -> 12 K, LAYERS weight layers, LeakyReLU.  K is 3, 5
// (the head layouts above) or 7, C a multiple of 32.  The encoder keeps in LDS what fits of the packed model: six
// layers of 128 filters fit without the CDF table, of 192 filters the first two layers (the other layers' weight
// tiles and, there, the table are read from global memory).
template <int MIXTURES, int C, int LAYERS>
struct NetAblation : NetPaper {
    static_assert((MIXTURES == 3 || MIXTURES == 5 || MIXTURES == 7) && C % 32 == 0 && C <= 192 && LAYERS >= 3 && LAYERS <= 7,
                  "unsupported shape");
    static constexpr int kLayers = LAYERS;
    static constexpr int K = MIXTURES;
    // 192 filters: a strip's activations and the next layer's take 192 registers, more than half of a lane's: with two waves to a
    // SIMD some 190 are spilled (4 images of 640x480: 882 us with 512 threads, 546 with 256).
    static constexpr int kEncodeThreads = C > 128 ? 256 : 512;
    static constexpr int kSharedCuLds = MIXTURES >= 7 || LAYERS >= 6 ? 7 : MIXTURES >= 5 ? 6 : 4;
    static constexpr unsigned kNarrowPercent = MIXTURES >= 7 ? 82 : MIXTURES >= 5 ? 88 : 91;
    static constexpr bool kKeepAwake = C >= 128, kKeepAwakeWide = C >= 128 && LAYERS > 4;
    static constexpr bool kSharedByCoefficient = C < 128;
    // (C = 192: a wave's weight slices alone are 264 registers; two workgroups per CU are never the better launch.)
    static constexpr unsigned kSharedAlonePercent = C > 128 ? 1000 : MIXTURES >= 7 ? 126 : MIXTURES >= 5 ? 107 : LAYERS >= 6 ? 114 : LAYERS <= 4 ? 104 : 101;
    static constexpr unsigned kSharedStepPercent = C > 128 ? 1000 : MIXTURES >= 7 ? 149 : MIXTURES >= 5 ? 135 : LAYERS >= 6 ? 141 : LAYERS <= 4 ? 130 : 123;
    __host__ __device__ static constexpr int dim(int l) { return l == 0 ? 36 : l == LAYERS ? 12 * MIXTURES : C; }
    __host__ __device__ static constexpr int ob(int l) { return (dim(l + 1) + 15) / 16; }
    __host__ __device__ static constexpr int kb(int l) { return (dim(l) + 31) / 32; }
    __host__ __device__ static constexpr int head_index(int g, int s) { return decoder_head_index<K>(g, s); }
};
using NetFewerLayers = NetAblation<3, 128, 4>;
using NetFewerFilters = NetAblation<3, 64, 5>;
using NetMoreMixtures = NetAblation<5, 128, 5>;
using NetMostMixtures = NetAblation<7, 128, 5>;
using NetMoreLayers = NetAblation<3, 128, 6>;
using NetMoreFilters = NetAblation<3, 192, 5>;

// Every canonical first-layer input sits in exactly one k-slot.
template <class Net>
constexpr bool inputs_placed_once() {
    for (int want = 0; want < Net::dim(0); ++want) {
        int n = 0;
        for (int kbi = 0; kbi < Net::kb(0); ++kbi)
            for (int g = 0; g < 4; ++g)
                for (int i = 0; i < 8; ++i) n += Net::in_index(kbi, g, i) == want ? 1 : 0;
        if (n != 1) return false;
    }
    return true;
}
static_assert(inputs_placed_once<NetWorkload>() && inputs_placed_once<NetPaper>() && inputs_placed_once<NetDiagonal>() &&
                  inputs_placed_once<NetFewerLayers>() &&
                  inputs_placed_once<NetFewerFilters>() && inputs_placed_once<NetMoreMixtures>() &&
                  inputs_placed_once<NetMostMixtures>() && inputs_placed_once<NetMoreLayers>() &&
                  inputs_placed_once<NetMoreFilters>(),
              "first-layer slot map");

constexpr int kBlockBytes = 64 * 16;  // one (out-block, k-block) A operand: 64 lanes x 8 bf16

// CDF table of the mixture's component distribution: F at z = (i - 768)/scale,
// i = 0..1536, as (value, forward difference).  scale = 128 for the Gaussian
// (|z| <= 6), 44 for the logistic of Eq. (8) (|z| <= 17.45, heavier tails).
constexpr int kLutEntries = 1537;
constexpr float kLutScaleGaussian = 128.0f;
constexpr float kLutScaleLogistic = 44.0f;
constexpr float kLutBias = 768.0f;
constexpr float kLutMax = 1536.0f;

// Packed model image: weight tiles layer by layer, fp32 biases (padded to the
// out-blocks), the CDF table, the table scale.
template <class Net>
struct Layout {
    __host__ __device__ static constexpr int w_off(int l) {
        int o = 0;
        for (int i = 0; i < l; ++i) o += Net::ob(i) * Net::kb(i) * kBlockBytes;
        return o;
    }
    static constexpr int kWeightBytes = w_off(Net::kLayers);
    __host__ __device__ static constexpr int b_off(int l) {
        int o = kWeightBytes;
        for (int i = 0; i < l; ++i) o += Net::ob(i) * 16 * 4;
        return o;
    }
    static constexpr int kLutOff = b_off(Net::kLayers);
    static constexpr int kLutScaleOff = kLutOff + (kLutEntries + 1) * 8;   // one float: table steps per unit of z
    static constexpr int kModelBytes = kLutScaleOff + 16;
    static constexpr int kHeadOB = Net::ob(Net::kLayers - 1);
    static constexpr int kHeadSlots = 4 * kHeadOB;                          // head registers per lane
    static_assert(kModelBytes % 16 == 0, "model image must be copyable in 16-byte pieces");
};
static_assert(Layout<NetWorkload>::kWeightBytes == 118784, "workload weight image size");

// The encoder's head.  A wave of the encoder takes a strip of 32 pixels, two MFMA tiles of 16; one exchange of rows of 16
// lanes per register (v_permlane16_swap) between the tiles' outputs gives every pixel two lanes, l and l + 32 ("halves"):
// half 0 holds lane groups 0 and 1 of both, half 1 groups 2 and 3.  The halves take a channel each, half 0 R and half 1 G, and
// share B's two CDF values, so that three evaluations per pixel and lane do for the strip's six per pixel (four where each lane
// group took a channel of its tile and a fourth group none).
// Register S of a half: its channel's 3 K parameters; in half 1 the K alphas; then B's 5 K values (parameters, betas, gammas),
// alternately in half 0 and half 1 of a register, from where both get them.  The last one of five mixtures does not fit there
// and stands in half 0 beside the alphas.
template <class Net>
struct EncHead {
    static constexpr int K = Net::K;
    static constexpr int kGroupSlots = Layout<Net>::kHeadSlots;       // registers of a lane group
    static constexpr int kSlots = 2 * kGroupSlots;
    static constexpr int kBItems = 5 * K;
    __host__ __device__ static constexpr int b_canonical(int b) { return b < 3 * K ? 6 * K + b : 10 * K + (b - 3 * K); }
    __host__ __device__ static constexpr int b_slot(int b) { return 4 * K + b / 2 < kSlots ? 4 * K + b / 2 : 3 * K + (4 * K + b / 2 - kSlots); }
    __host__ __device__ static constexpr int b_half(int b) { return 4 * K + b / 2 < kSlots ? b % 2 : 0; }
    // canonical head output in register S of half h, or -1
    __host__ __device__ static constexpr int index(int h, int S) {
        if (S < 3 * K) return 3 * K * h + S;
        if (h == 1 && S < 4 * K) return 9 * K + (S - 3 * K);
        for (int b = 0; b < kBItems; ++b) if (b_slot(b) == S && b_half(b) == h) return b_canonical(b);
        return -1;
    }
    // ... in register s of lane group g of a tile's outputs
    __host__ __device__ static constexpr int head_index(int g, int s) { return index(g >> 1, s + (g & 1) * kGroupSlots); }
    static constexpr bool placed_once() {
        for (int c = 0; c < Net::dim(Net::kLayers); ++c) {
            int n = 0;
            for (int g = 0; g < 4; ++g) for (int s = 0; s < kGroupSlots; ++s) n += head_index(g, s) == c ? 1 : 0;
            if (n != 1) return false;
        }
        return true;
    }
};
static_assert(EncHead<NetWorkload>::placed_once() && EncHead<NetPaper>::placed_once() && EncHead<NetMostMixtures>::placed_once(),
              "encoder's head layout");

// The head of the decoder with two workgroups per unit where Net::kSharedByCoefficient says so: groups 1 and 2 hold the first alphas and
// betas in the registers behind their channel's parameters, group 3 the others, one coefficient behind the other, then the gammas.  With
// five components the alphas, betas and gammas of a pixel are then a vector and a value each for a lane that takes them all (with
// component by component a value is read by itself, or with another in one instruction).
template <class Net>
struct SharedHead {
    static constexpr int K = Net::K, kSlots = Layout<Net>::kHeadSlots, kRoom = kSlots - 3 * K, kRest = K - kRoom;
    static_assert(kRoom >= 0 && kRest >= 0 && 2 * kRest + K <= kSlots, "the coefficients fit");
    __host__ __device__ static constexpr int head_index(int g, int s) {
        if (g < 3 && s < 3 * K) return 3 * K * g + s;
        if (g < 3) return g == 0 ? -1 : (8 + g) * K + s - 3 * K;
        if (s < kRest) return 9 * K + kRoom + s;
        if (s < 2 * kRest) return 10 * K + kRoom + s - kRest;
        return s < 2 * kRest + K ? 11 * K + s - 2 * kRest : -1;
    }
    static constexpr bool placed_once() {
        for (int c = 0; c < 12 * K; ++c) {
            int n = 0;
            for (int g = 0; g < 4; ++g) for (int s = 0; s < kSlots; ++s) n += head_index(g, s) == c ? 1 : 0;
            if (n != 1) return false;
        }
        return true;
    }
};
static_assert(SharedHead<NetWorkload>::placed_once() && SharedHead<NetFewerFilters>::placed_once(), "shared decoder's head layout");

// Feature index (within a 32-wide k-block) held in slot i of lane group g for
// the layers after the first: the two 16-row output tiles of the previous layer,
// as MFMA left them.
__host__ __device__ constexpr int kslot_feature(int g, int i) { return 16 * (i >> 2) + 4 * g + (i & 3); }

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0 .. N-1.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// ---------------------------------------------------------------------------
// bf16 helpers
// ---------------------------------------------------------------------------

// Hidden activations are carried as the sum of two bf16 numbers, a ~= hi + lo with
// hi = bf16(a), lo = bf16(a - hi) (both round to nearest even): 16 significant
// bits, so that the bf16 matrix cores reproduce the fp32 network to ~1e-5
// instead of ~1e-2.  Each weight tile is multiplied with hi and then with lo.
// ReLU as a signed integer maximum of the bit pattern (negative floats are negative
// integers), LeakyReLU as the median of {a, 0.01 a, +inf}: one instruction each, where
// fmaxf() would first re-canonicalise its operand.  (MFMA's NaN is a negative integer: ReLU makes it 0.)
template <bool LEAKY>
__device__ __forceinline__ float activation(float a) {
    if constexpr (LEAKY) return __builtin_amdgcn_fmed3f(a, 0.01f * a, __builtin_inff());
    else return __int_as_float(max(__float_as_int(a), 0));
}

typedef short bf16x4_bits_t __attribute__((ext_vector_type(4)));

// This lane's row of minus the 4x4 identity (rows repeat every four lanes), as bf16: the A operand of the split's subtraction.
__device__ __forceinline__ bf16x4_bits_t minus_identity(int lane) {
    const uint32_t one = 0xBF80u;                                    // -1
    u32x2_t v = {(lane & 2) ? 0u : ((lane & 1) ? one << 16 : one), (lane & 2) ? ((lane & 1) ? one << 16 : one) : 0u};
    asm volatile("" : "+v"(v));                                      // held in two registers, not made again where it is used
    return __builtin_bit_cast(bf16x4_bits_t, v);
}

// Applies the activation (ReLU, or LeakyReLU with slope 0.01) to two values and
// packs them: returns the hi pair, writes the lo pair.
template <bool LEAKY>
__device__ __forceinline__ uint32_t act_split_bf16(float a0, float a1, uint32_t& lo_pair) {
    a0 = activation<LEAKY>(a0);
    a1 = activation<LEAKY>(a1);
    const f32x2_t v = {a0, a1};
    const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
    const f32x2_t r = {a0 - __uint_as_float(hi << 16), a1 - __uint_as_float(hi & 0xFFFF0000u)};
    lo_pair = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2_t));
    return hi;
}

// The same for four values, with the subtractions on the matrix core: hi pairs and lo pairs.
// a - hi is one v_mfma_f32_4x4x4_16b_bf16, whose 16 blocks multiply, lane by lane, the lane's own four bf16 values with a
// 4x4 matrix: C - I hi, exact as the subtraction is (one product is not zero, and the difference has no more bits than a).
// Expanding hi and subtracting took eight vector instructions, a shift among them at half rate: 28 cycles for two waves
// of a SIMD against 8.3, and some 8 more where the matrix core changes between the two shapes.
template <bool LEAKY>
__device__ __forceinline__ void act_split4_bf16(const f32x4_t& acc, bf16x4_bits_t minus_one, u32x2_t& hi, u32x2_t& lo) {
    const f32x4_t a = {activation<LEAKY>(acc.x), activation<LEAKY>(acc.y), activation<LEAKY>(acc.z), activation<LEAKY>(acc.w)};
    const f32x2_t a01 = {a.x, a.y}, a23 = {a.z, a.w};
    hi.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(a01, bf16x2_t));
    hi.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(a23, bf16x2_t));
    f32x4_t r = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(minus_one, __builtin_bit_cast(bf16x4_bits_t, hi), a, 0, 0, 0);
    asm("" : "+v"(r));                                               // register allocation only: where the vector ALU reads it
    const f32x2_t r01 = {r.x, r.y}, r23 = {r.z, r.w};
    lo.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(r01, bf16x2_t));
    lo.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(r23, bf16x2_t));
}

// bf16 bit pattern of an integer 0..255 (exact).  The 1/256 input scaling is
// folded into the packed first-layer weights (a power of two, so exact).
__device__ __forceinline__ uint32_t byte_to_bf16(uint32_t x) {
    return __float_as_uint((float)x) >> 16;
}

// The same of a float that holds such an integer.
__device__ __forceinline__ uint16_t bf16_bits(float x) { return (uint16_t)(__float_as_uint(x) >> 16); }

// Four bytes of a run -> four bf16 (two packed pairs): the upper halves of the fp32 conversions.
__device__ __forceinline__ void run_to_bf16(uint32_t run, uint32_t& p01, uint32_t& p23) {
    const uint32_t sel = 0x07060302u;
    p01 = __builtin_amdgcn_perm(__float_as_uint((float)((run >> 8) & 0xFFu)), __float_as_uint((float)(run & 0xFFu)), sel);
    p23 = __builtin_amdgcn_perm(__float_as_uint((float)(run >> 24)), __float_as_uint((float)((run >> 16) & 0xFFu)), sel);
}

__device__ __forceinline__ f32x4_t mfma16(u32x4_t a, u32x4_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                    __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// The network on a strip of 32 pixels, two tiles of 16, held by one wave (encoder).
//   in[k-block][tile][0 = hi, 1 = lo]  B operands (8 bf16 per lane); the first layer's inputs are exact, their lo unused
//   out[out-block][tile]               raw head outputs, register 4 ob + i  <->  EncHead::head_index(lane >> 4, 4 ob + i)
// Accumulation order per output element: bias, then k-blocks 0,1,2,..., each hi then lo.
//
// A wave works through a layer in pairs of out-blocks (a pair is one k-block of the next layer) and k-block by k-block, all in
// the order written, which the scheduling barriers keep:
//   weights   are read two k-blocks ahead, across pairs and layers (`a`: those of the layer's first two), the next pair's
//             biases one k-block ahead;
//   split     the pair before (`last`; across layers too: it is the layer's last k-block) is activated and split into hi + lo
//             among this pair's MFMAs, three vector instructions beside one, the four subtractions on the matrix core together
//             (going from one MFMA shape to the other and back costs it some 8 cycles), and nothing is used right behind
//             the MFMA that makes it.
// Left to itself the compiler reads weights where they are used and waits for LDS in front of every other MFMA.
// ---------------------------------------------------------------------------
template <class Net, int L, int P, int KB>
struct KBlockAt {                      // layer, pair of out-blocks, k-block
    static constexpr int l = L, p = P, kb = KB;
    static constexpr bool valid = L < Net::kLayers;
    static constexpr int blocks = !valid ? 0 : 2 * P + 1 < Net::ob(L) ? 2 : 1;        // a layer of an odd number of out-blocks ends in half a pair
    static constexpr auto next() {
        if constexpr (!valid) return KBlockAt<Net, L, P, KB>{};
        else if constexpr (KB + 1 < Net::kb(L)) return KBlockAt<Net, L, P, KB + 1>{};
        else if constexpr (2 * P + 2 < Net::ob(L)) return KBlockAt<Net, L, P + 1, 0>{};
        else return KBlockAt<Net, L + 1, 0, 0>{};
    }
};
constexpr int kWeightsAhead = 2;       // k-blocks

// `model` holds the weight tiles of the first RESIDENT layers and, straight behind them, all biases (the packed image itself
// when RESIDENT is the number of layers); the other layers' tiles are read from the image at `rest`.
template <class Net, int RESIDENT>
struct EncoderNet {
    using Lay = Layout<Net>;
    const uint8_t* model;
    const uint8_t* rest;
    int lane;
    bf16x4_bits_t minus_one;

    template <class At>
    __device__ __forceinline__ void weights(At, u32x4_t (&a)[2]) const {
        const uint8_t* w = (At::l < RESIDENT ? model : rest) + lane * 16;
#pragma unroll
        for (int j = 0; j < At::blocks; ++j)
            a[j] = *reinterpret_cast<const u32x4_t*>(w + Lay::w_off(At::l) + ((2 * At::p + j) * Net::kb(At::l) + At::kb) * kBlockBytes);
    }
    template <class At>
    __device__ __forceinline__ void biases(At, f32x4_t (&b)[2]) const {
        const float* from = reinterpret_cast<const float*>(model + Lay::w_off(RESIDENT) + (Lay::b_off(At::l) - Lay::kWeightBytes)) + 4 * (lane >> 4);
#pragma unroll
        for (int j = 0; j < At::blocks; ++j) b[j] = *reinterpret_cast<const f32x4_t*>(from + 16 * (2 * At::p + j));
    }

    // The split of a pair, in pieces, eighths of its values: block e >> 2, tile (e >> 1) & 1, registers 2 (e & 1) and + 1.
    __device__ __forceinline__ void split_hi(f32x4_t (&v)[2][2], int e, u32x4_t (&to)[2][2]) const {
        f32x4_t& x = v[e >> 2][(e >> 1) & 1];
        const int i = 2 * (e & 1);
        const f32x2_t a = {activation<Net::kLeaky>(x[i]), activation<Net::kLeaky>(x[i + 1])};
        x[i] = a.x; x[i + 1] = a.y;
        to[(e >> 1) & 1][0][2 * (e >> 2) + (e & 1)] = __builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf16x2_t));
    }
    __device__ __forceinline__ void split_rest(f32x4_t (&v)[2][2], const u32x4_t (&to)[2][2]) const {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const u32x2_t h = {to[t][0][2 * j], to[t][0][2 * j + 1]};
                v[j][t] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(minus_one, __builtin_bit_cast(bf16x4_bits_t, h), v[j][t], 0, 0, 0);
            }
        }
    }
    __device__ __forceinline__ void split_lo(const f32x4_t (&v)[2][2], int e, u32x4_t (&to)[2][2]) const {
        const f32x4_t& x = v[e >> 2][(e >> 1) & 1];
        const f32x2_t a = {x[2 * (e & 1)], x[2 * (e & 1) + 1]};
        to[(e >> 1) & 1][1][2 * (e >> 2) + (e & 1)] = __builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf16x2_t));
    }
    // What of it goes behind MFMA M of a pair's NM (a layer's inputs are used from MFMA NM - 8 on, their lo from NM - 4 on).
    template <int M, int NM>
    __device__ __forceinline__ void split_piece(f32x4_t (&v)[2][2], u32x4_t (&to)[2][2]) const {
        constexpr int kHiPer = NM >= 24 ? 1 : NM >= 8 ? 2 : 4, kHi0 = NM >= 24 ? 2 : 1;
        constexpr int kRest = kHi0 + 8 / kHiPer - 1;
        constexpr int kLoPer = NM >= 24 ? 2 : NM >= 8 ? 4 : 8, kLo0 = NM >= 24 ? kRest + 3 : NM >= 16 ? kRest + 4 : NM >= 8 ? kRest + 2 : kRest + 1;
        static_assert(kLo0 + 8 / kLoPer <= (NM >= 16 ? NM - 4 : NM), "the split is done in time");
#pragma unroll
        for (int e = 0; e < 8; ++e) if (kHi0 + e / kHiPer == M) split_hi(v, e, to);
        if constexpr (kRest == M) {
            __builtin_amdgcn_sched_barrier(0);
            split_rest(v, to);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) if (kLo0 + e / kLoPer == M) split_lo(v, e, to);
        __builtin_amdgcn_sched_barrier(0);
    }

    // in: the layer's inputs; the last k-block's are still to be made of `last` (but in the first layer).  b: its first pair's biases.
    template <int L>
    __device__ __forceinline__ void layers(u32x4_t (&in)[Net::kb(L)][2][2], f32x4_t (&last)[2][2], u32x4_t (&a)[kWeightsAhead][2], f32x4_t (&b)[2],
                                           f32x4_t (&out)[Lay::kHeadOB][2]) const {
        constexpr bool kHead = L == Net::kLayers - 1;
        constexpr int NOB = Net::ob(L), NP = (NOB + 1) / 2, NKB = Net::kb(L), PARTS = L > 0 ? 2 : 1;
        static_assert(kHead || NOB == 2 * Net::kb(kHead ? L : L + 1), "two out-blocks form one k-block of the next layer");
        u32x4_t nxt[kHead ? 1 : NP][2][2];
        f32x4_t acc[2][2];
        static_for<0, NP>([&](auto pc) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value, NB = KBlockAt<Net, L, p, 0>::blocks, NM = NKB * PARTS * 4;
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j][0] = acc[j][1] = b[j];
            static_for<0, NKB>([&](auto kc) __attribute__((always_inline)) {
                constexpr int kb = decltype(kc)::value;
                using At = KBlockAt<Net, L, p, kb>;
                u32x4_t w[2];
#pragma unroll
                for (int j = 0; j < NB; ++j) w[j] = a[0][j];
                a[0][0] = a[1][0]; a[0][1] = a[1][1];
                weights(At::next().next(), a[1]);
                if constexpr (kb == (NKB > 1 ? NKB - 2 : 0)) biases(KBlockAt<Net, L, p, NKB - 1>::next(), b);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, 4 * PARTS>([&](auto mc) __attribute__((always_inline)) {
                    constexpr int m = decltype(mc)::value, part = m >> 2, j = (m >> 1) & 1, t = m & 1;
                    if constexpr (j < NB) acc[j][t] = mfma16(w[j], in[kb][t][part], acc[j][t]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (p == 0 && L > 0) split_piece<4 * PARTS * kb + m, NM>(last, in[NKB - 1]);
                    else if constexpr (p > 0 && !kHead) split_piece<4 * PARTS * kb + m, NM>(last, nxt[p - 1]);
                });
            });
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    if constexpr (kHead) out[2 * p + j][t] = acc[j][t];
                    last[j][t] = acc[j][t];
                }
            }
        });
        if constexpr (!kHead) layers<L + 1>(nxt, last, a, b, out);
    }

    __device__ __forceinline__ void run(u32x4_t (&in)[Net::kb(0)][2][2], f32x4_t (&out)[Lay::kHeadOB][2]) const {
        u32x4_t a[kWeightsAhead][2];
        f32x4_t b[2], last[2][2];
        using First = KBlockAt<Net, 0, 0, 0>;
        weights(First{}, a[0]);
        weights(First::next(), a[1]);
        biases(First{}, b);
        layers<0>(in, last, a, b, out);
    }
};

// ---------------------------------------------------------------------------
// Mixture parameters and the integer CDF (Eq. (1)-(4) of the paper).
// ---------------------------------------------------------------------------
template <int K>
struct ChanParams {
    float pi[K];   // mixture weights, softmax of the logits
    float mu[K];   // means, units of 1/256 of the grey range
    float a[K];    // table scale / sigma: table steps per unit of (edge - mu)
};

constexpr float kLog2e = 1.4426950408889634f;

// sigma = exp(clamp(log sigma, -8, 4)); a NaN counts as -8.  One instruction (fminf and fmaxf take three): the median of a NaN and two
// numbers is the smaller of the two, if the NaN is quiet (a signalling one counts as 4).  The matrix cores' results are: a head bias
// that is a signalling NaN arrives here as 0xFFC00000.  Values from elsewhere are made quiet first (cdf_tables_kernel).
__device__ __forceinline__ float clamp_log_sigma(float ls) { return __builtin_amdgcn_fmed3f(ls, -8.0f, 4.0f); }

// raw[0..K) logits, raw[K..2K) means, raw[2K..3K) log-sigmas of one channel.
template <int K>
__device__ __forceinline__ void channel_setup(const float (&raw)[3 * K], float lut_scale, ChanParams<K>& cp) {
    float m = raw[0];
#pragma unroll
    for (int k = 1; k < K; ++k) m = fmaxf(m, raw[k]);
    float e[K];
#pragma unroll
    for (int k = 0; k < K; ++k) e[k] = __builtin_amdgcn_exp2f((raw[k] - m) * kLog2e);
    float sum = e[0];
#pragma unroll
    for (int k = 1; k < K; ++k) sum = sum + e[k];
    const float inv = __builtin_amdgcn_rcpf(sum);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cp.pi[k] = e[k] * inv;
        cp.mu[k] = raw[K + k];
        const float ls = clamp_log_sigma(raw[2 * K + k]);
        cp.a[k] = __builtin_amdgcn_exp2f(-(ls * kLog2e)) * lut_scale;
    }
}

// One component of channel_setup: the same operations on the same inputs in the same order,
// so pi, mu, a equal cp.pi[k], cp.mu[k], cp.a[k] bit for bit.  logits[0..K) are the channel's
// logits; logit_k, mu_k, ls_k the component's own three head outputs.
template <int K>
__device__ __forceinline__ void channel_setup_one(const float (&logits)[K], float logit_k, float mu_k, float ls_k,
                                                  float lut_scale, float& pi, float& mu, float& a) {
    float m = logits[0];
#pragma unroll
    for (int k = 1; k < K; ++k) m = fmaxf(m, logits[k]);
    float e[K];
#pragma unroll
    for (int k = 0; k < K; ++k) e[k] = __builtin_amdgcn_exp2f((logits[k] - m) * kLog2e);
    float sum = e[0];
#pragma unroll
    for (int k = 1; k < K; ++k) sum = sum + e[k];
    const float inv = __builtin_amdgcn_rcpf(sum);
    pi = __builtin_amdgcn_exp2f((logit_k - m) * kLog2e) * inv;
    mu = mu_k;
    const float ls = clamp_log_sigma(ls_k);
    a = __builtin_amdgcn_exp2f(-(ls * kLog2e)) * lut_scale;
}

// Eq. (3): mu_g += alpha * r/256.   Eq. (4): mu_b += beta * r/256 + gamma * g/256.
template <int K>
__device__ __forceinline__ void couple_green(ChanParams<K>& cp, const float (&alpha)[K], float rhat) {
#pragma unroll
    for (int k = 0; k < K; ++k) cp.mu[k] = __builtin_fmaf(alpha[k], rhat, cp.mu[k]);
}
template <int K>
__device__ __forceinline__ void couple_blue(ChanParams<K>& cp, const float (&beta)[K], const float (&gamma)[K],
                                            float rhat, float ghat) {
#pragma unroll
    for (int k = 0; k < K; ++k) cp.mu[k] = __builtin_fmaf(gamma[k], ghat, __builtin_fmaf(beta[k], rhat, cp.mu[k]));
}

// Integer CDF at the lower edge of bin e (grey level e - 0.5), 1 <= e <= 255:
//   Cq(e) = e + min(floor(65280 * sum_k pi_k F(z_k)), 65280),  z_k = ((e-0.5)/256 - mu_k) / sigma_k.
// F (Phi, or the logistic CDF) is a table with linear interpolation at coordinate t = scale * z + 768,
// clamped to the table.  Entries are multiples of 2^-24 and the stored forward
// differences are exact, so one fma per lookup is non-decreasing in z; with
// pi_k >= 0 every later step (fma, floor) keeps that, hence Cq is strictly
// increasing in e and every symbol has frequency >= 1.
// In three parts, so that a caller can put other work between the table reads and their use: cq_lookup computes the
// table coordinates and issues the reads, cq_fractions needs the coordinates alone, cq_scaled interpolates, sums and scales.
template <int K>
struct CqLookup {
    float t[K];
    float2 td[K];
};

// Where entry i of the table lies in a copy of kSpreadLutBytes with 16 free bytes behind every 16 entries.  The decoder's
// 16 lanes of a pixel look up entries that lie equally far apart, and where that is a multiple of eight entries (eight for
// sigma = 1, the first sweep), four LDS banks would serve all of them.
__host__ __device__ constexpr uint32_t spread_at(uint32_t i) { return 8u * i + (i & ~15u); }
constexpr int kSpreadLutBytes = (int)spread_at(kLutEntries) + 8;
// Or four plain copies, a bank pair further on each, of which lanes 0 to 3 of the 16 read the first, lanes 4 to 7 the second and so on:
// entries that lie 8 / 2^k apart are then 2^k lanes apart on one bank in one copy at most.  One instruction a look-up less, for 49 KB.
constexpr int kLutCopies = 4, kLutCopyBytes = (((kLutEntries + 1) * 8 + 255) / 256) * 256 + 8;

// edge: the bin edge's position (2 e - 1) / 512, exact for every e.  TABLE: where the table is: at `lut`; a copy with free banks at LDS
// address 0 (an address the compiler knows: two instructions a look-up, a base it does not know would make it three); or a plain copy at
// LDS address `copy`.  The kernel that uses one in LDS has no static LDS, which would move its dynamic array: pcc_create refuses to
// go on with one that has.
enum class Table { kPlain, kSpread, kCopies };
template <int K, Table TABLE = Table::kPlain>
__device__ __forceinline__ void cq_lookup(const ChanParams<K>& cp, float edge, const float2* __restrict__ lut, CqLookup<K>& q, uint32_t copy = 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        q.t[k] = __builtin_amdgcn_fmed3f(__builtin_fmaf(edge - cp.mu[k], cp.a[k], kLutBias), 0.0f, kLutMax);
        const uint32_t i = (uint32_t)(int)q.t[k];                  // t >= 0: truncation is floor
        if constexpr (TABLE != Table::kPlain) {
            const f32x2_t v = *(const __attribute__((address_space(3))) f32x2_t*)(TABLE == Table::kSpread ? spread_at(i) : (i << 3) + copy);
            q.td[k].x = v.x; q.td[k].y = v.y;
        } else {
            q.td[k] = lut[i];
        }
    }
}

// What can be done while the reads are under way: t becomes its fraction.
template <int K>
__device__ __forceinline__ void cq_fractions(CqLookup<K>& q) {
#pragma unroll
    for (int k = 0; k < K; ++k) q.t[k] = __builtin_amdgcn_fractf(q.t[k]);
}

// 65280 min(sum, 1), whose floor is Cq(e) - e.  The sum is at least 0 and exceeds 1 by rounding at most, and 65280 times
// the minimum is what min(65280 sum, 65280) is.  A sum that is NaN (logits that are, or are infinite) counts as 1: all of
// the mass lies below bin 1 then.  (The result modifier of the last fma would limit the sum for nothing but make NaN 0.)
template <int K>
__device__ __forceinline__ float cq_scaled(const ChanParams<K>& cp, CqLookup<K>& q) {
    static_assert(K == 3 || K == 5 || K == 7, "the scheduling barrier below lists the table reads explicitly");
    float2 (&td)[K] = q.td;
    // Scheduling only: all table reads are in flight before the first is used
    // (one LDS latency per evaluation instead of K).
    if constexpr (K == 7) {
        asm volatile("" : "+v"(td[0].x), "+v"(td[0].y), "+v"(td[1].x), "+v"(td[1].y), "+v"(td[2].x), "+v"(td[2].y),
                          "+v"(td[3].x), "+v"(td[3].y), "+v"(td[4].x), "+v"(td[4].y), "+v"(td[5].x), "+v"(td[5].y),
                          "+v"(td[6].x), "+v"(td[6].y));
    } else if constexpr (K == 5) {
        asm volatile("" : "+v"(td[0].x), "+v"(td[0].y), "+v"(td[1].x), "+v"(td[1].y), "+v"(td[2].x), "+v"(td[2].y),
                          "+v"(td[3].x), "+v"(td[3].y), "+v"(td[4].x), "+v"(td[4].y));
    } else {
        asm volatile("" : "+v"(td[0].x), "+v"(td[0].y), "+v"(td[1].x), "+v"(td[1].y), "+v"(td[2].x), "+v"(td[2].y));
    }
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float phi = __builtin_fmaf(q.t[k], td[k].y, td[k].x);
        acc = __builtin_fmaf(cp.pi[k], phi, acc);
    }
    return fminf(acc, 1.0f) * 65280.0f;
}

template <int K>
__device__ __forceinline__ uint32_t cq_eval(const ChanParams<K>& cp, int e, const float2* __restrict__ lut) {
    CqLookup<K> q;
    cq_lookup<K>(cp, (float)(2 * e - 1) * (1.0f / 512.0f), lut, q);
    cq_fractions<K>(q);
    return (uint32_t)e + (uint32_t)cq_scaled<K>(cp, q);       // not negative: the conversion's truncation is the floor
}

template <int K>
__device__ __forceinline__ uint32_t cq_full(const ChanParams<K>& cp, int e, const float2* __restrict__ lut) {
    if (e <= 0) return 0u;
    if (e >= 256) return 65536u;
    return cq_eval<K>(cp, e, lut);
}

// ---------------------------------------------------------------------------
// rANS (one stream per image row): 64-bit state in [2^31, 2^63), 16-bit
// frequencies, 32-bit renormalisation words.
// ---------------------------------------------------------------------------
constexpr uint64_t kRansL = 1ull << 31;

}  // namespace pcc
