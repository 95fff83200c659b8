// Sparse convolution on the matrix cores of gfx950 (CDNA4).
//
// The same result as the tile kernel (kernels.hip), organised as a product: output channels x outputs, summed over
// (channel, tap).  The stored weights stand in a dense table with zeros between them (MatrixWeights), in the order the
// matrix instructions take them: v_mfma_f32_32x32x16_f16 multiplies 32 output channels x 16 input channels of one tap with
// 16 input channels x 32 outputs.  At 90 % sparsity nine tenths of the products are with zeros, yet it is the faster way:
// the tile kernel is bound by its LDS reads (16 bytes for 4 to 8 multiply-adds a lane) at 30 to 40 TFLOP/s of stored
// weights, where this kernel does 600 to 1100 TFLOP/s of all weights in binary16 (256 -> 512 channels, 28 x 28, batch 128,
// 90 %: 569 us by the tile kernel, 208 us here) and 200 to 330 in fp32 (256 -> 256, 14 x 14, batch 256, 70 %: 430 and 172 us).
//
// Tile.  A workgroup of four wavefronts owns consecutive outputs of the batch and keeps, chunk by chunk of channels, the
// lattice elements they touch in LDS, 8 channels of one position to a 16-byte element: a tap is an LDS offset, so the
// tile is loaded once for all R * S taps, and a fragment of inputs is one ds_read_b128 a lane, 32 consecutive elements
// for 32 consecutive outputs (outputs alone: no lane works on padding; a row's end costs a bank conflict, up to half of the
// LDS cycles, which are a third to a half of the time).  A wavefront's MK x NP fragments share MK weight and NP input fragments per
// step: 2 x 4 is what 256 registers hold.  Weight fragments come straight from L2 (each is used by one wavefront of the
// workgroup, or few), AHEAD steps before their use.
//
// Few outputs (a batch of one to some ten images, small maps) leave most CUs without a tile, and a wavefront alone on its SIMD takes some
// 240 clocks a step, the latencies of its weights and inputs, for 32 to 128 of products.  So there (binary16) eight wavefronts share the channels of a
// tile of 32 x 32 or 32 x 64: up to four times the workgroups, two wavefronts a SIMD, and chunks of twice the channels, a memory
// latency each.  1381 -> 385 channels, 14 x 14, one image, 70 %: 25.2 us by the tile kernel, 18.4 by four wavefronts, 9.5 so; 205 -> 100,
// 8 x 8, 5 x 5 taps, batch 26: 16.4 by four, 9.9; VGG-16's 512 -> 512 on 2 x 2, batch 256: 18.1 and 14.3.
//
// Order of the loads.  Vector loads return in order, so a weight fragment that is asked for after the loads of the next
// chunk's inputs waits for those.  All of a chunk's input loads are therefore issued together at its start, behind the
// weights of its first AHEAD steps, and those steps stand outside the loop: there the compiler can count exactly which
// loads are out (in the loop it would have to assume the fewest, and waited for everything at every step: 331 -> 243 us on
// the layer above).  For the same reason the number of loads does not depend on run-time conditions: FLY blocks of 64
// elements x 8 channels a wavefront (or of 64 runs of pixels x 8 channels: "Wide staging" below), of which the absent ones are
// out of the descriptor's range.
//
// fp32 layers.  A value is the sum of two binary16 numbers to 2^-23 of it; three of the four products of two such sums are
// multiplied (the fourth is 2^-22 of the result or less), smallest first.  binary16 has few exponents, so the weights of an
// output channel are scaled by a power of two of their own (those below 2^-16 of the largest, which two pieces do not hold, are
// few: they stand in a list and are multiplied as fp32; so are all weights of rows of few, which are more exact so), and the
// inputs by one for each image of the tile, taken from the image's largest magnitude in the first chunk.  The low piece of an
// input is kept times 2^12 and meets the high piece of the weight times 2^-12: so 29 binary orders of magnitude hold every value
// to 2^-23 (kWindow; without that factor 17).
//  * An input above its image's window is left out, and its chunk is multiplied once more with only what was left out, under
//    a scale that fits it, as often as something is left.
//  * An input below the window takes part with 11 bits.  Its place is marked, and if an output that sees a marked place has a
//    sum so small that what such inputs lack could be more than 2^-23 of its terms, they are taken out of the sums again and
//    multiplied in the same way.  (Normally distributed inputs: one tile in two thousand has such an input, and one in some
//    ten thousand repeats a chunk for it.)
// So every output has fp32's precision whatever else is in its tile, and no image's sums depend on another image.  Measured
// (256 -> 256, 14 x 14, batch 256, 70 %): this care is 3 % of the 180 us; 620 us for inputs spread evenly over 50 binary orders of
// magnitude, 275 if the second half of the channels is a million times the first.
// The sum of a chunk is added to that of the chunks before it, which keeps the
// rounding below that of a sum over all terms: 1.6e-7 of the result (2-norm, against 64 bits) for the layer above, 4.6e-7
// by the tile kernel.
//
// Non-finite inputs.  The table's zeros meet every input of the receptive field, so exactly the outputs with an input that
// is not finite have a sum that is not: those are summed again over the stored weights alone (a mask says which), one after
// the other, a lane a row, about 50 us each for 2304 columns.  Measured on the layer above (430 us by the tile kernel): 180 us,
// with one NaN (nine outputs of four wavefronts) 610, with nothing but NaN 5000.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "internal.h"

namespace sc {

namespace {

typedef _Float16 half2 __attribute__((ext_vector_type(2)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

#define SC_LDS __attribute__((address_space(3)))
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
__device__ __forceinline__ unsigned lds_address(const unsigned char* in_lds)
{
    return (unsigned)(unsigned long long)(const SC_LDS unsigned char*)(in_lds);
}
// The kernel's argument block read anew, through a pointer the compiler cannot trace back to it: for code that runs seldom or
// late.  Loaded with the rest at the kernel's start, what it needs would be spilled across the whole multiply loop.
__device__ __forceinline__ const MatrixArgs& late_arguments()
{
    auto p = (const __attribute__((address_space(4))) MatrixArgs*)(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(p));
    return *(const MatrixArgs*)(p);
}
__device__ __forceinline__ half8 lds_read(unsigned address) { return *(const SC_LDS half8*)(address); }
__device__ __forceinline__ void lds_write(unsigned address, half8 v) { *(SC_LDS half8*)(address) = v; }
template <typename V>
__device__ __forceinline__ void lds_put(unsigned address, V v) { *(SC_LDS V*)(address) = v; }
template <typename V>
__device__ __forceinline__ V lds_get(unsigned address) { return *(const SC_LDS V*)(address); }
#pragma clang diagnostic pop

// n / d for 0 <= n < 2^31 with the multiplier prepared on the host.
// (Without a case for d = 1, which became a branch each, some twenty before a kernel's first loads: VGG-16 of 32-pixel images 2 % less
// time in binary16, 1 % in fp32.)
__device__ __forceinline__ int fdiv(int n, const FastDiv& f)
{
    return (int)(__umulhi((unsigned)n << 1, f.mul) >> f.shift);
}

// One input value (as it lies in memory) through a buffer descriptor; out-of-range offsets read as zero.
template <typename T>
struct Raw;
template <>
struct Raw<_Float16> {
    typedef unsigned short type;
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rs, unsigned off, unsigned soff)
    {
        return __builtin_amdgcn_raw_buffer_load_b16(rs, (int)off, (int)soff, 0);
    }
};
template <>
struct Raw<float> {
    typedef unsigned type;
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rs, unsigned off, unsigned soff)
    {
        return __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, (int)soff, 0);
    }
};

// Eq. 1 for one output (i, j) of image u and the lane's row k over the stored weights alone.  All lanes of the wavefront take the
// same output: they load an input each and hand it round; only under inputs that are not finite the mask is asked.  Four steps'
// loads are on their way at once.
template <typename T>
__device__ __forceinline__ float stored_sum(const MatrixArgs& a, int u, int k, int i, int j, int lane)
{
    const T* x = static_cast<const T*>(a.x) + (size_t)u * a.C * a.H * a.W;
    constexpr int kParts = sizeof(T) == 4 ? 2 : 1, kGo = 4;
    const _Float16* w = static_cast<const _Float16*>(a.weights) + (size_t)(k >> 5) * a.stream_steps * kParts * 512 + (k & 31) * 8;
    const int exponent = kParts == 2 ? -a.row_exp[k] : 0;
    float sum = 0.f;
#pragma unroll 1
    for (int t = 0; t < a.stream_steps; t += kGo) {
        half8 weight[kGo][kParts][2];
        float in[kGo];
        int col[kGo];                                   // of the step's first channel
#pragma unroll
        for (int q = 0; q < kGo; ++q) {
            const int group = (t + q) / a.RS, tap = t + q - group * a.RS, r = tap / a.S, s = tap - r * a.S;
            const int c = group * 16 + lane, yy = i * a.stride + r - a.pad, xx = j * a.stride + s - a.pad;
            const bool inside = (t + q < a.stream_steps) & (lane < 16) & (c < a.C) & ((unsigned)yy < (unsigned)a.H) & ((unsigned)xx < (unsigned)a.W);
            in[q] = inside ? (float)x[((size_t)c * a.H + yy) * a.W + xx] : 0.f;
            col[q] = group * 16 * a.RS + tap;
#pragma unroll
            for (int p = 0; p < kParts; ++p)
#pragma unroll
                for (int h = 0; h < 2; ++h)             // (steps past the last: the table goes on further than that)
                    weight[q][p][h] = *reinterpret_cast<const half8*>(w + ((size_t)(t + q) * kParts + p) * 512 + h * 256);
        }
#pragma unroll
        for (int q = 0; q < kGo; ++q) {
            const bool ok = __builtin_fabsf(in[q]) <= 3.402823466e38f;
            const float real = ok ? in[q] : 0.f;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                float v = (float)weight[q][0][c >> 3][c & 7];
                if constexpr (kParts == 2) v = ldexpf(v + (float)weight[q][1][c >> 3][c & 7], exponent);
                sum = __builtin_fmaf(v, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(real), c)), sum);
            }
            unsigned long long others = __ballot(!ok);
#pragma unroll 1
            while (others) {
                const int c = __builtin_ctzll(others), at = col[q] + c * a.RS;
                others &= others - 1;
                const _Float16* one = w + (size_t)(t + q) * kParts * 512 + (c >> 3) * 256 + (c & 7);
                float v = (float)one[0];
                if constexpr (kParts == 2) v = ldexpf(v + (float)one[512], exponent);
                if (a.mask[(size_t)k * a.mask_words + (at >> 5)] >> (at & 31) & 1u)
                    sum = __builtin_fmaf(v, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(in[q]), c)), sum);
            }
        }
        if (!__ballot(sum == sum)) break;               // nothing changes a NaN
    }
    if constexpr (kParts == 2) {
        auto add = [&](const MatrixWeights::Small& w1) {
            const int r = w1.tap / a.S, yy = i * a.stride + r - a.pad, xx = j * a.stride + w1.tap - r * a.S - a.pad;
            if (w1.row == (k & 31) && yy >= 0 && yy < a.H && xx >= 0 && xx < a.W)
                sum = __builtin_fmaf(ldexpf(w1.weight, -a.row_exp[k]), (float)x[((size_t)w1.c * a.H + yy) * a.W + xx], sum);
        };
#pragma unroll 1
        for (int e = 0; e < MatrixWeights::kSlots; ++e) add(a.slots[(k >> 5) * MatrixWeights::kSlots + e]);
#pragma unroll 1
        for (int e = a.small_first[k >> 5]; e < a.small_first[(k >> 5) + 1]; ++e) add(a.small[e]);
    }
    return sum;
}

// fp32 inputs.  A window of binary orders of magnitude [base, base + kWindow) (biased exponents) whose values, scaled to
// 2^-14 .. 2^15, are held by the two pieces to 2^-23 of them, the low one times kLowScale.  In it the high piece is a normal
// number: the matrix instruction takes subnormal ones as what they are, but aligns their products as if they were 2^-14, and
// drops what then lies below fp32 (2^-38 of the other factor).  The first window leaves room for chunks kRoom orders above the
// first.
constexpr int kWindow = 29, kRoom = 2;
constexpr float kLowScale = 4096.f;
constexpr int kDefaultTop = 134;      // nothing seen to take a window from: values below 2^7
constexpr int kMaxApart = 64;         // windows further apart than this share no sum: the image's outputs are summed by themselves

__device__ __forceinline__ float window_scale(int base) { return __uint_as_float((unsigned)(240 - base) << 23); }
__device__ __forceinline__ int window_base(float scale) { return 240 - (int)(__float_as_uint(scale) >> 23); }
// the lowest window that ends with the biased exponent `last`; subnormal inputs are below any
__device__ __forceinline__ int window_ending(int last) { return last + 1 - kWindow > 1 ? last + 1 - kWindow : 1; }
// magnitudes (as bits) [low, high) of a window
__device__ __forceinline__ unsigned window_low(int base) { return (unsigned)base << 23; }
__device__ __forceinline__ unsigned window_high(int base) { return (unsigned)(base + kWindow < 255 ? base + kWindow : 255) << 23; }

// Eight inputs in two pieces each under a window's scale.  (By hand: the compiler takes half as many instructions again.)
__device__ __forceinline__ void cut(const float (&x)[8], float scale, half8& hi, half8& lo)
{
    uint4v high, low;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        unsigned h, l;
        float t0, t1;
        asm("v_fma_mixlo_f16 %0, %4, %6, 0\n\t"
            "v_fma_mixhi_f16 %0, %5, %6, 0\n\t"
            "v_mul_f32 %2, %4, %7\n\t"
            "v_mul_f32 %3, %5, %7\n\t"
            "v_fma_mixlo_f16 %1, %0, %8, %2 op_sel_hi:[1,0,0]\n\t"
            "v_fma_mixhi_f16 %1, %0, %8, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
            "s_nop 0"
            : "=&v"(h), "=&v"(l), "=&v"(t0), "=&v"(t1)
            : "v"(x[2 * j]), "v"(x[2 * j + 1]), "v"(scale), "v"(scale * kLowScale), "s"(-kLowScale));
        high[j] = h;
        low[j] = l;
    }
    hi = __builtin_bit_cast(half8, high);
    lo = __builtin_bit_cast(half8, low);
}

// The windows of one image of the tile, in LDS.
struct ImageWindow {
    float first;           // scale of the first window
    float scale;           // the present one's
    unsigned low, high;    // the present one's magnitudes
    unsigned above, below; // largest magnitude left to do above the first window, and below
};
static_assert(sizeof(ImageWindow) == kImageWindowBytes, "what the plan reserves in LDS");

// The window of the next round: from the largest magnitude that is left, those above the first window before those below.
__device__ __forceinline__ void next_window(ImageWindow& w)
{
    const int first = window_base(w.first);
    const unsigned top = w.above ? w.above : w.below;
    w.low = w.high = 0u;
    if (!top) return;
    const int base = window_ending((int)(top >> 23));
    const unsigned low = window_low(base), high = window_high(base);
    w.scale = window_scale(base);
    if (w.above) {
        w.low = low < window_high(first) ? window_high(first) : low;
        w.high = high;
        w.above = 0u;
    } else {
        w.low = top < low ? 1u : low;                       // (subnormal ones: a window by themselves)
        w.high = top < low ? low : high < window_low(first) ? high : window_low(first);
        w.below = 0u;
    }
}
// The window's values can be added to the sums: it is near enough to the first one, and its values are normal numbers.
__device__ __forceinline__ bool summable(const ImageWindow& w)
{
    const int by = window_base(w.scale) - window_base(w.first);
    return by >= -kMaxApart && by <= kMaxApart && w.high > window_low(1);
}

}  // namespace

// Wavefronts of a workgroup.
template <int KS>
constexpr int kWaves = KS > 4 ? KS : 4;

// Wavefronts a SIMD holds at least: the smallest variant (1 x 1 layers mostly, which load and store more than they multiply)
// would take 130 registers, fits 128 without scratch, and four of it are faster than three (64 -> 256 channels, 56 x 56, binary16: 47 and
// 55 us; 40 layers 1.5 % in the mean, one 2 % slower).
template <typename T, int MK, int NP, int AHEAD, int FLY, int KS, bool WIDE>
constexpr int kResident = sizeof(T) == 2 && MK * NP == 4 && AHEAD == 2 && FLY <= 2 && KS == 1 && !WIDE ? 4 : 2;

template <typename T, int MK, int NP, int AHEAD, int FLY, int KS, bool WIDE>
__global__ __launch_bounds__(64 * kWaves<KS>, (kResident<T, MK, NP, AHEAD, FLY, KS, WIDE>)) void matrix_kernel(const MatrixArgs a)
{
    using raw = typename Raw<T>::type;
    constexpr int kPx = WIDE ? 8 / (int)sizeof(T) : 1;          // pixels of a channel a lane stages
    using staged = std::conditional_t<WIDE, uint2v, raw>;
    constexpr bool kSplit = sizeof(T) == 4;
    constexpr int kParts = kSplit ? 2 : 1;      // binary16 pieces a value is held in
    constexpr int kW = kWaves<KS>, kThreads = 64 * kW;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, half = lane >> 5;
    const int bid = blockIdx.x;
    const int item = (bid & 7) * (int)(gridDim.x >> 3) + (bid >> 3);
    if (item >= a.ntiles * a.kblocks) return;
    // (tile, channel block) pairs are cut into 8 contiguous ranges, one per XCD, numbered so that the larger of input and
    // weight table is read by as few XCDs as can be: tile-major, an XCD reads its tiles' input and the whole table,
    // block-major the other way round
    const int major = a.block_major ? a.ntiles : a.kblocks;
    const int outer = item / major, inner = item - outer * major;
    const int tile = a.block_major ? inner : outer, kb = a.block_major ? outer : inner;
    // KS = 1: the wavefronts share the tile's output channels and outputs out among them; KS = 4 (8): each works on the
    // whole tile for a quarter (an eighth) of every chunk's channels
    const int wk = KS == 1 ? wave & (a.WK - 1) : 0, wp = KS == 1 ? wave >> a.logWK : 0;
    const int ks = KS == 1 ? 0 : wave;
    const int kf0 = (kb * a.WK + wk) * MK;      // first block of 32 output channels of this wavefront

    // Bias and scale of the workgroup's rows, in LDS for the store step: loaded from memory there they would cost a latency
    // each workgroup, and at each row wait for the stores before it (loads and stores share one counter).
    const int rows = (KS == 1 ? a.WK : 1) * MK * 32;
    float* row_bias = reinterpret_cast<float*>(smem + a.meet_at + 64);
    int* row_exp = reinterpret_cast<int*>(smem + a.meet_at + 64) + rows;
    // kSplit: the first small weights of the workgroup's blocks, the windows of its images
    MatrixWeights::Small* slots = reinterpret_cast<MatrixWeights::Small*>(smem + a.meet_at + 64 + 8 * rows);
    ImageWindow* images = reinterpret_cast<ImageWindow*>(slots + rows / 32 * MatrixWeights::kSlots);
    unsigned* marks = reinterpret_cast<unsigned*>(images + a.images);                          // kSplit: a bit per lattice element
    unsigned* meet = reinterpret_cast<unsigned*>(smem + a.meet_at);   // kSplit: [0..1] chunks (modulo 64) with values that the
                                                                      // first windows do not hold, [2] some sum is short of them,
                                                                      // [3] how many values are below them
    float my_bias = 0.f;      // (a row a thread; on their way while the first chunk's inputs are)
    if (tid < rows && kb * rows + tid < a.K) {
        if (a.bias) my_bias = a.bias[kb * rows + tid];
        if constexpr (kSplit) row_exp[tid] = a.row_exp[kb * rows + tid];
    }
    if constexpr (kSplit)     // (no register to spare for it there)
    {
        if (tid < rows) row_bias[tid] = my_bias;
        if (tid < rows / 32 * MatrixWeights::kSlots) {
            const int at = kb * rows / 32 * MatrixWeights::kSlots + tid;
            slots[tid] = at < a.KF * MatrixWeights::kSlots ? a.slots[at] : MatrixWeights::Small{-1, 0, 0, 0.f};
        }
        for (int i = tid; i < a.images; i += kThreads) images[i].above = 0u;
        for (int i = tid; i < a.EB * 2; i += kThreads) marks[i] = 0u;
        if (tid < 4) meet[tid] = 0u;
    }

    // outputs of the tile and where their receptive fields start in the lattice
    const int o0 = tile * a.PT;
    auto lattice = [&](int o) {
        const int u = fdiv(o, a.fd_EF);
        const int rem = o - u * a.EF;
        const int i = fdiv(rem, a.fd_F);
        return (u * a.Hs + i * a.stride) * a.Wp + (rem - i * a.F) * a.stride;
    };
    const int q0 = lattice(o0);
    const int u0 = fdiv(o0, a.fd_EF);
    const unsigned lds0 = lds_address(smem);
    const unsigned plane = (unsigned)a.EB * 64u * 16u;           // bytes of one group of 8 channels
    const unsigned part = plane * (unsigned)a.CG;                // bytes of one piece of a buffer
    const unsigned buffer = part * kParts;
    auto image_of = [&](int o, const MatrixArgs& a) { return fdiv(o < a.nout ? o : a.nout - 1, a.fd_EF) - u0; };   // counted from the tile's first
    unsigned at[NP];
#pragma unroll
    for (int np = 0; np < NP; ++np) {
        const int o = o0 + (wp * NP + np) * 32 + (lane & 31);
        at[np] = lds0 + (unsigned)(lattice(o < a.nout ? o : a.nout - 1) - q0) * 16u + ((unsigned)half + (unsigned)(ks * a.own_groups) * 2u) * plane;
    }

    // ---- weights: one stream of steps per block of 32 output channels
    constexpr size_t frag = 64 * 8;                              // halves of one fragment
    const size_t stream = (size_t)a.stream_steps * kParts * frag;
    const _Float16* wa[MK];
    // the wavefront's first group of 16 channels of a chunk.  (Eight wavefronts: past the last one, the first of those that the
    // table holds behind it, whatever the chunk lacks: they meet zeros of the input.)
    auto group_of = [&](int ch, const MatrixArgs& a) __attribute__((always_inline)) {
        const int g = ch * (a.CG / 2) + ks * a.own_groups;
        if constexpr (KS > 4) return g < a.groups ? g : a.groups;
        return g;
    };
    auto weights_of = [&](int ch, const MatrixArgs& a) __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)                          // blocks past the last repeat it (never stored)
            wa[mk] = static_cast<const _Float16*>(a.weights) + (size_t)(kf0 + mk < a.KF ? kf0 + mk : a.KF - 1) * stream +
                     (size_t)(group_of(ch, a) * a.RS) * kParts * frag;
    };
    weights_of(0, a);
    // from the end of a chunk's steps of this wavefront to the next chunk's first
    const ptrdiff_t skip = KS == 1 ? 0 : (ptrdiff_t)((a.CG / 2 - a.own_groups) * a.RS) * (ptrdiff_t)(kParts * frag);
    const unsigned lane8 = (unsigned)lane * 8u;
    half8 A[AHEAD][MK][kParts];
    auto load_a = [&](half8(&dst)[MK][kParts]) __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) {
#pragma unroll
            for (int p = 0; p < kParts; ++p) dst[mk][p] = *reinterpret_cast<const half8*>(wa[mk] + p * frag + lane8);
            wa[mk] += kParts * frag;
        }
    };

    // ---- staging: blocks of 64 lattice elements x 8 channels
    const unsigned chan_bytes = (unsigned)(a.H * a.W) * (unsigned)sizeof(T);
    const size_t img_bytes = (size_t)a.C * chan_bytes;
    const size_t base_off = (size_t)u0 * img_bytes;
    const size_t remain = (size_t)a.N * img_bytes - base_off;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(a.x)) + base_off, 0, remain > 0x80000000ull ? 0x80000000u : (unsigned)remain, 0x00020000);
    const int nblk = a.CG * a.EB;               // blocks of a chunk
    // Wide staging.  The address unit takes some 20 clocks for a load of 64 lanes, 2 bytes each or 8 (512 -> 512 channels, 4 x 4,
    // binary16, batch 256: of 37.6 us, 13 were these loads).  So where planes are whole runs of kPx pixels, a lane takes runs: all
    // pixels of the tile's lattice elements are consecutive, images one behind the other, and the padding between them, which no
    // run holds, is cleared once.  (That layer's best split: 37.5 -> 26.4 us; in fp32, batch 128: 51.3 -> 37.1.)  A block is 64
    // runs, those of all channel groups one behind the other.  Inputs start at any element, as vector memory loads 8 bytes from
    // any address: 2 bytes off a word that layer takes 24.8 us for 23.6 (single pixels: 33.3), 2 x 2 maps 21.4 for 18.0.
    // Planes that are not whole runs end in one that overlaps the run before it (ragged_runs: 173 -> 354 channels, 25 x 25, binary16,
    // 91 %, batch 5: 17.2 -> 13.8 us).
    const int nwide = WIDE ? (a.CG * a.quads + 63) >> 6 : 0;
    int quad0 = 0;                              // the tile's first run
    if constexpr (WIDE) {
        const int Y = fdiv(q0, a.fd_Wp), X = q0 - Y * a.Wp - a.pad, y = Y - fdiv(Y, a.fd_Hs) * a.Hs - a.pad;
        const int inside = y < 0 ? 0 : y * a.W + (X < 0 ? 0 : X < a.W ? X : a.W);
        quad0 = u0 * a.plane_quads + (inside < a.H * a.W ? inside : a.H * a.W) / kPx;
    }
    const int blocks = WIDE ? nwide : nblk;     // what the wavefronts share
    staged st[FLY][8];
    // run b * 64 + lane: its channel group, image and first pixel.  (The last run of a plane that is not whole ones begins
    // before the one before it ends: both write the same there.)
    auto run_of = [&](int b, int& cg, int& u, int& at, const MatrixArgs& a) __attribute__((always_inline)) {
        const int n = b * 64 + lane;
        cg = fdiv(n, a.fd_quads);
        const int quad = quad0 + n - cg * a.quads;
        u = fdiv(quad, a.fd_plane_quads);
        at = (quad - u * a.plane_quads) * kPx;
        at = at < a.last_run ? at : a.last_run;
    };
    auto load_runs = [&](uint2v(&dst)[8], int ch, int b, const MatrixArgs& a) __attribute__((always_inline)) {
        int cg, u, at;
        run_of(b, cg, u, at, a);
        const bool ok = (u < a.N) & (cg < a.CG) & (ch < a.nchunks);
        const unsigned off = (unsigned)(u - u0) * (unsigned)img_bytes + (unsigned)(cg * 8) * chan_bytes + (unsigned)at * (unsigned)sizeof(T);
        const int left = ok ? a.C - (ch * a.CG + cg) * 8 : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int c = ch * a.CG * 8 + j;                     // (the descriptor's range is what lies behind this channel: it has to be there)
            const unsigned from = c < a.C ? (unsigned)c * chan_bytes : 0u;
            dst[j] = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rs, j < left ? (int)off : (int)0x80000000u, (int)from, 0));
        }
    };
    // the loads of block b of chunk ch; absent blocks (and channels past the last) are out of the descriptor's range
    // and read as zero, so that nothing here is a branch
    auto load_block = [&](raw(&dst)[8], int ch, int b, const MatrixArgs& a) __attribute__((always_inline)) {
        const int cg = fdiv(b, a.fd_EB), eb = b - cg * a.EB;
        const int L = q0 + eb * 64 + lane;
        const int Y = fdiv(L, a.fd_Wp), X = L - Y * a.Wp - a.pad;
        const int u = fdiv(Y, a.fd_Hs), yy = Y - u * a.Hs - a.pad;
        const bool ok = (u < a.N) & ((unsigned)yy < (unsigned)a.H) & ((unsigned)X < (unsigned)a.W) & (b < nblk) & (ch < a.nchunks);
        const unsigned at0 = (unsigned)(u - u0) * (unsigned)img_bytes + (unsigned)(yy * a.W + X) * (unsigned)sizeof(T);
        const unsigned off = ok ? at0 : 0x80000000u;
        const int c0 = (ch * a.CG + cg) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = c0 + j < a.C;
            dst[j] = Raw<T>::load(rs, in ? off : 0x80000000u, in ? (unsigned)(c0 + j) * chan_bytes : 0u);
        }
    };
    // kSplit: the image of the lane's element of block b, counted from the tile's first
    auto image_of_block = [&](int b, const MatrixArgs& a) __attribute__((always_inline)) {
        const int cg = fdiv(b, a.fd_EB), eb = b - cg * a.EB;
        return fdiv(fdiv(q0 + eb * 64 + lane, a.fd_Wp), a.fd_Hs) - u0;
    };
    bool outside = false;                       // kSplit: some value is not in its image's window
    auto store_element = [&](const raw(&src)[8], float scale, unsigned to) __attribute__((always_inline)) {
        half8 hi, lo;
        if constexpr (kSplit) {
            unsigned least = ~0u;               // of twice the magnitude bits, less one: zeros are the largest
            float most = 0.f, x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                x[j] = __uint_as_float(src[j]);
                const unsigned twice = ((unsigned)src[j] << 1) - 1u;
                least = twice < least ? twice : least;
            }
#pragma unroll
            for (int j = 0; j < 8; j += 2)      // (fmaxf would first make every operand a quiet number)
                asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(x[j]), "v"(x[j + 1]));
            cut(x, scale, hi, lo);
            const int base = window_base(scale);
            outside = outside | (most >= __uint_as_float(window_high(base))) | (least < ((unsigned)base << 24) - 1u);
            lds_write(to + part, lo);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) __builtin_memcpy(reinterpret_cast<char*>(&hi) + 2 * j, &src[j], 2);
        }
        lds_write(to, hi);
    };
    auto store_block = [&](const raw(&src)[8], float scale, int buf, int b) __attribute__((always_inline)) {
        const int cg = fdiv(b, a.fd_EB), eb = b - cg * a.EB;
        store_element(src, scale, lds0 + (unsigned)buf * buffer + (unsigned)cg * plane + (unsigned)(eb * 64 + lane) * 16u);
    };
    auto store_runs = [&](const uint2v(&src)[8], float scale, int buf, int b) __attribute__((always_inline)) {
        int cg, u, at;
        run_of(b, cg, u, at, a);
        const int y = fdiv(at, a.fd_W), x = at - y * a.W;
        const int e0 = (u * a.Hs + a.pad + y) * a.Wp + a.pad + x - q0;
        const unsigned to = lds0 + (unsigned)buf * buffer + (unsigned)cg * plane;
#pragma unroll
        for (int p = 0; p < kPx; ++p) {
            const int e = e0 + p + (x + p >= a.W ? a.Wp - a.W : 0);            // (a run goes over a row's end once at most)
            raw one[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if constexpr (kSplit) one[j] = src[j][p];
                else one[j] = (raw)(src[j][p / 2] >> (p % 2 * 16));
            }
            if ((cg < a.CG) & ((unsigned)e < (unsigned)(a.EB * 64))) store_element(one, scale, to + (unsigned)e * 16u);
        }
    };
    // kSplit: this wavefront's blocks of a chunk once more, value by value.  First round: without what is above its image's
    // window, and with 11 bits of what is below it, which is marked and counted.  Later rounds: of the values above the first
    // window, or of those below it, only what is in the present window; between the two, under an empty window, those below it
    // as they were first but with their signs turned, which takes them out of the sums (11 bits by 11: exactly).  The largest
    // of what is left is remembered.  (Values that are not finite belong to the first round.)
    auto restage = [&](int ch, int buf, bool first) __attribute__((always_inline)) {
        const MatrixArgs& a = late_arguments();
        auto again_element = [&](const raw(&src)[8], int cg, int e, ImageWindow& w) __attribute__((always_inline)) {
            const unsigned to = lds0 + (unsigned)buf * buffer + (unsigned)cg * plane + (unsigned)e * 16u;
            const int base = window_base(w.first);
            const unsigned low = w.low, high = w.high, bottom = window_low(base), top = window_high(base);
            const bool lows = !first & (low < top), out = lows & (low == high) & (low != 0u);
            unsigned left = 0u;
            int strays = 0;
            float x[8];
            half8 hi, lo, eleven;                                 // eleven: values below the window, low pieces only
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const unsigned bits = (unsigned)src[j], m = bits & 0x7fffffffu;
                const float v = __uint_as_float(out ? bits ^ 0x80000000u : bits);
                const bool stray = (m < bottom) & (m != 0u), high_one = (m >= top) & (m < 0x7f800000u);
                const bool in = first ? !stray & !high_one : (lows ? stray & !out : high_one) & (m - low < high - low);
                x[j] = in ? v : 0.f;
                const float y = ((first | out) & stray) ? v * (w.scale * kLowScale) : 0.f;
                eleven[j] = (_Float16)(__builtin_fabsf(y) >= 0x1p-14f ? y : 0.f);
                const bool rest = first ? high_one : (lows ? stray : high_one) & (m < low);
                left = (rest & (m > left)) ? m : left;
                strays += stray;
            }
            cut(x, w.scale, hi, lo);
#pragma unroll
            for (int j = 0; j < 8; ++j) lo[j] += eleven[j];       // (one of the two is zero)
            lds_write(to, hi);
            lds_write(to + part, lo);
            if (left) atomicMax(lows ? &w.below : &w.above, left);
            if (first) {
                if (strays) {
                    atomicOr(&marks[e >> 5], 1u << (e & 31));
                    atomicAdd(&meet[3], (unsigned)strays);
                }
                if (strays | (int)left) atomicOr(&meet[ch >> 5 & 1], 1u << (ch & 31));
            }
        };
#pragma unroll 1
        for (int b = wave; b < blocks; b += kW) {
            if constexpr (WIDE) {
                uint2v src[8];
                load_runs(src, ch, b, a);
                int cg, u, at;
                run_of(b, cg, u, at, a);
                const int y = fdiv(at, a.fd_W), x = at - y * a.W;
                const int e0 = (u * a.Hs + a.pad + y) * a.Wp + a.pad + x - q0;
#pragma unroll 1
                for (int p = 0; p < kPx; ++p) {
                    const int e = e0 + p + (x + p >= a.W ? a.Wp - a.W : 0);
                    raw one[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) one[j] = p ? src[j][1] : src[j][0];
                    if ((cg < a.CG) & ((unsigned)e < (unsigned)(a.EB * 64))) again_element(one, cg, e, images[u - u0]);
                }
            } else {
                raw src[8];
                load_block(src, ch, b, a);
                const int cg = fdiv(b, a.fd_EB), eb = b - cg * a.EB;
                again_element(src, cg, eb * 64 + lane, images[image_of_block(b, a)]);
            }
        }
    };
    auto load = [&](staged(&dst)[8], int ch, int b) __attribute__((always_inline)) {
        if constexpr (WIDE) load_runs(dst, ch, b, a);
        else load_block(dst, ch, b, a);
    };
    // kSplit: the image of what the lane stages in block b, counted from the tile's first (past its last: not stored)
    auto staged_image = [&](int b) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            int cg, u, at;
            run_of(b, cg, u, at, a);
            return u - u0;
        } else {
            return image_of_block(b, a);
        }
    };
    auto staged_scale = [&](int b) __attribute__((always_inline)) {
        const int image = staged_image(b);
        return images[!WIDE || image < a.images ? image : 0].first;
    };
    auto fetch = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FLY; ++i) load(st[i], ch, wave + kW * i);
    };
    float scale[kSplit ? FLY : 1];              // kSplit: of the blocks in flight
    auto take_scales = [&]() __attribute__((always_inline)) {
        if constexpr (kSplit) {
#pragma unroll
            for (int i = 0; i < FLY; ++i)
                if (wave + kW * i < blocks) scale[i] = staged_scale(wave + kW * i);
        }
    };
    auto deposit = [&](int ch, int buf) __attribute__((always_inline)) {
        auto store = [&](const staged(&src)[8], float scale, int b) __attribute__((always_inline)) {
            if constexpr (WIDE) store_runs(src, scale, buf, b);
            else store_block(src, scale, buf, b);
        };
#pragma unroll
        for (int i = 0; i < FLY; ++i)
            if (wave + kW * i < blocks) store(st[i], scale[kSplit ? i : 0], wave + kW * i);
        for (int b = wave + kW * FLY; b < blocks; b += kW) {      // what does not fit in flight
            staged more[8];
            load(more, ch, b);
            store(more, kSplit ? staged_scale(b) : 0.f, b);
        }
        if constexpr (kSplit) {
            if (__builtin_expect(__ballot(outside) != 0, 0)) {
                restage(ch, buf, true);
                outside = false;
            }
        }
    };

    // kSplit: the first windows, from the largest finite magnitudes of the loads in flight
    auto first_windows = [&]() __attribute__((always_inline)) {
        __syncthreads();                                         // the table is cleared
#pragma unroll
        for (int i = 0; i < FLY; ++i) {
            unsigned top = 0;
            auto see = [&](unsigned bits) __attribute__((always_inline)) {
                const unsigned m = bits & 0x7fffffffu;
                top = ((m < 0x7f800000u) & (m > top)) ? m : top;
            };
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if constexpr (WIDE) see(st[i][j][0]), see(st[i][j][1]);
                else see((unsigned)st[i][j]);
            }
            const int image = staged_image(wave + kW * i);
            if (top && (!WIDE || image < a.images)) atomicMax(&images[image].above, top);           // (absent blocks hold zeros)
        }
        __syncthreads();
        for (int i = tid; i < a.images; i += kThreads) {
            const unsigned top = images[i].above;
            const int last = top ? (int)(top >> 23) + kRoom : kDefaultTop - 1;
            const int base = window_ending(last < 254 ? last : 254);
            images[i] = ImageWindow{window_scale(base), window_scale(base), window_low(base), window_high(base), 0u, 0u};
        }
        __syncthreads();
    };

    auto for_steps = [&](auto& step, int t, int ch, bool more) __attribute__((always_inline)) {
        if constexpr (KS > 1) {   // the weights asked for during a chunk's last steps are the next chunk's
            ptrdiff_t jump = 0;
            if (more && t + AHEAD >= a.own_steps) jump = KS > 4 ? (ptrdiff_t)((group_of(ch + 1, a) - group_of(ch, a) - a.own_groups) * a.RS) * (ptrdiff_t)(kParts * frag) : skip;
#pragma unroll
            for (int mk = 0; mk < MK; ++mk) wa[mk] += jump;
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) step(A[i]);
    };

    float16v acc[MK][NP];
    float16v sum[kSplit ? MK : 1][kSplit ? NP : 1];   // kSplit: the chunks before this one
    half8 B[NP][kParts];
    constexpr int kMK = KS > 1 ? 1 : MK, kNP = KS > 1 ? 1 : NP;   // pairs a wavefront finishes
    unsigned bad = 0;   // one bit per np: the sums of the lane's output np are not to be had this way
    float apart[kSplit ? NP : 1];                     // kSplit: from the present window's scale to the first one's
#pragma unroll
    for (int np = 0; np < (kSplit ? NP : 1); ++np) apart[np] = 1.f;
#pragma unroll
    for (int mk = 0; mk < MK; ++mk)
#pragma unroll
        for (int np = 0; np < NP; ++np)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc[mk][np][i] = 0.f;
                if constexpr (kSplit) sum[mk][np][i] = 0.f;
            }
    fetch(0);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load_a(A[i]);
    if constexpr (WIDE) {                                // the padding is cleared while the first loads are on their way
        const half8 zero = {};
        const unsigned all = a.padded ? (a.nchunks > 1 ? 2u : 1u) * buffer : 0u;
        for (unsigned i = (unsigned)tid * 16u; i < all; i += (unsigned)kThreads * 16u) lds_write(lds0 + i, zero);
    }
    if constexpr (kSplit) first_windows();
    take_scales();
    if constexpr (WIDE && !kSplit)
        if (a.padded) __syncthreads();                   // the padding is cleared (kSplit: behind the windows' barriers)
    deposit(0, 0);
    if constexpr (!kSplit)
        if (tid < rows) row_bias[tid] = my_bias;
    __syncthreads();

    auto chunk = [&](int ch, auto more) __attribute__((always_inline)) {
        constexpr bool kMore = decltype(more)::value;
        if constexpr (kMore) fetch(ch + 1);
        const unsigned here = (unsigned)(ch & 1) * buffer;
        auto read_b = [&](int np, unsigned o) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < kParts; ++p) B[np][p] = lds_read(at[np] + o + (unsigned)p * part);
        };
#pragma unroll
        for (int np = 0; np < NP; ++np) read_b(np, here);
        int r = 0, s = 0;
        unsigned group = here;                               // the 16 channels the step is at
        const unsigned end = here + (unsigned)(2 * a.own_groups) * plane;
        auto step = [&](half8(&W)[MK][kParts]) __attribute__((always_inline)) {
            // where the next step reads (after the chunk's last one: somewhere in the chunk, unused)
            ++s;
            const bool row_done = s == a.S;
            s = row_done ? 0 : s;
            r += row_done ? 1 : 0;
            const bool group_done = r == a.R;
            r = group_done ? 0 : r;
            group += group_done ? 2 * plane : 0u;
            group = group >= end ? here : group;
            const unsigned off = group + (unsigned)(r * a.Wp + s) * 16u;
#pragma unroll
            for (int np = 0; np < NP; ++np) {
                if constexpr (kSplit) {
#pragma unroll
                    for (int mk = 0; mk < MK; ++mk) acc[mk][np] = __builtin_amdgcn_mfma_f32_32x32x16_f16(W[mk][1], B[np][0], acc[mk][np], 0, 0, 0);
#pragma unroll
                    for (int mk = 0; mk < MK; ++mk)
                        acc[mk][np] = __builtin_amdgcn_mfma_f32_32x32x16_f16(W[mk][0] * (_Float16)(1.f / kLowScale), B[np][1], acc[mk][np], 0, 0, 0);
                }
#pragma unroll
                for (int mk = 0; mk < MK; ++mk) acc[mk][np] = __builtin_amdgcn_mfma_f32_32x32x16_f16(W[mk][0], B[np][0], acc[mk][np], 0, 0, 0);
                // The reads stay where they are, between this fragment's products and the next one's, which hide them.  (The
                // compiler moved a step's products together and its reads behind them, where the next step waited for them:
                // 128 -> 256 channels, 8 x 8, binary16, batch 256: 22.0 -> 19.2 us; 512 -> 512, 4 x 4, fp32, batch 128: 58.4 -> 51.3.)
                __builtin_amdgcn_sched_barrier(0);
                read_b(np, off);
                __builtin_amdgcn_sched_barrier(0);
            }
            load_a(W);
        };
        // the first steps stand by themselves: their weights were asked for before the loads of the next chunk
        for_steps(step, 0, ch, kMore);
        for (int t = AHEAD; t < a.own_steps; t += AHEAD) for_steps(step, t, ch, kMore);
        if constexpr (kSplit) {
#pragma unroll
            for (int mk = 0; mk < MK; ++mk)
#pragma unroll
                for (int np = 0; np < NP; ++np) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        sum[mk][np][i] = kMore ? sum[mk][np][i] + acc[mk][np][i] : __builtin_fmaf(acc[mk][np][i], apart[np], sum[mk][np][i]);
                        acc[mk][np][i] = 0.f;
                    }
                }
        }
        if constexpr (kMore) deposit(ch + 1, (ch + 1) & 1);
        __syncthreads();
    };
    // kSplit: some image has inputs, or parts of some, that are left to do (every wavefront gets the same answer)
    auto anything_left = [&](const MatrixArgs& a) __attribute__((always_inline)) {
        unsigned some = 0;
        __syncthreads();
        for (int i = 0; i < a.images; ++i) some |= images[i].above | images[i].below;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane((int)some) != 0;
    };
    // kSplit: an output of the lane sees a marked input, and a sum of it is so small that what the products with such inputs
    // lack may be more than 2^-23 of its terms' magnitudes, which are no less than the sum: of each, 2^-11 for the low piece's
    // rounding and as much for the weight's low piece, of less than 2^-14 times a weight of less than 2^15
    auto short_sums = [&](const MatrixArgs& a) __attribute__((always_inline)) {
        unsigned sees = 0;
#pragma unroll
        for (int np = 0; np < NP; ++np)
#pragma unroll 1
            for (int t = 0; t < a.RS; ++t) {
                const int e = (int)((at[np] - lds0) % plane >> 4) + t / a.S * a.Wp + t % a.S;
                sees |= (marks[e >> 5] >> (e & 31) & 1u) << np;
            }
        const unsigned strays = meet[3];
        const float floor = 16384.f * (float)(strays < (unsigned)a.longest ? strays : (unsigned)a.longest);
        bool yes = false;
#pragma unroll
        for (int np = 0; np < NP; ++np)
#pragma unroll
            for (int mk = 0; mk < MK; ++mk)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    yes |= (sees >> np & 1u) & !(__builtin_fabsf(sum[mk][np][i]) >= floor) &
                           ((kf0 + mk) * 32 + half * 4 + (i >> 2) * 8 + (i & 3) < a.K);
        return yes;
    };
    int last = 0;
    for (; last + 1 < a.nchunks; ++last) chunk(last, std::true_type{});
    // kSplit: chunks of which the first windows did not hold everything are multiplied again, round after round with the
    // windows of what is still left (each round holds every image's largest, so it ends with less)
    unsigned long long again = 0;                     // those chunks, modulo 64
    if constexpr (kSplit)                             // (all chunks have been staged)
        again = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)meet[1]) << 32) |
                (unsigned)__builtin_amdgcn_readfirstlane((int)meet[0]);
    // kSplit: the small weights are multiplied as fp32, two columns a product.  The inputs of the first ones are on their way
    // during the last chunk.
    bool few[MK];
    float few_w[MK][2], few_x[MK][2][NP];
    auto small_input = [&](const MatrixWeights::Small& w, int np, const MatrixArgs& a) __attribute__((always_inline)) {
        const int o = o0 + (wp * NP + np) * 32 + (lane & 31), oo = o < a.nout ? o : a.nout - 1;
        const int u = fdiv(oo, a.fd_EF), rem = oo - u * a.EF, i = fdiv(rem, a.fd_F), r = w.tap / a.S;
        const int yy = i * a.stride + r - a.pad, xx = (rem - i * a.F) * a.stride + w.tap - r * a.S - a.pad;
        const bool in = (w.row >= 0) & ((unsigned)yy < (unsigned)a.H) & ((unsigned)xx < (unsigned)a.W);
        return in ? (float)static_cast<const T*>(a.x)[(((size_t)u * a.C + w.c) * a.H + yy) * a.W + xx] : 0.f;
    };
    if constexpr (kSplit) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) {
            const MatrixWeights::Small* mine = slots + (wk * MK + mk) * MatrixWeights::kSlots;
            few[mk] = ks == 0 && __builtin_amdgcn_readfirstlane(mine->row) >= 0;
            if (!few[mk]) continue;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const MatrixWeights::Small w = mine[q * 2 + half];
                few_w[mk][q] = w.row == (lane & 31) ? w.weight : 0.f;
#pragma unroll
                for (int np = 0; np < NP; ++np) few_x[mk][q][np] = small_input(w, np, late_arguments());
            }
        }
    }
    bool begun = false, short_of = false;             // short_of: the values below the windows are needed in full, and not yet looked for
    for (;;) {
        chunk(last, std::false_type{});
        if constexpr (!kSplit) {
            break;
        } else {
            if (__builtin_expect(!again, 1)) break;
            if (!begun) {
                begun = true;
                if (short_sums(late_arguments())) meet[2] = 1u;
                __syncthreads();
                short_of = __builtin_amdgcn_readfirstlane((int)meet[2]) != 0;
                last = a.nchunks;
            }
            do ++last;
            while (last < a.nchunks && !(again >> (last & 63) & 1u));
            if (last >= a.nchunks) {                              // the next round
                const MatrixArgs& a = late_arguments();
                const bool some = anything_left(a);
                if (!some && !short_of) break;
                for (int i = tid; i < a.images; i += kThreads) {
                    if (some) {
                        next_window(images[i]);
                    } else {                                      // those below: out of the sums
                        images[i].low = images[i].high = window_low(window_base(images[i].first));
                        images[i].scale = images[i].first;
                    }
                }
                short_of = short_of & some;
                __syncthreads();
#pragma unroll
                for (int np = 0; np < NP; ++np) {
                    const ImageWindow& w = images[image_of(o0 + (wp * NP + np) * 32 + (lane & 31), a)];
                    apart[np] = summable(w) ? __uint_as_float((unsigned)(127 + window_base(w.scale) - window_base(w.first)) << 23) : 0.f;
                    if (w.high && !summable(w)) bad |= 1u << np;
                }
                last = 0;
                while (!(again >> (last & 63) & 1u)) ++last;
            }
            weights_of(last, late_arguments());
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) load_a(A[i]);
            restage(last, last & 1, false);
            __syncthreads();
        }
    }
    if constexpr (kSplit) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) {
            if (!few[mk]) continue;
            const MatrixArgs& a = late_arguments();
            float scale[NP];
#pragma unroll
            for (int np = 0; np < NP; ++np) scale[np] = images[image_of(o0 + (wp * NP + np) * 32 + (lane & 31), a)].first;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int np = 0; np < NP; ++np)
                    sum[mk][np] = __builtin_amdgcn_mfma_f32_32x32x2f32(few_w[mk][q], few_x[mk][q][np] * scale[np], sum[mk][np], 0, 0, 0);
            const int end = a.small_first[kf0 + mk + 1];
#pragma unroll 1
            for (int e = a.small_first[kf0 + mk]; e < end; e += 8) {
                float weight[4], x[4][NP];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int mine = e + q * 2 + half;
                    MatrixWeights::Small w = a.small[mine < end ? mine : e];
                    if (mine >= end) w.row = -1;
                    weight[q] = w.row == (lane & 31) ? w.weight : 0.f;
#pragma unroll
                    for (int np = 0; np < NP; ++np) x[q][np] = small_input(w, np, a) * scale[np];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int np = 0; np < NP; ++np)
                        sum[mk][np] = __builtin_amdgcn_mfma_f32_32x32x2f32(weight[q], x[q][np], sum[mk][np], 0, 0, 0);
            }
        }
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int np = 0; np < NP; ++np) acc[mk][np] = sum[mk][np];
    }
    if constexpr (KS > 1) {
        // the wavefronts' sums of a (mk, np) pair meet at the wavefront with the pair's number, always added in
        // the same order (nobody reads the tile any more: its place is free)
        constexpr int kPairs = MK * NP;
        static_assert(kPairs <= KS, "a pair a wavefront at most");
        float* meeting = reinterpret_cast<float*>(smem);
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int np = 0; np < NP; ++np)
#pragma unroll
                for (int i = 0; i < 16; ++i) meeting[((ks * kPairs + mk * NP + np) * 16 + i) * 64 + lane] = acc[mk][np][i];
        __syncthreads();
        if (wave < kPairs) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float v = meeting[((size_t)wave * 16 + i) * 64 + lane];
#pragma unroll
                for (int q = 1; q < KS; ++q) v += meeting[(((size_t)q * kPairs + wave) * 16 + i) * 64 + lane];
                acc[0][0][i] = v;
            }
        }
        __syncthreads();
        if (kPairs < KS && wave >= kPairs) return;
        bad = bad >> (wave % NP) & 1u;
    }
#pragma unroll
    for (int np = 0; np < kNP; ++np) {
        // (a value that is not finite makes 0 * value, and every sum with it, a NaN: one instruction a value, in two chains; 128 values
        // compared one by one took 1.3 to 1.6 us, 0.4 so)
        float none[2] = {0.f, 0.f};
#pragma unroll
        for (int mk = 0; mk < kMK; ++mk)
#pragma unroll
            for (int i = 0; i < 16; ++i) none[i & 1] = __builtin_fmaf(acc[mk][np][i], 0.f, none[i & 1]);
        const float all = none[0] + none[1];
        bad |= all == all ? 0u : 1u << np;
    }
    bad |= (unsigned)__shfl_xor((int)bad, 32);           // the lane that holds the other rows of the same outputs

    // ---- store
    // (binary16 layers store faster without: 64 -> 256 channels, 56 x 56, batch 128: 95 us, and 102 with the arguments read late here)
    const MatrixArgs& la = [&]() -> const MatrixArgs& {
        if constexpr (kSplit) return late_arguments();
        return a;
    }();
    // (kSplit, and the variant of 128 registers: the lane's number is asked for anew: kept since the kernel's start it would be spilled)
    int late_lane = lane;
    if constexpr (kSplit || kResident<T, MK, NP, AHEAD, FLY, KS, WIDE> == 4) {
        late_lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(late_lane));
    }
    const int late_half = late_lane >> 5;
    T* __restrict__ y = static_cast<T*>(la.y);
    const int kfirst = (kf0 + (KS > 1 ? wave / NP : 0)) * 32;                  // first output channel and
    const int ofirst = o0 + (wp * NP + (KS > 1 ? wave % NP : 0)) * 32;         // first output of the wavefront's sums
    const int krow0 = kfirst + late_half * 4;
    // section 3: bias, then activation.  (The larger of a number and a NaN is the number: one instruction with ReLU and without, and
    // a NaN becomes 0 under ReLU, as where it is compared with 0.)
    const float least = la.relu ? 0.f : __builtin_nanf("");
    auto finish = [&](float v, float b) __attribute__((always_inline)) { return __builtin_fmaxf(v + b, least); };
    // What the table holds for the lane's 16 rows of a fragment, in registers before the fragment's first store (read
    // inside the branches below, each of them would wait for its own).
    const int table_row = kfirst - kb * rows + late_half * 4;
    float4 bias[4];
    int4 rexp[4];
    auto take_rows = [&](int mk) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bias[q] = *reinterpret_cast<const float4*>(row_bias + table_row + mk * 32 + q * 8);
            asm volatile("" : "+v"(bias[q].x), "+v"(bias[q].y), "+v"(bias[q].z), "+v"(bias[q].w));
            if constexpr (kSplit) {
                rexp[q] = *reinterpret_cast<const int4*>(row_exp + table_row + mk * 32 + q * 8);
                asm volatile("" : "+v"(rexp[q].x), "+v"(rexp[q].y), "+v"(rexp[q].z), "+v"(rexp[q].w));
            }
        }
    };
    auto at4 = [](const auto& v, int i) __attribute__((always_inline)) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; };
    auto unscale = [&](int o) __attribute__((always_inline)) {                 // kSplit: the exponent its sums lack, but for the row's
        if constexpr (kSplit) return window_base(images[image_of(o, la)].first) - 113;
        return 0;
    };
    auto scaled = [&](float v, int i, int exponent) __attribute__((always_inline)) {
        if constexpr (kSplit) v = ldexpf(v, exponent - at4(rexp[i >> 2], i & 3));
        return finish(v, at4(bias[i >> 2], i & 3));
    };
    // Outputs in runs.  A store of 64 lanes takes the address unit some 20 clocks, 2 bytes each or 16, and 32 binary16 outputs of a
    // row are half a cache line.  So where planes are whole runs of 16 (8) bytes, a block of 32 rows goes through the tile's
    // place in LDS, and a lane stores a run of one row, past the caches: the launch does not read it again.  (64 -> 256 channels,
    // 56 x 56, binary16, batch 128, 257 MB: 90 -> 83 us with runs, 61 with runs past the caches; 256 -> 512, 28 x 28: 254 -> 244 and
    // 240; 256 -> 256, 14 x 14, fp32, batch 256: 200 -> 200 and 194; all by launches repeated on the same buffers.  With inputs that
    // change from launch to launch the first takes 87 us one by one and 56 so.)
    constexpr int kPitch = kNP * 32 * (int)sizeof(T) + 16;
    auto put_runs = [&](int mk, auto run) __attribute__((always_inline)) {
        using Run = decltype(run);
        constexpr int kRun = (int)(sizeof(Run) / sizeof(T)), kRuns = kNP * 32 / kRun;           // outputs of a run, runs of a row
        const MatrixArgs& la = late_arguments();
        int own = late_lane;
        asm volatile("" : "+v"(own));            // (what follows is not worked out before, nor for both kinds of runs)
        const int row = own / kRuns, o = ofirst + own % kRuns * kRun;
        const unsigned from = lds0 + (unsigned)((wave * 32 + row) * kPitch) + (unsigned)(own % kRuns) * (unsigned)sizeof(Run);
        Run v[32 * kRuns / 64];
#pragma unroll
        for (int r = 0; r < 32 * kRuns / 64; ++r) v[r] = lds_get<Run>(from + (unsigned)(r * (64 / kRuns) * kPitch));
#pragma unroll
        for (int r = 0; r < 32 * kRuns / 64; ++r) asm volatile("" : "+v"(v[r]));       // (not read in the branches, one wait each)
        const int u = fdiv(o, la.fd_EF), k = kfirst + mk * 32 + row;
        Run* to = reinterpret_cast<Run*>(static_cast<T*>(la.y) + ((size_t)u * la.K + k) * la.EF + (o - u * la.EF));
        const int rows_left = o < la.nout ? la.K - k : 0;
        const size_t step = (size_t)(64 / kRuns) * la.EF / kRun;
#pragma unroll
        for (int r = 0; r < 32 * kRuns / 64; ++r) {
            if (r * (64 / kRuns) < rows_left) {
                if constexpr (sizeof(Run) == 16) __builtin_nontemporal_store(v[r], to + r * step);
                else to[r * step] = v[r];
            }
        }
    };
    // Pooled outputs in runs.  A wavefront's outputs are whole pairs of rows, so its maxima are consecutive too.  One by one each of
    // a fragment's 16 registers takes a store of which a quarter of the lanes hold something, and on rows of 16 or fewer a trip through
    // LDS for the row below: 14.4 us of 36 (128 -> 128 channels, 16 x 16, binary16, batch 256; 64 -> 64, 32 x 32: 7.1 of 31), 3.2
    // (3.5) so.  So all outputs go to LDS as above and a lane reads the windows of a run.  (Rows of two have windows of half
    // a word in two rows; they stay one by one.)
    auto put_pooled = [&](int mk, auto run) {
        using Run = decltype(run);
        constexpr int kRun = (int)(sizeof(Run) / sizeof(T)), kRuns = kNP * 8 / kRun, kAll = 32 * kRuns;
        constexpr int kPasses = kAll > 64 ? kAll / 64 : 1;
        using Pair = std::conditional_t<kSplit, uint2v, unsigned>;             // two maxima
        const MatrixArgs& la = late_arguments();
        int own = late_lane;
        asm volatile("" : "+v"(own));
        const int row = own / kRuns & 31, F = la.F, logQ = __builtin_ctz((unsigned)F) - 2;     // F / 4 windows of two in a row
        const unsigned from = lds0 + (unsigned)((wave * 32 + row) * kPitch), below = (unsigned)F * (unsigned)sizeof(T);
        auto two = [&](unsigned at) __attribute__((always_inline)) -> Pair {
            if constexpr (kSplit) {
                const float4v a = lds_get<float4v>(at), b = lds_get<float4v>(at + below);
                const float p = a.x > b.x ? a.x : b.x, q = a.y > b.y ? a.y : b.y, r = a.z > b.z ? a.z : b.z, s = a.w > b.w ? a.w : b.w;
                return Pair{__float_as_uint(p > q ? p : q), __float_as_uint(r > s ? r : s)};
            } else {
                const half4 a = lds_get<half4>(at), b = lds_get<half4>(at + below), m = __builtin_elementwise_max(a, b);
                return __builtin_bit_cast(unsigned, __builtin_elementwise_max(half2{m[0], m[2]}, half2{m[1], m[3]}));
            }
        };
        Run v[kPasses];
#pragma unroll
        for (int r = 0; r < kPasses; ++r)
#pragma unroll
            for (int t = 0; t < kRun / 2; ++t) {
                const int n = (own % kRuns * kRun >> 1) + t, p = n >> logQ, q = n & ((1 << logQ) - 1);
                const Pair pair = two(from + (unsigned)(r * (64 / kRuns) * kPitch) + (unsigned)(p * 2 * F + q * 4) * (unsigned)sizeof(T));
                if constexpr (kSplit) v[r][2 * t] = pair[0], v[r][2 * t + 1] = pair[1];
                else v[r][t] = pair;
            }
#pragma unroll
        for (int r = 0; r < kPasses; ++r) asm volatile("" : "+v"(v[r]));
        const int o = ofirst + own % kRuns * kRun * 4, u = fdiv(o, la.fd_EF), k = kfirst + mk * 32 + row;
        const int plane_out = la.EF >> 2;
        Run* to = reinterpret_cast<Run*>(static_cast<T*>(la.y) + ((size_t)u * la.K + k) * plane_out + ((o - u * la.EF) >> 2));
        const int rows_left = o < la.nout && (kAll >= 64 || own < kAll) ? la.K - k : 0;
        const size_t step = (size_t)(64 / kRuns) * plane_out / kRun;
#pragma unroll
        for (int r = 0; r < kPasses; ++r) {
            if (r * (64 / kRuns) < rows_left) {
                if constexpr (sizeof(Run) == 16) __builtin_nontemporal_store(v[r], to + r * step);
                else to[r * step] = v[r];
            }
        }
    };
    const bool in_runs = late_arguments().out_runs && __ballot(bad != 0) == 0;
    // (the sums as they are: else the compiler copies them apart before the branch, and the smallest variant spills)
#pragma unroll
    for (int mk = 0; mk < kMK; ++mk)
#pragma unroll
        for (int np = 0; np < kNP; ++np) asm volatile("" : "+v"(acc[mk][np]));
    if (in_runs) {
#pragma unroll
        for (int mk = 0; mk < kMK; ++mk) {
            take_rows(mk);
            unsigned to = lds0 + (unsigned)((wave * 32 + late_half * 4) * kPitch) + (unsigned)(late_lane & 31) * (unsigned)sizeof(T);
            asm volatile("" : "+v"(to));         // (the rest of an address is the instruction's offset, not two additions a value:
                                                 // with ReLU by one instruction 4.7 -> 3.3 us for 2 x 4 fragments)
#pragma unroll
            for (int np = 0; np < kNP; ++np) {
                const int exponent = unscale(ofirst + np * 32 + (late_lane & 31));
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    lds_put(to + (unsigned)(((i >> 2) * 8 + (i & 3)) * kPitch + np * 32 * (int)sizeof(T)), (T)scaled(acc[mk][np][i], i, exponent));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (late_arguments().pool) {
                if (late_arguments().out_runs == 16) put_pooled(mk, uint4v{});
                else put_pooled(mk, uint2v{});
            } else {
                if (late_arguments().out_runs == 16) put_runs(mk, uint4v{});
                else put_runs(mk, uint2v{});
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    } else
#pragma unroll
    for (int mk = 0; mk < kMK; ++mk) {
        take_rows(mk);
        if (!la.pool) {
#pragma unroll
            for (int np = 0; np < kNP; ++np) {
                const int o = ofirst + np * 32 + (late_lane & 31);
                const int u = fdiv(o, la.fd_EF);
                const bool valid = o < la.nout && !((bad >> np) & 1u);
                const int exponent = unscale(o);
                T* to = y + ((size_t)u * la.K + krow0) * la.EF + (o - u * la.EF);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int kr = mk * 32 + (i >> 2) * 8 + (i & 3);
                    if (krow0 + kr < la.K && valid) to[(size_t)kr * la.EF] = (T)scaled(acc[mk][np][i], i, exponent);
                }
            }
        } else {
            // 2 x 2 maximum: the wavefront's outputs hold whole pairs of rows of F outputs (the planner's condition).  The
            // value below is F / 32 registers or F lanes away, the one to the right one lane.  (Scale, bias and activation
            // are monotonic: they are applied to the largest of the four sums.)
            const int F = la.F, apart = F >> 5;
            const size_t plane_out = (size_t)(la.E >> 1) * (F >> 1);
#pragma unroll
            for (int np = 0; np < kNP; ++np) {
                if (apart && ((np / apart) & 1)) continue;
                unsigned wrong = bad >> np;
                if (apart == 1 && np + 1 < kNP) wrong |= bad >> (np + 1 < kNP ? np + 1 : 0);
                if (apart == 2 && np + 2 < kNP) wrong |= bad >> (np + 2 < kNP ? np + 2 : 0);
                wrong &= 1u;
                if (!apart) wrong |= (unsigned)__shfl_xor((int)wrong, F);
                wrong |= (unsigned)__shfl_xor((int)wrong, 1);
                const int o = ofirst + np * 32 + (late_lane & 31);
                const int u = fdiv(o, la.fd_EF);
                const int rem = o - u * la.EF, i0 = fdiv(rem, la.fd_F), j0 = rem - i0 * F;
                const bool valid = o < la.nout && !wrong && !((i0 | j0) & 1);
                const int exponent = unscale(o);
                T* to = y + ((size_t)u * la.K + krow0) * plane_out + (size_t)(i0 >> 1) * (F >> 1) + (j0 >> 1);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int kr = mk * 32 + (i >> 2) * 8 + (i & 3);
                    float v = acc[mk][np][i];
                    float below = v;
                    if (apart == 1) below = acc[mk][np + 1 < kNP ? np + 1 : np][i];
                    if (apart == 2) below = acc[mk][np + 2 < kNP ? np + 2 : np][i];
                    if (!apart) below = __shfl_xor(v, F);
                    v = below > v ? below : v;
                    const float right = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));   // lane ^ 1
                    v = right > v ? right : v;
                    if (krow0 + kr < la.K && valid) to[(size_t)kr * plane_out] = (T)scaled(v, i, exponent);
                }
            }
        }
    }
    // ---- outputs whose receptive field holds a value that is not finite: the zeros of the dense table met it as well.
    // Summed once more over the stored weights alone, one output after the other, a lane a row.
    if (__builtin_expect(__ballot(bad != 0) != 0, 0)) {
        const MatrixArgs& la = late_arguments();
#pragma unroll 1
        for (int np = 0; np < kNP; ++np) {
            unsigned todo = (unsigned)__ballot((bad >> np) & 1u);      // the upper half repeats the lower
#pragma unroll 1
            while (todo) {
                const int o = ofirst + np * 32 + __builtin_ctz(todo);
                todo &= todo - 1;
                if (o >= la.nout) continue;
                const int u = fdiv(o, la.fd_EF);
                const int rem = o - u * la.EF, i0 = fdiv(rem, la.fd_F), j0 = rem - i0 * la.F;
                const int k = kfirst + lane < la.K ? kfirst + lane : la.K - 1;
                float v = 0.f;
#pragma unroll 1
                for (int q = 0; q < (la.pool ? 4 : 1); ++q) {
                    const float w = stored_sum<T>(la, u, k, la.pool ? (i0 & ~1) + (q >> 1) : i0, la.pool ? (j0 & ~1) + (q & 1) : j0, lane);
                    v = q == 0 || w > v ? w : v;
                }
                if (lane >= kMK * 32 || kfirst + lane >= la.K) continue;
                T* to = la.pool ? y + ((size_t)u * la.K + k) * ((size_t)(la.E >> 1) * (la.F >> 1)) + (size_t)(i0 >> 1) * (la.F >> 1) + (j0 >> 1)
                                : y + ((size_t)u * la.K + k) * la.EF + rem;
                *to = (T)finish(v, la.bias ? la.bias[k] : 0.f);
            }
        }
    }
}

namespace {

template <typename T, int MK, int NP, int AHEAD, int FLY, int KS, bool WIDE>
int launch_one(const MatrixArgs& a, int grid, int lds, hipStream_t s)
{
    auto fn = matrix_kernel<T, MK, NP, AHEAD, FLY, KS, WIDE>;
    if (lds > 64 * 1024) {
        // more than 64 KB of dynamic LDS has to be allowed per kernel and device: once, for the whole 160 KB
        static std::atomic<unsigned long long> allowed{0};   // one bit per device ordinal
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return (int)e;
        const unsigned long long bit = dev < 64 ? 1ull << dev : 0ull;
        if (!(allowed.load(std::memory_order_relaxed) & bit)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return (int)e;
            allowed.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    hipLaunchKernelGGL(fn, dim3(grid), dim3(64 * kWaves<KS>), lds, s, a);
    return (int)hipGetLastError();
}

template <typename T, int MK, int NP, int KS>
int launch_fly(const MatrixArgs& a, const MatrixPlan& p, hipStream_t s)
{
    constexpr int unit = sizeof(T) == 4 ? 1 : 2;
    if (a.own_steps % p.ahead) return (int)hipErrorInvalidValue;
    if (stages_runs(p, sizeof(T))) {      // (from any element on: vector memory takes 8 bytes at any address)
        const int kind = p.ahead * 10 + p.wide_fly;
        if (kind == 21) return launch_one<T, MK, NP, 2, 1, KS, true>(a, p.grid, p.lds_bytes, s);
        if (kind == 31) return launch_one<T, MK, NP, 3, 1, KS, true>(a, p.grid, p.lds_bytes, s);
        if constexpr (MK * NP * (unit == 1 ? 2 : 1) < 8) {           // (registers)
            if (kind == 22) return launch_one<T, MK, NP, 2, 2, KS, true>(a, p.grid, p.lds_bytes, s);
            if (kind == 32) return launch_one<T, MK, NP, 3, 2, KS, true>(a, p.grid, p.lds_bytes, s);
        }
        return (int)hipErrorInvalidValue;
    }
    const int kind = p.ahead * 10 + p.fly / unit;
    if constexpr (unit == 2 || KS == 1) {     // (four wavefronts that share the channels have two fp32 blocks in flight at least)
        if (kind == 31) return launch_one<T, MK, NP, 3, unit, KS, false>(a, p.grid, p.lds_bytes, s);
        if (kind == 21) return launch_one<T, MK, NP, 2, unit, KS, false>(a, p.grid, p.lds_bytes, s);
    }
    switch (kind) {
        case 32: return launch_one<T, MK, NP, 3, 2 * unit, KS, false>(a, p.grid, p.lds_bytes, s);
        case 33: return launch_one<T, MK, NP, 3, 3 * unit, KS, false>(a, p.grid, p.lds_bytes, s);
        case 22: return launch_one<T, MK, NP, 2, 2 * unit, KS, false>(a, p.grid, p.lds_bytes, s);
        case 23: return launch_one<T, MK, NP, 2, 3 * unit, KS, false>(a, p.grid, p.lds_bytes, s);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace

}  // namespace sc
