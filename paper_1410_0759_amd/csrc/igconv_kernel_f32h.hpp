// fp32 convolution (forward; backward data with unit stride) on the 16-bit matrix pipes, every operand as two binary16
// numbers, with the gathered operand read from a staged patch of the zero-extended image.
//
//     x * 2^e = h + m / 2^11,   h = f16(x * 2^e), m = f16((x * 2^e - h) * 2^11)
// (11 + 11 significant bits and m's sign: x itself for three operands out of four, else one unit of its last place off),
// and a product as h*h' + (h*m' + m*h') / 2^11; the product left out is up to 2^-22 of it.  (A binary16 number and its residual times 2^11:
// Ootomo and Yokota, Recovering single precision accuracy from Tensor Cores while surpassing the FP32 theoretical peak performance, 2022.)
// Where three bfloat16 parts (igconv_kernel_f32s.hpp) need six products, this takes three.  What is lost has either sign where operands differ in their low
// bits, and is made up for in the sums: those of a chunk of 144 indices (16 channels, nine taps) are formed in accumulators of their own, h*h' apart
// from the two small products, and added up in a third one - fewer roundings at the full sum's size.  Where all operands of a sum have the same low bits
// it is lost on one side: up to 2^-21 of the sum of magnitudes, however long the sum.  Forward, 64x56x56 -> 64, 3x3, errors against 64 bits, three parts and two:
// normal weights over uniform images 1.3e-7 and 1.1e-7, over images of k / 255 1.4e-7 and 1.2e-7; all operands 1 + 2^-11 2.6e-8 and 2.4e-7, all 0.1
// 1.0e-8 and 1.6e-7, all 1 + 3001 * 2^-23 4.8e-8 and 3.7e-7.
//
// The exponent e is that of the chunk: the movers take the largest magnitude of the patch (of the filter rows) once it has
// arrived, before any of it is written, and scale it to [2^14, 2^15); the factor 2^-(e + e') goes into the addition to
// the third accumulator.  No range is assumed and none is kept from chunk to chunk.  What leaves it: an operand below 2^-13 after scaling
// (below 2^-28 of its chunk's largest) loses up to 2^-36.  The movers note each lane's smallest operand that is not zero; from the lanes that have such
// operands, and from the largest sum of magnitudes of a filter row, follows what a sum of the tile may be off by (off_by).  Results below 2^22 times that,
// not finite, or not zero but below 2^-100 are multiplied again (halves_mend): with fp32 multiply-adds, one by one; more than 24 of a wavefront's 4096
// with an exponent for each column; and what that leaves one by one, or, more than 24 again, all with the fp32 instruction.  Zeros are asked about
// only where an operand was below 2^-19, and pass where their whole filter row or window is zero.
// us, 128x64x56x56 -> 64, 3x3, backward data (every tile with such an operand multiplied again -> this): log-normal gradients, sigma 2 130 -> 128, 2.5
// 291 -> 137, 3 733 -> 150, with maps of zeros 739 -> 150; normal ones 134 -> 131.  -> 70 maps, one weight of 1e-12: 1152 -> 195, without it 207 -> 193.
// What still costs: tiles over images whose gradients differ, 384x13x13 -> 256, by 10^4 833 -> 281, by 10^6 845 -> 463 (alike 126); windows of
// zeros beside an operand far below the others (1286 -> 420, 150 without it).
//
// The reduction is ordered (16 channels, group of nine taps, tap, channel).  A tile's whole range of pixels of the
// zero-extended image goes to LDS once per 16 channels, and all R*S taps read their operands from it at shifted
// pixels.  The nine floats of a (row, channel, group) of the filter are contiguous in either pass (forward: row k, channel c;
// backward data: row c, channel k, the taps walked backwards).  Where R*S is no multiple of nine the last group begins at
// R*S - 9 and the taps it shares with the one before are zero.
//
// The filter is split once per call, into the caller's workspace, in the order in which the tiles read it (split_filter below:
// [row block][chunk][tap][part][half of the channels][row][8 channels], and each chunk's exponent and count).
//
// Measured, us and error against 64 bits, 128 images unless said, three bfloat16 parts -> this with the filter's split: 64x56x56 -> 64, 3x3
// 160 -> 117, 1.3e-7 -> 1.1e-7 (backward data 149 -> 111); 384x13x13 -> 256, 3x3 203 -> 143, 3.4e-7 -> 1.6e-7 (163 -> 117); 96x64x64 -> 128,
// 9x9, 32 images 1206 -> 569, 5.5e-7 -> 2.1e-7 (1621 -> 723); 96x27x27 -> 256, 5x5 647 -> 320 (750 -> 386); 64x224x224 -> 64, 3x3, 4
// images 124 -> 83.  What bounds it: with many taps the matrix pipes at the clocks that power leaves (350 TFLOP/s); with nine the
// requests and the splitting of the patch (the first layer without them 87 us, with neither MFMAs nor their waits 77) and 17 us of epilogues.
// (The filter split by the movers as well, in each tile, from registers: 137 us where this took 121, the 9x9 layer 1230; a barrier per
// step instead of per chunk: 121 instead of 110; 128 x 128 tiles level.)
//
// Four multiplying wavefronts, one that copies the split filter to LDS (loads straight into LDS, 16 bytes per lane) and three that
// move the patch; one workgroup per compute unit (LDS), persistent.  A step is three taps, a chunk three steps, one barrier each (WHOLE: one per chunk,
// with two stages of a chunk's filter):
//   filter, step q: request step q + 1 (three stages), wait for step q;
//   patch, in a 16-channel block's last chunk: the next block's - largest and smallest magnitude (end of step 0), split and write
//     every other item (steps 1 and 2), requesting the same item of the block after (nine taps: of the one after that, so
//     that its loads have four steps to arrive);
//   multipliers run one step behind: they pass the barrier that ends step q + 1 in the middle of step q's last tap.
// Where at most half of the compute units would have a tile more than the others, those tiles go as two halves of 128 columns (more than
// nine taps), a block of 32 columns per wavefront instead of two: 96x64x64 -> 128, 9x9, 32 images (784 tiles on 256 units) 570 -> 533 us, channels
// innermost 571 -> 537; 48x40x40 -> 60, 5x5, 100 images level.  (Nine taps: a chunk of half a tile takes nearly as long, 64x56x56 -> 64 with tanh 120 -> 124.)
// LDS: filter [stage][tap of 3][part][half][row][8 channels], patch [stage][part][half][pixel][8 channels]: a fragment is
// 32 neighbouring 16-byte pieces per half wavefront, and a tap a distance the same for all lanes.
#ifndef IGCONV_KERNEL_F32H_HPP_
#define IGCONV_KERNEL_F32H_HPP_

#include "igconv_kernel_f32s.hpp"

namespace igc {

using f16x8 = _Float16 __attribute__((ext_vector_type(8)));

// Scale of a chunk of one operand, from its largest magnitude (bits).
struct HalvesScale {
    int e;           // operands times 2^e
    float s, t;      // 2^e, 2^(e + 11)
    uint32_t below;  // bits of the magnitude under which an operand loses something
};
__device__ __forceinline__ HalvesScale halves_scale(uint32_t largest) {
    HalvesScale r;
    const int e = 141 - (int)(largest >> 23);   // the largest to [2^14, 2^15); within 2^60 either way the factors stay normal
    r.e = e < -60 ? -60 : (e > 60 ? 60 : e);
    r.s = __builtin_bit_cast(float, (uint32_t)(127 + r.e) << 23);
    r.t = __builtin_bit_cast(float, (uint32_t)(138 + r.e) << 23);
    r.below = (uint32_t)(114 - r.e) << 23;
    return r;
}

// x0, x1 as two pairs of binary16 numbers (x0's part in the low half): six instructions.
__device__ __forceinline__ void halves_pair(float x0, float x1, const HalvesScale &sc, uint32_t &h, uint32_t &m) {
    const float t0 = x0 * sc.t, t1 = x1 * sc.t;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(x0), "s"(sc.s));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(x1), "s"(sc.s));
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(m) : "v"(h), "s"(-2048.f), "v"(t0));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(m) : "v"(h), "s"(-2048.f), "v"(t1));
}

// Largest magnitude and, of those that are not zero, smallest one (twice its bits, less one) of a thread's operands.
struct HalvesSeen {
    float largest = 0.f;
    uint32_t smallest = ~0u;
};
__device__ __forceinline__ void look_at(HalvesSeen &seen, float x0, float x1) {
    // (the compiler's maximum would quiet both operands first; a NaN shows in the sums)
    asm("v_max3_f32 %0, %0, abs(%1), abs(%2)" : "+v"(seen.largest) : "v"(x0), "v"(x1));
    const uint32_t u0 = (__builtin_bit_cast(uint32_t, x0) << 1) - 1u, u1 = (__builtin_bit_cast(uint32_t, x1) << 1) - 1u;
    const uint32_t u = u0 < u1 ? u0 : u1;
    seen.smallest = seen.smallest < u ? seen.smallest : u;
}
__device__ __forceinline__ uint32_t wave_largest(uint32_t v) {
    auto reduce = [&](auto ctrl_c) __attribute__((always_inline)) {
        const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl_c)::value, 0xF, 0xF, true);
        v = v > other ? v : other;
    };
    reduce(std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8: lane 15 of each row of 16 has the row's
    reduce(std::integral_constant<int, 0x112>{});
    reduce(std::integral_constant<int, 0x114>{});
    reduce(std::integral_constant<int, 0x118>{});
    reduce(std::integral_constant<int, 0x142>{});   // row_bcast 15 and 31: lane 63 has the wavefront's
    reduce(std::integral_constant<int, 0x143>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// The wavefront's largest magnitude to LDS for the other moving wavefronts.
__device__ __forceinline__ void publish_largest(uint8_t *slot, const HalvesSeen &seen, int lane) {
    const uint32_t big = wave_largest(__builtin_bit_cast(uint32_t, seen.largest));
    if (lane == 0) *reinterpret_cast<uint32_t *>(slot) = big;
}
// Beside a count of operands that lost something: one of them was below 2^-19 after scaling.  Then sums of zero are asked about too: else each
// operand has 17 bits and more, and a sum of zero has no products but zeros, or some that cancel.
constexpr uint32_t kFarBelow = 1u << 31;
__device__ __forceinline__ uint32_t far_below(uint32_t below) { return below - (6u << 23); }
// Lanes whose smallest operand (as in HalvesSeen) is under a magnitude.
__device__ __forceinline__ uint64_t lanes_under(uint32_t smallest, uint32_t magnitude) { return __ballot(smallest < 2u * magnitude - 1u); }
__device__ __forceinline__ HalvesScale read_scale(const uint8_t *slots) {   // of the four moving wavefronts
    const u32x4 b = *reinterpret_cast<const u32x4 *>(slots);
    const uint32_t b0 = b[0] > b[1] ? b[0] : b[1], b1 = b[2] > b[3] ? b[2] : b[3];
    return halves_scale((uint32_t)__builtin_amdgcn_readfirstlane((int)(b0 > b1 ? b0 : b1)));
}
__device__ __forceinline__ uint32_t count_lossy(float x, uint32_t below) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x) & 0x7FFFFFFFu;
    return (uint32_t)__popcll(__ballot(u != 0u && u < below));
}

// True when a lane's sums call for a second look: one is infinite or NaN, or below 2^-100 or `limit` - zeros only where they are asked about.
template <int MB, int NB>
__device__ __forceinline__ bool outside_halves_range(const f32x16 (&sums)[MB][NB], float limit, bool zeros_too) {
    float nan = 0.f;   // (as outside_split_range of igconv_kernel_f32s.hpp)
    const uint32_t zero_passes = zeros_too ? 0u : ~0u;
    uint32_t small = ~0u;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float a = sums[mb][nb][v];
                nan = __builtin_fmaf(a, 0.f, nan);
                const uint32_t u = (__builtin_bit_cast(uint32_t, a) << 1) + zero_passes;
                small = small < u ? small : u;
            }
    const uint32_t least = __builtin_bit_cast(uint32_t, 0x1p-100f) << 1, other = __builtin_bit_cast(uint32_t, limit) << 1;
    return nan != 0.f || small < (least > other ? least : other);
}

// A sum over the wavefront, the same in every lane.
template <class T>
__device__ __forceinline__ T wave_sum(T s) {
    auto add = [&](auto ctrl_c) __attribute__((always_inline)) {
        s += __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, s), decltype(ctrl_c)::value, 0xF, 0xF, true));
    };
    add(std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8: see wave_largest
    add(std::integral_constant<int, 0x112>{});
    add(std::integral_constant<int, 0x114>{});
    add(std::integral_constant<int, 0x118>{});
    add(std::integral_constant<int, 0x142>{});
    add(std::integral_constant<int, 0x143>{});
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 63));
}

// First tap of group g: the last group ends with the filter.
__host__ __device__ __forceinline__ int halves_first_tap(int g, int taps) { return 9 * g < taps - 9 ? 9 * g : taps - 9; }

// Chunk of a row block of the split filter: exponent, operands that lost something (144 at most: no result meets more; kFarBelow) and, from bit 8 on, the
// largest sum of a row's magnitudes, scaled (at most 144 * 2^15).
struct HalvesChunk {
    int e;
    uint32_t lossy_sum;
};

// The results that operands with something lost could have touched, multiplied again one by one: four at a time, the wavefront's lanes along
// their reduction.  get(g, v), set(g, v, s): result v of the lane's block g; counts(g, v): whether it is stored;
// sums(which, from, s): the sums of result which[i] (16 g + v) of lane from[i].  limit(g, v): see the callers.  Results that are zero are, where
// they are asked about (asked(g): a bit each), handed to zeros(bits) first, which strikes out those whose zero is right.  False, and nothing done, when there
// are more than MOST left (then the blocks are cheaper as a whole).
template <int G, int MOST, class Limit, class Asked, class Get, class Set, class Counts, class Zeros, class Sums>
__device__ __forceinline__ bool mend_results(Limit limit, Asked asked, int lane, Get get, Set set, Counts counts, Zeros zeros, Sums sums) {
    uint32_t bad[G], zero[G];   // one bit per result
    uint32_t any_zero = 0;
    int left = 0;
    auto count = [&](const uint32_t (&bits)[G]) __attribute__((always_inline)) {
        int n = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) n += __builtin_popcount(bits[g]);
        return wave_sum(n);
    };
    static_for<G>([&](auto gc) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        bad[g] = zero[g] = 0u;
        static_for<16>([&](auto vc) __attribute__((always_inline)) {
            constexpr int v = decltype(vc)::value;
            const float a = __builtin_fabsf(get(gc, vc));
            const uint32_t bit = counts(gc, vc) ? 1u << v : 0u;
            const float least = limit(gc, vc);
            zero[g] |= a == 0.f ? bit : 0u;
            bad[g] |= a >= (least > 0x1p-100f ? least : 0x1p-100f) && a < __builtin_inff() ? 0u : bit;   // (NaN: bad)
        });
        bad[g] &= ~zero[g];
        zero[g] &= asked(gc);
        any_zero |= zero[g];
    });
    left = count(bad);
    if (left > MOST) return false;
    if (__any(any_zero != 0u)) {
        zeros(zero);
        left += count(zero);
        if (left > MOST) return false;
#pragma unroll
        for (int g = 0; g < G; ++g) bad[g] |= zero[g];
    }
#pragma clang loop unroll(disable)
    while (left > 0) {
        int first = -1;   // this lane's next one
#pragma unroll
        for (int g = G - 1; g >= 0; --g)
            if (bad[g] != 0u) first = g * 16 + __builtin_ctz(bad[g]);
        uint64_t lanes = __ballot(first >= 0);
        int which[4], from[4];
        float s[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // (fewer than four left: the first again)
            from[i] = lanes != 0u ? __builtin_ctzll(lanes) : from[0];
            which[i] = __builtin_amdgcn_readlane(first, from[i]);
            left -= lanes != 0u ? 1 : 0;
            lanes &= lanes - 1u;
        }
        sums(which, from, s);
        float mended = 0.f;
        bool mine = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            mended = lane == from[i] ? s[i] : mended;
            mine = mine || lane == from[i];
        }
        const int at = mine ? first : -1;
        static_for<G>([&](auto gc) __attribute__((always_inline)) {
            constexpr int g = decltype(gc)::value;
            static_for<16>([&](auto vc) __attribute__((always_inline)) {
                constexpr int v = decltype(vc)::value;
                set(gc, vc, at == g * 16 + v ? mended : get(gc, vc));
            });
            bad[g] = at >= 0 && at / 16 == g ? bad[g] & (bad[g] - 1u) : bad[g];
        });
    }
    return true;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) | (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
}

// NHWC: channel-fastest x (16-byte loads of channels) and y (lanes along output channels in the epilogue).
// SETS: patches in registers, 2 (nine taps: a chunk is a block) or 1 (more).  WHOLE: one barrier per chunk, where two stages of
// a chunk's filter fit (nine taps).
template <int BM_, int BN_, int WM_, int WN_, int PIX_, bool NHWC_, int SETS_, bool WHOLE_>
struct HalvesPatchConfig {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, PIX = PIX_, SETS = SETS_;
    static constexpr bool NHWC = NHWC_, SWAP = NHWC_, WHOLE = WHOLE_;
    static constexpr bool HALVES = SETS == 1;   // the last tiles may go as halves
    static constexpr int THREADS = 512, BK = 144, MOVERS = 3;
    static constexpr int A_PLANE = BM * 16, A_PART = 2 * A_PLANE, A_TAP = 2 * A_PART, A_STAGE = (WHOLE ? 9 : 3) * A_TAP;
    static constexpr int B_PLANE = PIX * 16, B_PART = 2 * B_PLANE, B_STAGE = 2 * B_PART;
    static constexpr int B_BASE = (WHOLE ? 2 : 3) * A_STAGE;
    static constexpr int SLOT_B = B_BASE + 2 * B_STAGE;   // largest magnitudes of the patch [parity of the block][wavefront]
    static constexpr int SLOT_C = SLOT_B + 32;            // 2^-(e + e') [parity of the chunk]
    // [parity of the tile]: patch operands of each moving wavefront that lost something, what a sum may be off by for all the patch's, for the filter's
    static constexpr int SLOT_N = SLOT_C + 16;
    static constexpr int LDS_BYTES = SLOT_N + 64;
    static constexpr int TM = BM / WM, TN = BN / WN, MB = TM / 32, NB = TN / 32;
    static constexpr int COPIES = A_STAGE / 1024;         // loads into LDS per step
    static constexpr int BLOCKS = PIX / 64;               // of 64 pixels
    static constexpr int ITEMS = (2 * BLOCKS + MOVERS - 1) / MOVERS;   // (block, half of the channels) per moving wavefront
    static_assert(WM * WN == 4 && BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "four wavefronts of 32x32 blocks");
    static_assert(BM == 64 && PIX % 64 == 0 && COPIES < 64 && !(WHOLE && SETS == 1), "shares of the moving wavefronts");
    static_assert(LDS_BYTES <= 160 * 1024 && B_PART < 65536, "LDS budget, offsets of the LDS instructions");
};

#if defined(__HIP_DEVICE_COMPILE__)
// All sums of a wavefront's blocks with v_mfma_f32_32x32x2_f32 straight from global memory: four taps as the filter stores them (they are next to each other:
// see gather_mode_ok) of four channels at a time, the next ones requested meanwhile.  Half wavefronts have channels of their own.
// (Index by index as sums_in_fp32 goes, a division for each and the filter element by element, a tile of 64x56x56 -> 64 took 100 us.)
template <bool SWAP, int MB, int NB>
__device__ __forceinline__ void halves_in_fp32(const ConvKernelParams &p, f32x16 (&acc)[MB][NB], int krow0, int col0, int half, int l32) {
    constexpr int CH = 2;   // channels of a half wavefront per round
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    const bool rev = (p.flip != 0) != (p.wsTapS < 0);   // (see the kernel)
    uint32_t rowoff[MB], colbase[NB];
    int h0[NB], w0[NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int row = krow0 + mb * 32 + l32;
        rowoff[mb] = row < p.K ? (uint32_t)row * (uint32_t)p.wsRow * 4u : kOutOfRange;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int j = col0 + nb * 32 + l32;
        const uint32_t jj = j < p.NPQ ? (uint32_t)j : 0u, n = magic_div(jj, p.mPQ), rem = jj - n * (uint32_t)p.PQ, pp = magic_div(rem, p.mQ), qq = rem - pp * (uint32_t)p.Q;
        h0[nb] = j < p.NPQ ? (int)pp * p.u - p.pad_h : -(1 << 20);
        w0[nb] = (int)qq * p.v - p.pad_w;
        colbase[nb] = (n * (uint32_t)p.xsN + (uint32_t)((int)pp * p.u - p.pad_h) * (uint32_t)p.xsH + (uint32_t)w0[nb] * (uint32_t)p.xsW) * 4u;
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;
    struct Operands { f32x4 a[CH][MB]; float b[CH][NB][4]; };
    int tap0 = 0, c0 = 0;   // of the round to be requested
    auto request = [&](Operands &o) __attribute__((always_inline)) {
        uint32_t xo[NB][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int at = rev ? p.RS - 1 - (tap0 + t) : tap0 + t;   // (past the last tap: outside every window)
            const uint32_t tr = magic_div((uint32_t)(at < 0 ? 0 : at), p.mS), ts = (uint32_t)at - tr * (uint32_t)p.S;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const bool ok = tap0 + t < p.RS && (uint32_t)(h0[nb] + (int)tr) < (uint32_t)p.H && (uint32_t)(w0[nb] + (int)ts) < (uint32_t)p.W;
                xo[nb][t] = ok ? colbase[nb] + (tr * (uint32_t)p.xsH + ts * (uint32_t)p.xsW) * 4u : kOutOfRange;
            }
        }
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const int c = c0 + e * 2 + half;
            const bool live = c < p.C;
            const uint32_t wc = ((uint32_t)c * (uint32_t)p.wsRed + (uint32_t)tap0) * 4u, xc = (uint32_t)c * (uint32_t)p.xsC * 4u;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {   // (taps past the last one: multiplied by zero below)
                const uint32_t at = live && rowoff[mb] != kOutOfRange ? rowoff[mb] + wc : kOutOfRange;
                o.a[e][mb] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, at, 0, 0));
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t at = live && xo[nb][t] != kOutOfRange ? xo[nb][t] + xc : kOutOfRange;
                    o.b[e][nb][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, at, 0, 0));
                }
        }
        if ((c0 += 2 * CH) >= p.C) {
            c0 = 0;
            tap0 += 4;
        }
    };
    int tap_now = 0, c_now = 0;   // of the round being multiplied
    auto multiply = [&](const Operands &o) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (tap_now + t >= p.RS) break;   // (what was read in their place may be another row's infinity)
#pragma unroll
            for (int e = 0; e < CH; ++e)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const float a = o.a[e][mb][t], b = o.b[e][nb][t];
                        if constexpr (SWAP) acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(b, a, acc[mb][nb], 0, 0, 0);
                        else acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[mb][nb], 0, 0, 0);
                    }
        }
        if ((c_now += 2 * CH) >= p.C) {
            c_now = 0;
            tap_now += 4;
        }
    };
    Operands o0, o1;
    request(o0);
#pragma clang loop unroll(disable)
    for (int left = (p.RS + 3) / 4 * ((p.C + 2 * CH - 1) / (2 * CH)); left > 0; left -= 2) {
        request(o1);
        multiply(o0);
        request(o0);
        multiply(o1);
    }
}

// x0, x1 as two pairs of binary16 numbers, each lane with a scale of its own.
__device__ __forceinline__ void halves_pair_lanes(float x0, float x1, const HalvesScale &sc, uint32_t &h, uint32_t &m) {
    const float t0 = x0 * sc.t, t1 = x1 * sc.t;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(x0), "v"(sc.s));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(x1), "v"(sc.s));
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(m) : "v"(h), "s"(-2048.f), "v"(t0));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(m) : "v"(h), "s"(-2048.f), "v"(t1));
}

// All sums of a wavefront's blocks over the split filter again, every column of the gathered operand - read from global memory - with
// an exponent of its own for three taps of 16 channels: columns of images that are small beside others of the tile lose nothing then.  limit: 2^22 times what
// the sums of this lane's column of each block may be off by; far: a bit per block as kFarBelow.
template <bool SWAP, int MB, int NB>
__device__ __forceinline__ void halves_by_columns(const ConvKernelParams &p, f32x16 (&total)[MB][NB], float (&limit)[NB], uint32_t *far, int krow0, int col0,
                                                  int half, int l32) {
    constexpr int BM = 64;
    static_assert(MB == 2, "a wavefront has a whole row block");
    const int groups = (p.RS + 8) / 9, nch = (p.C + 15) / 16, chunks = groups * nch, row_block = krow0 / BM;
    const uint32_t filter_bytes = (uint32_t)p.tilesM * (uint32_t)chunks * (9u * BM * 64u);   // (below 2^31: see gather_mode_ok)
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.halves), 0, filter_bytes, kBufferWord3);
    using ConstantChunk = const __attribute__((address_space(4))) uint64_t;
    ConstantChunk *const table = (ConstantChunk *)(uintptr_t)(static_cast<const char *>(p.halves) + filter_bytes) + (size_t)row_block * (size_t)chunks;
    const bool rev = (p.flip != 0) != (p.wsTapS < 0);   // (see the kernel)
    const uint32_t lane_at = (uint32_t)(half * (BM * 16) + l32 * 16);
    static_for<NB>([&](auto nbc) __attribute__((always_inline)) {
        constexpr int nb = decltype(nbc)::value;
        const int j = col0 + nb * 32 + l32;
        const uint32_t jj = j < p.NPQ ? (uint32_t)j : 0u, n = magic_div(jj, p.mPQ), rem = jj - n * (uint32_t)p.PQ, pp = magic_div(rem, p.mQ), qq = rem - pp * (uint32_t)p.Q;
        const int h0 = j < p.NPQ ? (int)pp * p.u - p.pad_h : -(1 << 20), w0 = (int)qq * p.v - p.pad_w;
        const uint32_t base = (n * (uint32_t)p.xsN + (uint32_t)((int)pp * p.u - p.pad_h) * (uint32_t)p.xsH + (uint32_t)w0 * (uint32_t)p.xsW) * 4u;
        f32x16 sum[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[mb][v] = 0.f;
        float off = 0.f;
        bool far_off = false;
        // three taps of a chunk at a time: their patch operands and the first block's rows are requested while the ones before are multiplied
        const int thirds = chunks * 3;
        float x[3][8];
        auto request_x = [&](int at3) __attribute__((always_inline)) {
            const int chunk = at3 / 3, cb = chunk / groups, first = halves_first_tap(chunk - cb * groups, p.RS) + (at3 - chunk * 3) * 3;
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int at = rev ? p.RS - 1 - (first + t) : first + t;
                const uint32_t tr = magic_div((uint32_t)at, p.mS), ts = (uint32_t)at - tr * (uint32_t)p.S;
                const bool ok = at3 < thirds && (uint32_t)(h0 + (int)tr) < (uint32_t)p.H && (uint32_t)(w0 + (int)ts) < (uint32_t)p.W;
                const uint32_t from = base + (tr * (uint32_t)p.xsH + ts * (uint32_t)p.xsW) * 4u;
#pragma unroll
                for (int e = 0; e < 8; ++e) {   // (beyond the last channel, where the filter is zero, nothing)
                    const int c = cb * 16 + half * 8 + e;
                    x[t][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, ok && c < p.C ? from + (uint32_t)c * (uint32_t)p.xsC * 4u : kOutOfRange, 0, 0));
                }
            }
        };
        u32x4 a[2][3][2];   // [block of rows][tap][part]
        auto request_a = [&](int at3, auto mbc) __attribute__((always_inline)) {   // (past the last one: beyond the row block, or zero)
            constexpr int mb = decltype(mbc)::value;
            const uint32_t from = ((uint32_t)(row_block * chunks) * 3u + (uint32_t)at3) * (3u * BM * 64u) + mb * 512u;
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int part = 0; part < 2; ++part)
                    a[mb][t][part] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, lane_at + (t * (BM * 64u) + part * (BM * 32u)), from, 0));
        };
        request_x(0);
        request_a(0, std::integral_constant<int, 0>{});
#pragma clang loop unroll(disable)
        for (int at3 = 0; at3 < thirds; ++at3) {
            HalvesSeen seen;
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int e = 0; e < 8; e += 2) look_at(seen, x[t][e], x[t][e + 1]);
            // (the other half wavefront has the column's other eight channels)
            const uint32_t here = __builtin_bit_cast(uint32_t, seen.largest), there = (uint32_t)__shfl_xor((int)here, 32), least = (uint32_t)__shfl_xor((int)seen.smallest, 32);
            const HalvesScale sc = halves_scale(here > there ? here : there);
            const uint32_t smallest = seen.smallest < least ? seen.smallest : least;
            u32x4 bh[3], bm[3];
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t h, m;
                    halves_pair_lanes(x[t][2 * q], x[t][2 * q + 1], sc, h, m);
                    bh[t][q] = h; bm[t][q] = m;
                }
            // (requests return in order: the second block's rows before the next patch operands)
            request_a(at3, std::integral_constant<int, 1>{});
            __builtin_amdgcn_sched_barrier(0);
            request_x(at3 + 1);
            __builtin_amdgcn_sched_barrier(0);
            const uint64_t entry = table[at3 / 3];   // HalvesChunk
            const uint32_t lossy = (uint32_t)(entry >> 32);
            const float c = __builtin_bit_cast(float, (uint32_t)(127 - (int)(uint32_t)entry - sc.e) << 23), c14 = c * 0x1p-14f;
            off = __builtin_fmaf((float)((lossy & 255u) << 15), c14, off);
            if (smallest < 2u * sc.below - 1u) off = __builtin_fmaf((float)(lossy >> 8 & 0x7FFFFFu), c14, off);
            far_off = far_off || (lossy & kFarBelow) != 0u || smallest < 2u * far_below(sc.below) - 1u;
            static_for<MB>([&](auto mbc) __attribute__((always_inline)) {
                constexpr int mb = decltype(mbc)::value;
                f32x16 acc = {}, low = {};
                auto product = [&](u32x4 rows, u32x4 column, f32x16 &to) __attribute__((always_inline)) {
                    const f16x8 fa = __builtin_bit_cast(f16x8, rows), fb = __builtin_bit_cast(f16x8, column);
                    if constexpr (SWAP) to = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb, fa, to, 0, 0, 0);
                    else to = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa, fb, to, 0, 0, 0);
                };
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    product(a[mb][t][0], bm[t], low);
                    product(a[mb][t][1], bh[t], low);
                    product(a[mb][t][0], bh[t], acc);
                }
                if constexpr (mb == 0) request_a(at3 + 1, std::integral_constant<int, 0>{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float cv = SWAP ? __shfl(c, v / 4 * 8 + v % 4 + half * 4) : c;
                    sum[mb][v] = __builtin_fmaf(__builtin_fmaf(low[v], 0x1p-11f, acc[v]), cv, sum[mb][v]);
                }
            });
        }
        limit[nb] = off;
        *far |= far_off ? 1u << nb : 0u;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) total[mb][nb] = sum[mb];
    });
}

// The sums of a tile's results that are out of range or that something lost could have touched, one by one or - many of them -
// all blocks of the wavefront (see the head of the file).  limit: 2^22 times what a sum may be off by.  A sum of zero is right where its whole row or window of operands is zero.
// n_end: first column beyond the tile's.  A call: inlined, its registers spilled in the tiles that need none of it (64x56x56 -> 64, channels innermost 120 -> 131 us).
constexpr int kForwardMost = 24;   // 384x13x13 -> 256, backward data: four results 13 us, all of a wavefront's by columns 95, with the fp32 instruction 330
using KernelArguments = const __attribute__((address_space(4))) ConvKernelParams;
template <bool SWAP, int MB, int NB>
__device__ __attribute__((noinline)) void halves_mend(uint64_t arguments, f32x16 *blocks, float limit, bool zeros_too, int n_end, int krow0, int col0) {
    ConvKernelParams p = *(KernelArguments *)(uintptr_t)uniform64(arguments);
    p.NPQ = __builtin_amdgcn_readfirstlane(n_end);
    krow0 = __builtin_amdgcn_readfirstlane(krow0);
    col0 = __builtin_amdgcn_readfirstlane(col0);
    limit = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, limit)));
    zeros_too = __builtin_amdgcn_readfirstlane((int)zeros_too) != 0;
    f32x16 total[MB][NB];
#pragma unroll
    for (int g = 0; g < MB * NB; ++g) total[g / NB][g % NB] = blocks[g];
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    auto get = [&](auto gc, auto vc) __attribute__((always_inline)) {
        const float a = total[decltype(gc)::value / NB][decltype(gc)::value % NB][decltype(vc)::value];
        return a;
    };
    auto set = [&](auto gc, auto vc, float a) __attribute__((always_inline)) { total[decltype(gc)::value / NB][decltype(gc)::value % NB][decltype(vc)::value] = a; };
    auto in_block = [](int v, int h) { return v / 4 * 8 + v % 4 + h * 4; };   // row (SWAP: column) of a block
    auto counts = [&](auto gc, auto vc) __attribute__((always_inline)) {
        constexpr int mb = decltype(gc)::value / NB, nb = decltype(gc)::value % NB, v = decltype(vc)::value;
        return krow0 + mb * 32 + (SWAP ? l32 : in_block(v, half)) < p.K && col0 + nb * 32 + (SWAP ? in_block(v, half) : l32) < p.NPQ;
    };
    // reduction index k: offsets of its filter element and of its tap's pixel, the tap
    struct Index { uint32_t ao, so; int tr, ts; };
    auto decode = [&](uint32_t k) __attribute__((always_inline)) {
        const uint32_t c = magic_div(k, p.mRS), rs = k - c * (uint32_t)p.RS, r = magic_div(rs, p.mS), sx = rs - r * (uint32_t)p.S;
        Index x;
        x.tr = (int)(p.flip ? (uint32_t)p.R - 1u - r : r);
        x.ts = (int)(p.flip ? (uint32_t)p.S - 1u - sx : sx);
        x.ao = (c * (uint32_t)p.wsRed + (uint32_t)p.wTap0 + r * (uint32_t)p.wsTapR + sx * (uint32_t)p.wsTapS) * 4u;
        x.so = (c * (uint32_t)p.xsC + (uint32_t)x.tr * (uint32_t)p.xsH + (uint32_t)x.ts * (uint32_t)p.xsW) * 4u;
        return x;
    };
    struct Window { int h0, w0; uint32_t base; };
    auto window = [&](int j) __attribute__((always_inline)) {
        const uint32_t n = magic_div((uint32_t)j, p.mPQ), rem = (uint32_t)j - n * (uint32_t)p.PQ, pp = magic_div(rem, p.mQ), qq = rem - pp * (uint32_t)p.Q;
        Window w;
        w.h0 = (int)pp * p.u - p.pad_h;
        w.w0 = (int)qq * p.v - p.pad_w;
        w.base = (n * (uint32_t)p.xsN + (uint32_t)w.h0 * (uint32_t)p.xsH + (uint32_t)w.w0 * (uint32_t)p.xsW) * 4u;
        return w;
    };
    auto load_w = [&](bool ok, uint32_t rowoff, const Index &x) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, ok ? rowoff + x.ao : kOutOfRange, 0, 0));
    };
    auto load_x = [&](bool ok, const Window &w, const Index &x) __attribute__((always_inline)) {
        ok = ok && (uint32_t)(w.h0 + x.tr) < (uint32_t)p.H && (uint32_t)(w.w0 + x.ts) < (uint32_t)p.W;
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, ok ? w.base + x.so : kOutOfRange, 0, 0));
    };
    // Rows of zeros: the lanes along a row, as far as the first operand that is not zero.  Then windows of zeros: a lane on each.
    auto zeros = [&](uint32_t (&zero)[MB * NB]) __attribute__((always_inline)) {
        // (row or column) r of block i of 32: its results' bits
        auto strike_lanes = [&](int i, uint32_t which, bool rows) __attribute__((always_inline)) {   // along the lanes: a bit per lane
#pragma unroll
            for (int g = 0; g < MB * NB; ++g)
                if ((rows ? g / NB : g % NB) == i && ((which >> l32) & 1u) != 0u) zero[g] = 0u;
        };
        auto strike_results = [&](int i, uint32_t which, bool rows) __attribute__((always_inline)) {   // along the results of a lane
            uint32_t bits = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) bits |= ((which >> in_block(v, half)) & 1u) << v;
#pragma unroll
            for (int g = 0; g < MB * NB; ++g)
                if ((rows ? g / NB : g % NB) == i) zero[g] &= ~bits;
        };
        // which rows (columns) of block i have such results
        auto present_lanes = [&](int i, bool rows) __attribute__((always_inline)) {
            uint32_t bits = 0;
#pragma unroll
            for (int g = 0; g < MB * NB; ++g)
                if ((rows ? g / NB : g % NB) == i) bits |= zero[g];
            const uint64_t m = __ballot(bits != 0u);
            return (uint32_t)m | (uint32_t)(m >> 32);
        };
        auto present_results = [&](int i, bool rows) __attribute__((always_inline)) {
            uint32_t bits = 0, found = 0;
#pragma unroll
            for (int g = 0; g < MB * NB; ++g)
                if ((rows ? g / NB : g % NB) == i) bits |= zero[g];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint64_t m = __ballot((bits >> v) & 1u);
                found |= ((uint32_t)m != 0u ? 1u : 0u) << in_block(v, 0) | ((m >> 32) != 0u ? 1u : 0u) << in_block(v, 1);
            }
            return found;
        };
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            uint32_t rows = SWAP ? present_lanes(mb, true) : present_results(mb, true), all_zero = 0;
#pragma clang loop unroll(disable)
            while (rows != 0u) {
                const int r = __builtin_ctz(rows);
                rows &= rows - 1u;
                const uint32_t rowoff = (uint32_t)(krow0 + mb * 32 + r) * (uint32_t)p.wsRow * 4u;
                bool found = false;
#pragma clang loop unroll(disable)
                for (int k0 = 0; k0 < p.CRS && !found; k0 += 512) {
                    float a[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int k = k0 + e * 64 + lane;
                        a[e] = load_w(k < p.CRS, rowoff, decode((uint32_t)k));
                    }
                    bool some = false;
#pragma unroll
                    for (int e = 0; e < 8; ++e) some = some || a[e] != 0.f;
                    found = __any(some);
                }
                all_zero |= found ? 0u : 1u << r;
            }
            if (SWAP) strike_lanes(mb, all_zero, true);
            else strike_results(mb, all_zero, true);
        }
        // (a lane on column l32 of block `half`, then of the two blocks after)
        static_assert(NB % 2 == 0, "two blocks of columns at a time");
#pragma unroll
        for (int nb = 0; nb < NB; nb += 2) {
            const uint32_t c0 = SWAP ? present_results(nb, false) : present_lanes(nb, false), c1 = SWAP ? present_results(nb + 1, false) : present_lanes(nb + 1, false);
            bool open = (((half ? c1 : c0) >> l32) & 1u) != 0u;
            const bool asked = open;
            const int j = col0 + (nb + half) * 32 + l32;
            const Window w = window(j < p.NPQ ? j : p.NPQ - 1);
#pragma clang loop unroll(disable)
            for (int rs = 0; rs < p.RS && __any(open); ++rs) {   // tap by tap
                const uint32_t tr = magic_div((uint32_t)rs, p.mS), ts = (uint32_t)rs - tr * (uint32_t)p.S;
                const bool inside = (uint32_t)(w.h0 + (int)tr) < (uint32_t)p.H && (uint32_t)(w.w0 + (int)ts) < (uint32_t)p.W;
                const uint32_t at = w.base + (tr * (uint32_t)p.xsH + ts * (uint32_t)p.xsW) * 4u;
#pragma clang loop unroll(disable)
                for (int c = 0; c < p.C && __any(open); c += 32) {
                    float b[32];
                    const uint32_t from = open && inside ? at + (uint32_t)c * (uint32_t)p.xsC * 4u : kOutOfRange;
#pragma unroll
                    for (int e = 0; e < 32; ++e)   // (beyond the last channel: the last again)
                        b[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, from, (uint32_t)(c + e < p.C ? e : p.C - 1 - c) * (uint32_t)p.xsC * 4u, 0));
                    bool some = false;
#pragma unroll
                    for (int e = 0; e < 32; ++e) some = some || b[e] != 0.f;
                    open = open && !some;
                }
            }
            const uint64_t m = __ballot(asked && open);   // (still open: all of it is zero)
            if (SWAP) {
                strike_results(nb, (uint32_t)m, false);
                strike_results(nb + 1, (uint32_t)(m >> 32), false);
            } else {
                strike_lanes(nb, (uint32_t)m, false);
                strike_lanes(nb + 1, (uint32_t)(m >> 32), false);
            }
        }
    };
    auto sums = [&](const int (&which)[4], const int (&from)[4], float (&s)[4]) __attribute__((always_inline)) {
        uint32_t rowoff[4];
        Window w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int g = which[i] >> 4, r = in_block(which[i] & 15, from[i] >> 5), l = from[i] & 31;
            rowoff[i] = (uint32_t)(krow0 + g / NB * 32 + (SWAP ? l : r)) * (uint32_t)p.wsRow * 4u;
            w[i] = window(col0 + g % NB * 32 + (SWAP ? r : l));
            s[i] = 0.f;
        }
#pragma clang loop unroll(disable)
        for (int k0 = 0; k0 < p.CRS; k0 += 192) {
            float a[3][4], b[3][4];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const int k = k0 + e * 64 + lane;
                const Index x = decode((uint32_t)k);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a[e][i] = load_w(k < p.CRS, rowoff[i], x);
                    b[e][i] = load_x(k < p.CRS, w[i], x);
                }
            }
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] = __builtin_fmaf(a[e][i], b[e][i], s[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = wave_sum(s[i]);
    };
    bool done = mend_results<MB * NB, kForwardMost>([&](auto, auto) { return limit; }, [&](auto) { return zeros_too ? 0xFFFFu : 0u; }, lane, get, set, counts, zeros, sums);
    int infinite = 0;   // or NaN: no exponent helps
    static_for<MB * NB>([&](auto gc) __attribute__((always_inline)) {
        static_for<16>([&](auto vc) __attribute__((always_inline)) { infinite += __builtin_fabsf(get(gc, vc)) < __builtin_inff() ? 0 : 1; });
    });
    if (!done && wave_sum(infinite) <= kForwardMost) {
        float limits[NB];
        uint32_t far = 0;
        halves_by_columns<SWAP, MB, NB>(p, total, limits, &far, krow0, col0, half, l32);
        // (SWAP: a lane's results have columns of their own)
        auto limit_of = [&](auto gc, auto vc) __attribute__((always_inline)) {
            const float own = limits[decltype(gc)::value % NB];
            return SWAP ? __shfl(own, in_block(decltype(vc)::value, half)) : own;
        };
        auto asked = [&](auto gc) __attribute__((always_inline)) {
            const bool own = (far >> (decltype(gc)::value % NB) & 1u) != 0u;
            if (!SWAP) return own ? 0xFFFFu : 0u;
            const uint32_t columns = (uint32_t)__ballot(own);
            uint32_t bits = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) bits |= ((columns >> in_block(v, half)) & 1u) << v;
            return bits;
        };
        done = mend_results<MB * NB, kForwardMost>(limit_of, asked, lane, get, set, counts, zeros, sums);
    }
    if (!done) halves_in_fp32<SWAP, MB, NB>(p, total, krow0, col0, half, l32);
#pragma unroll
    for (int g = 0; g < MB * NB; ++g) blocks[g] = total[g / NB][g % NB];
}
#endif

template <class Cfg>
__global__ __launch_bounds__(512, 2) void igconv_f32h_kernel(const ConvKernelParams p) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernel's name and signature only)
    constexpr int BM = Cfg::BM, BN = Cfg::BN, MB = Cfg::MB, NB = Cfg::NB, ITEMS = Cfg::ITEMS, SETS = Cfg::SETS;

    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int l32 = lane & 31;

    // persistent workgroups, tiles numbered in contiguous ranges per XCD (see igconv_kernel.hpp)
    const int wg_xcd = (int)(blockIdx.x % 8u), wg_local = (int)(blockIdx.x / 8u);
    const int tiles_total = p.tilesM * p.tilesN;
    // Work item: the tile; with HALVES four times the tile, and 0 - all of it -, 1 or 2 - its left or right half.  (The last p.halvedPerXcd tiles of an
    // XCD's range, which would be one more for some of the compute units, go as halves: see the head of the file.)
    constexpr int PARTS = Cfg::HALVES ? 4 : 1;
    const int none = Cfg::HALVES ? tiles_total * 4 : tiles_total;
    auto work_number = [&](int i) {
        const int local = wg_local + i * p.wgsPerXcd;
        if constexpr (Cfg::HALVES) {
            const int whole_tiles = p.tilesPerXcd - p.halvedPerXcd, past = local - whole_tiles;
            const int t = wg_xcd * p.tilesPerXcd + (past < 0 ? local : whole_tiles + past / 2);
            return past < 2 * p.halvedPerXcd && t < tiles_total ? t * 4 + (past < 0 ? 0 : 1 + past % 2) : none;
        } else {
            const int t = wg_xcd * p.tilesPerXcd + local;
            return local < p.tilesPerXcd && t < tiles_total ? t : tiles_total;
        }
    };
    if (work_number(0) >= none) return;
    const int groups = (p.RS + 8) / 9;            // of nine taps
    const int nch = (p.C + 15) / 16;              // blocks of 16 channels; the split filter is zero beyond the last channel
    auto first_tap = [&](int g) { return halves_first_tap(g, p.RS); };
    // columns of a work item: [first, end); where an image's pixels are tiled by themselves its last tile is cut short.  (A right half with none:
    // the last column, of which nothing is stored.)
    auto work_columns = [&](int work, int *first, int *end) {
        const int tn = work / PARTS / p.tilesM, part = work % PARTS;
        if (p.imageTiles == 0) {
            *first = tn * BN;
            *end = p.NPQ;
        } else {
            const int image = tn / p.imageTiles;
            *first = image * p.PQ + (tn - image * p.imageTiles) * BN;
            *end = (image + 1) * p.PQ;
        }
        bool some = true;
        if (part == 1) *end = *end < *first + BN / 2 ? *end : *first + BN / 2;
        if (part == 2) {
            *end = *end < *first + BN ? *end : *first + BN;
            some = *first + BN / 2 < *end;
            *first = some ? *first + BN / 2 : *end - 1;
        }
        return some;
    };
    // first pixel of column j's window as a flat index into the zero-extended images
    auto window_start = [&](uint32_t j) {
        const uint32_t n = magic_div(j, p.mPQ);
        const uint32_t rem = j - n * (uint32_t)p.PQ;
        const uint32_t pp = magic_div(rem, p.mQ);
        const uint32_t qq = rem - pp * (uint32_t)p.Q;
        return n * (uint32_t)p.HpWp + pp * (uint32_t)(p.u * p.Wp) + qq * (uint32_t)p.v;
    };

    const int chunks = nch * groups;
    int rem = 0;
    for (int i = 0; work_number(i) < none; ++i) rem += chunks;   // chunks of all tiles of this workgroup

    if (wave == 4) {
        // ================================ filter ================================
        const uint32_t block_bytes = (uint32_t)(chunks * 9 * Cfg::A_TAP);   // of a row block
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.halves), 0, (uint32_t)p.tilesM * block_bytes, kBufferWord3);
        const uint32_t voff = (uint32_t)lane * 16u;
        constexpr int STEPS = Cfg::WHOLE ? 1 : 3;
        int it = 0, left = chunks * STEPS;   // of the step to be requested: tile, steps of it that are left
        uint32_t from = (uint32_t)(work_number(0) / PARTS % p.tilesM) * block_bytes;
        auto request = [&](auto stage_c) __attribute__((always_inline)) {
            uint8_t *const dst = lds + decltype(stage_c)::value * Cfg::A_STAGE;
#pragma unroll
            for (int i = 0; i < Cfg::COPIES; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void *)(dst + i * 1024), 16, voff, from + i * 1024u, 0, 0);
            from += Cfg::A_STAGE;
            if (--left == 0) {   // (past the last tile: its first steps again; nothing of them is multiplied)
                left = chunks * STEPS;
                const int next = work_number(++it);
                from = next < none ? (uint32_t)(next / PARTS % p.tilesM) * block_bytes : 0u;
            }
        };
        if constexpr (Cfg::WHOLE) {
            split_barrier();
            auto chunk = [&](auto stage_c) __attribute__((always_inline)) {
                request(stage_c);
                __builtin_amdgcn_s_waitcnt(0x0F70);
                split_barrier();
            };
            for (;;) {
                chunk(std::integral_constant<int, 0>{});
                if (--rem <= 0) break;
                chunk(std::integral_constant<int, 1>{});
                if (--rem <= 0) break;
            }
            split_barrier();
            return;
        }
        request(std::integral_constant<int, 0>{});
        split_barrier();
        for (int s = rem; s > 0; --s)
            static_for<3>([&](auto jc) __attribute__((always_inline)) {
                request(std::integral_constant<int, (decltype(jc)::value + 1) % 3>{});
                constexpr int later = Cfg::COPIES;   // (the step requested just now may stay in flight)
                __builtin_amdgcn_s_waitcnt(0x0F70 | (later & 15) | ((later >> 4) << 14));
                split_barrier();
            });
        __builtin_amdgcn_s_waitcnt(0x0F70);   // no request may still be on its way into LDS when it is given away
        split_barrier();                       // (the multipliers' last step passes one more)
        return;
    }
    if (wave > 4) {
        // ================================ patch ================================
        const int mw = wave - 5;
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        using ConstantChunk = const __attribute__((address_space(4))) uint64_t;   // (written by the kernel before: read through scalar loads)
        ConstantChunk *const table = (ConstantChunk *)(uintptr_t)(static_cast<const char *>(p.halves) + (size_t)p.tilesM * (size_t)chunks * (9 * Cfg::A_TAP));
        // item i of this wavefront: 64 pixels (block n / 2) and one half (n % 2) of the 16 channels, n = 3 i + mw
        uint32_t b_voff[ITEMS];
        float b_reg[SETS][ITEMS][8];
        int items = 0, held[SETS];   // items of the block to be requested, of those in registers, next one first

        auto setup_patch = [&](int work) {
            int n0, n_end;
            work_columns(work, &n0, &n_end);
            const uint32_t g_first = __builtin_amdgcn_readfirstlane(window_start((uint32_t)n0));
            const int j_last = n0 + BN - 1 < n_end ? n0 + BN - 1 : n_end - 1;
            const uint32_t g_end = __builtin_amdgcn_readfirstlane(window_start((uint32_t)j_last)) +
                                   (uint32_t)((p.R - 1) * p.Wp + p.S);   // one past the tile's last pixel
            items = (int)(g_end - g_first + 63u) / 64 * 2;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const uint32_t g = g_first + (uint32_t)((3 * i + mw) / 2 * 64 + lane);
                const uint32_t n = magic_div(g, p.mHpWp);
                const uint32_t rem_ = g - n * (uint32_t)p.HpWp;
                const uint32_t hp = magic_div(rem_, p.mWp);
                const uint32_t wp = rem_ - hp * (uint32_t)p.Wp;
                const uint32_t h = hp - (uint32_t)p.pad_h, w = wp - (uint32_t)p.pad_w;   // wrap below 0 -> huge
                const bool ok = g < g_end && h < (uint32_t)p.H && w < (uint32_t)p.W;    // (g < g_end implies n < N)
                b_voff[i] = ok ? (n * (uint32_t)p.xsN + h * (uint32_t)p.xsH + w * (uint32_t)p.xsW) * 4u : kOutOfRange;
            }
        };
        // Offsets of the channels that the even (odd) items of block cb have: one set for all of them, worked out when their turn comes.
        // (Per load they took three scalar instructions and, kept for both halves, moves out of spilled registers, 350 of 1150 instructions per chunk:
        // 384x13x13 -> 256, 128 images, 143 -> 134 us, 64x56x56 -> 64, 3x3, backward data 110.5 -> 109.5.  Channel-fastest, two loads per item, that gains nothing.)
        struct Channels { uint32_t off[8]; };
        auto channels_of = [&](uint32_t cb, int odd) __attribute__((always_inline)) {
            Channels r = {};
            if constexpr (!Cfg::NHWC) {
                const uint32_t c = cb * 16u + (uint32_t)((odd + mw) % 2 * 8);
#pragma unroll
                for (int e = 0; e < 8; ++e) {   // (beyond the last channel, where the filter is zero, the last one again)
                    const uint32_t k = c + (uint32_t)e < (uint32_t)p.C - 1u ? c + (uint32_t)e : (uint32_t)p.C - 1u;
                    r.off[e] = k * (uint32_t)p.xsC * 4u;
                }
            }
            return r;
        };
        // request item i of the patch of block cb
        auto request_b = [&](auto set_c, int i, uint32_t cb, const Channels &ch) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            if constexpr (Cfg::NHWC) {
                const uint32_t c = cb * 16u + (uint32_t)((3 * i + mw) % 2 * 8);
#pragma unroll
                for (int e = 0; e < 2; ++e) {   // (beyond the last channel the last four again)
                    const uint32_t k = c + (uint32_t)e * 4u < (uint32_t)p.C - 4u ? c + (uint32_t)e * 4u : (uint32_t)p.C - 4u;
                    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xbuf, b_voff[i], k * 4u, 0));
#pragma unroll
                    for (int q = 0; q < 4; ++q) b_reg[set][i][e * 4 + q] = v[q];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    b_reg[set][i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, b_voff[i], ch.off[e], 0));
            }
        };
        // split item i and write it into the stage at byte offset `stage`
        HalvesScale sb;
        auto convert_b = [&](auto set_c, int i, int stage) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            u32x4 bh, bm;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t h, m;
                halves_pair(b_reg[set][i][2 * q], b_reg[set][i][2 * q + 1], sb, h, m);
                bh[q] = h; bm[q] = m;
            }
            const int n = 3 * i + mw;
            uint8_t *const dst = lds + Cfg::B_BASE + stage + n % 2 * Cfg::B_PLANE + n / 2 * 1024 + lane * 16;
            *reinterpret_cast<u32x4 *>(dst) = bh;
            *reinterpret_cast<u32x4 *>(dst + Cfg::B_PART) = bm;
        };
        uint32_t small_b = 0;   // smallest magnitude of what is in registers (this lane's, as in HalvesSeen)
        // Products of one result that this wavefront's lost operands could touch, counted from above (a lane with a small one may have as many as it
        // holds; a block has 144 indices per group).
        uint32_t lossy_b = 0, far_a = 0, far_b = 0;
        float off_a = 0.f, off_b = 0.f;   // 2^22 times what a sum may be off by for lost operands of the filter, for any of the patch
        auto look_at_patch = [&](auto set_c, int parity) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            HalvesSeen seen;
            static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                if (3 * i + mw < held[0])
#pragma unroll
                    for (int e = 0; e < 8; e += 2) look_at(seen, b_reg[set][i][e], b_reg[set][i][e + 1]);
            });
            publish_largest(lds + Cfg::SLOT_B + parity * 16 + mw * 4, seen, lane);
            small_b = seen.smallest;
        };
        auto scale_patch = [&](int parity) __attribute__((always_inline)) {
            sb = read_scale(lds + Cfg::SLOT_B + parity * 16);
            const uint64_t small = lanes_under(small_b, sb.below);
            if (small != 0u) {
                const uint32_t n = (uint32_t)__popcll(small) * (8u * ITEMS), most = 144u * (uint32_t)groups;
                lossy_b += n < most ? n : most;   // (far below 2^31: the split filter has fewer chunks)
                if (lanes_under(small_b, far_below(sb.below)) != 0u) far_b = kFarBelow;
            }
        };

        // where the chunk being written and the block being requested are
        int it = 0, cb = 0, g = 0;
        int b_it = 0, b_cb = 0;
        // f(item, its channels): the even items, then the odd ones; channel-fastest, where two items in a row read the same pixels' lines, as they come
        auto in_order = [&](auto f) __attribute__((always_inline)) {
            if constexpr (Cfg::NHWC) {
                static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { f(ic, Channels{}); });
            } else {
                static_for<2>([&](auto oc) __attribute__((always_inline)) {
                    constexpr int odd = decltype(oc)::value;
                    const Channels ch = channels_of((uint32_t)b_cb, odd);
                    static_for<(ITEMS + 1 - odd) / 2>([&](auto ic) __attribute__((always_inline)) { f(std::integral_constant<int, decltype(ic)::value * 2 + odd>{}, ch); });
                });
            }
        };
        // (past the last tile the last one's operands are requested again; nothing of them is multiplied)
        auto next_block = [&]() {
            if (++b_cb == nch) {
                b_cb = 0;
                if (work_number(++b_it) < none) setup_patch(work_number(b_it));
            }
        };
        int e_patch;                 // exponent of the block being multiplied
        int stage = 0;               // byte offset of its patch's stage
        uint32_t n_chunk = 0;        // chunks so far
        int n_block = 0;             // blocks so far
        uint32_t entry = (uint32_t)(work_number(0) / PARTS % p.tilesM) * (uint32_t)chunks;   // this chunk's in the table
        auto publish_scale = [&](bool tile_begins) __attribute__((always_inline)) {   // the chunk's, for the multipliers
            if (mw == 0) {
                const uint64_t t = table[entry];   // HalvesChunk
                const uint32_t n = (uint32_t)(t >> 32), c = (uint32_t)(127 - (int)(uint32_t)t - e_patch) << 23;
                const float c14 = __builtin_bit_cast(float, c) * 0x1p-14f;   // (2^-36 * 2^22)
                off_a = __builtin_fmaf((float)((n & 255u) << 15), c14, tile_begins ? 0.f : off_a);
                off_b = __builtin_fmaf((float)(n >> 8 & 0x7FFFFFu), c14, tile_begins ? 0.f : off_b);
                far_a = (tile_begins ? 0u : far_a) | (n & kFarBelow);
                if (lane == 0) *reinterpret_cast<uint32_t *>(lds + Cfg::SLOT_C + (n_chunk & 1u) * 4u) = c;
            }
        };
        auto publish_lossy = [&]() __attribute__((always_inline)) {   // the tile's
            uint8_t *const slot = lds + Cfg::SLOT_N + (it & 1) * 32;
            if (lane == 0) {
                *reinterpret_cast<uint32_t *>(slot + mw * 4) = lossy_b | far_a | far_b;
                if (mw == 0) *reinterpret_cast<float *>(slot + 12) = off_b;
                if (mw == 0) *reinterpret_cast<float *>(slot + 16) = off_a;
            }
        };
        auto next_chunk = [&]() __attribute__((always_inline)) {
            ++n_chunk;
            ++entry;
            if (++g == groups) {
                g = 0;
                if (++cb == nch) {
                    cb = 0;
                    const int next = work_number(++it);
                    entry = next < none ? (uint32_t)(next / PARTS % p.tilesM) * (uint32_t)chunks : 0u;
                }
            }
        };
        // (Requests stand under no condition but the compile-time ones: with any other the compiler, which counts the loads in
        // flight, would wait for those just requested as well.  `block_end`: the block's last chunk.)
        auto chunk = [&](auto par_c, auto end_c) __attribute__((always_inline)) {
            constexpr int par = decltype(par_c)::value;
            constexpr bool block_end = decltype(end_c)::value;
            using Blk = std::integral_constant<int, SETS == 2 ? par ^ 1 : 0>;   // the next block's patch
            static_for<3>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                if constexpr (j == 0) {
                    publish_scale(cb == 0 && g == 0);
                    if (block_end && cb == nch - 1) publish_lossy();
                }
                if constexpr (j == 1 && block_end) {
                    if (cb == nch - 1) lossy_b = far_b = 0;   // (from here on the next tile's)
                    scale_patch((n_block + 1) & 1);
                }
                if constexpr (j > 0 && block_end) {
                    const Channels ch = channels_of((uint32_t)b_cb, j - 1);
                    static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) {
                        constexpr int i = decltype(ic)::value;
                        if constexpr (i % 2 == j - 1) {
                            if (3 * i + mw < held[0]) convert_b(Blk{}, i, Cfg::B_STAGE - stage);
                            request_b(Blk{}, i, (uint32_t)b_cb, ch);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    });
                }
                if constexpr (j == 0 && block_end) look_at_patch(Blk{}, (n_block + 1) & 1);
                split_barrier();
            });
            if constexpr (block_end) {
                e_patch = sb.e;
                stage = Cfg::B_STAGE - stage;
                ++n_block;
                if constexpr (SETS == 2) held[0] = held[1];
                held[SETS - 1] = items;
                next_block();
            }
            next_chunk();
        };
        // One barrier per chunk: the chunk's own patch is split and written, the same registers requested for the block
        // after the next, the next one's magnitudes taken.
        auto whole_chunk = [&](auto par_c) __attribute__((always_inline)) {
            constexpr int par = decltype(par_c)::value;
            if (cb == 0) lossy_b = far_b = 0;
            scale_patch(par);
            e_patch = sb.e;
            publish_scale(cb == 0);
            if (cb == nch - 1) publish_lossy();
            in_order([&](auto ic, const Channels &ch) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                if (3 * i + mw < held[0]) convert_b(par_c, i, par * Cfg::B_STAGE);
                request_b(par_c, i, (uint32_t)b_cb, ch);
                __builtin_amdgcn_sched_barrier(0);
            });
            held[0] = held[SETS - 1];
            held[SETS - 1] = items;
            next_block();
            look_at_patch(std::integral_constant<int, par ^ 1>{}, par ^ 1);
            split_barrier();
            next_chunk();
        };
        // the first block's patch
        using S0 = std::integral_constant<int, 0>;
        auto request_patch = [&](auto set_c, int h) __attribute__((always_inline)) {
            held[h] = items;
            in_order([&](auto ic, const Channels &ch) __attribute__((always_inline)) { request_b(set_c, decltype(ic)::value, (uint32_t)b_cb, ch); });
            next_block();
        };
        if (lane == 0 && mw == 0)   // (the unused fourth wavefront's)
            for (int i = 0; i < 2; ++i)
                *reinterpret_cast<uint32_t *>(lds + Cfg::SLOT_B + i * 16 + 12) = 0u;
        setup_patch(work_number(0));
        request_patch(S0{}, 0);
        if constexpr (SETS == 2) request_patch(std::integral_constant<int, 1>{}, 1);
        look_at_patch(S0{}, 0);
        split_barrier();
        if constexpr (Cfg::WHOLE) {
            for (;;) {
                whole_chunk(S0{});
                if (--rem <= 0) break;
                whole_chunk(std::integral_constant<int, 1>{});
                if (--rem <= 0) break;
            }
            split_barrier();
            return;
        }
        scale_patch(0);
        e_patch = sb.e;
        static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { if (3 * decltype(ic)::value + mw < held[0]) convert_b(S0{}, decltype(ic)::value, 0); });
        if constexpr (SETS == 2) held[0] = held[1];
        request_patch(S0{}, SETS - 1);
        auto any_chunk = [&](auto par_c) __attribute__((always_inline)) {
            if constexpr (SETS == 2) chunk(par_c, std::true_type{});   // (nine taps: every one)
            else if (g == groups - 1) chunk(par_c, std::true_type{});
            else chunk(par_c, std::false_type{});
        };
        for (;;) {
            any_chunk(std::integral_constant<int, 0>{});
            if (--rem <= 0) break;
            any_chunk(std::integral_constant<int, 1>{});
            if (--rem <= 0) break;
        }
        split_barrier();                       // (the multipliers' last step passes one more)
        return;
    }

    // ================================ multipliers ================================
    const int wm = wave % Cfg::WM, wn = wave / Cfg::WM;
    constexpr int M = MB * NB;
    u32x4 ah[2][MB], am[MB], bh[NB], bm[NB];
    f32x16 total[MB][NB], acc[MB][NB], low[MB][NB];
    // filter operands of the chunk's first tap (step j of a chunk has stage j; WHOLE: the chunks alternate)
    int fa = half * Cfg::A_PLANE + (wm * Cfg::TM + l32) * 16;
    int a_other = Cfg::WHOLE ? Cfg::A_STAGE : 0;
    int fb[NB], fb_next[NB];                                    // patch operands of tap offset 0: this chunk, the next one
    int b_other = Cfg::B_STAGE;                                 // distance to the patch's other stage
    // the storage order of the taps is that of the filter; where in the window one reads: reversed for eq. 2, and for
    // the exchanged filter of backward data, whose gather walks the taps backwards
    const bool rev = (p.flip != 0) != (p.wsTapS < 0);
    const int in_row = rev ? -16 : 16, to_row = (rev ? -1 : 1) * (p.Wp - p.S + 1) * 16;   // from tap to tap, bytes
    auto tap_position = [&](int g, int *s) {   // column and offset of group g's first tap
        const uint32_t tap = (uint32_t)first_tap(g);
        const uint32_t r = magic_div(tap, p.mS);
        *s = (int)(tap - r * (uint32_t)p.S);
        const int o = (int)r * p.Wp + *s;
        return (rev ? (p.R - 1) * p.Wp + p.S - 1 - o : o) * 16;
    };
    auto columns = [&](int work, int stage_offset, int (&f)[NB]) {
        int n0, n_end;
        work_columns(work, &n0, &n_end);
        const uint32_t g_first = __builtin_amdgcn_readfirstlane(window_start((uint32_t)n0));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            int j = n0 + wn * Cfg::TN + nb * 32 + l32;
            if constexpr (Cfg::HALVES) j -= work % PARTS != 0 ? wn * (Cfg::TN / 2) : 0;   // (the second half of its blocks is not read)
            // columns past the end are never stored; let them read the last column's window
            const uint32_t rel = window_start((uint32_t)(j < n_end ? j : n_end - 1)) - g_first;
            f[nb] = Cfg::B_BASE + stage_offset + half * Cfg::B_PLANE + (int)rel * 16;
        }
    };
    auto read = [&](int at) __attribute__((always_inline)) { return *reinterpret_cast<const u32x4 *>(lds + at); };
    // product 0: h*m', 1: m*h', 2: h*h'; block j: column block first
    auto mfma = [&](int prod, int set, int j, bool fresh) __attribute__((always_inline)) {
        const int mb = j % MB, nb = j / MB;
        const f16x8 a = __builtin_bit_cast(f16x8, prod == 1 ? am[mb] : ah[set][mb]);
        const f16x8 b = __builtin_bit_cast(f16x8, prod == 0 ? bm[nb] : bh[nb]);
        f32x16 &sum = prod == 2 ? acc[mb][nb] : low[mb][nb];
        const f32x16 zero = {};
        if constexpr (Cfg::SWAP) sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, a, fresh ? zero : sum, 0, 0, 0);
        else sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, fresh ? zero : sum, 0, 0, 0);
    };
    float c_cur = 0.f, c_before = 0.f;   // 2^-(e + e') of this chunk, of the one before
    uint32_t c_largest = 0, n_chunk = 0;
    // The nine taps of a chunk.  The h*h' sums of the chunk before join the total during the first two products of
    // the first tap, this chunk's small ones during the last product of the last tap; each accumulator then starts from zero.
    auto chunk = [&](int off, int s, int off_next) __attribute__((always_inline)) {
        uint32_t c_bits = 0;
        static_for<9>([&](auto tc) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value, set = t & 1;
            constexpr bool last = t % 3 == 2;
            const int a_next = fa + (t == 8 ? a_other : (t + 1) * Cfg::A_TAP);
            const bool wrap = s + 1 == p.S;
            const int off_after = t == 8 ? off_next : off + (wrap ? to_row : in_row);
            s = wrap ? 0 : s + 1;
            const int (&f)[NB] = t == 8 ? fb_next : fb;
            if constexpr (t == 1) c_bits = *reinterpret_cast<const uint32_t *>(lds + Cfg::SLOT_C + (n_chunk & 1u) * 4u);
            static_for<3 * M>([&](auto sc) __attribute__((always_inline)) {
                constexpr int i = decltype(sc)::value;
                if constexpr (i == 0) bh[NB - 1] = read(fb[NB - 1] + off);
                if constexpr ((Cfg::WHOLE ? t == 8 : last) && i == M) split_barrier();
                // the next tap's fragments: bm after product 0, ah any time, am after product 1, bh after its blocks of product 2
                if constexpr (i >= M && i < 2 * M) {
                    constexpr int r0 = (i - M) * (NB + MB) / M, r1 = (i - M + 1) * (NB + MB) / M;
                    static_for<r1 - r0>([&](auto rc) __attribute__((always_inline)) {
                        constexpr int r = r0 + decltype(rc)::value;
                        if constexpr (r < NB) bm[r] = read(f[r] + off_after + Cfg::B_PART);
                        else ah[set ^ 1][r - NB] = read(a_next + (r - NB) * 512);
                    });
                }
                if constexpr (i >= 2 * M) {
                    constexpr int r0 = (i - 2 * M) * MB / M, r1 = (i - 2 * M + 1) * MB / M;
                    static_for<r1 - r0>([&](auto rc) __attribute__((always_inline)) {
                        constexpr int r = r0 + decltype(rc)::value;
                        am[r] = read(a_next + r * 512 + Cfg::A_PART);
                    });
                    if constexpr ((i - 2 * M) % MB == 0 && i > 2 * M) bh[(i - 2 * M) / MB - 1] = read(f[(i - 2 * M) / MB - 1] + off_after);
                }
                mfma(i / M, set, i % M, t == 0 && i < 3 * M && (i < M || i >= 2 * M));
                if constexpr (t == 0 && i < 2 * M) {
                    constexpr int mb = (i / 2) % MB, nb = (i / 2) / MB;
#pragma unroll
                    for (int v = 0; v < 8; ++v)
                        total[mb][nb][(i % 2) * 8 + v] = __builtin_fmaf(acc[mb][nb][(i % 2) * 8 + v], c_before, total[mb][nb][(i % 2) * 8 + v]);
                }
                if constexpr (t == 8 && i >= 2 * M) {
                    constexpr int mb = (i - 2 * M) % MB, nb = (i - 2 * M) / MB;
                    const float c_low = c_cur * 0x1p-11f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) total[mb][nb][v] = __builtin_fmaf(low[mb][nb][v], c_low, total[mb][nb][v]);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (t == 4) {
                c_bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)c_bits);
                c_cur = __builtin_bit_cast(float, c_bits);
                c_largest = c_largest > c_bits ? c_largest : c_bits;
            }
            off = off_after;
        });
        fa += a_other;
        a_other = -a_other;
        // (the next chunk's first fragments sit in set 1)
        c_before = c_cur;
        ++n_chunk;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) ah[0][mb] = ah[1][mb];
    };
    // The same of half a tile: one block of columns per wavefront, the other's registers of bh for the next tap's.
    auto half_chunk = [&](int off, int s, int off_next) __attribute__((always_inline)) {
        static_assert(NB == 2 && MB == 2, "one block of columns, registers for two");
        uint32_t c_bits = 0;
        static_for<9>([&](auto tc) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value, set = t & 1;
            constexpr bool last = t % 3 == 2;
            const int a_next = fa + (t == 8 ? a_other : (t + 1) * Cfg::A_TAP);
            const bool wrap = s + 1 == p.S;
            const int off_after = t == 8 ? off_next : off + (wrap ? to_row : in_row);
            s = wrap ? 0 : s + 1;
            const int f = t == 8 ? fb_next[0] : fb[0];
            if constexpr (t == 1) c_bits = *reinterpret_cast<const uint32_t *>(lds + Cfg::SLOT_C + (n_chunk & 1u) * 4u);
            static_for<6>([&](auto sc) __attribute__((always_inline)) {
                constexpr int i = decltype(sc)::value, prod = i / 2, mb = i % 2;
                if constexpr ((Cfg::WHOLE ? t == 8 : last) && i == 2) split_barrier();
                // the next tap's fragments: bm after product 0, ah and bh any time, am after product 1
                if constexpr (i == 2) {
                    bh[set ^ 1] = read(f + off_after);
                    bm[0] = read(f + off_after + Cfg::B_PART);
                }
                if constexpr (i == 3) {
                    ah[set ^ 1][0] = read(a_next);
                    ah[set ^ 1][1] = read(a_next + 512);
                }
                if constexpr (i >= 4) am[mb] = read(a_next + mb * 512 + Cfg::A_PART);
                const f16x8 a = __builtin_bit_cast(f16x8, prod == 1 ? am[mb] : ah[set][mb]);
                const f16x8 b = __builtin_bit_cast(f16x8, prod == 0 ? bm[0] : bh[set]);
                f32x16 &sum = prod == 2 ? acc[mb][0] : low[mb][0];
                const f32x16 zero = {};
                constexpr bool fresh = t == 0 && prod != 1;
                if constexpr (Cfg::SWAP) sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, a, fresh ? zero : sum, 0, 0, 0);
                else sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, fresh ? zero : sum, 0, 0, 0);
                if constexpr (t == 0 && i < 4)
#pragma unroll
                    for (int v = 0; v < 8; ++v)
                        total[i / 2][0][i % 2 * 8 + v] = __builtin_fmaf(acc[i / 2][0][i % 2 * 8 + v], c_before, total[i / 2][0][i % 2 * 8 + v]);
                if constexpr (t == 8 && i >= 4) {
                    const float c_low = c_cur * 0x1p-11f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) total[mb][0][v] = __builtin_fmaf(low[mb][0][v], c_low, total[mb][0][v]);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (t == 4) {
                c_bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)c_bits);
                c_cur = __builtin_bit_cast(float, c_bits);
                c_largest = c_largest > c_bits ? c_largest : c_bits;
            }
            off = off_after;
        });
        fa += a_other;
        a_other = -a_other;
        // (the next chunk's first fragments sit in set 1)
        c_before = c_cur;
        ++n_chunk;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) ah[0][mb] = ah[1][mb];
        bh[0] = bh[1];
    };
    __builtin_amdgcn_s_setprio(2);   // the MFMA stream goes first where both kinds of wavefront want to issue
    split_barrier();
    split_barrier();
    columns(work_number(0), 0, fb);
    int s0;
    int off0 = tap_position(0, &s0);
    auto first_fragments = [&]() __attribute__((always_inline)) {   // of the next chunk
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            ah[0][mb] = read(fa + mb * 512);
            am[mb] = read(fa + mb * 512 + Cfg::A_PART);
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            bm[nb] = read(fb[nb] + off0 + Cfg::B_PART);
            if (nb < NB - 1) bh[nb] = read(fb[nb] + off0);
        }
    };
    first_fragments();
    for (int it = 0;; ++it) {
        const int work = work_number(it);
        if (work >= none) break;
        const bool half_tile = Cfg::HALVES && work % PARTS != 0;
        int n0, n_end;
        [[maybe_unused]] const bool some = work_columns(work, &n0, &n_end);
        const int krow0 = (work / PARTS % p.tilesM) * BM + wm * Cfg::TM;
        int col0 = n0 + wn * Cfg::TN;
        if constexpr (Cfg::HALVES)
            if (half_tile) {
                col0 -= wn * (Cfg::TN / 2);
                n_end = !some ? 0 : (n_end < col0 + Cfg::TN / 2 ? n_end : col0 + Cfg::TN / 2);   // (the wavefront's)
            }
        float bvec[MB];
        load_bias<MB>(p, krow0, l32, bvec);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][nb][v] = total[mb][nb][v] = 0.f;
        c_largest = 0;
        const int next = work_number(it + 1);
        auto multiply = [&](auto one) __attribute__((always_inline)) {   // (a loop for each kind of chunk)
            for (int c = 0; c < nch; ++c)
                for (int g = 0; g < groups; ++g) {
                    int s_next;
                    const int off_next = tap_position(g + 1 < groups ? g + 1 : 0, &s_next);
                    if (g + 1 < groups) {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) fb_next[nb] = fb[nb];
                    } else {
                        if (c + 1 < nch) {
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) fb_next[nb] = fb[nb] + b_other;
                        } else {
                            columns(next < none ? next : work, b_other < 0 ? 0 : Cfg::B_STAGE, fb_next);
                        }
                        b_other = -b_other;
                    }
                    one(off0, s0, off_next);
                    off0 = off_next;
                    s0 = s_next;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) fb[nb] = fb_next[nb];
                }
        };
        if (Cfg::HALVES && half_tile) multiply([&](int off, int tap, int next_off) __attribute__((always_inline)) { half_chunk(off, tap, next_off); });
        else multiply([&](int off, int tap, int next_off) __attribute__((always_inline)) { chunk(off, tap, next_off); });
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) total[mb][nb][v] = __builtin_fmaf(acc[mb][nb][v], c_before, total[mb][nb][v]);
        // What a sum may be off by, times 2^22: each lost operand of the patch by 2^-36 times one of the filter's - as many as were counted, below 2^15
        // each, or all of the row's -, each of the filter's by 2^-36 * 2^15; scaled.
        const u32x4 lossy = *reinterpret_cast<const u32x4 *>(lds + Cfg::SLOT_N + (it & 1) * 32);
        const uint32_t count = (lossy[0] & ~kFarBelow) + (lossy[1] & ~kFarBelow) + (lossy[2] & ~kFarBelow);
        const bool zeros_too = __builtin_amdgcn_readfirstlane((int)((lossy[0] | lossy[1] | lossy[2]) & kFarBelow)) != 0;
        const uint32_t all_bits = lossy[3];   // (a bit cast of the vector's element itself takes element 0)
        const float counted = (float)count * 2.f * __builtin_bit_cast(float, c_largest), all = __builtin_bit_cast(float, all_bits);
        float off_by = *reinterpret_cast<const float *>(lds + Cfg::SLOT_N + (it & 1) * 32 + 16) + (count == 0u ? 0.f : (counted < all ? counted : all));
        off_by = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, off_by)));
        ConvKernelParams pt = p;
        pt.NPQ = n_end;
        // (rows beyond the last one are zero and would always be asked about: they count as large)
        const bool ragged = zeros_too && krow0 + Cfg::TM > p.K;
        if (__builtin_expect(ragged, 0)) {
            const int rows = p.K - krow0 - (Cfg::SWAP ? l32 : half * 4);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        total[mb][nb][v] = mb * 32 + (Cfg::SWAP ? 0 : v / 4 * 8 + v % 4) < rows ? total[mb][nb][v] : 3e38f;
        }
        if (Cfg::HALVES && half_tile) {   // (the other blocks count as large, and are not stored)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) total[mb][NB - 1][v] = 3e38f;
        }
        if (__builtin_expect(__any(outside_halves_range<MB, NB>(total, off_by, zeros_too)), 0)) {
            f32x16 blocks[MB * NB];
#pragma unroll
            for (int g = 0; g < MB * NB; ++g) blocks[g] = total[g / NB][g % NB];
            halves_mend<Cfg::SWAP, MB, NB>((uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr(), blocks, off_by, zeros_too, n_end, krow0, col0);
#pragma unroll
            for (int g = 0; g < MB * NB; ++g) total[g / NB][g % NB] = blocks[g];
            first_fragments();   // (again: not held across the call)
        }
        const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, kBufferWord3);
        store_tile<Cfg::SWAP, MB, NB>(pt, ybuf, total, bvec, krow0, col0, half, l32);
    }
#endif
}

}  // namespace igc
#endif
