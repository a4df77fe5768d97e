// fp32 backward filter on the 16-bit matrix pipes: dw = dy . D_m^T with every float operand as two binary16 parts
// (igconv_kernel_f32h.hpp: what the parts hold, what three products leave out of one of floats), unit horizontal stride, rows of three taps and more.
// Rows are feature maps k of dy, 64 per tile; columns come in units of (32 channels, three neighbouring taps of a filter row),
// two units per tile; the reduction runs over output pixels (n,p,q) in chunks of 128 and is cut into ranges, one
// (tile, range) after another per workgroup (igconv_kernel_wgrad.hpp).
//
// Why this shape.  The kernel by tap (igconv_kernel_wgrad_f32s.hpp) is bound by its moving wavefronts: an element of x is fetched
// and split once for every tap.  Here the pixels of x that a chunk's three taps read - 128 and two more per output row - are split
// once into LDS, 136 elements of splitting per 12288 products; one tap more is a read from LDS at the next pixel.
//
// Measured, us, three bfloat16 parts or fp32 instruction -> this, 128 images: 64x56x56 -> 64, 3x3 256 -> 135 (error against 64 bits 1.1e-6 -> 3.3e-7),
// channels innermost 784 -> 128; 384x13x13 -> 256, 3x3 234 -> 198 (4.4e-7 -> 3.9e-7); 96x27x27 -> 256, 5x5 822 -> 546; 96x64x64 -> 128, 9x9, 32 images 1419 -> 768
// (1.2e-6 -> 8.2e-7).
// What bounds it: instruction issue of the moving wavefronts, one per SIMD, about 750 instructions of 5.3 cycles per chunk (binary16
// fused multiply-adds take 9.3) where the MFMAs take 2304: 9400 cycles in all at 64x56x56; without its loads 106 us, without its MFMAs 132.
// Chunks of 64 pixels took 214 us, an item's eight loads together instead of among the splitting of the next one 822 (9x9),
// a kernel argument read where it is used instead of all at once 178.
//
// LDS holds both operands pixel by pixel, [operand][stage][part][block of 32 rows][8 rows][pixel][row of 8]: movers read 16
// neighbouring pixels of 32 rows with eight loads and write 16 bytes per lane and part; the multipliers, whose
// reduction index is the pixel, read four pixels at a time with the transposing LDS read (ds_read_b64_tr_b16: lane i of 16 gets
// element i % 4 of the words that lanes i / 4, i / 4 + 4, ... address).  A row of pixels in the other order would let no tap but
// every eighth be read in 16 bytes.
//
// Four multiplying wavefronts (one of the two units, one half of a chunk's pixels each: 64 x 32 x 3 taps, h*h' and the small
// products in accumulators of their own) and four moving ones; one barrier per chunk, two stages.  The two pixel halves' sums meet in
// LDS when a range ends.  Movers work on three chunks at once: pixel offsets of the one after next but one are
// decoded (one pixel per lane, into a table), loads of the one after next are requested, the next one's largest magnitude is taken,
// the chunk itself is split and written.
//
// Exponents.  As in the forward kernel an operand is scaled by a power of two, here kept from chunk to chunk of a range while the
// chunk's largest magnitude, scaled, stays within [2^13, 2^15) (it is put into [2^13, 2^14) when it does not; the sums so far are then
// multiplied by the ratio, which the multipliers have time for), and at most 2^40 finer than that of the range's largest chunk.  Operands below 2^-13
// after scaling lose up to 2^-36; the movers count the lanes that have some, and with them, per chunk, what a sum may be off by.  Results below 2^22 times that, not
// finite, or not zero but below 2^-100 are multiplied again one by one, more than 96 of a wavefront's 6144 all with the fp32 instruction (wgrad_halves_mend);
// zeros as in the forward kernel.
// us, 128x64x56x56 -> 64, 3x3 (scaled to [2^6, 2^15), every range with such an operand multiplied again -> this): normal 154 -> 154; one gradient of 1e-11
// 791 -> 175 with a map of zeros; log-normal gradients, sigma 2 820 -> 162, with maps of zeros 825 -> 161, 2.5 880 -> 185 and 222, 3 875 -> 215 and 258;
// images whose gradients differ by up to 10^12 787 -> 222.
#ifndef IGCONV_KERNEL_WGRAD_F32H_HPP_
#define IGCONV_KERNEL_WGRAD_F32H_HPP_

#include "igconv_kernel_f32h.hpp"

namespace igc {

// NHWC: both tensors channel-fastest (16-byte loads of channels).
template <bool NHWC_>
struct WgradHalvesConfig {
    static constexpr bool NHWC = NHWC_;
    static constexpr int BM = 64, BN = 64, BK = 128, TAPS = 3, PIX = 160, THREADS = 512;
    static constexpr int A_PLANE = BK * 16 + 64, B_PLANE = PIX * 16 + 64;   // (eight rows; 64 bytes more: neighbouring planes in other banks)
    static constexpr int A_BLOCK = 4 * A_PLANE, B_BLOCK = 4 * B_PLANE;      // 32 rows
    static constexpr int A_PART = 2 * A_BLOCK, B_PART = 2 * B_BLOCK;
    static constexpr int A_STAGE = 2 * A_PART, B_STAGE = 2 * B_PART, B_BASE = 2 * A_STAGE;
    static constexpr int SUMS = 2 * A_STAGE + 2 * B_STAGE;                     // eight of the second pixel half's sums [unit][register][lane]
    static constexpr int SUM_ROUNDS = TAPS * 2 * 2;
    static constexpr int TABLE = SUMS + 2 * 8 * 256;           // [parity][pixel of the patch: unit 0, unit 1; pixel of dy] offsets
    static constexpr int TABLE_BYTES = (2 * PIX + BK) * 4;
    static constexpr int POS = TABLE + 2 * TABLE_BYTES;        // [chunk % 4][pixel]: distance of its window in the patch
    static constexpr int SLOT_MAX = POS + 4 * BK * 4;          // largest magnitudes [parity][dy, x][wavefront]
    static constexpr int SLOT_E = SLOT_MAX + 64;               // e + e' [parity of the chunk]
    static constexpr int SLOT_N = SLOT_E + 16;                 // what a sum may be off by [parity of the range][wavefront]; sign: kFarBelow
    static constexpr int LDS_BYTES = SLOT_N + 32;
    static constexpr int A_ITEMS = BK / 16 * 2 / 4, B_ITEMS = PIX / 16 * 2 / 4, ITEMS = A_ITEMS + B_ITEMS;   // of 16 pixels x 32 rows, per moving wavefront
    static_assert(LDS_BYTES <= 160 * 1024 && A_STAGE + A_PART + A_BLOCK + 256 < 65536 && B_STAGE + B_PART + 32 < 65536, "LDS budget, offsets of the LDS instructions");
};

// Row (channel) that stands at position `at` (of 0..31) of the block beginning at `first`: eights beyond the last
// whole one are the last eight again; *ours: not one that an earlier position has.
__device__ __forceinline__ int wgrad_row(int first, int at, int count, bool *ours) {
    const int begin = first + (at & ~7), from = begin < count - 8 ? begin : count - 8;
    *ours = from + (at & 7) >= begin;
    return from + (at & 7);
}

// A wavefront's blocks over its share of the output pixels [j_begin, j_end) - 64 of every `apart` - with the fp32 instruction straight from global memory.
__device__ __forceinline__ void wgrad_halves_in_fp32(const ConvKernelParams &p, f32x16 (&acc)[3][2], int m0, int c0, int tap_h, int tap_w, int j_begin,
                                                     int j_end, int part, int apart, int half, int l32) {
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    bool ours;
    uint32_t rowoff[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) rowoff[mb] = (uint32_t)wgrad_row(m0 + mb * 32, l32, p.K, &ours) * (uint32_t)p.wsRow * 4u;
    const uint32_t coloff = (uint32_t)wgrad_row(c0, l32, p.NPQ, &ours) * (uint32_t)p.xsN * 4u;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][mb][v] = 0.f;
#pragma clang loop unroll(disable)
    for (int jb = j_begin + part * 64; jb < j_end; jb += apart)
#pragma clang loop unroll(disable)
        for (int i = 0; i < 64; i += 2) {
            const uint32_t j = (uint32_t)(jb + i + half);
            const bool live = (int)j < j_end;
            const uint32_t n = magic_div(j, p.mRS);
            const uint32_t rem = j - n * (uint32_t)p.RS;
            const uint32_t pp = magic_div(rem, p.mS);
            const uint32_t qq = rem - pp * (uint32_t)p.S;
            const uint32_t hh = pp * (uint32_t)p.redMulH + (uint32_t)tap_h;
            const uint32_t ao = (n * (uint32_t)p.wsRed + pp * (uint32_t)p.wsTapR + qq * (uint32_t)p.wsTapS) * 4u;
            float a[2], b[3];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                a[mb] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, live ? rowoff[mb] + ao : kOutOfRange, 0, 0));
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const uint32_t ww = qq + (uint32_t)(tap_w + t);
                const bool ok = live && hh < (uint32_t)p.H && ww < (uint32_t)p.W;
                const uint32_t xo = (n * (uint32_t)p.xsC + hh * (uint32_t)p.xsH + ww * (uint32_t)p.xsW) * 4u;
                b[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, ok ? coloff + xo : kOutOfRange, 0, 0));
            }
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) acc[t][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mb], b[t], acc[t][mb], 0, 0, 0);
        }
}

#if defined(__HIP_DEVICE_COMPILE__)
// One bit per lane of a half wavefront, set in either of the two.
__device__ __forceinline__ uint32_t nonzero_lanes(uint32_t v) {
    const uint64_t m = __ballot(v != 0u);
    return (uint32_t)m | (uint32_t)(m >> 32);
}
// A wavefront's blocks of a range: where they are.
struct WgradMend {
    int m0, c0, tap_h, tap_w, j_begin, j_end, part, apart;   // (its share: 64 of every `apart` pixels, from part * 64 on)
    bool live;        // (not one that fills up a pair of units)
    bool zeros_too;   // (mend_results)
};

// As halves_mend of the forward kernel: the sums that are out of range or that something lost could have touched, one by one or all.
__device__ __attribute__((noinline)) void wgrad_halves_mend(uint64_t arguments, f32x16 *blocks, float limit, WgradMend where) {
    ConvKernelParams p = *(KernelArguments *)(uintptr_t)uniform64(arguments);
    auto uniform = [](auto &v) __attribute__((always_inline)) { v = __builtin_bit_cast(std::remove_reference_t<decltype(v)>, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v))); };
    uniform(limit);
    uniform(where.m0); uniform(where.c0); uniform(where.tap_h); uniform(where.tap_w); uniform(where.j_begin); uniform(where.j_end); uniform(where.part); uniform(where.apart);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    f32x16 acc[3][2];
#pragma unroll
    for (int g = 0; g < 6; ++g) acc[g / 2][g % 2] = blocks[g];
    auto get = [&](auto gc, auto vc) __attribute__((always_inline)) {
        const float a = acc[decltype(gc)::value / 2][decltype(gc)::value % 2][decltype(vc)::value];
        return a;
    };
    auto set = [&](auto gc, auto vc, float a) __attribute__((always_inline)) { acc[decltype(gc)::value / 2][decltype(gc)::value % 2][decltype(vc)::value] = a; };
    auto in_block = [](int v, int h) { return v / 4 * 8 + v % 4 + h * 4; };   // row of a block
    auto counts = [&](auto, auto) { return where.live; };
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    // a lane's output pixel: its offset in dy, of its window in x; the window's place
    struct Pixel { uint32_t ao, xo; bool live, row; uint32_t w; };
    auto pixel = [&](int j) __attribute__((always_inline)) {
        const uint32_t n = magic_div((uint32_t)j, p.mRS), rem = (uint32_t)j - n * (uint32_t)p.RS, pp = magic_div(rem, p.mS), qq = rem - pp * (uint32_t)p.S;
        const uint32_t h = pp * (uint32_t)p.redMulH + (uint32_t)where.tap_h;
        Pixel x;
        x.live = j < where.j_end;
        x.row = x.live && h < (uint32_t)p.H;
        x.w = qq + (uint32_t)where.tap_w;
        x.ao = (n * (uint32_t)p.wsRed + pp * (uint32_t)p.wsTapR + qq * (uint32_t)p.wsTapS) * 4u;
        x.xo = (n * (uint32_t)p.xsC + h * (uint32_t)p.xsH + x.w * (uint32_t)p.xsW) * 4u;
        return x;
    };
    auto load_dy = [&](const Pixel &x, uint32_t rowoff) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, x.live ? rowoff + x.ao : kOutOfRange, 0, 0));
    };
    auto load_x = [&](const Pixel &x, uint32_t coloff, int t) __attribute__((always_inline)) {
        const bool ok = x.row && x.w + (uint32_t)t < (uint32_t)p.W;
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, ok ? coloff + x.xo + (uint32_t)(t * p.xsW) * 4u : kOutOfRange, 0, 0));
    };
    auto rowoff_of = [&](int mb, int r) __attribute__((always_inline)) {
        bool ours;
        return (uint32_t)wgrad_row(where.m0 + mb * 32, r, p.K, &ours) * (uint32_t)p.wsRow * 4u;
    };
    auto coloff_of = [&](int c) __attribute__((always_inline)) {
        bool ours;
        return (uint32_t)wgrad_row(where.c0, c, p.NPQ, &ours) * (uint32_t)p.xsN * 4u;
    };
    const int j_first = where.j_begin + where.part * 64 + lane;
    // Maps, then channels, of zeros: the lanes along the pixels, as far as the first operand that is not zero.
    auto zeros = [&](uint32_t (&zero)[6]) __attribute__((always_inline)) {
        uint64_t rows = 0, all_zero = 0;   // (bit 32 mb + r)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            const uint32_t asked = zero[mb] | zero[2 + mb] | zero[4 + mb];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint64_t m = __ballot((asked >> v) & 1u);
                rows |= (uint64_t)(((uint32_t)m != 0u ? 1u : 0u) << in_block(v, 0) | ((m >> 32) != 0u ? 1u : 0u) << in_block(v, 1)) << (32 * mb);
            }
        }
#pragma clang loop unroll(disable)
        while (rows != 0u) {   // four at a time (fewer left: the last again)
            uint32_t rowoff[4], found = 0;
            int r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                r[i] = rows != 0u ? __builtin_ctzll(rows) : r[i > 0 ? i - 1 : 0];
                rows &= rows - 1u;
                rowoff[i] = rowoff_of(r[i] >> 5, r[i] & 31);
            }
#pragma clang loop unroll(disable)
            for (int j = j_first; __any(j < where.j_end) && found != 15u; j += 6 * where.apart) {
                float a[6][4];
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    const Pixel x = pixel(j + e * where.apart);
#pragma unroll
                    for (int i = 0; i < 4; ++i) a[e][i] = load_dy(x, rowoff[i]);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    bool some = false;
#pragma unroll
                    for (int e = 0; e < 6; ++e) some = some || a[e][i] != 0.f;
                    found |= __any(some) ? 1u << i : 0u;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) all_zero |= ((found >> i) & 1u) != 0u ? 0u : (uint64_t)1 << r[i];
        }
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            uint32_t bits = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) bits |= (((uint32_t)(all_zero >> (32 * mb)) >> in_block(v, half)) & 1u) << v;
#pragma unroll
            for (int t = 0; t < 3; ++t) zero[t * 2 + mb] &= ~bits;
        }
        uint32_t channels = nonzero_lanes(zero[0] | zero[1] | zero[2] | zero[3] | zero[4] | zero[5]), some_in[3] = {~0u, ~0u, ~0u};
#pragma clang loop unroll(disable)
        while (channels != 0u) {   // two at a time, three taps
            const int c0 = __builtin_ctz(channels);
            channels &= channels - 1u;
            const int c1 = channels != 0u ? __builtin_ctz(channels) : c0;
            channels &= channels - 1u;
            const uint32_t coloff[2] = {coloff_of(c0), coloff_of(c1)};
            uint32_t found = 0;
#pragma clang loop unroll(disable)
            for (int j = j_first; __any(j < where.j_end) && found != 63u; j += 4 * where.apart) {
                float b[4][6];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const Pixel x = pixel(j + e * where.apart);
#pragma unroll
                    for (int i = 0; i < 6; ++i) b[e][i] = load_x(x, coloff[i / 3], i % 3);
                }
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    bool some = false;
#pragma unroll
                    for (int e = 0; e < 4; ++e) some = some || b[e][i] != 0.f;
                    found |= __any(some) ? 1u << i : 0u;
                }
            }
#pragma unroll
            for (int i = 0; i < 6; ++i) some_in[i % 3] &= ((found >> i) & 1u) != 0u ? ~0u : ~(1u << (i < 3 ? c0 : c1));
        }
#pragma unroll
        for (int g = 0; g < 6; ++g) zero[g] = ((some_in[g / 2] >> l32) & 1u) != 0u ? zero[g] : 0u;
    };
    auto sums = [&](const int (&which)[4], const int (&from)[4], float (&s)[4]) __attribute__((always_inline)) {
        uint32_t rowoff[4], coloff[4];
        int tap[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int g = which[i] >> 4;
            rowoff[i] = rowoff_of(g % 2, in_block(which[i] & 15, from[i] >> 5));
            coloff[i] = coloff_of(from[i] & 31);
            tap[i] = g / 2;
            s[i] = 0.f;
        }
#pragma clang loop unroll(disable)
        for (int j = j_first; __any(j < where.j_end); j += 4 * where.apart) {
            float a[4][4], b[4][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const Pixel x = pixel(j + e * where.apart);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a[e][i] = load_dy(x, rowoff[i]);
                    b[e][i] = load_x(x, coloff[i], tap[i]);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] = __builtin_fmaf(a[e][i], b[e][i], s[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = wave_sum(s[i]);
    };
    const bool zeros_too = __builtin_amdgcn_readfirstlane((int)where.zeros_too) != 0;
    // (64x56x56 -> 64: four results 13 us, a range's blocks 700)
    if (!mend_results<6, 96>([&](auto, auto) { return limit; }, [&](auto) { return zeros_too ? 0xFFFFu : 0u; }, lane, get, set, counts, zeros, sums))
        wgrad_halves_in_fp32(p, acc, where.m0, where.c0, where.tap_h, where.tap_w, where.j_begin, where.j_end, where.part, where.apart, half, l32);
#pragma unroll
    for (int g = 0; g < 6; ++g) blocks[g] = acc[g / 2][g % 2];
}

// What a moving wavefront of the filter kernels knows of its operands: the exponents of dy (a) and of the patch (b) that the chunk being written is split
// by, and what a sum may be off by for what they lost.
struct WgradScales {
    int ea = 0, eb = 0, e_low = 0, e_high = 0;
    bool set_a = false, set_b = false, begun = false;
    float off_by = 0.f;      // 2^22 times what a sum of the chain may be off by for this wavefront's operands that lost something
    uint32_t far = 0;        // kFarBelow: one of them far below the others
    HalvesScale sa = {}, sb = {};

    // the largest magnitude of all moving wavefronts
    static __device__ __forceinline__ uint32_t largest_of(const uint8_t *slots) {
        const u32x4 s = *reinterpret_cast<const u32x4 *>(slots);
        const uint32_t s0 = s[0] > s[1] ? s[0] : s[1], s1 = s[2] > s[3] ? s[2] : s[3];
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(s0 > s1 ? s0 : s1));
    }
    // an exponent out of bounds?  (zeros say nothing)
    static __device__ __forceinline__ bool fits(uint32_t largest, int e, bool set) { return largest == 0 || (set && (uint32_t)((int)(largest >> 23) - 140 + e) <= 1u); }
    static __device__ __forceinline__ void choose(uint32_t largest, int &e, bool &set) {
        const int w = 140 - (int)(largest >> 23);
        e = w < -60 ? -60 : (w > 60 ? 60 : w);
        set = true;
    }
    static __device__ __forceinline__ HalvesScale scale_of(int e) {
        HalvesScale r;
        r.e = e;
        r.s = __builtin_bit_cast(float, (uint32_t)(127 + e) << 23);
        r.t = __builtin_bit_cast(float, (uint32_t)(138 + e) << 23);
        r.below = (uint32_t)(114 - e) << 23;
        return r;
    }
    // The next chunk, of a new chain of sums if `first`.  slots: the wavefronts' largest magnitudes of dy, then of the patch; small_a, small_b: this lane's
    // smallest ones.  A lost operand may have touched as many of a result's products as the lane's pixels are: A_LANE of dy, B_LANE of the patch, for all
    // lanes not more than A_MOST and 64; each by 2^-36 of the other operand's largest.
    template <int A_LANE, int A_MOST, int B_LANE>
    __device__ __forceinline__ void next(const uint8_t *slots, bool first, uint32_t small_a, uint32_t small_b) {
        const uint32_t la = largest_of(slots), lb = largest_of(slots + 16);
        if (first || !fits(la, ea, set_a) || !fits(lb, eb, set_b)) {
            if (first) {
                set_a = set_b = begun = false;
                off_by = 0.f;
                far = 0;
            }
            if (!fits(la, ea, set_a)) choose(la, ea, set_a);
            if (!fits(lb, eb, set_b)) choose(lb, eb, set_b);
            if (set_a && set_b) {   // (before that all products are zero)
                // A chunk far below the range's largest gets no finer unit than 2^-40 of that one's: sums multiplied up by more could leave the float range.
                // Those multiplied down by more than 2^-70 could lose something.
                const int over = begun && ea + eb > e_low + 40 ? ea + eb - (e_low + 40) : 0, of_a = over < ea + 100 ? over : ea + 100;
                ea -= of_a;
                eb -= over - of_a;
                const int e = ea + eb;
                if (begun && e_high - e > 70) off_by += __builtin_ldexpf(2.f, -e);
                e_low = !begun || e < e_low ? e : e_low;
                e_high = !begun || e > e_high ? e : e_high;
                begun = true;
            }
            sa = scale_of(ea);
            sb = scale_of(eb);
        }
        const uint64_t under_a = lanes_under(small_a, sa.below), under_b = lanes_under(small_b, sb.below);
        if ((under_a | under_b) != 0u) {
            const int na = A_LANE * __popcll(under_a), nb = B_LANE * __popcll(under_b);
            // (none times infinity would be NaN)
            if (na != 0) off_by += (float)(na < A_MOST ? na : A_MOST) * __builtin_ldexpf(__builtin_bit_cast(float, lb), -ea - 14);   // (times 2^22)
            if ((lanes_under(small_a, far_below(sa.below)) | lanes_under(small_b, far_below(sb.below))) != 0u) far = kFarBelow;
            if (nb != 0) off_by += (float)(nb < 64 ? nb : 64) * __builtin_ldexpf(__builtin_bit_cast(float, la), -eb - 14);
        }
    }
};
// What a sum of a chain may be off by, of all moving wavefronts; zeros_too: sums of zero are in question as well.
__device__ __forceinline__ float wgrad_off_by(const uint8_t *slots, bool *zeros_too) {
    const u32x4 s = *reinterpret_cast<const u32x4 *>(slots);
    float off_by = 0.f;
    uint32_t far = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t slot = s[i];
        off_by += __builtin_bit_cast(float, slot & ~kFarBelow);
        far |= slot & kFarBelow;
    }
    *zeros_too = __builtin_amdgcn_readfirstlane((int)far) != 0;
    return off_by;
}
#endif

// p.Wp: pixels of a row of the patch (output columns and two), p.HpWp: output rows; p.PQ: blocks of 32 channels;
// p.tilesN: pairs of units; otherwise as for the kernels by tap.
template <class Cfg>
__global__ __launch_bounds__(512, 2) void igconv_wgrad_f32h_kernel(const ConvKernelParams p) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernel's name and signature only)
    constexpr int BK = Cfg::BK, PIX = Cfg::PIX, ITEMS = Cfg::ITEMS;

    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // persistent workgroups over (tile, range) numbers in contiguous ranges per XCD (see igconv_kernel_wgrad.hpp)
    const int wg_xcd = (int)(blockIdx.x % 8u), wg_local = (int)(blockIdx.x / 8u);
    const int tiles_mn = p.tilesM * p.tilesN;
    const int tiles_total = tiles_mn * p.splits;
    auto tile_number = [&](int i) {
        const int local = wg_local + i * p.wgsPerXcd;
        const int t = wg_xcd * p.tilesPerXcd + local;
        return local < p.tilesPerXcd && t < tiles_total ? t : tiles_total;
    };
    if (tile_number(0) >= tiles_total) return;
    const int per = p.stepsPerSplit < 2 ? 2 : p.stepsPerSplit;   // chunks of a range (even: the stage alternates)
    const int groups = (p.Q + 2) / 3;                            // of three taps in a filter row (p.Q of them; the last ones overlap)
    const int units = p.R * groups * p.PQ;
    struct Unit { int c0, r, s0, skip, tap_h, tap_w; bool live; };
    struct Tile { int m0, u0, split; };
    auto tile_of = [&](int number) {
        if (number >= tiles_total) number = 0;   // (no tile: any; nothing of it is multiplied)
        Tile t;
        t.split = number / tiles_mn;
        const int tile = number - t.split * tiles_mn;
        t.m0 = (tile % p.tilesM) * Cfg::BM;
        t.u0 = tile / p.tilesM * 2;
        return t;
    };
    auto unit_of = [&](int u) {
        Unit r;
        r.live = u < units;
        if (!r.live) u = units - 1;
        const int rg = u / p.PQ;
        r.c0 = (u - rg * p.PQ) * 32;
        r.r = rg / groups;
        const int s_first = (rg - r.r * groups) * 3;
        r.s0 = s_first < p.Q - 3 ? s_first : p.Q - 3;
        r.skip = s_first - r.s0;   // storage taps that another unit has
        r.tap_h = (p.flip ? p.R - 1 - r.r : r.r) - p.pad_h;
        r.tap_w = (p.flip ? p.Q - 3 - r.s0 : r.s0) - p.pad_w;
        return r;
    };
    int ntiles = 0;
    while (tile_number(ntiles) < tiles_total) ++ntiles;

    if (wave >= 4) {
        // ================================ movers ================================
        const int mw = wave - 4;
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        const int px = lane & 15, plane = lane >> 4;   // within an item
        // ---- A chunk's pixels: offsets in the patch (wavefronts 0 to 2) and in dy (2 and 3), distances of the windows (0 and 1).
        // The parameters of this are read again for each chunk, all at once: kept, they would drive the strides of the loads out
        // of the scalar registers.
        struct Decode {
            Magic mQ, mRow, mP, mPQ;
            int32_t pixels, Wp, P, Q, PQ, down, H, W, xN, xH, xW, yN, yP, yQ;
        };
        auto decode_parameters = [&]() __attribute__((always_inline)) {
            using Params = const __attribute__((address_space(4))) ConvKernelParams;
            uint64_t at = (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(at));
            Params *const q = (Params *)at;
            Decode d;
            d.mQ = Magic{q->mS.mul, q->mS.shift}; d.mRow = Magic{q->mWp.mul, q->mWp.shift};
            d.mP = Magic{q->mHpWp.mul, q->mHpWp.shift}; d.mPQ = Magic{q->mRS.mul, q->mRS.shift};
            d.pixels = q->CRS; d.Wp = q->Wp; d.P = q->HpWp; d.Q = q->S; d.PQ = q->RS; d.down = q->redMulH; d.H = q->H; d.W = q->W;
            d.xN = q->xsC; d.xH = q->xsH; d.xW = q->xsW; d.yN = q->wsRed; d.yP = q->wsTapR; d.yQ = q->wsTapS;
            return d;
        };
        struct Span { int j0, j_last; uint32_t g0, length; };   // first and last pixel; first window, patch length (to the last window's end)
        auto span_of = [&](const Decode &d, int j0) __attribute__((always_inline)) {
            Span s;
            const int jf = j0 < d.pixels ? j0 : d.pixels - 1;
            s.j0 = j0;
            s.j_last = j0 + BK - 1 < d.pixels ? j0 + BK - 1 : d.pixels - 1;
            s.g0 = (uint32_t)jf + 2u * magic_div((uint32_t)jf, d.mQ);
            s.length = (uint32_t)s.j_last + 2u * magic_div((uint32_t)s.j_last, d.mQ) + 3u - s.g0;
            return s;
        };
        int t_it = 0, t_c = 0, t_j0 = 0;
        int t_h[2], t_w[2];
        auto table_tile = [&]() {
            const Tile t = tile_of(tile_number(t_it));
            t_j0 = t.split * per * BK;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const Unit r = unit_of(t.u0 + u);
                t_h[u] = r.tap_h;
                t_w[u] = r.tap_w;
            }
        };
        table_tile();
        auto write_table = [&](const Decode &d, int parity) __attribute__((always_inline)) {
            uint8_t *const table = lds + Cfg::TABLE + parity * Cfg::TABLE_BYTES;
            const Span s = span_of(d, t_j0);
            if (mw < 3) {
                const int at = mw * 64 + lane;
                const uint32_t g = s.g0 + (uint32_t)at;
                const uint32_t row = magic_div(g, d.mRow), col = g - row * (uint32_t)d.Wp;
                const uint32_t n = magic_div(row, d.mP), pp = row - n * (uint32_t)d.P;
                const uint32_t image = n * (uint32_t)d.xN, down = pp * (uint32_t)d.down;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t h = down + (uint32_t)t_h[u], w = col + (uint32_t)t_w[u];   // (below zero: huge)
                    const bool ok = (uint32_t)at < s.length && h < (uint32_t)d.H && w < (uint32_t)d.W;
                    if (at < PIX)
                        *reinterpret_cast<uint32_t *>(table + u * PIX * 4 + at * 4) = ok ? (image + h * (uint32_t)d.xH + w * (uint32_t)d.xW) * 4u : kOutOfRange;
                }
            }
            if (mw >= 2) {
                const int at = (mw - 2) * 64 + lane;
                const uint32_t j = (uint32_t)(t_j0 + at);
                const uint32_t row = magic_div(j, d.mQ), qq = j - row * (uint32_t)d.Q;
                const uint32_t n = magic_div(j, d.mPQ), pp = row - n * (uint32_t)d.P;
                *reinterpret_cast<uint32_t *>(table + 2 * PIX * 4 + at * 4) =
                    (int)j < d.pixels ? (n * (uint32_t)d.yN + pp * (uint32_t)d.yP + qq * (uint32_t)d.yQ) * 4u : kOutOfRange;
            }
            t_j0 += BK;
            if (++t_c == per) {
                t_c = 0;
                ++t_it;
                table_tile();
            }
            return s;
        };
        auto write_positions = [&](const Decode &d, const Span &s, int slot) __attribute__((always_inline)) {
            if (mw < 2) {
                const int at = mw * 64 + lane, j = s.j0 + at < s.j_last ? s.j0 + at : s.j_last;
                *reinterpret_cast<uint32_t *>(lds + Cfg::POS + slot * BK * 4 + at * 4) = ((uint32_t)j + 2u * magic_div((uint32_t)j, d.mQ) - s.g0) * 16u;
            }
        };

        // ---- requests.  Item i, dy: block i % 2, pixels 16 (4 (i / 2) + mw) ..; patch: n = 4 (i - A_ITEMS) + mw, unit n % 2, pixels n / 2 * 16 ..
        float reg[2][ITEMS][8];
        uint32_t rowoff[2], choff;
        int r_it = 0, r_c = 0;
        auto request_tile = [&]() {
            const Tile t = tile_of(tile_number(r_it));
            const int at = plane * 8;
            bool ours;
#pragma unroll
            for (int i = 0; i < 2; ++i) rowoff[i] = (uint32_t)wgrad_row(t.m0 + i * 32, at, p.K, &ours) * (uint32_t)p.wsRow * 4u;
            choff = (uint32_t)wgrad_row(unit_of(t.u0 + (mw & 1)).c0, at, p.NPQ, &ours) * (uint32_t)p.xsN * 4u;
        };
        request_tile();
        uint32_t row_step[8], ch_step[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            row_step[e] = (uint32_t)(e * p.wsRow) * 4u;
            ch_step[e] = (uint32_t)(e * p.xsN) * 4u;
        }
        constexpr int PIXELS = Cfg::A_ITEMS / 2 + Cfg::B_ITEMS;   // different pixels of a thread's items
        uint32_t pixel_at[PIXELS];
        auto read_table = [&](int parity) __attribute__((always_inline)) {
            const uint8_t *const table = lds + Cfg::TABLE + parity * Cfg::TABLE_BYTES;
#pragma unroll
            for (int i = 0; i < PIXELS; ++i)
                pixel_at[i] = *reinterpret_cast<const uint32_t *>(i < Cfg::A_ITEMS / 2 ? table + 2 * PIX * 4 + ((i * 4 + mw) * 16 + px) * 4
                                                                                      : table + (mw & 1) * PIX * 4 + (((4 * (i - Cfg::A_ITEMS / 2) + mw) >> 1) * 16 + px) * 4);
        };
        // quarter q of item i's loads
        auto request = [&](auto set_c, auto ic, int q) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value, i = decltype(ic)::value;
            constexpr bool of_dy = i < Cfg::A_ITEMS;
            const uint32_t off = pixel_at[of_dy ? i / 2 : i - Cfg::A_ITEMS / 2] + (of_dy ? rowoff[i & 1] : choff);
            const __amdgpu_buffer_rsrc_t buf = of_dy ? wbuf : xbuf;
            if constexpr (Cfg::NHWC) {
                if (q & 1) return;
                const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, off + (uint32_t)q * 8u, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) reg[set][i][q * 2 + e] = v[e];
            } else {
#pragma unroll
                for (int e = 2 * q; e < 2 * q + 2; ++e) reg[set][i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(buf, off, of_dy ? row_step[e] : ch_step[e], 0));
            }
        };
        auto request_item = [&](auto set_c, auto ic) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) request(set_c, ic, q);
        };
        auto next_request = [&]() __attribute__((always_inline)) {
            if (++r_c == per) {
                r_c = 0;
                ++r_it;
                request_tile();
            }
        };
        auto sixteens = [](const Span &s) { return (int)(s.length + 15u) / 16; };   // of pixels of the patch
        constexpr auto always = [](int i) { return i < Cfg::A_ITEMS || (4 * (i - Cfg::A_ITEMS) + 3) / 2 < (BK + 2 + 15) / 16; };   // (whatever the chunk)
        auto held = [&](auto ic, int ng) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            if constexpr (always(i)) return true;
            else return (4 * (i - Cfg::A_ITEMS) + mw) / 2 < ng;
        };

        // ---- magnitudes and scales
        HalvesSeen seen_a, seen_b;          // of the next chunk's operands
        uint32_t small_a = 0, small_b = 0;  // this lane's smallest ones of this chunk
        auto look = [&](auto set_c, auto ic, int q) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value, i = decltype(ic)::value;
            look_at(i < Cfg::A_ITEMS ? seen_a : seen_b, reg[set][i][2 * q], reg[set][i][2 * q + 1]);
        };
        auto look_at_item = [&](auto set_c, auto ic, int ng) __attribute__((always_inline)) {
            if (held(ic, ng))
#pragma unroll
                for (int q = 0; q < 4; ++q) look(set_c, ic, q);
        };
        auto publish = [&](int parity) __attribute__((always_inline)) {
            const uint32_t a = wave_largest(__builtin_bit_cast(uint32_t, seen_a.largest)), b = wave_largest(__builtin_bit_cast(uint32_t, seen_b.largest));
            if (lane == 0) {
                *reinterpret_cast<uint32_t *>(lds + Cfg::SLOT_MAX + parity * 32 + mw * 4) = a;
                *reinterpret_cast<uint32_t *>(lds + Cfg::SLOT_MAX + parity * 32 + 16 + mw * 4) = b;
            }
            small_a = seen_a.smallest;
            small_b = seen_b.smallest;
            seen_a = HalvesSeen{};
            seen_b = HalvesSeen{};
        };
        int it = 0, c = 0;                       // range and chunk being written
        WgradScales scale;
        auto scales = [&](int parity) __attribute__((always_inline)) {
            // (of the 64 pixels that a result's sum takes from the chunk - half of it - this wavefront has 16 of dy, one per lane and map, and up to 64 of the
            // patch, five per lane and channel at most)
            scale.next<1, 16, Cfg::B_ITEMS>(lds + Cfg::SLOT_MAX + parity * 32, c == 0, small_a, small_b);
            if (mw == 0 && lane == 0) *reinterpret_cast<int *>(lds + Cfg::SLOT_E + parity * 4) = scale.ea + scale.eb;
            if (c == per - 1 && lane == 0)
                *reinterpret_cast<uint32_t *>(lds + Cfg::SLOT_N + (it & 1) * 16 + mw * 4) = __builtin_bit_cast(uint32_t, scale.off_by) | scale.far;
        };
        u32x4 part_h, part_m;
        auto convert = [&](auto set_c, auto ic, int q) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value, i = decltype(ic)::value;
            uint32_t h, m;
            halves_pair(reg[set][i][2 * q], reg[set][i][2 * q + 1], i < Cfg::A_ITEMS ? scale.sa : scale.sb, h, m);
            part_h[q] = h; part_m[q] = m;
        };
        auto write_item = [&](auto ic, int parity) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            constexpr bool of_dy = i < Cfg::A_ITEMS;
            const int n = 4 * (i - Cfg::A_ITEMS) + mw;
            uint8_t *const dst = lds + parity * (of_dy ? Cfg::A_STAGE : Cfg::B_STAGE) + (of_dy ? i % 2 * Cfg::A_BLOCK + plane * Cfg::A_PLANE + ((i / 2 * 4 + mw) * 16 + px) * 16
                                                               : Cfg::B_BASE + (mw & 1) * Cfg::B_BLOCK + plane * Cfg::B_PLANE + ((n >> 1) * 16 + px) * 16);
            *reinterpret_cast<u32x4 *>(dst) = part_h;
            *reinterpret_cast<u32x4 *>(dst + (of_dy ? Cfg::A_PART : Cfg::B_PART)) = part_m;
        };
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        // Requests stand under no condition: the compiler counts the loads in flight.  An item of the next chunk is looked at just
        // before the same item of the chunk after it is requested: as many loads stay in flight all along.
        int n_chunk = 0;   // this one's number
        Span span[3];   // of this chunk, the next one, the one after it
        auto interval = [&](auto par_c) __attribute__((always_inline)) {
            constexpr int par = decltype(par_c)::value;
            using Other = std::integral_constant<int, par ^ 1>;
            const Decode d = decode_parameters();
            read_table(par);
            const int ng = sixteens(span[0]), ng_after = sixteens(span[1]);
            write_positions(d, span[1], ++n_chunk & 3);   // (the multipliers may still be reading those of the chunk before this one)
            span[0] = span[1];
            span[1] = span[2];
            span[2] = write_table(d, par ^ 1);
            scales(par);
            __builtin_amdgcn_sched_barrier(0);
            // (an item's loads among the splitting of the next one: eight together wait for the other moving wavefronts')
            static_for<ITEMS + 1>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                using Before = std::integral_constant<int, i - 1>;
                if constexpr (i < ITEMS && !always(i)) {
                    if (held(ic, ng)) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) convert(par_c, ic, q);
                        write_item(ic, par);
                    }
                    look_at_item(Other{}, ic, ng_after);
                }
                static_for<4>([&](auto qc) __attribute__((always_inline)) {
                    constexpr int q = decltype(qc)::value;
                    if constexpr (i < ITEMS && always(i)) {
                        convert(par_c, ic, q);
                        look(Other{}, ic, q);
                    }
                    if constexpr (i > 0) request(par_c, Before{}, q);
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (i < ITEMS && always(i)) write_item(ic, par);
            });
            next_request();
            publish(par ^ 1);
            if (c == 1 && it > 0)
                for (int i = 0; i < 2 * Cfg::SUM_ROUNDS; ++i) split_barrier();   // (the range before: its sums meet)
            if (++c == per) {
                c = 0;
                ++it;
            }
            split_barrier();
        };
        // before the first interval: tables of three chunks, requests of two, magnitudes of one
        {
            const Decode d = decode_parameters();
            span[0] = write_table(d, 0);
            span[1] = write_table(d, 1);
            write_positions(d, span[0], 0);
            split_barrier();
            read_table(0);
            static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { request_item(S0{}, ic); });
            next_request();
            read_table(1);
            static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { request_item(S1{}, ic); });
            next_request();
            split_barrier();
            span[2] = write_table(d, 0);
            static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { look_at_item(S0{}, ic, sixteens(span[0])); });
            publish(0);
            split_barrier();
        }
        for (int left = ntiles * per; left > 0; left -= 2) {
            interval(S0{});
            interval(S1{});
        }
        split_barrier();                       // (the multipliers' last chunk passes one more)
        for (int i = 0; i < 2 * Cfg::SUM_ROUNDS; ++i) split_barrier();   // (the last range's sums meet)
        return;
    }

    // ================================ multipliers ================================
    const int half = lane >> 5, l32 = lane & 31;
    const int wn = wave & 1, ph = wave >> 1;   // unit, half of a chunk's pixels
    f32x16 acc[3][2], low[3][2];
    u32x4 ah[2][2], am[2], bh[2], bm[2];
    // the transposing read: this lane addresses pixel (lane >> 2) % 4 of four (half 1: eight further on), four rows of the block
    const int quad = lane & 3, sixteen = (lane >> 4) & 1, pixel = half * 8 + ((lane >> 2) & 3);
    const int in_block = sixteen * 2 + (quad >> 1), in_plane = (quad & 1) * 8;
    const int a_lane = in_block * Cfg::A_PLANE + in_plane + (ph * 64 + pixel) * 16;
    const int b_lane = Cfg::B_BASE + wn * Cfg::B_BLOCK + in_block * Cfg::B_PLANE + in_plane;
    int pos_now = Cfg::POS + (ph * 64 + pixel) * 4, pos_next = pos_now + BK * 4, n_chunk = 0;   // of this chunk, the next one
    int b_at[2], pos[2];   // [four of eight pixels]: of this sixteen, of the next one
    using s16x4 = short __attribute__((ext_vector_type(4)));
    using Words = __attribute__((address_space(3))) s16x4 *;
    auto read4 = [&](int at) __attribute__((always_inline)) {
        return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Words)(lds + at)));
    };
    auto read_a = [&](int stage, int ks, int part, int mb) __attribute__((always_inline)) {
        const int at = a_lane + stage * Cfg::A_STAGE + part * Cfg::A_PART + mb * Cfg::A_BLOCK + ks * 256;
        const u32x2 lo = read4(at), hi = read4(at + 64);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    };
    auto read_b = [&](int stage, int part, int t) __attribute__((always_inline)) {
        const int at = stage * Cfg::B_STAGE + part * Cfg::B_PART + t * 16;
        const u32x2 lo = read4(b_at[0] + at), hi = read4(b_at[1] + at);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    };
    auto read_positions = [&](int from, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) pos[q] = *reinterpret_cast<const int *>(lds + from + ks * 64 + q * 16);
    };
    auto take_positions = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) b_at[q] = b_lane + pos[q];
    };
    int e_read = 0;
    // product 0: m*h', 1: h*m', 2: h*h'
    auto chunk = [&](auto stage_c) __attribute__((always_inline)) {
        constexpr int stage = decltype(stage_c)::value;
        static_for<12>([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value, ks = u / 3, t = u % 3, set = u & 1, aset = ks & 1;
            constexpr bool last = u == 11;
            static_for<6>([&](auto sc) __attribute__((always_inline)) {
                constexpr int i = decltype(sc)::value, prod = i / 2, mb = i % 2;
                constexpr int to = last ? stage ^ 1 : stage, kn = (ks + 1) % 4;   // where the next sixteen pixels are
                if constexpr (t == 0 && i == 0) read_positions(ks == 3 ? pos_next : pos_now, kn);
                if constexpr (last && i == 2) split_barrier();
                if constexpr (t == 2 && i == (last ? 2 : 0)) take_positions();
                // the next tap's patch operands; the next sixteen pixels' operands of dy (m after product 0 of the last tap)
                if constexpr (i == (last ? 2 : 0)) bh[set ^ 1] = read_b(to, 0, (t + 1) % 3);
                if constexpr (i == (last ? 5 : 1)) bm[set ^ 1] = read_b(to, 1, (t + 1) % 3);
                if constexpr (t == 2 && !last && i < 2) ah[aset ^ 1][i] = read_a(to, kn, 0, i);
                if constexpr (t == 2 && (i == 2 || i == 3)) am[i - 2] = read_a(to, kn, 1, i - 2);
                if constexpr (last && i == 4) {
                    ah[0][0] = read_a(to, 0, 0, 0);
                    ah[0][1] = read_a(to, 0, 0, 1);
                    e_read = *reinterpret_cast<const int *>(lds + Cfg::SLOT_E + to * 4);
                }
                const f16x8 a = __builtin_bit_cast(f16x8, prod == 0 ? am[mb] : ah[aset][mb]);
                const f16x8 b = __builtin_bit_cast(f16x8, prod == 1 ? bm[set] : bh[set]);
                f32x16 &sum = prod == 2 ? acc[t][mb] : low[t][mb];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, sum, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        pos_now = pos_next;
        pos_next += (++n_chunk & 3) == 3 ? -3 * BK * 4 : BK * 4;
    };
    // before the first chunk
    __builtin_amdgcn_s_setprio(2);   // the MFMA stream goes first where both kinds of wavefront want to issue
    split_barrier();
    split_barrier();
    split_barrier();
    split_barrier();
    read_positions(pos_now, 0);
    take_positions();
    e_read = *reinterpret_cast<const int *>(lds + Cfg::SLOT_E);
    auto first_fragments = [&](int stage) __attribute__((always_inline)) {   // of a range
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            am[mb] = read_a(stage, 0, 1, mb);
            ah[0][mb] = read_a(stage, 0, 0, mb);
        }
        bh[0] = read_b(stage, 0, 0);
        bm[0] = read_b(stage, 1, 0);
    };
    first_fragments(0);
    for (int it = 0; it < ntiles; ++it) {
        const Tile tile = tile_of(tile_number(it));
        const Unit unit = unit_of(tile.u0 + wn);
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][mb][v] = low[t][mb][v] = 0.f;
        int e_sum = __builtin_amdgcn_readfirstlane(e_read);
        auto rescale = [&]() __attribute__((always_inline)) {
            const int e = __builtin_amdgcn_readfirstlane(e_read);
            if (e == e_sum) return;
            const int by = e - e_sum;
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        acc[t][mb][v] = __builtin_ldexpf(acc[t][mb][v], by);
                        low[t][mb][v] = __builtin_ldexpf(low[t][mb][v], by);
                    }
            e_sum = e;
        };
        for (int c = 0; c < per; c += 2) {
            if (c > 0) rescale();
            chunk(std::integral_constant<int, 0>{});
            rescale();
            chunk(std::integral_constant<int, 1>{});
        }
        // sums of the range's pixels that this wavefront has
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][mb][v] = __builtin_ldexpf(__builtin_fmaf(low[t][mb][v], 0x1p-11f, acc[t][mb][v]), -e_sum);
        bool zeros_too;
        const float off_by = wgrad_off_by(lds + Cfg::SLOT_N + (it & 1) * 16, &zeros_too);
        if (__builtin_expect(__any(outside_halves_range<3, 2>(acc, off_by, zeros_too)), 0)) {
            const long long jb = (long long)tile.split * per * BK, je = jb + (long long)per * BK;
            WgradMend m;
            m.m0 = tile.m0; m.c0 = unit.c0; m.tap_h = unit.tap_h; m.tap_w = unit.tap_w;
            m.j_begin = jb < p.CRS ? (int)jb : p.CRS;
            m.j_end = je < p.CRS ? (int)je : p.CRS;
            m.part = ph;
            m.apart = BK;
            m.live = unit.live;
            m.zeros_too = zeros_too;
            f32x16 blocks[6];
#pragma unroll
            for (int g = 0; g < 6; ++g) blocks[g] = acc[g / 2][g % 2];
            wgrad_halves_mend((uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr(), blocks, off_by, m);
#pragma unroll
            for (int g = 0; g < 6; ++g) acc[g / 2][g % 2] = blocks[g];
            first_fragments(0);   // (again: not held across the call)
        }
        float *const sums = reinterpret_cast<float *>(lds + Cfg::SUMS) + wn * (8 * 64) + lane;
        static_for<Cfg::SUM_ROUNDS>([&](auto rc) __attribute__((always_inline)) {
            constexpr int t = decltype(rc)::value / 4, mb = decltype(rc)::value / 2 % 2, v0 = decltype(rc)::value % 2 * 8;
            if (ph == 1)
#pragma unroll
                for (int v = 0; v < 8; ++v) sums[v * 64] = acc[t][mb][v0 + v];
            split_barrier();
            if (ph == 0)
#pragma unroll
                for (int v = 0; v < 8; ++v) acc[t][mb][v0 + v] += sums[v * 64];
            split_barrier();
        });
        if (ph == 0 && unit.live) {
            const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(static_cast<char *>(p.y) + (size_t)tile.split * p.ySplitBytes, 0, p.y_bytes, kBufferWord3);
            bool c_ours;
            const int channel = wgrad_row(unit.c0, l32, p.NPQ, &c_ours);
            const uint32_t col = (uint32_t)channel * (uint32_t)p.ysQ + (uint32_t)(unit.r * p.Q + unit.s0);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    bool k_ours;
                    const int row = wgrad_row(tile.m0 + mb * 32, (v / 4) * 8 + half * 4 + v % 4, p.K, &k_ours);
                    const uint32_t at = ((uint32_t)row * (uint32_t)p.ysK + col) * 4u;
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        const int tap = p.flip ? 2 - t : t;
                        const uint32_t off = c_ours && k_ours && tap >= unit.skip ? at + (uint32_t)tap * 4u : kOutOfRange;
                        float out = p.alpha * acc[t][mb][v];
                        if (p.beta != 0.f) out += p.beta * __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ybuf, off, 0, 0));
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, out), ybuf, off, 0, 0);
                    }
                }
        }
    }
#endif
}

}  // namespace igc
#endif
