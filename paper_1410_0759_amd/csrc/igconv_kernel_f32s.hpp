// fp32 implicit-GEMM kernel (forward pass, backward data) on the bfloat16 matrix pipes: every float operand is
// written as a sum of three bfloat16 numbers,
//     x = h + m + l,   h = bf16(x), m = bf16(x - h), l = bf16(x - h - m)
// (8 + 8 + 8 significant bits: the sum is x itself), and a product of two floats as the six products of parts
// that reach 2^-24 of it: l*h', h*l', m*m', m*h', h*m', h*h' (the three left out are below 2^-26).  A product of two
// bfloat16 numbers is exact in fp32 and the matrix instruction accumulates in fp32, like the fp32 one.
//
// Why: v_mfma_f32_32x32x2_f32 gives 157 TFLOP/s dense and shares the vector unit (no vector instruction runs
// beside it), v_mfma_f32_32x32x16_bf16 gives 2517: six of the latter do the work of eight of the former in 192 cycles
// instead of 512, and the vector unit stays free for the gather and for the splitting.  Error against 64-bit results:
// smaller than the fp32 instruction's, because the large sums are rounded once per 16 reduction indices.  Measured, 128
// images, fp32 instruction -> this kernel: 384x13x13 -> 256, 3x3 293 -> 268 us, error 7.9e-7 -> 2.7e-7; 96x27x27 -> 256, 5x5 880 ->
// 654 us, 6.6e-7 -> 2.2e-7; 96x64x64 -> 128, 9x9 6.0 -> 4.15 ms, 1.2e-6 -> 4.2e-7.  (Published: Henry, Tang, Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019.)
//
// Division of labour, as in igconv_kernel_bf16s.hpp: four multiplying wavefronts (operand fragments from LDS, MFMAs,
// epilogue) and MOVERS moving ones (gather, splitting, LDS writes), one barrier per step of BK reduction indices.
// LDS tiles hold [row][part][k], k contiguous, rows 16 bytes apart beyond that (an odd number of 16-byte units: the
// 16-byte reads of 16 consecutive rows meet no bank conflict), two stages.
//
// Movers: the offsets of a step's BK reduction indices - where their tap lies relative to a window's origin, the
// tap's coordinates, where the filter element lies in a filter row - are decoded one index per lane a step ahead and
// left in a small table in LDS, private to the wavefront; the gather reads them back as broadcasts.  The
// window test is the packed 16-bit comparison of igconv_kernel.hpp (any filter size, pad, stride).
//
// Values outside bfloat16's reach.  An infinite operand, or a finite one that rounds to infinity, has a NaN among its
// parts, which its sums show.  The parts of a small operand lose what bfloat16's denormals (multiples of 2^-133) cannot hold:
// conversions and matrix instructions keep denormals, so that x - h - m is l, with at most eight significant bits, unless
// it is itself a float denormal (some |x| < 2^-103).  l is therefore taken as its upper half, and a lower half that is not zero
// says that something was lost, less than 2^-133; the movers gather those, and the largest magnitude (SplitSeen).  A sum of n
// products of a tile that lost something is off by less than n * 2^-132 times the largest operand.  A wavefront some of whose
// sums are smaller than 2^24 times that - half a unit of their last place - multiplies its blocks again with the fp32
// instruction straight from global memory (no LDS, no barrier), as it does where a sum is not finite, or not zero but below
// 2^-100.  Slow where it happens: with every sum NaN, 96x64x64 -> 128, 9x9, 32 images 1.2 -> 5.5 ms, backward filter 1.4 -> 8.1 ms;
// 128x384x13x13 -> 256, 3x3 0.20 -> 1.18 ms.
#ifndef IGCONV_KERNEL_F32S_HPP_
#define IGCONV_KERNEL_F32S_HPP_

#include "igconv_instantiate.hpp"

namespace igc {

// What a moving thread's operands were like: the bits their parts lost (low halves; see the head of the file), and the
// largest magnitude.  Per pair of operands one `or` and one maximum beside eleven instructions of splitting: a layer's
// forward and both backward passes, without and with them, 9x9, 128x96x64x64 -> 128 16.5 and 17.4 ms; 3x3, 128x64x56x56 -> 64
// (staged patch) 694 and 702 us.  (Class tests of both remainders in place of the `or`, two vector and two scalar
// instructions: 18.1 ms and 708 us.)
struct SplitSeen {
    uint32_t lost = 0;
    float largest = 0.f;
};
constexpr int kSeenBytes = 8;   // of one wavefront and tile in LDS

// x0, x1 as three pairs of bfloat16 numbers (x0's part in the low half)
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t &h, uint32_t &m, uint32_t &l, SplitSeen &seen) {
    using f32x2 = float __attribute__((ext_vector_type(2)));
    using bf16x2 = __bf16 __attribute__((ext_vector_type(2)));
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x0, x1}), bf16x2));
    const float r0 = x0 - __builtin_bit_cast(float, h << 16), r1 = x1 - __builtin_bit_cast(float, h & 0xFFFF0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{r0, r1}), bf16x2));
    const float s0 = r0 - __builtin_bit_cast(float, m << 16), s1 = r1 - __builtin_bit_cast(float, m & 0xFFFF0000u);
    const uint32_t t0 = __builtin_bit_cast(uint32_t, s0), t1 = __builtin_bit_cast(uint32_t, s1);
    l = __builtin_amdgcn_perm(t1, t0, 0x07060302u);   // the upper halves
    seen.lost |= t0 | t1;
    // (the compiler's maximum would quiet both operands first; a NaN shows in the sums)
    asm("v_max3_f32 %0, %0, abs(%1), abs(%2)" : "+v"(seen.largest) : "v"(x0), "v"(x1));
}

// Leaves it in LDS for the multipliers (once per tile, before a barrier); the tile's operands have all been split.
__device__ __forceinline__ void publish_seen(uint8_t *slot, SplitSeen &seen) {
    uint32_t big = __builtin_bit_cast(uint32_t, seen.largest);   // (not negative: ordered like the integers)
    auto reduce = [&](auto ctrl_c) __attribute__((always_inline)) {
        const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)big, decltype(ctrl_c)::value, 0xF, 0xF, true);
        big = big > other ? big : other;
    };
    reduce(std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8: lane 15 of each row of 16 has the row's
    reduce(std::integral_constant<int, 0x112>{});
    reduce(std::integral_constant<int, 0x114>{});
    reduce(std::integral_constant<int, 0x118>{});
    reduce(std::integral_constant<int, 0x142>{});   // row_bcast 15 and 31: lane 63 has the wavefront's
    reduce(std::integral_constant<int, 0x143>{});
    const uint32_t inexact = __any((seen.lost & 0xFFFFu) != 0u) ? 1u : 0u;
    if ((threadIdx.x & 63u) == 63u) *reinterpret_cast<u32x2 *>(slot) = u32x2{inexact, big};
    seen.lost = 0;   // (the largest magnitude may only grow: that of the tiles before bounds this one's too)
}

// The multipliers' side: sums of `terms` products smaller than this in magnitude (its bits) may be off; 0 when the tile's
// parts are exact.  `slots` of `count` wavefronts.
template <int count>
__device__ __forceinline__ uint32_t inexact_below(const uint8_t *slots, int terms) {
    uint32_t inexact = 0, big = 0;
#pragma unroll
    for (int i = 0; i < count; ++i) {
        const u32x2 s = *reinterpret_cast<const u32x2 *>(slots + i * kSeenBytes);
        inexact |= s[0];
        big = big > s[1] ? big : s[1];
    }
    if (__builtin_amdgcn_readfirstlane(inexact) == 0) return 0;
    const float largest = __builtin_bit_cast(float, big < 0x7F800000u ? big : 0x7F800000u);
    return __builtin_bit_cast(uint32_t, (float)terms * (largest * 0x1p-108f));
}

// BM x BN tile, WM x WN multiplying wavefronts.  VECA: the filter is read in its own order with 16-byte loads, else
// element by element through the row / reduction / tap strides.  PADDED: window test (else pad 0).
template <int BM_, int BN_, int BK_, int WM_, int WN_, bool SWAP_, bool VECA_, bool PADDED_, int MOVERS_>
struct SplitConfig {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, MOVERS = MOVERS_;
    static constexpr bool SWAP = SWAP_, VECA = VECA_, PADDED = PADDED_;
    static constexpr int THREADS = 256 + 64 * MOVERS;
    static constexpr int PART = BK * 2;                 // bytes of one part of a row
    static constexpr int ROW = 3 * PART + 16;
    static constexpr int A_BYTES = BM * ROW, B_BYTES = BN * ROW, STAGE = A_BYTES + B_BYTES;
    static constexpr int RING = BK * 12;                // per moving wavefront: BK entries (offset, tap), BK filter offsets
    static constexpr int SEEN = 2 * STAGE + MOVERS * RING;   // [parity of the tile][moving wavefront]
    static constexpr int LDS_USED = SEEN + 2 * MOVERS * kSeenBytes;
    // workgroups per compute unit: one or two (three would leave a wavefront 85 registers); the allocation says so.  (Two, the
    // 64 x 128 tiles: 128 registers, a dozen of the multiplying wavefronts' values spill to scratch around the epilogue.)
    static constexpr int WGS = (160 * 1024) / LDS_USED >= 2 ? 2 : 1;
    static constexpr int LDS_BYTES = (160 * 1024) / LDS_USED >= 3 ? 64 * 1024 : LDS_USED;
    static constexpr int WAVES_PER_SIMD = WGS * THREADS / 256;
    static constexpr int TM = BM / WM, TN = BN / WN, MB = TM / 32, NB = TN / 32;
    static constexpr int G = BK / 16;                   // groups of 16 reduction indices per step
    static constexpr int CG = BN / 64, KPARTS = MOVERS / CG, KPT = BK / KPARTS;
    static_assert(WM * WN == 4 && BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "four wavefronts of 32x32 blocks");
    static_assert(MOVERS % CG == 0 && KPT % 8 == 0, "a moving lane writes whole 16-byte pieces");
    static_assert(G == 1 || G == 2, "fragment sets alternate from group to group");
    static_assert((ROW / 16) % 2 == 1 && LDS_BYTES <= 160 * 1024, "LDS rows, LDS budget");
};

// The sums of a wavefront's blocks over the reduction indices [k_begin, k_end), with v_mfma_f32_32x32x2_f32 straight
// from global memory (see the head of the file).  krow0, col0: the first row and column of the blocks.
template <bool SWAP, int MB, int NB>
__device__ __forceinline__ void sums_in_fp32(const ConvKernelParams &p, f32x16 (&acc)[MB][NB], int krow0, int col0, int k_begin,
                                             int k_end, int half, int l32) {
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    uint32_t rowoff[MB], colbase[NB];
    int h0[NB], w0[NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int row = krow0 + mb * 32 + l32;
        rowoff[mb] = (uint32_t)(row < p.K ? row : 0) * (uint32_t)p.wsRow * 4u;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int j = col0 + nb * 32 + l32;
        const uint32_t jj = j < p.NPQ ? (uint32_t)j : 0u;
        const uint32_t n = magic_div(jj, p.mPQ);
        const uint32_t rem = jj - n * (uint32_t)p.PQ;
        const uint32_t pp = magic_div(rem, p.mQ);
        const uint32_t qq = rem - pp * (uint32_t)p.Q;
        h0[nb] = (int)pp * p.u - p.pad_h;
        w0[nb] = (int)qq * p.v - p.pad_w;
        colbase[nb] = (n * (uint32_t)p.xsN + (uint32_t)h0[nb] * (uint32_t)p.xsH + (uint32_t)w0[nb] * (uint32_t)p.xsW) * 4u;
        if (j >= p.NPQ) h0[nb] = -(1 << 20);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;
#pragma clang loop unroll(disable)
    for (int k0 = k_begin; k0 < k_end; k0 += 4) {
        float a[2][MB], b[2][NB];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t i = (uint32_t)(k0 + 2 * e + half);
            const bool live = (int)i < k_end;
            const uint32_t c = magic_div(i, p.mRS);
            const uint32_t rs = i - c * (uint32_t)p.RS;
            const uint32_t r = magic_div(rs, p.mS);
            const uint32_t sx = rs - r * (uint32_t)p.S;
            const int tr = (int)(p.flip ? (uint32_t)p.R - 1u - r : r), ts = (int)(p.flip ? (uint32_t)p.S - 1u - sx : sx);
            const uint32_t ao = (c * (uint32_t)p.wsRed + (uint32_t)p.wTap0 + r * (uint32_t)p.wsTapR + sx * (uint32_t)p.wsTapS) * 4u;
            const uint32_t so = (c * (uint32_t)p.xsC + (uint32_t)tr * (uint32_t)p.xsH + (uint32_t)ts * (uint32_t)p.xsW) * 4u;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                a[e][mb] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, live ? rowoff[mb] + ao : kOutOfRange, 0, 0));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const bool ok = live && (uint32_t)(h0[nb] + tr) < (uint32_t)p.H && (uint32_t)(w0[nb] + ts) < (uint32_t)p.W;
                b[e][nb] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, ok ? colbase[nb] + so : kOutOfRange, 0, 0));
            }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    if constexpr (SWAP)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[e][nb], a[e][mb], acc[mb][nb], 0, 0, 0);
                    else
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e][mb], b[e][nb], acc[mb][nb], 0, 0, 0);
                }
    }
}

// True when a lane's sums call for sums_in_fp32: one is infinite or NaN (times zero gives NaN, which every addition
// keeps), or not zero but below 2^-100, or - zeros too - below what `inexact` (the bits of a magnitude) says.
template <int MB, int NB>
__device__ __forceinline__ bool outside_split_range(const f32x16 (&acc)[MB][NB], uint32_t inexact) {
    float nan = 0.f;
    // twice the magnitude's bits; where the parts are exact one less, so that zero is the largest
    const uint32_t zero_passes = inexact == 0 ? ~0u : 0u;
    uint32_t small = ~0u;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float a = acc[mb][nb][v];   // (a bit cast of the vector's element itself takes element 0)
                nan = __builtin_fmaf(a, 0.f, nan);
                const uint32_t u = (__builtin_bit_cast(uint32_t, a) << 1) + zero_passes;
                small = small < u ? small : u;
            }
    const uint32_t limit = __builtin_bit_cast(uint32_t, 0x1p-100f) << 1, other = inexact << 1;
    return nan != 0.f || small < (limit > other ? limit : other);
}

// Workgroup barrier after this wavefront's LDS reads and writes are done; global requests stay in flight.
__device__ __forceinline__ void split_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The multiplying wavefronts' part, shared with the backward-filter kernel (igconv_kernel_wgrad_f32s.hpp).
template <class Cfg>
struct SplitMultiplier {
    static constexpr int MB = Cfg::MB, NB = Cfg::NB, G = Cfg::G, ROW = Cfg::ROW, PART = Cfg::PART;
    static constexpr int M = MB * NB;                       // MFMAs per product of parts
    static constexpr int NR1 = 2 * MB + 2 * NB;             // fragments read during products 1 to 3: al, ah, bh, bl
    const uint8_t *lds;
    int fa, fb;
    // Fragments: the h parts of the next group load while this group multiplies (two sets); the m and l parts have
    // one set each, loaded again as soon as this group's products no longer need them.
    u32x4 ah[2][MB], bh[2][NB], am[MB], bm[NB], al[MB], bl[NB];
    // Sums of the h*h' products, and of the five others: kept apart until the end of the reduction, the large sums are
    // rounded once per 16 reduction indices (six times with one accumulator: backward filter over 128x56x56 pixels, 64x64
    // maps, error against 64 bits 6.0e-7 instead of 3.0e-6; the fp32 instruction 1.1e-6).
    f32x16 acc[MB][NB], low[MB][NB];

    __device__ __forceinline__ void init(const uint8_t *lds_, int wm, int wn, int half, int l32) {
        lds = lds_;
        fa = (wm * Cfg::TM + l32) * ROW + half * 16;
        fb = Cfg::A_BYTES + (wn * Cfg::TN + l32) * ROW + half * 16;
    }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][nb][v] = low[mb][nb][v] = 0.f;
    }
    __device__ __forceinline__ void finish() {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][nb][v] += low[mb][nb][v];
    }
    __device__ __forceinline__ void read_frag(int stage, int g, int set, int i) {
        const uint8_t *const A = lds + stage * Cfg::STAGE + fa + g * 32, *const B = lds + stage * Cfg::STAGE + fb + g * 32;
        if (i < MB) al[i] = *reinterpret_cast<const u32x4 *>(A + i * 32 * ROW + 2 * PART);
        else if (i < 2 * MB) ah[set][i - MB] = *reinterpret_cast<const u32x4 *>(A + (i - MB) * 32 * ROW);
        else if (i < 2 * MB + NB) bh[set][i - 2 * MB] = *reinterpret_cast<const u32x4 *>(B + (i - 2 * MB) * 32 * ROW);
        else if (i < NR1) bl[i - 2 * MB - NB] = *reinterpret_cast<const u32x4 *>(B + (i - 2 * MB - NB) * 32 * ROW + 2 * PART);
        else if (i < NR1 + MB) am[i - NR1] = *reinterpret_cast<const u32x4 *>(A + (i - NR1) * 32 * ROW + PART);
        else bm[i - NR1 - MB] = *reinterpret_cast<const u32x4 *>(B + (i - NR1 - MB) * 32 * ROW + PART);
    }
    __device__ __forceinline__ void mfma(int prod, int set, int j) {
        const int mb = j / NB, nb = j % NB;
        const bf16x8 a = __builtin_bit_cast(bf16x8, prod == 0 ? al[mb] : (prod == 2 || prod == 3 ? am[mb] : ah[set][mb]));
        const bf16x8 b = __builtin_bit_cast(bf16x8, prod == 1 ? bl[nb] : (prod == 2 || prod == 4 ? bm[nb] : bh[set][nb]));
        f32x16 &sum = prod == 5 ? acc[mb][nb] : low[mb][nb];
        if constexpr (Cfg::SWAP) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, sum, 0, 0, 0);
        else sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, sum, 0, 0, 0);
    }
    // Group g of a step: products l*h', h*l', m*m', m*h', h*m', h*h' (small ones first), M MFMAs each; between them
    // the reads of the next group - al once product 0 is issued, bl after product 1, am after 3, bm after 4.  In a
    // step's last group the barrier comes before the first of those reads (this step's own reads are done).
    template <int set, int stage, int g>
    __device__ __forceinline__ void group() {
        constexpr bool last = g == G - 1;
        constexpr int nstage = last ? stage ^ 1 : stage, ng = last ? 0 : g + 1;
        static_for<6 * M>([&](auto mc) __attribute__((always_inline)) {
            constexpr int s = decltype(mc)::value;
            if constexpr (last && s == M) split_barrier();
            if constexpr (s >= M && s < 4 * M) {
                constexpr int r0 = (s - M) * NR1 / (3 * M), r1 = (s - M + 1) * NR1 / (3 * M);
                static_for<r1 - r0>([&](auto ic) __attribute__((always_inline)) { read_frag(nstage, ng, set ^ 1, r0 + decltype(ic)::value); });
            }
            if constexpr (s >= 4 * M && s < 5 * M) {
                constexpr int r0 = (s - 4 * M) * MB / M, r1 = (s - 4 * M + 1) * MB / M;
                static_for<r1 - r0>([&](auto ic) __attribute__((always_inline)) { read_frag(nstage, ng, set ^ 1, NR1 + r0 + decltype(ic)::value); });
            }
            if constexpr (s >= 5 * M) {
                constexpr int r0 = (s - 5 * M) * NB / M, r1 = (s - 5 * M + 1) * NB / M;
                static_for<r1 - r0>([&](auto ic) __attribute__((always_inline)) { read_frag(nstage, ng, set ^ 1, NR1 + MB + r0 + decltype(ic)::value); });
            }
            mfma(s / M, set, s % M);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    template <int stage>
    __device__ __forceinline__ void step() {
        if constexpr (G == 1) {
            group<stage, stage, 0>();
        } else {
            group<0, stage, 0>();
            group<1, stage, 1>();
        }
    }
    // the movers' two intervals before the first step, then that step's first fragments
    __device__ __forceinline__ void prime() {
        split_barrier();
        split_barrier();
#pragma unroll
        for (int i = 0; i < 3 * (MB + NB); ++i) read_frag(0, 0, 0, i);
    }
    __device__ __forceinline__ void steps(int nsteps) {
        for (int t = 0; t < nsteps; t += 2) {
            step<0>();
            step<1>();
        }
        finish();
    }
};

#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernels' names and signatures only)
// `block`: the workgroup's number within its problem
template <class Cfg>
__device__ __forceinline__ void f32s_body(const ConvKernelParams &p, uint32_t block) {
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, MB = Cfg::MB, NB = Cfg::NB, KPT = Cfg::KPT;
    constexpr int ROW = Cfg::ROW, PART = Cfg::PART, STAGE = Cfg::STAGE;

    __shared__ __attribute__((aligned(16))) uint8_t lds[Cfg::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int l32 = lane & 31;

    // persistent workgroups, tiles numbered in contiguous ranges per XCD (see igconv_kernel.hpp); the reduction is never cut
    const int wg_xcd = (int)(block % 8u), wg_local = (int)(block / 8u);
    const int tiles_total = p.tilesM * p.tilesN;
    auto tile_number = [&](int i) {
        const int local = wg_local + i * p.wgsPerXcd;
        const int t = wg_xcd * p.tilesPerXcd + local;
        return local < p.tilesPerXcd && t < tiles_total ? t : tiles_total;
    };
    if (tile_number(0) >= tiles_total) return;
    // steps per tile (even: the stage alternates; a problem without any - a backward-data phase that meets no tap - runs
    // two steps of zeros)
    const int nsteps = p.stepsPerSplit < 2 ? 2 : p.stepsPerSplit;

    // Interval i of the movers (each ends with a barrier): request step i, write step i - 1 to its stage.  The
    // multipliers pass barrier i + 1 in the middle of step i - 1: the reads of that step's stage are then done, and
    // step i is complete in the other one.  Two intervals come before the first step; two more than there are
    // steps are run.
    if (wave >= 4) {
        // ================================ movers ================================
        const int mw = wave - 4;
        const int mtid = tid - 256;
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        const int jl = (mw % Cfg::CG) * 64 + lane;      // this lane's column of the tile
        const int kpart = mw / Cfg::CG;                 // this wavefront's run of KPT reduction indices
        uint8_t *const ring = lds + 2 * STAGE + mw * Cfg::RING;

        u16x2 hw0;                 // (p*u - pad_h, q*v - pad_w) packed; 0x8000 in the row field: column beyond NPQ
        uint32_t colbase = 0;      // byte offset of the window origin (unpadded: the out-of-range marker beyond NPQ)
        u16x2 hw_max;
        hw_max[1] = (uint16_t)(p.H - 1);
        hw_max[0] = (uint16_t)(p.W - 1);

        // filter tile: 16-byte pieces of a row (four reduction indices), or pairs of reduction indices
        constexpr int A_UNIT = Cfg::VECA ? 4 : 2, A_UPR = BK / A_UNIT;
        constexpr int A_TOTAL = BM * A_UPR, A_PASSES = (A_TOTAL + 64 * Cfg::MOVERS - 1) / (64 * Cfg::MOVERS);
        constexpr bool A_PARTIAL = A_TOTAL % (64 * Cfg::MOVERS) != 0;
        static_assert((64 * Cfg::MOVERS) % A_UPR == 0, "a thread's reduction indices are the same in all its passes");
        const int a_kk = (mtid % A_UPR) * A_UNIT;
        const int a_row0 = mtid / A_UPR;
        constexpr int A_RSTEP = 64 * Cfg::MOVERS / A_UPR;
        uint32_t a_voff[A_PASSES];

        u32x4 a_vec[2][Cfg::VECA ? A_PASSES : 1];
        float a_sca[2][Cfg::VECA ? 1 : A_PASSES][2];
        float b_val[2][KPT];

        auto setup_tile = [&](int tile) {
            const int m0 = (tile % p.tilesM) * BM, n0 = (tile / p.tilesM) * BN;
            const int j = n0 + jl;
            const bool cv = j < p.NPQ;
            const uint32_t jj = cv ? (uint32_t)j : 0u;
            const uint32_t n = magic_div(jj, p.mPQ);
            const uint32_t rem = jj - n * (uint32_t)p.PQ;
            const uint32_t pp = magic_div(rem, p.mQ);
            const uint32_t qq = rem - pp * (uint32_t)p.Q;
            const int h0 = (int)pp * p.u - p.pad_h, w0 = (int)qq * p.v - p.pad_w;
            colbase = (n * (uint32_t)p.xsN + (uint32_t)h0 * (uint32_t)p.xsH + (uint32_t)w0 * (uint32_t)p.xsW) * 4u;
            hw0[1] = (uint16_t)(cv ? h0 : 0x8000);
            hw0[0] = (uint16_t)w0;
            if (!Cfg::PADDED && !cv) colbase = kOutOfRange;
            // (rows beyond K are never stored: they may read row 0)
#pragma unroll
            for (int ps = 0; ps < A_PASSES; ++ps) {
                const int row = m0 + a_row0 + ps * A_RSTEP;
                a_voff[ps] = (uint32_t)(row < p.K ? row : 0) * (uint32_t)(Cfg::VECA ? p.CRS : p.wsRow) * 4u + (Cfg::VECA ? (uint32_t)a_kk * 4u : 0u);
            }
        };
        // The offsets of a step's reduction indices, one per lane, are stepped from step to step: (c, r, s) advance by
        // BK = dc*RS + dr*S + ds with a carry from s to r and one from r to c.
        const int dl = lane & (BK - 1);
        const uint32_t dc = magic_div((uint32_t)BK, p.mRS), drem = (uint32_t)BK - dc * (uint32_t)p.RS;
        const uint32_t dr = magic_div(drem, p.mS), ds = drem - dr * (uint32_t)p.S;
        const uint32_t sH = (uint32_t)(p.flip ? -p.xsH : p.xsH) * 4u, sW = (uint32_t)(p.flip ? -p.xsW : p.xsW) * 4u, sC = (uint32_t)p.xsC * 4u;
        const uint32_t so_step = dc * sC + dr * sH + ds * sW, so_s = sH - (uint32_t)p.S * sW, so_r = sC - (uint32_t)p.R * sH;
        const uint32_t ao_step = (dc * (uint32_t)p.wsRed + dr * (uint32_t)p.wsTapR + ds * (uint32_t)p.wsTapS) * 4u;
        const uint32_t ao_s = (uint32_t)(p.wsTapR - p.S * p.wsTapS) * 4u, ao_r = (uint32_t)(p.wsRed - p.R * p.wsTapR) * 4u;
        uint32_t st_i = (uint32_t)dl, st_tap, st_so, st_ao;   // index; (r << 16) | s; offset in x; offset in a filter row
        {
            const uint32_t c = magic_div(st_i, p.mRS);
            const uint32_t rs = st_i - c * (uint32_t)p.RS;
            const uint32_t r = magic_div(rs, p.mS);
            const uint32_t sx = rs - r * (uint32_t)p.S;
            st_tap = (r << 16) | sx;
            st_so = c * sC + (p.flip ? (uint32_t)((p.R - 1) * p.xsH + (p.S - 1) * p.xsW) * 4u : 0u) + r * sH + sx * sW;
            st_ao = (c * (uint32_t)p.wsRed + (uint32_t)p.wTap0 + r * (uint32_t)p.wsTapR + sx * (uint32_t)p.wsTapS) * 4u;
        }
        const uint32_t first_tap = st_tap, first_so = st_so, first_ao = st_ao;
        const uint32_t tap_flip = p.flip ? ~0u : 0u, tap_base = p.flip ? ((uint32_t)(p.R - 1) << 16 | (uint32_t)(p.S - 1)) + 1u : 0u;
        const uint32_t n_live = p.ksteps > 0 ? (uint32_t)p.CRS : 0u;
        // leave the current step's offsets in the ring.  An index past the end has a tap that is never inside the image
        // resp. an out-of-range offset, and an out-of-range filter offset.
        auto put_offsets = [&]() {
            const bool live = st_i < n_live;
            if constexpr (Cfg::PADDED) {
                const u32x2 e = {st_so, live ? (st_tap ^ tap_flip) + tap_base : 0x80000000u};
                *reinterpret_cast<u32x2 *>(ring + dl * 8) = e;
            } else {
                *reinterpret_cast<uint32_t *>(ring + dl * 4) = live ? st_so : kOutOfRange;
            }
            if constexpr (!Cfg::VECA) *reinterpret_cast<uint32_t *>(ring + BK * 8 + dl * 4) = live ? st_ao : kOutOfRange;
        };
        // to the next step, or back to the first one
        auto advance = [&](bool first) {
            uint32_t tap = st_tap + ((dr << 16) | ds);
            const bool cs = (tap & 0xFFFFu) >= (uint32_t)p.S;
            tap += cs ? 0x10000u - (uint32_t)p.S : 0u;
            const bool cr = tap >= (uint32_t)p.R << 16;
            tap -= cr ? (uint32_t)p.R << 16 : 0u;
            st_tap = first ? first_tap : tap;
            st_so = first ? first_so : st_so + so_step + (cs ? so_s : 0u) + (cr ? so_r : 0u);
            if constexpr (!Cfg::VECA) st_ao = first ? first_ao : st_ao + ao_step + (cs ? ao_s : 0u) + (cr ? ao_r : 0u);
            st_i = first ? (uint32_t)dl : st_i + (uint32_t)BK;
        };
        // this thread's offsets of the step to be requested next
        constexpr int NENT = Cfg::PADDED ? KPT / 2 : KPT / 4;
        u32x4 ent[NENT];
        uint32_t a_off[2] = {0, 0};
        auto get_offsets = [&]() {
#pragma unroll
            for (int q = 0; q < NENT; ++q) ent[q] = *reinterpret_cast<const u32x4 *>(ring + kpart * KPT * (Cfg::PADDED ? 8 : 4) + 16 * q);
            if constexpr (!Cfg::VECA) {
                const u32x2 t = *reinterpret_cast<const u32x2 *>(ring + BK * 8 + a_kk * 4);
                a_off[0] = t[0];
                a_off[1] = t[1];
            }
        };
        // request number i of a step
        constexpr int A_LOADS = Cfg::VECA ? A_PASSES : 2 * A_PASSES, NLD = A_LOADS + KPT;
        auto request = [&](auto set_c, int i) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            if (i < A_LOADS) {
                if constexpr (Cfg::VECA)
                    a_vec[set][i] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, a_voff[i] + a_off[0], 0, 0);
                else
                    a_sca[set][i / 2][i % 2] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, a_voff[i / 2] + a_off[i % 2], 0, 0));
            } else {
                const int e = i - A_LOADS;
                uint32_t vo;
                if constexpr (Cfg::PADDED) {
                    const u16x2 hw = hw0 + __builtin_bit_cast(u16x2, (uint32_t)ent[e / 2][2 * (e % 2) + 1]);
                    const u16x2 cl = __builtin_elementwise_min(hw, hw_max);
                    const bool ok = __builtin_bit_cast(uint32_t, cl) == __builtin_bit_cast(uint32_t, hw);
                    vo = ok ? colbase + ent[e / 2][2 * (e % 2)] : kOutOfRange;
                } else {
                    // (a dead index in a dead column: the markers cancel and the sum is some valid offset; such a column
                    // is never stored)
                    vo = colbase + ent[e / 4][e % 4];
                }
                b_val[set][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, vo, 0, 0));
            }
        };
        // piece i of splitting what has arrived in `set` and writing it to the stage of that number: the filter's passes,
        // then pairs of the gathered run
        constexpr int NCV = A_PASSES + KPT / 2;
        u32x4 bh, bm, bl;
        SplitSeen seen;
        // of tile number `it` of this workgroup
        auto publish = [&](int it) { publish_seen(lds + Cfg::SEEN + ((it & 1) * Cfg::MOVERS + mw) * kSeenBytes, seen); };
        auto convert = [&](auto set_c, int i) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            uint8_t *const A = lds + set * STAGE, *const B = A + Cfg::A_BYTES;
            if (i < A_PASSES) {
                const int row = a_row0 + i * A_RSTEP;
                uint8_t *const dst = A + row * ROW + a_kk * 2;
                if constexpr (Cfg::VECA) {
                    const f32x4 v = __builtin_bit_cast(f32x4, a_vec[set][i]);
                    uint32_t h0, m0, l0, h1, m1, l1;
                    split_pair(v[0], v[1], h0, m0, l0, seen);
                    split_pair(v[2], v[3], h1, m1, l1, seen);
                    if (!A_PARTIAL || row < BM) {
                        *reinterpret_cast<u32x2 *>(dst) = u32x2{h0, h1};
                        *reinterpret_cast<u32x2 *>(dst + PART) = u32x2{m0, m1};
                        *reinterpret_cast<u32x2 *>(dst + 2 * PART) = u32x2{l0, l1};
                    }
                } else {
                    uint32_t h, m, l;
                    split_pair(a_sca[set][i][0], a_sca[set][i][1], h, m, l, seen);
                    if (!A_PARTIAL || row < BM) {
                        *reinterpret_cast<uint32_t *>(dst) = h;
                        *reinterpret_cast<uint32_t *>(dst + PART) = m;
                        *reinterpret_cast<uint32_t *>(dst + 2 * PART) = l;
                    }
                }
            } else {
                const int q = i - A_PASSES;
                uint32_t h, m, l;
                split_pair(b_val[set][2 * q], b_val[set][2 * q + 1], h, m, l, seen);
                bh[q % 4] = h; bm[q % 4] = m; bl[q % 4] = l;
                if (q % 4 == 3) {
                    uint8_t *const dst = B + jl * ROW + kpart * (KPT * 2) + (q / 4) * 16;
                    *reinterpret_cast<u32x4 *>(dst) = bh;
                    *reinterpret_cast<u32x4 *>(dst + PART) = bm;
                    *reinterpret_cast<u32x4 *>(dst + 2 * PART) = bl;
                }
            }
        };
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        // One interval: request a step into `set` (its offsets are in registers), bring the offsets of the one after
        // (`first`: the next tile's first step) to registers, write the step before (other set).  Requests and conversions
        // alternate, so that the address unit works beside the vector unit and every request has a whole interval to arrive.
        // `done`: the step written is the last one of the tile of that number (-1: of none).
        auto interval = [&](auto set_c, auto other_c, int tau, bool first, int done) __attribute__((always_inline)) {
            if constexpr (Cfg::VECA)
                a_off[0] = (uint32_t)(tau * BK + a_kk) < n_live ? (uint32_t)(tau * BK) * 4u : kOutOfRange;
            advance(first);
            put_offsets();
            __builtin_amdgcn_sched_barrier(0);
            static_for<NCV>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                constexpr int r0 = i * NLD / NCV, r1 = (i + 1) * NLD / NCV;
                static_for<r1 - r0>([&](auto rc) { request(set_c, r0 + decltype(rc)::value); });
                convert(other_c, i);
                __builtin_amdgcn_sched_barrier(0);
            });
            get_offsets();
            if (done >= 0) publish(done);
            split_barrier();
        };
        // (what the first interval writes lands in a stage that is not read before it is written again)
#pragma unroll
        for (int e = 0; e < KPT; ++e) b_val[1][e] = 0.f;
#pragma unroll
        for (int ps = 0; ps < A_PASSES; ++ps) {
            if constexpr (Cfg::VECA) a_vec[1][ps] = u32x4{0u, 0u, 0u, 0u};
            else a_sca[1][ps][0] = a_sca[1][ps][1] = 0.f;
        }
        setup_tile(tile_number(0));
        put_offsets();
        get_offsets();
        int it = 1;
        for (;; ++it) {
            const int next = tile_number(it);
            for (int t = 0; t < nsteps; t += 2) {
                interval(S0{}, S1{}, t, false, t == 0 ? it - 2 : -1);
                interval(S1{}, S0{}, t + 1, t + 2 >= nsteps, -1);
            }
            if (next >= tiles_total) break;
            setup_tile(next);
        }
        static_for<NCV>([&](auto ic) { convert(S1{}, decltype(ic)::value); });
        publish(it - 1);
        split_barrier();
        split_barrier();                       // (the multipliers' last step passes one more)
        return;
    }

    // ================================ multipliers ================================
    const int wm = wave % Cfg::WM, wn = wave / Cfg::WM;
    SplitMultiplier<Cfg> mult;
    mult.init(lds, wm, wn, half, l32);
    __builtin_amdgcn_s_setprio(2);   // the MFMA stream goes first where both kinds of wavefront want to issue
    mult.prime();
    for (int it = 0;; ++it) {
        const int tile = tile_number(it);
        if (tile >= tiles_total) break;
        const int krow0 = (tile % p.tilesM) * BM + wm * Cfg::TM, col0 = (tile / p.tilesM) * BN + wn * Cfg::TN;
        float bvec[MB];
        load_bias<MB>(p, krow0, l32, bvec);
        mult.zero();
        mult.steps(nsteps);
        // (written two barriers ago or more, and not again for two tiles)
        const uint32_t inexact = inexact_below<Cfg::MOVERS>(lds + Cfg::SEEN + (it & 1) * Cfg::MOVERS * kSeenBytes, p.CRS);
        if (__any(outside_split_range<MB, NB>(mult.acc, inexact)))
            sums_in_fp32<Cfg::SWAP, MB, NB>(p, mult.acc, krow0, col0, 0, p.ksteps > 0 ? p.CRS : 0, half, l32);
        const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, kBufferWord3);
        store_tile<Cfg::SWAP, MB, NB>(p, ybuf, mult.acc, bvec, krow0, col0, half, l32);
    }
}
#endif

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::WAVES_PER_SIMD) void igconv_f32s_kernel(const ConvKernelParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
    f32s_body<Cfg>(p, blockIdx.x);
#endif
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::WAVES_PER_SIMD) void igconv_f32s_phases_kernel(const ConvPhaseParams) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t block;
    const ConvKernelParams p = phase_of_workgroup(&block);
    f32s_body<Cfg>(p, block);
#endif
}

// Instantiates the kernels of IGC_F32S_LIST and defines the group GROUP (variant 4: operands split).
#define IGC_F32S_INSTANTIATE(NAME, BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS, GMODE) \
    template __global__ void igconv_f32s_kernel<SplitConfig<BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS>>(const ConvKernelParams); \
    IGC_F32S_PHASES_##VECA##_##PADDED(IGC_F32S_CONFIG(BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS))
// (backward data only: filter through strides, window test)
#define IGC_F32S_CONFIG(...) SplitConfig<__VA_ARGS__>
#define IGC_F32S_PHASES_false_true(...) template __global__ void igconv_f32s_phases_kernel<__VA_ARGS__>(const ConvPhaseParams);
#define IGC_F32S_PHASES_true_true(...)
#define IGC_F32S_PHASES_false_false(...)
#define IGC_F32S_PHASES_true_false(...)
#define IGC_F32S_ROW(NAME, BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS, GMODE)                 \
    {NAME, false, BM, BN, BK, SWAP, VECA, GMODE,                                                  \
     SplitConfig<BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS>::THREADS,                        \
     SplitConfig<BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS>::LDS_BYTES,                      \
     &launch_f32s<SplitConfig<BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS>>, 4, false, 512,    \
     f32s_phases_launcher<SplitConfig<BM, BN, BK, WM, WN, SWAP, VECA, PADDED, MOVERS>>()},
template <class Cfg>
inline int launch_f32s(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_f32s_kernel<Cfg>, "igconv_f32s_kernel", p, grid, Cfg::THREADS, stream);
}
template <class Cfg>
inline int launch_f32s_phases(const ConvPhaseParams &p, int grid, void *stream) {
    return launch_checked(&igconv_f32s_phases_kernel<Cfg>, "igconv_f32s_phases_kernel", p, grid, Cfg::THREADS, stream);
}
template <class Cfg>
constexpr auto f32s_phases_launcher() -> int (*)(const ConvPhaseParams &, int, void *) {
    if constexpr (!Cfg::VECA && Cfg::PADDED) return &launch_f32s_phases<Cfg>;
    else return nullptr;
}
#if !defined(__HIP_DEVICE_COMPILE__)
#define IGC_F32S_INSTANCES(GROUP)                                 \
    IGC_F32S_LIST(IGC_F32S_INSTANTIATE)                           \
    static const KernelInfo kRows[] = {IGC_F32S_LIST(IGC_F32S_ROW)}; \
    const KernelGroup GROUP = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#else
#define IGC_F32S_INSTANCES(GROUP) IGC_F32S_LIST(IGC_F32S_INSTANTIATE)
#endif

}  // namespace igc
#endif
