// fp32 nine-tap convolution (forward; backward data with unit stride) on the bfloat16 matrix pipes, every operand split
// into three bfloat16 parts (why, and the error: igconv_kernel_f32s.hpp), with the gathered operand read from a staged
// patch of the zero-extended image instead of being gathered tap by tap.
//
// What the tap-by-tap kernel spends its time on is not the MFMAs but the moving wavefronts: every element of x is
// requested and split once per tap.  Here the reduction is ordered (16 channels, tap, channel): a tile's whole range of
// pixels of the zero-extended image goes to LDS once per 16 channels, split, and the nine taps read their operands from
// it at shifted pixels; elements of the gathered side are requested and split nine times less often.  The nine floats of
// a (row, channel) pair of the filter are contiguous in either pass (forward: row k, channel c; backward data: row c,
// channel k, the taps walked backwards); they are loaded once per 16 channels - 16 + 16 + 4 bytes - and handed out tap by
// tap from registers.  (A forward row's 72 floats of eight channels as eighteen aligned 16-byte loads: 2 to 9 % slower.)
//
// Measured, best kernel with the fp32 instruction -> this one: 128x64x56x56 -> 64 223 -> 149 us, 128x384x13x13 -> 256 293 -> 198,
// 64x128x28x28 -> 128 120 -> 74, 128x512x7x7 -> 512 261 -> 140, 32x256x14x14 -> 256 69 -> 49; 64x64x56x56 -> 64 channel-fastest 236 -> 89; error
// against 64 bits 3.4e-7 -> 1.3e-7 on the first.  What bounds it: power.  On zeros the first took 122 us where it took 163 on data
// (the clocks stay up), and 115 with the movers requesting and splitting nothing; 17 us were the tiles' epilogues.
//
// Four multiplying and four moving wavefronts, one workgroup per compute unit (LDS), persistent.  A step is three taps of
// 16 channels, one barrier each:
//   movers, step q = 3s + j (chunk s of 16 channels, taps 3j..3j+2): request a third of chunk s+1's filter rows and
//   pixels, split and write the filter parts of this step (stage q & 1) and the third of the pixels requested one step
//   ago (the patch of chunk s+1, stage (s+1) & 1; its last third in the first step of chunk s+1).
//   multipliers run one step behind: they pass barrier 4 + q in the middle of step q's last tap, when their reads of
//   that step are done; step q + 1 is then complete.
// LDS: [stage][tap of 3][part][row][16 channels] for the filter, [stage][part][pixel][16 channels] for the patch; the two
// 16-byte halves of an entry are swapped on every other group of eight (16-byte reads of consecutive entries meet no
// bank conflict, igconv_kernel_bf16c.hpp).
#ifndef IGCONV_KERNEL_F32P_HPP_
#define IGCONV_KERNEL_F32P_HPP_

#include "igconv_kernel_f32s.hpp"

namespace igc {

// NHWC: channel-fastest x (16-byte loads of channels) and y (lanes along output channels in the epilogue).
template <int BM_, int BN_, int WM_, int WN_, int PIX_, bool NHWC_>
struct SplitPatchConfig {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, PIX = PIX_;
    static constexpr bool NHWC = NHWC_, SWAP = NHWC_;
    static constexpr int THREADS = 512, CH = 16, TAPS = 9, BK = CH * TAPS;
    static constexpr int A_PART = BM * 32, A_TAP = 3 * A_PART, A_STAGE = 3 * A_TAP;
    static constexpr int B_PART = PIX * 32, B_STAGE = 3 * B_PART;
    static constexpr int B_BASE = 2 * A_STAGE;
    static constexpr int SEEN = 2 * (A_STAGE + B_STAGE);   // [parity of the tile][filter, patch][moving wavefront]
    static constexpr int LDS_BYTES = SEEN + 2 * 2 * 4 * kSeenBytes;
    static constexpr int TM = BM / WM, TN = BN / WN, MB = TM / 32, NB = TN / 32;
    static constexpr int CPT = BM / 16;                 // channels of a filter row per moving thread (of 256)
    static constexpr int NPASS = PIX / 128;             // passes of 256 (pixel, half) items over the patch
    static_assert(WM * WN == 4 && BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "four wavefronts of 32x32 blocks");
    static_assert((CPT == 4 || CPT == 8) && PIX % 128 == 0 && NPASS >= 3 && NPASS <= 6, "shares of the moving threads");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

template <class Cfg>
__global__ __launch_bounds__(512, 2) void igconv_f32p_kernel(const ConvKernelParams p) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernel's name and signature only)
    constexpr int BM = Cfg::BM, BN = Cfg::BN, MB = Cfg::MB, NB = Cfg::NB, CPT = Cfg::CPT, NPASS = Cfg::NPASS;

    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int l32 = lane & 31;

    // persistent workgroups, tiles numbered in contiguous ranges per XCD (see igconv_kernel.hpp)
    const int wg_xcd = (int)(blockIdx.x % 8u), wg_local = (int)(blockIdx.x / 8u);
    const int tiles_total = p.tilesM * p.tilesN;
    auto tile_number = [&](int i) {
        const int local = wg_local + i * p.wgsPerXcd;
        const int t = wg_xcd * p.tilesPerXcd + local;
        return local < p.tilesPerXcd && t < tiles_total ? t : tiles_total;
    };
    if (tile_number(0) >= tiles_total) return;
    const int nch = p.ksteps;            // chunks of 16 channels (at least one)
    // first pixel of column j's window as a flat index into the zero-extended images
    auto window_start = [&](uint32_t j) {
        const uint32_t n = magic_div(j, p.mPQ);
        const uint32_t rem = j - n * (uint32_t)p.PQ;
        const uint32_t pp = magic_div(rem, p.mQ);
        const uint32_t qq = rem - pp * (uint32_t)p.Q;
        return n * (uint32_t)p.HpWp + pp * (uint32_t)(p.u * p.Wp) + qq * (uint32_t)p.v;
    };
    // byte offset of (row or pixel number, 16-byte half) in a part
    auto swz = [](int idx, int hf) { return idx * 32 + ((hf ^ ((idx >> 3) & 1)) << 4); };

    if (wave >= 4) {
        // ================================ movers ================================
        const int mw = wave - 4;
        const int mtid = tid - 256;
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        // filter: this thread's CPT channels of one row
        const int a_row = mtid / (16 / CPT), a_sub = mtid % (16 / CPT);
        const int a_dst = swz(a_row, a_sub * CPT / 8) + (CPT == 4 ? (a_sub & 1) * 8 : 0);
        uint32_t a_voff = 0;
        float a_reg[2][CPT * 9];
        // patch: pass i of this wavefront covers 64 pixels and one half of the channels
        int b_dst[NPASS];
        uint32_t b_voff[NPASS];
        float b_reg[2][2][8];
#pragma unroll
        for (int i = 0; i < NPASS; ++i) {
            const int idx = i * 4 + mw;
            b_dst[i] = Cfg::B_BASE + swz((idx >> 1) * 64 + lane, idx & 1);
        }
        auto setup_tile = [&](int tile) {
            const int m0 = (tile % p.tilesM) * BM, n0 = (tile / p.tilesM) * BN;
            const int row = m0 + a_row < p.K ? m0 + a_row : 0;   // (rows beyond K are never stored: they may read row 0)
            a_voff = ((uint32_t)row * (uint32_t)p.wsRow + (uint32_t)(a_sub * CPT) * (uint32_t)p.wsRed) * 4u;
            const uint32_t g_first = __builtin_amdgcn_readfirstlane(window_start((uint32_t)n0));
            const int j_last = n0 + BN - 1 < p.NPQ ? n0 + BN - 1 : p.NPQ - 1;
            const uint32_t g_end = __builtin_amdgcn_readfirstlane(window_start((uint32_t)j_last)) +
                                   (uint32_t)((p.R - 1) * p.Wp + p.S);   // one past the tile's last pixel
#pragma unroll
            for (int i = 0; i < NPASS; ++i) {
                const int idx = i * 4 + mw;
                const uint32_t g = g_first + (uint32_t)((idx >> 1) * 64 + lane);
                const uint32_t n = magic_div(g, p.mHpWp);
                const uint32_t rem = g - n * (uint32_t)p.HpWp;
                const uint32_t hp = magic_div(rem, p.mWp);
                const uint32_t wp = rem - hp * (uint32_t)p.Wp;
                const uint32_t h = hp - (uint32_t)p.pad_h, w = wp - (uint32_t)p.pad_w;   // wrap below 0 -> huge
                const bool ok = g < g_end && h < (uint32_t)p.H && w < (uint32_t)p.W;    // (g < g_end implies n < N)
                b_voff[i] = ok ? (n * (uint32_t)p.xsN + h * (uint32_t)p.xsH + w * (uint32_t)p.xsW) * 4u : kOutOfRange;
            }
        };
        // request part j (of three) of the filter rows of chunk rc into set `set`
        constexpr int NA = 3 * CPT;    // loads per chunk
        auto request_a = [&](auto set_c, int i, uint32_t rc) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            const int e = i / 3, q = i % 3;
            const uint32_t so = (rc * 16u + (uint32_t)e) * (uint32_t)p.wsRed * 4u;
            if (q < 2) {
                const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, a_voff + (uint32_t)q * 16u, so, 0));
#pragma unroll
                for (int c = 0; c < 4; ++c) a_reg[set][e * 9 + q * 4 + c] = v[c];
            } else {
                a_reg[set][e * 9 + 8] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, a_voff + 32u, so, 0));
            }
        };
        // request pass `i` of the patch of chunk rc: slot `sl` of set `set`; channel e of the eight, or all of them
        constexpr int NBL = Cfg::NHWC ? 2 : 8;
        auto request_b = [&](auto set_c, int sl, int i, int e, uint32_t rc) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            const uint32_t c = rc * 16u + (uint32_t)(((i * 4 + mw) & 1) * 8);
            if constexpr (Cfg::NHWC) {
                const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xbuf, b_voff[i], (c + (uint32_t)e * 4u) * 4u, 0));
#pragma unroll
                for (int q = 0; q < 4; ++q) b_reg[set][sl][e * 4 + q] = v[q];
            } else {
                b_reg[set][sl][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, b_voff[i], (c + (uint32_t)e) * (uint32_t)p.xsC * 4u, 0));
            }
        };
        // The patch runs ahead of the filter, so that each has its own (SplitSeen; `operand` 0: filter, 1: patch); of tile number `it`.
        SplitSeen seen[2];
        auto publish = [&](int it, int operand) {
            publish_seen(lds + Cfg::SEEN + (((it & 1) * 2 + operand) * 4 + mw) * kSeenBytes, seen[operand]);
        };
        // split and write: filter, pair q of tap t (of the chunk in `set`) into stage `st`
        uint32_t ph[CPT / 2], pm[CPT / 2], pl[CPT / 2];
        auto convert_a = [&](auto set_c, int st, int t, int q) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            split_pair(a_reg[set][2 * q * 9 + t], a_reg[set][(2 * q + 1) * 9 + t], ph[q], pm[q], pl[q], seen[0]);
            if (q == CPT / 2 - 1) {
                uint8_t *const dst = lds + st * Cfg::A_STAGE + (t % 3) * Cfg::A_TAP + a_dst;
                if constexpr (CPT == 8) {
                    *reinterpret_cast<u32x4 *>(dst) = u32x4{ph[0], ph[1], ph[2], ph[3]};
                    *reinterpret_cast<u32x4 *>(dst + Cfg::A_PART) = u32x4{pm[0], pm[1], pm[2], pm[3]};
                    *reinterpret_cast<u32x4 *>(dst + 2 * Cfg::A_PART) = u32x4{pl[0], pl[1], pl[2], pl[3]};
                } else {
                    *reinterpret_cast<u32x2 *>(dst) = u32x2{ph[0], ph[1]};
                    *reinterpret_cast<u32x2 *>(dst + Cfg::A_PART) = u32x2{pm[0], pm[1]};
                    *reinterpret_cast<u32x2 *>(dst + 2 * Cfg::A_PART) = u32x2{pl[0], pl[1]};
                }
            }
        };
        // ... patch, pair q of slot `sl` of set `set` = pass i, into stage `st`
        u32x4 bh, bm, bl;
        auto convert_b = [&](auto set_c, int st, int sl, int i, int q) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            uint32_t h, m, l;
            split_pair(b_reg[set][sl][2 * q], b_reg[set][sl][2 * q + 1], h, m, l, seen[1]);
            bh[q] = h; bm[q] = m; bl[q] = l;
            if (q == 3) {
                uint8_t *const dst = lds + st * Cfg::B_STAGE + b_dst[i];
                *reinterpret_cast<u32x4 *>(dst) = bh;
                *reinterpret_cast<u32x4 *>(dst + Cfg::B_PART) = bm;
                *reinterpret_cast<u32x4 *>(dst + 2 * Cfg::B_PART) = bl;
            }
        };
        uint32_t rc = 0;             // chunk of the tile whose operands are requested
        int it = 0;                  // its tile
        // step j of chunk s (par: s & 1).  Third j of the patch: passes j and j + 3.  Where rc is 0, s is the last chunk of the
        // tile before: all of its patch has been split after step 0, all of its filter rows after step 2.
        auto step = [&](auto par_c, auto j_c) __attribute__((always_inline)) {
            constexpr int par = decltype(par_c)::value, j = decltype(j_c)::value;
            constexpr int q = (par + j) & 1;                            // parity of 3s + j
            constexpr int jc = (j + 2) % 3, stc = j == 0 ? par : par ^ 1;   // third of the patch to write, its stage
            using Cur = std::integral_constant<int, par>;
            using Nxt = std::integral_constant<int, par ^ 1>;
            using Req = std::integral_constant<int, q>;
            using Got = std::integral_constant<int, q ^ 1>;
            constexpr int PR = j + 3 < NPASS ? 2 : 1, PC = jc + 3 < NPASS ? 2 : 1;   // passes of the two thirds
            constexpr int A0 = NA * j / 3, A1 = NA * (j + 1) / 3;
            constexpr int NLD = A1 - A0 + PR * NBL, NCA = 3 * (CPT / 2), NCV = NCA + PC * 4;
            static_for<NCV>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                constexpr int r0 = i * NLD / NCV, r1 = (i + 1) * NLD / NCV;
                static_for<r1 - r0>([&](auto rc_) __attribute__((always_inline)) {
                    constexpr int r = r0 + decltype(rc_)::value;
                    if constexpr (r < PR * NBL) request_b(Req{}, r / NBL, j + 3 * (r / NBL), r % NBL, rc);
                    else request_a(Nxt{}, A0 + r - PR * NBL, rc);
                });
                if constexpr (i < NCA) convert_a(Cur{}, q, 3 * j + i / (CPT / 2), i % (CPT / 2));
                else convert_b(Got{}, stc, (i - NCA) / 4, jc + 3 * ((i - NCA) / 4), (i - NCA) % 4);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (j != 1 && rc == 0 && it > 0) publish(it - 1, j == 0 ? 1 : 0);
            split_barrier();
        };
        int rem = 0;
        for (int i = 0; tile_number(i) < tiles_total; ++i) rem += nch;   // chunks of all tiles of this workgroup
        auto chunk = [&](auto par_c) __attribute__((always_inline)) {
            step(par_c, std::integral_constant<int, 0>{});
            step(par_c, std::integral_constant<int, 1>{});
            step(par_c, std::integral_constant<int, 2>{});
            if (++rc == (uint32_t)nch) {
                rc = 0;   // (after the last tile its first chunk is requested again; nothing of it is multiplied)
                if (tile_number(++it) < tiles_total) setup_tile(tile_number(it));
            }
        };
        // (what is written before the first operands have arrived lands in stages that are written again before they are read)
#pragma unroll
        for (int i = 0; i < CPT * 9; ++i) a_reg[1][i] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) b_reg[0][0][i] = b_reg[0][1][i] = 0.f;
        setup_tile(tile_number(0));
        for (;;) {   // chunks s = -1 .. number of chunks - 1
            chunk(std::integral_constant<int, 1>{});
            if (--rem < 0) break;
            chunk(std::integral_constant<int, 0>{});
            if (--rem < 0) break;
        }
        split_barrier();                       // (the multipliers' last step passes one more)
        return;
    }

    // ================================ multipliers ================================
    const int wm = wave % Cfg::WM, wn = wave / Cfg::WM;
    constexpr int M = MB * NB, NR1 = 2 * MB + 2 * NB;     // see SplitMultiplier
    u32x4 ah[2][MB], bh[2][NB], am[MB], bm[NB], al[MB], bl[NB];
    f32x16 acc[MB][NB], low[MB][NB];
    const uint8_t *fa = lds + swz(wm * Cfg::TM + l32, half);                   // filter operands, this step's stage
    const uint8_t *fa_other = fa + Cfg::A_STAGE;
    const uint8_t *fb[NB][9];                                                  // patch operands per tap, this chunk's stage
    int b_other = Cfg::B_STAGE;                                                // distance to the other stage
    // the storage order of the taps is that of the filter; where in the window one reads: reversed for eq. 2, and for
    // the exchanged filter of backward data, whose gather walks the taps backwards
    const bool rev = (p.flip != 0) != (p.wsTapS < 0);
    auto setup_columns = [&](int n0) {
        const uint32_t g_first = __builtin_amdgcn_readfirstlane(window_start((uint32_t)n0));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int j = n0 + wn * Cfg::TN + nb * 32 + l32;
            // columns past the end are never stored; let them read the last column's window
            const uint32_t rel = window_start((uint32_t)(j < p.NPQ ? j : p.NPQ - 1)) - g_first;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const uint32_t r = magic_div((uint32_t)t, p.mS);
                const uint32_t sx = (uint32_t)t - r * (uint32_t)p.S;
                const uint32_t tr = rev ? (uint32_t)p.R - 1u - r : r, ts = rev ? (uint32_t)p.S - 1u - sx : sx;
                fb[nb][t] = lds + Cfg::B_BASE + (b_other < 0 ? Cfg::B_STAGE : 0) + swz((int)(rel + tr * (uint32_t)p.Wp + ts), half);
            }
        }
    };
    // fragment i of tap t (a: the filter's stage; b: the patch operands' addresses)
    auto read_frag = [&](const uint8_t *a, const uint8_t *const (&b)[NB], int tl, int set, int i) __attribute__((always_inline)) {
        const uint8_t *const A = a + tl * Cfg::A_TAP;
        if (i < MB) al[i] = *reinterpret_cast<const u32x4 *>(A + 2 * Cfg::A_PART + i * 1024);
        else if (i < 2 * MB) ah[set][i - MB] = *reinterpret_cast<const u32x4 *>(A + (i - MB) * 1024);
        else if (i < 2 * MB + NB) bh[set][i - 2 * MB] = *reinterpret_cast<const u32x4 *>(b[i - 2 * MB]);
        else if (i < NR1) bl[i - 2 * MB - NB] = *reinterpret_cast<const u32x4 *>(b[i - 2 * MB - NB] + 2 * Cfg::B_PART);
        else if (i < NR1 + MB) am[i - NR1] = *reinterpret_cast<const u32x4 *>(A + Cfg::A_PART + (i - NR1) * 1024);
        else bm[i - NR1 - MB] = *reinterpret_cast<const u32x4 *>(b[i - NR1 - MB] + Cfg::B_PART);
    };
    auto mfma = [&](int prod, int set, int j) __attribute__((always_inline)) {
        const int mb = j / NB, nb = j % NB;
        const bf16x8 a = __builtin_bit_cast(bf16x8, prod == 0 ? al[mb] : (prod == 2 || prod == 3 ? am[mb] : ah[set][mb]));
        const bf16x8 b = __builtin_bit_cast(bf16x8, prod == 1 ? bl[nb] : (prod == 2 || prod == 4 ? bm[nb] : bh[set][nb]));
        f32x16 &sum = prod == 5 ? acc[mb][nb] : low[mb][nb];
        if constexpr (Cfg::SWAP) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, sum, 0, 0, 0);
        else sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, sum, 0, 0, 0);
    };
    // The nine taps of a chunk; products and order of the reads as in SplitMultiplier.  The ninth tap requests the next
    // chunk's first fragments.  b_next: where that chunk's first tap reads.
    auto chunk = [&](const uint8_t *const (&b_next)[NB]) __attribute__((always_inline)) {
        static_for<9>([&](auto tc) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value, set = t & 1;
            constexpr bool last = t % 3 == 2;
            // (steps alternate between the two stages: this tap's step and the one after)
            const uint8_t *const a_cur = (t / 3) & 1 ? fa_other : fa, *const a_nxt = (t / 3) & 1 ? fa : fa_other;
            const uint8_t *b[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) b[nb] = t < 8 ? fb[nb][t < 8 ? t + 1 : 0] : b_next[nb];
            const uint8_t *const (&bref)[NB] = b;
            static_for<6 * M>([&](auto mc) __attribute__((always_inline)) {
                constexpr int s = decltype(mc)::value;
                if constexpr (last && s == M) split_barrier();
                constexpr int r0 = s < M ? 0 : s < 4 * M ? (s - M) * NR1 / (3 * M) : s < 5 * M ? NR1 + (s - 4 * M) * MB / M : NR1 + MB + (s - 5 * M) * NB / M;
                constexpr int r1 = s < M ? 0 : s < 4 * M ? (s - M + 1) * NR1 / (3 * M) : s < 5 * M ? NR1 + (s - 4 * M + 1) * MB / M : NR1 + MB + (s - 5 * M + 1) * NB / M;
                static_for<r1 - r0>([&](auto ic) __attribute__((always_inline)) {
                    read_frag(last ? a_nxt : a_cur, bref, (t + 1) % 3, set ^ 1, r0 + decltype(ic)::value);
                });
                mfma(s / M, set, s % M);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        // three steps on: the filter stages have changed places; the patch too; the first fragments sit in set 1
        const uint8_t *const f = fa;
        fa = fa_other;
        fa_other = f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int t = 0; t < 9; ++t) fb[nb][t] += b_other;
        b_other = -b_other;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) ah[0][mb] = ah[1][mb];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bh[0][nb] = bh[1][nb];
    };
    __builtin_amdgcn_s_setprio(2);   // the MFMA stream goes first where both kinds of wavefront want to issue
    for (int i = 0; i < 4; ++i) split_barrier();
    setup_columns((tile_number(0) / p.tilesM) * BN);
    {
        const uint8_t *b[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) b[nb] = fb[nb][0];
        const uint8_t *const (&bref)[NB] = b;
#pragma unroll
        for (int i = 0; i < 3 * (MB + NB); ++i) read_frag(fa, bref, 0, 0, i);
    }
    for (int it = 0;; ++it) {
        const int tile = tile_number(it);
        if (tile >= tiles_total) break;
        const int krow0 = (tile % p.tilesM) * BM + wm * Cfg::TM, col0 = (tile / p.tilesM) * BN + wn * Cfg::TN;
        float bvec[MB];
        load_bias<MB>(p, krow0, l32, bvec);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][nb][v] = low[mb][nb][v] = 0.f;
        const uint8_t *b_next[NB];
        const uint8_t *const (&bref)[NB] = b_next;
        for (int c = 1; c < nch; ++c) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) b_next[nb] = fb[nb][0] + b_other;
            chunk(bref);
        }
        // the last chunk requests the next tile's first fragments
        const int next = tile_number(it + 1);
        {
            const int n0 = (next < tiles_total ? next : tile) / p.tilesM * BN;
            const uint32_t g_first = __builtin_amdgcn_readfirstlane(window_start((uint32_t)n0));
            const uint32_t r = rev ? (uint32_t)(p.R - 1) : 0u, sx = rev ? (uint32_t)(p.S - 1) : 0u;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int j = n0 + wn * Cfg::TN + nb * 32 + l32;
                const uint32_t rel = window_start((uint32_t)(j < p.NPQ ? j : p.NPQ - 1)) - g_first;
                b_next[nb] = lds + Cfg::B_BASE + (b_other < 0 ? 0 : Cfg::B_STAGE) + swz((int)(rel + r * (uint32_t)p.Wp + sx), half);
            }
        }
        chunk(bref);
        if (next < tiles_total) setup_columns((next / p.tilesM) * BN);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][nb][v] += low[mb][nb][v];
        const uint32_t inexact = inexact_below<8>(lds + Cfg::SEEN + (it & 1) * 8 * kSeenBytes, p.CRS);
        if (__any(outside_split_range<MB, NB>(acc, inexact))) sums_in_fp32<Cfg::SWAP, MB, NB>(p, acc, krow0, col0, 0, p.CRS, half, l32);
        const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, kBufferWord3);
        store_tile<Cfg::SWAP, MB, NB>(p, ybuf, acc, bvec, krow0, col0, half, l32);
    }
#endif
}

}  // namespace igc
#endif
