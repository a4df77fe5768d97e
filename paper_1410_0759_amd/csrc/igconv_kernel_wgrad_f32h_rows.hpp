// fp32 backward filter on the 16-bit matrix pipes, filters of three rows of three taps and more at unit strides: as
// igconv_kernel_wgrad_f32h.hpp (operands as two binary16 parts, layout of LDS, exponents, results looked at again), with three filter
// rows by three taps of 32 channels per tile.
//
// Why this shape.  That kernel is bound by its moving wavefronts, which split 134 pixels of x per chunk and channel for three taps of one filter
// row, and 128 of dy.  Three filter rows read the same pixels of x but for two output rows more: with the patch extended by
// them, 250 pixels at 56 per row and 200 at 13, a chunk's splitting serves 288 columns instead of 192, 0.9 of it for 1.5 times the products.
// A row of the filter is a wavefront of its own, over all pixels of a chunk: three multiplying wavefronts (64 maps x 32 channels x three taps,
// h*h' and the small products apart), four moving ones, and one that decodes the pixels of the chunks to come for them, which was a third
// of their instructions and the waits between them.
//
// A patch that spans two images holds two rows more; where those do not fit the chunks keep to one image each (p.imageTiles).
//
// Precision: a chain of sums here has all of a chunk's pixels, there half of them, so a range is summed in pieces (p.stepsPerChain) where its
// chain would be longer than there; the second piece is added to the first one's results where they are.
//
// Measured, us, that kernel -> this, 128 images: 64x56x56 -> 64, 3x3 152 -> 123 (error against 64 bits 3.4e-7 -> 3.1e-7 in a training step), channels
// innermost 137 -> 122; 384x13x13 -> 256, 3x3 198 -> 140 (4.1e-7 -> 3.8e-7); 96x27x27 -> 256, 5x5 550 -> 494; 96x64x64 -> 128, 9x9 3050 -> 2300 (350
// TFLOP/s; 1.7e-6 -> 1.1e-6).
// What bounds it: the moving wavefronts' instructions still, about 880 per chunk, beside the MFMAs (4608 of about 6150 cycles per chunk at 9x9), and the
// clock that is left, 1.6 GHz (2340 us, of zeros 1850): without the multiplying wavefronts' work 70 to 75 % of the time, without the loads 74 (9x9) to 88 %.  With the decoding in the movers, five of them, 1400 instructions and
// 2650 us (9x9); parts stored in dw's order 30 us more at 64x56x56.
#ifndef IGCONV_KERNEL_WGRAD_F32H_ROWS_HPP_
#define IGCONV_KERNEL_WGRAD_F32H_ROWS_HPP_

#include "igconv_kernel_wgrad_f32h.hpp"

namespace igc {

// NHWC: both tensors channel-fastest (16-byte loads of channels).
template <bool NHWC_>
struct WgradHalvesRowsConfig {
    static constexpr bool NHWC = NHWC_;
    static constexpr int BM = 64, BN = 32, BK = 128, PIX = kWgradRowsPatch, THREADS = 512;
    static constexpr int A_PLANE = BK * 16 + 64, B_PLANE = PIX * 16 + 64;   // (eight rows; 64 bytes more: neighbouring planes in other banks)
    static constexpr int A_BLOCK = 4 * A_PLANE;                              // 32 rows
    static constexpr int A_PART = 2 * A_BLOCK, B_PART = 4 * B_PLANE;
    static constexpr int A_STAGE = 2 * A_PART, B_STAGE = 2 * B_PART, B_BASE = 2 * A_STAGE;
    static constexpr int TABLE = B_BASE + 2 * B_STAGE;         // [parity][pixel of the patch; pixel of dy] offsets
    static constexpr int TABLE_BYTES = (PIX + BK) * 4;
    static constexpr int POS = TABLE + 2 * TABLE_BYTES;        // [chunk % 4][pixel]: distance of its window in the patch
    static constexpr int SIXTEENS = POS + 4 * BK * 4;          // [chunk % 4] of pixels in the patch
    static constexpr int SLOT_MAX = SIXTEENS + 16;             // largest magnitudes [parity][dy, x][wavefront]
    static constexpr int SLOT_N = SLOT_MAX + 64;               // what a sum may be off by [parity of the piece][wavefront]; sign: kFarBelow
    static constexpr int SLOT_E = SLOT_N + 32;                 // e + e' [parity of the chunk]
    static constexpr int LDS_BYTES = SLOT_E + 16;
    static constexpr int A_ITEMS = BK / 16 * 2 / 4, B_ITEMS = PIX / 16 / 4, ITEMS = A_ITEMS + B_ITEMS;   // of 16 pixels x 32 rows, per moving wavefront
    static_assert(PIX % 64 == 0 && TABLE % 16 == 0 && SLOT_MAX % 16 == 0, "whole items, alignment");
    static_assert(LDS_BYTES <= 160 * 1024 && A_STAGE + A_PART + A_BLOCK + 7 * 256 + 64 < 65536 && B_STAGE + B_PART + 32 < 65536, "LDS budget, offsets of the LDS instructions");
};

// p.Wp: pixels of a row of the patch (output columns and two), p.HpWp: its rows per image (output rows and two); p.PQ: blocks of 32
// channels; p.tilesN: units; p.imageTiles: chunks per image where none spans two, else 0; p.stepsPerChain: chunks whose products one chain of sums
// takes; otherwise as for the kernels by tap.
template <class Cfg>
__global__ __launch_bounds__(512, 2) void igconv_wgrad_f32h_rows_kernel(const ConvKernelParams p) {
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
    const int chains = (per + p.stepsPerChain - 1) / p.stepsPerChain;      // of a range: its sums are added up in this many pieces, one after the other
    struct Unit { int c0, r0, s0, skip_r, skip_s, tap_h, tap_w; };
    struct Tile { int m0, unit, split, number; };
    auto tile_of = [&](int number) {
        if (number >= tiles_total) number = 0;   // (no tile: any; nothing of it is multiplied)
        Tile t;
        t.split = number / tiles_mn;
        const int tile = number - t.split * tiles_mn;
        t.number = tile;
        t.m0 = (tile % p.tilesM) * Cfg::BM;
        t.unit = tile / p.tilesM;
        return t;
    };
    auto unit_of = [&](int u) {
        Unit r;
        const int rg = u / p.PQ;
        r.c0 = (u - rg * p.PQ) * 32;
        const int g = rg / groups, r_first = g * 3, s_first = (rg - g * groups) * 3;
        r.r0 = r_first < p.R - 3 ? r_first : p.R - 3;
        r.s0 = s_first < p.Q - 3 ? s_first : p.Q - 3;
        r.skip_r = r_first - r.r0;   // storage rows and taps that another unit has
        r.skip_s = s_first - r.s0;
        r.tap_h = (p.flip ? p.R - 3 - r.r0 : r.r0) - p.pad_h;
        r.tap_w = (p.flip ? p.Q - 3 - r.s0 : r.s0) - p.pad_w;
        return r;
    };
    // piece i of this workgroup's work: a chain of sums
    auto steps_of = [&](int i) {
        const int left = per - i % chains * p.stepsPerChain;
        return left < p.stepsPerChain ? left : p.stepsPerChain;
    };
    int ntiles = 0;
    while (tile_number(ntiles) < tiles_total) ++ntiles;
    const int pieces = ntiles * chains;

    if (wave == 3) {
        // ================ a chunk's pixels: offsets in the patch and in dy, distances of the windows ================
        struct Span { int j0, j_last; uint32_t g0, length; };   // first and last pixel; first window, patch length (to the last window's end)
        struct Cursor { int piece, c, j0, in_image; };              // the next chunk of a kind of work: piece, chunk of it, first pixel
        auto start = [&](Cursor &k) {
            const Tile t = tile_of(tile_number(k.piece / chains));
            const int chunk = t.split * per + k.piece % chains * p.stepsPerChain;
            const int n = p.imageTiles ? chunk / p.imageTiles : 0;
            k.c = 0;
            k.in_image = p.imageTiles ? chunk - n * p.imageTiles : 0;
            k.j0 = p.imageTiles ? n * p.RS + k.in_image * BK : chunk * BK;
        };
        auto distance = [&](uint32_t j) __attribute__((always_inline)) {   // of pixel j's window from the first image's first: rows of two pixels more, images of two rows more
            return j + 2u * magic_div(j, p.mS) + 2u * (uint32_t)p.Wp * magic_div(j, p.mRS);
        };
        auto span_of = [&](int j0) __attribute__((always_inline)) {
            Span s;
            const int jf = j0 < p.CRS ? j0 : p.CRS - 1;
            s.j0 = j0;
            int end = p.CRS;
            if (p.imageTiles) end = ((int)magic_div((uint32_t)jf, p.mRS) + 1) * p.RS;
            s.j_last = j0 + BK < end ? j0 + BK - 1 : end - 1;
            s.g0 = distance((uint32_t)jf);
            s.length = j0 < p.CRS ? distance((uint32_t)s.j_last) + 2u * (uint32_t)p.Wp + 3u - s.g0 : 0u;
            return s;
        };
        Cursor table_at{0, 0, 0, 0};
        int t_h, t_w;
        auto table_piece = [&]() {
            start(table_at);
            const Unit r = unit_of(tile_of(tile_number(table_at.piece / chains)).unit);
            t_h = r.tap_h;
            t_w = r.tap_w;
        };
        table_piece();
        auto write_table = [&](int chunk) __attribute__((always_inline)) {
            uint8_t *const table = lds + Cfg::TABLE + (chunk & 1) * Cfg::TABLE_BYTES;
            const Span s = span_of(table_at.j0);
            auto patch = [&](int at) __attribute__((always_inline)) {
                const uint32_t g = s.g0 + (uint32_t)at;
                const uint32_t row = magic_div(g, p.mWp), col = g - row * (uint32_t)p.Wp;
                const uint32_t n = magic_div(row, p.mHpWp);
                const uint32_t h = row - n * (uint32_t)p.HpWp + (uint32_t)t_h, w = col + (uint32_t)t_w;   // (below zero: huge)
                const bool ok = (uint32_t)at < s.length && h < (uint32_t)p.H && w < (uint32_t)p.W;
                *reinterpret_cast<uint32_t *>(table + at * 4) = ok ? (n * (uint32_t)p.xsC + h * (uint32_t)p.xsH + w * (uint32_t)p.xsW) * 4u : kOutOfRange;
            };
#pragma unroll
            for (int at = 0; at < PIX; at += 64) patch(at + lane);
#pragma unroll
            for (int at = lane; at < BK; at += 64) {
                const uint32_t j = (uint32_t)(s.j0 + at);
                const uint32_t row = magic_div(j, p.mS), qq = j - row * (uint32_t)p.S;
                const uint32_t n = magic_div(j, p.mRS), pp = row - n * (uint32_t)(p.HpWp - 2);
                *reinterpret_cast<uint32_t *>(table + PIX * 4 + at * 4) =
                    (int)j <= s.j_last ? (n * (uint32_t)p.wsRed + pp * (uint32_t)p.wsTapR + qq * (uint32_t)p.wsTapS) * 4u : kOutOfRange;
            }
            if (lane == 0) *reinterpret_cast<int *>(lds + Cfg::SIXTEENS + (chunk & 3) * 4) = (int)(s.length + 15u) / 16;
            table_at.j0 += BK;
            if (p.imageTiles && ++table_at.in_image == p.imageTiles) {
                table_at.in_image = 0;
                table_at.j0 = s.j_last + 1;
            }
            if (++table_at.c == steps_of(table_at.piece)) {
                ++table_at.piece;
                table_piece();
            }
            return s;
        };
        auto write_positions = [&](const Span &s, int chunk) __attribute__((always_inline)) {
#pragma unroll
            for (int at = lane; at < BK; at += 64) {
                const int j = s.j0 + at < s.j_last ? s.j0 + at : s.j_last;
                // (a chunk past the end: any pixels inside the patch, of zeros)
                *reinterpret_cast<uint32_t *>(lds + Cfg::POS + ((chunk & 3) * BK + at) * 4) = s.length ? (distance((uint32_t)j) - s.g0) * 16u : 0u;
            }
        };
        // ahead of the movers: tables of three chunks, positions of one
        Span next = write_table(0), after = write_table(1);
        write_positions(next, 0);
        next = after;
        split_barrier();
        split_barrier();
        after = write_table(2);
        split_barrier();
        for (int n = 0; n < ntiles * per; ++n) {
            write_positions(next, n + 1);     // (the multipliers may still be reading those of the chunk before this one)
            next = after;
            after = write_table(n + 3);
            split_barrier();
        }
        split_barrier();                       // (the multipliers' last chunk passes one more)
        return;
    }
    if (wave >= 4) {
        // ================================ movers ================================
        const int mw = wave - 4;
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        const int px = lane & 15, plane = lane >> 4;   // within an item
        // ---- requests.  Item i, dy: block of rows i % 2, pixels 16 (4 (i / 2) + mw) ..; patch: pixels 16 (4 (i - A_ITEMS) + mw) ..
        float reg[2][ITEMS][8];
        uint32_t rowoff[2], choff;
        int r_piece = 0, r_c = 0;
        auto request_piece = [&]() {
            const Tile t = tile_of(tile_number(r_piece / chains));
            const int at = plane * 8;
            bool ours;
#pragma unroll
            for (int i = 0; i < 2; ++i) rowoff[i] = (uint32_t)wgrad_row(t.m0 + i * 32, at, p.K, &ours) * (uint32_t)p.wsRow * 4u;
            choff = (uint32_t)wgrad_row(unit_of(t.unit).c0, at, p.NPQ, &ours) * (uint32_t)p.xsN * 4u;
        };
        request_piece();
        int r_steps = steps_of(0);
        uint32_t row_step[8], ch_step[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            row_step[e] = (uint32_t)(e * p.wsRow) * 4u;
            ch_step[e] = (uint32_t)(e * p.xsN) * 4u;
        }
        constexpr int PIXELS = Cfg::A_ITEMS / 2 + Cfg::B_ITEMS;   // different pixels of a thread's items
        uint32_t pixel_at[PIXELS];
        auto read_table = [&](int parity) __attribute__((always_inline)) {
            const uint8_t *const table = lds + Cfg::TABLE + parity * Cfg::TABLE_BYTES + (mw * 16 + px) * 4;
#pragma unroll
            for (int i = 0; i < PIXELS; ++i)
                pixel_at[i] = *reinterpret_cast<const uint32_t *>(i < Cfg::A_ITEMS / 2 ? table + PIX * 4 + i * 256 : table + (i - Cfg::A_ITEMS / 2) * 256);
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
            if (++r_c == r_steps) {
                r_c = 0;
                ++r_piece;
                request_piece();
                r_steps = steps_of(r_piece);
            }
        };
        // (whatever the chunk: 128 pixels in rows of nine and more span 155 pixels of the patch)
        constexpr auto always = [](int i) { return i < Cfg::A_ITEMS || 4 * (i - Cfg::A_ITEMS) + 3 < 155 / 16; };
        auto held = [&](auto ic, int ng) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            if constexpr (always(i)) return true;
            else return 4 * (i - Cfg::A_ITEMS) + mw < ng;
        };
        auto sixteens = [&](int chunk) __attribute__((always_inline)) {
            return __builtin_amdgcn_readfirstlane(*reinterpret_cast<const int *>(lds + Cfg::SIXTEENS + (chunk & 3) * 4));
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
        int it = 0, c = 0;                       // piece and chunk of it being written
        WgradScales scale;
        int steps_now = steps_of(0);             // chunks of the piece being written
        auto scales = [&](int parity) __attribute__((always_inline)) {
            // (of the 128 pixels that a result's sum takes from the chunk this wavefront has at most 32 of dy, two per lane and map, and 64 of the
            // patch, four per lane and channel)
            scale.next<2, 32, Cfg::B_ITEMS>(lds + Cfg::SLOT_MAX + parity * 32, c == 0, small_a, small_b);
            if (mw == 0 && lane == 0) *reinterpret_cast<int *>(lds + Cfg::SLOT_E + parity * 4) = scale.ea + scale.eb;
            if (c == steps_now - 1 && lane == 0)
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
            uint8_t *const dst = lds + parity * (of_dy ? Cfg::A_STAGE : Cfg::B_STAGE) + (of_dy ? i % 2 * Cfg::A_BLOCK + plane * Cfg::A_PLANE + (i / 2 * 4 + mw) * 256
                                                               : Cfg::B_BASE + plane * Cfg::B_PLANE + (4 * (i - Cfg::A_ITEMS) + mw) * 256) + px * 16;
            *reinterpret_cast<u32x4 *>(dst) = part_h;
            *reinterpret_cast<u32x4 *>(dst + (of_dy ? Cfg::A_PART : Cfg::B_PART)) = part_m;
        };
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        // Requests stand under no condition: the compiler counts the loads in flight.  An item of the next chunk is looked at just
        // before the same item of the chunk after it is requested: as many loads stay in flight all along.
        int n_chunk = 0;   // the number of the one being written
        auto interval = [&](auto par_c) __attribute__((always_inline)) {
            constexpr int par = decltype(par_c)::value;
            using Other = std::integral_constant<int, par ^ 1>;
            read_table(par);
            const int ng = sixteens(n_chunk), ng_after = sixteens(n_chunk + 1);
            ++n_chunk;
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
            if (++c == steps_now) {
                c = 0;
                ++it;
                steps_now = steps_of(it);
            }
            split_barrier();
        };
        // before the first interval: requests of two chunks, magnitudes of one
        split_barrier();
        read_table(0);
        static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { request_item(S0{}, ic); });
        next_request();
        read_table(1);
        static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { request_item(S1{}, ic); });
        next_request();
        split_barrier();
        static_for<ITEMS>([&](auto ic) __attribute__((always_inline)) { look_at_item(S0{}, ic, sixteens(0)); });
        publish(0);
        split_barrier();
        for (int left = ntiles * per; left > 0; left -= 2) {
            interval(S0{});
            interval(S1{});
        }
        split_barrier();                       // (the multipliers' last chunk passes one more)
        return;
    }

    // ================================ multipliers ================================
    const int half = lane >> 5, l32 = lane & 31;
    // (the wavefront's number: its row of the patch, of three)
    f32x16 acc[3][2], low[3][2];
    u32x4 ah[2][2], am[2], bh[2], bm[2];
    // the transposing read: this lane addresses pixel (lane >> 2) % 4 of four (half 1: eight further on), four rows of the block
    const int quad = lane & 3, sixteen = (lane >> 4) & 1, pixel = half * 8 + ((lane >> 2) & 3);
    const int in_block = sixteen * 2 + (quad >> 1), in_plane = (quad & 1) * 8;
    const int a_lane = in_block * Cfg::A_PLANE + in_plane + pixel * 16;
    const int b_lane = Cfg::B_BASE + in_block * Cfg::B_PLANE + in_plane + wave * p.Wp * 16;
    int pos_now = Cfg::POS + pixel * 4, pos_next = pos_now + BK * 4, n_chunk = 0;   // of this chunk, the next one
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
        static_for<24>([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value, ks = u / 3, t = u % 3, set = u & 1, aset = ks & 1;
            constexpr bool last = u == 23;
            static_for<6>([&](auto sc) __attribute__((always_inline)) {
                constexpr int i = decltype(sc)::value, prod = i / 2, mb = i % 2;
                constexpr int to = last ? stage ^ 1 : stage, kn = (ks + 1) % 8;   // where the next sixteen pixels are
                if constexpr (t == 0 && i == 0) read_positions(ks == 7 ? pos_next : pos_now, kn);
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
    auto first_fragments = [&](int stage) __attribute__((always_inline)) {   // of a piece
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            am[mb] = read_a(stage, 0, 1, mb);
            ah[0][mb] = read_a(stage, 0, 0, mb);
        }
        bh[0] = read_b(stage, 0, 0);
        bm[0] = read_b(stage, 1, 0);
    };
    first_fragments(0);
    for (int it = 0; it < pieces; ++it) {
        const Tile tile = tile_of(tile_number(it / chains));
        const Unit unit = unit_of(tile.unit);
        const int steps = steps_of(it);
        const bool live = (p.flip ? 2 - wave : wave) >= unit.skip_r;      // (else another unit has this filter row)
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
        for (int c = 0; c < steps; c += 2) {
            if (c > 0) rescale();
            chunk(std::integral_constant<int, 0>{});
            rescale();
            chunk(std::integral_constant<int, 1>{});
        }
        // sums of the piece's pixels
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][mb][v] = __builtin_ldexpf(__builtin_fmaf(low[t][mb][v], 0x1p-11f, acc[t][mb][v]), -e_sum);
        bool zeros_too;
        const float off_by = wgrad_off_by(lds + Cfg::SLOT_N + (it & 1) * 16, &zeros_too);
        if (__builtin_expect(__any(outside_halves_range<3, 2>(acc, off_by, zeros_too)), 0)) {
            auto first_pixel = [&](int chunk) {
                const long long j = p.imageTiles ? (long long)(chunk / p.imageTiles) * p.RS + chunk % p.imageTiles * BK : (long long)chunk * BK;
                return j < p.CRS ? (int)j : p.CRS;
            };
            const int chunk = tile.split * per + it % chains * p.stepsPerChain;
            WgradMend m;
            m.m0 = tile.m0; m.c0 = unit.c0; m.tap_h = unit.tap_h + wave; m.tap_w = unit.tap_w;
            m.j_begin = first_pixel(chunk);
            m.j_end = first_pixel(chunk + steps);
            m.part = 0;
            m.apart = 64;
            m.live = live;
            m.zeros_too = zeros_too;
            f32x16 blocks[6];
#pragma unroll
            for (int g = 0; g < 6; ++g) blocks[g] = acc[g / 2][g % 2];
            wgrad_halves_mend((uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr(), blocks, off_by, m);
#pragma unroll
            for (int g = 0; g < 6; ++g) acc[g / 2][g % 2] = blocks[g];
            first_fragments(0);   // (again: not held across the call)
        }
        // The first chain of a range is written where the range's sums belong, the others are added to what is there.
        const bool more = it % chains != 0;
        if (more) __builtin_amdgcn_s_waitcnt(0x0F70);     // (this wavefront's own results)
        const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(static_cast<char *>(p.y) + (size_t)tile.split * p.ySplitBytes, 0, p.y_bytes, kBufferWord3);
        if (live && p.ysN != 0) {
            // A part in the workspace, in the order of the accumulators (WgradRowsPart): 16 bytes per lane, whole lines.  (In dw's order a store
            // meets 36 bytes apart and a line is written by three wavefronts: 15 us per piece at 64x56x56 -> 64, 3x3.)
            const uint32_t first = (uint32_t)(tile.number * 3 + wave) * (uint32_t)(6 * 16 * 64 * 4) + (uint32_t)lane * 16u;
            static_for<24>([&](auto gc) __attribute__((always_inline)) {
                constexpr int g = decltype(gc)::value, t = g / 8, mb = g / 4 % 2, v = g % 4 * 4;
                f32x4 out;
#pragma unroll
                for (int e = 0; e < 4; ++e) out[e] = p.alpha * acc[t][mb][v + e];
                if (more) out += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ybuf, first, (uint32_t)(g * 1024), 0));
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out), ybuf, first, (uint32_t)(g * 1024), 0);
            });
        } else if (live) {
            const float beta = more ? 1.f : p.beta;
            bool c_ours;
            const int channel = wgrad_row(unit.c0, l32, p.NPQ, &c_ours);
            const uint32_t col = (uint32_t)channel * (uint32_t)p.ysQ + (uint32_t)((unit.r0 + (p.flip ? 2 - wave : wave)) * p.Q + unit.s0);
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
                        const uint32_t off = c_ours && k_ours && tap >= unit.skip_s ? at + (uint32_t)tap * 4u : kOutOfRange;
                        float out = p.alpha * acc[t][mb][v];
                        if (beta != 0.f) out += beta * __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ybuf, off, 0, 0));
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, out), ybuf, off, 0, 0);
                    }
                }
        }
    }
#endif
}

}  // namespace igc
#endif
