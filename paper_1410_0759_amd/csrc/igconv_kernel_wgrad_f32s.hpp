// fp32 backward filter on the bfloat16 matrix pipes: dw = dy . D_m^T with every float operand split into three
// bfloat16 parts (why, and what it does to the error: igconv_kernel_f32s.hpp, whose multiplying half this kernel uses as
// it is).  Rows are feature maps k of dy, columns (tap, channel) with one tap per column tile (gather mode 8), the reduction runs over
// output pixels (n,p,q) and is cut into ranges, one (tile, range) after another per workgroup (igconv_kernel_wgrad.hpp).
// Measured, 128 images, fp32 instruction -> this kernel: 384x13x13 -> 256, 3x3 320 -> 240 us; 96x27x27 -> 256, 5x5 1151 -> 837;
// 96x64x64 -> 128, 9x9 8.0 -> 5.9 ms; error against 64 bits 1.0e-6 -> 5.0e-7, 1.7e-6 -> 8.7e-7, 2.5e-6 -> 1.2e-6.  64 x 64 tiles
// (64 maps and channels) were level (250 us) and few channels (11x11, stride 4, columns (c,r,s)) slower (127 -> 142): not built.
// Where the fp32 kernels stay ahead (channels innermost, strides, narrow rows): see validate_backward_filter in igconv_api.cpp.
//
// Movers: 16 lanes stand for a step's 32 reduction indices, two consecutive ones each, so that a pair becomes one dword
// of each part; four rows (columns) per request.  The two indices' offsets in dy and in x (tap shift and window test
// folded in) are the same for all rows resp. columns; the pass's row or column goes into the scalar offset, so that a
// request costs no vector instruction.  (n,p,q) is stepped from step to step by additions with two
// carries, one index per lane, and handed to the lanes that need it through a table in LDS private to the wavefront.
#ifndef IGCONV_KERNEL_WGRAD_F32S_HPP_
#define IGCONV_KERNEL_WGRAD_F32S_HPP_

#include "igconv_kernel_f32s.hpp"

namespace igc {

template <int BM_, int BN_, int WM_, int WN_>
struct WgradSplitConfig {
    static constexpr int BM = BM_, BN = BN_, BK = 32, WM = WM_, WN = WN_, MOVERS = 4;
    static constexpr bool SWAP = false;
    static constexpr int THREADS = 256 + 64 * MOVERS;
    static constexpr int PART = BK * 2, ROW = 3 * PART + 16;
    static constexpr int A_BYTES = BM * ROW, B_BYTES = BN * ROW, STAGE = A_BYTES + B_BYTES;
    static constexpr int RING = BK * 8;                 // per moving wavefront: BK entries (offset in x, offset in dy)
    static constexpr int SEEN = 2 * STAGE + MOVERS * RING;   // [parity of the (tile, range)][moving wavefront]
    static constexpr int LDS_USED = SEEN + 2 * MOVERS * kSeenBytes;
    static constexpr int WGS = (160 * 1024) / LDS_USED >= 2 ? 2 : 1;   // workgroups per compute unit: one or two
    static constexpr int LDS_BYTES = (160 * 1024) / LDS_USED >= 3 ? 64 * 1024 : LDS_USED;
    static constexpr int WAVES_PER_SIMD = WGS * THREADS / 256;
    static constexpr int TM = BM / WM, TN = BN / WN, MB = TM / 32, NB = TN / 32;
    static constexpr int G = BK / 16;
    static constexpr int ROWS_PER_PASS = 4 * MOVERS, AP = BM / ROWS_PER_PASS, BP = BN / ROWS_PER_PASS;
    static_assert(WM * WN == 4 && BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "four wavefronts of 32x32 blocks");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// A wavefront's blocks over the reduction indices [k_begin, k_end) with the fp32 instruction straight from global memory
// (for operands outside bfloat16's reach).  tap_h, tap_w: the tile's tap relative to the window origin.
template <class Cfg>
__device__ __forceinline__ void wgrad_sums_in_fp32(const ConvKernelParams &p, f32x16 (&acc)[Cfg::MB][Cfg::NB], int krow0, int col0,
                                                   int tap_h, int tap_w, int k_begin, int k_end, int half, int l32) {
    constexpr int MB = Cfg::MB, NB = Cfg::NB;
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    uint32_t rowoff[MB], coloff[NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int row = krow0 + mb * 32 + l32;
        rowoff[mb] = (uint32_t)(row < p.K ? row : 0) * (uint32_t)p.wsRow * 4u;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const uint32_t col = (uint32_t)(col0 + nb * 32 + l32 < p.NPQ ? col0 + nb * 32 + l32 : 0);
        coloff[nb] = col * (uint32_t)p.xsN * 4u;
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
            const uint32_t n = magic_div(i, p.mRS);
            const uint32_t rem = i - n * (uint32_t)p.RS;
            const uint32_t pp = magic_div(rem, p.mS);
            const uint32_t qq = rem - pp * (uint32_t)p.S;
            const uint32_t hh = pp * (uint32_t)p.redMulH + (uint32_t)tap_h, ww = qq * (uint32_t)p.redMulW + (uint32_t)tap_w;
            const bool ok = live && hh < (uint32_t)p.H && ww < (uint32_t)p.W;
            const uint32_t xo = (n * (uint32_t)p.xsC + hh * (uint32_t)p.xsH + ww * (uint32_t)p.xsW) * 4u;
            const uint32_t ao = (n * (uint32_t)p.wsRed + pp * (uint32_t)p.wsTapR + qq * (uint32_t)p.wsTapS) * 4u;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                a[e][mb] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, live ? rowoff[mb] + ao : kOutOfRange, 0, 0));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                b[e][nb] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, ok ? coloff[nb] + xo : kOutOfRange, 0, 0));
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e][mb], b[e][nb], acc[mb][nb], 0, 0, 0);
    }
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::WAVES_PER_SIMD) void igconv_wgrad_f32s_kernel(const ConvKernelParams p) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernel's name and signature only)
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, MB = Cfg::MB, NB = Cfg::NB, AP = Cfg::AP, BP = Cfg::BP;
    constexpr int ROW = Cfg::ROW, PART = Cfg::PART, STAGE = Cfg::STAGE, RPP = Cfg::ROWS_PER_PASS;

    __shared__ __attribute__((aligned(16))) uint8_t lds[Cfg::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int l32 = lane & 31;

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
    const int nsteps = p.stepsPerSplit < 2 ? 2 : p.stepsPerSplit;   // per range (even: the stage alternates)
    // a (tile, range) number -> first row, first channel, tap and range
    struct Tile { int m0, n0, tap, tap_h, tap_w, split; };
    auto tile_of = [&](int tile) {
        Tile t{};
        t.split = tile / tiles_mn;
        tile -= t.split * tiles_mn;
        t.m0 = (tile % p.tilesM) * BM;
        const uint32_t tn = (uint32_t)(tile / p.tilesM);
        const uint32_t tap = magic_div(tn, p.mPQ);   // (PQ: channel blocks per tap; Q, R: the filter's S, R)
        const uint32_t r = magic_div(tap, p.mQ);
        const uint32_t sx = tap - r * (uint32_t)p.Q;
        t.tap = (int)tap;
        t.tap_h = (int)(p.flip ? (uint32_t)p.R - 1u - r : r) - p.pad_h;
        t.tap_w = (int)(p.flip ? (uint32_t)p.Q - 1u - sx : sx) - p.pad_w;
        t.n0 = (int)(tn - tap * (uint32_t)p.PQ) * BN;
        return t;
    };

    if (wave >= 4) {
        // ================================ movers ================================
        const int mw = wave - 4;
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        const int kp = lane & 15;                          // this lane's pair of a step's reduction indices
        const int lrow = (lane >> 4) + 4 * mw;             // its row (column) within a pass
        uint8_t *const ring = lds + 2 * STAGE + mw * Cfg::RING;
        const uint32_t a_lane = (uint32_t)lrow * (uint32_t)p.wsRow * 4u;
        const uint32_t b_lane = (uint32_t)lrow * (uint32_t)p.xsN * 4u;
        uint32_t sa[AP], sb[BP];      // scalar offsets of the passes (a scalar offset never exceeds the buffer's size)
        float a_val[2][AP][2], b_val[2][BP][2];

        // (n, p, q) of one index per lane: n in the offsets, (p << 16) | q apart
        const int dl = lane & (BK - 1);
        const uint32_t sN = (uint32_t)p.xsC * 4u, sP = (uint32_t)(p.redMulH * p.xsH) * 4u, sQ = (uint32_t)(p.redMulW * p.xsW) * 4u;
        const uint32_t dN = (uint32_t)p.wsRed * 4u, dP = (uint32_t)p.wsTapR * 4u, dQ = (uint32_t)p.wsTapS * 4u;
        const uint32_t qn = (uint32_t)p.S, qp = magic_div((uint32_t)p.RS, p.mS);   // output columns and rows
        const uint32_t dn = magic_div((uint32_t)BK, p.mRS), drem = (uint32_t)BK - dn * (uint32_t)p.RS;
        const uint32_t dp = magic_div(drem, p.mS), dq = drem - dp * qn;
        const uint32_t x_step = dn * sN + dp * sP + dq * sQ, x_q = sP - qn * sQ, x_p = sN - qp * sP;
        const uint32_t y_step = dn * dN + dp * dP + dq * dQ, y_q = dP - qn * dQ, y_p = dN - qp * dP;
        uint32_t st_i = 0, st_pq = 0, st_x = 0, st_y = 0;
        int tap_h = 0, tap_w = 0;
        uint32_t tap_off = 0;
        uint32_t a_off[2], b_off[2];   // this lane's pair: offsets of the step to be requested next

        auto put_offsets = [&]() {
            const bool live = st_i < (uint32_t)p.CRS;
            const uint32_t hh = (st_pq >> 16) * (uint32_t)p.redMulH + (uint32_t)tap_h;   // (wraps below zero: fails the test)
            const uint32_t ww = (st_pq & 0xFFFFu) * (uint32_t)p.redMulW + (uint32_t)tap_w;
            const bool ok = live && hh < (uint32_t)p.H && ww < (uint32_t)p.W;
            *reinterpret_cast<u32x2 *>(ring + dl * 8) = u32x2{ok ? st_x + tap_off : kOutOfRange, live ? st_y : kOutOfRange};
        };
        auto get_offsets = [&]() {
            const u32x4 t = *reinterpret_cast<const u32x4 *>(ring + kp * 16);
            b_off[0] = t[0] + b_lane; a_off[0] = t[1] + a_lane;
            b_off[1] = t[2] + b_lane; a_off[1] = t[3] + a_lane;
        };
        auto advance = [&]() {
            st_pq += (dp << 16) | dq;
            const bool cq = (st_pq & 0xFFFFu) >= qn;
            st_pq += cq ? 0x10000u - qn : 0u;
            const bool cp = st_pq >= qp << 16;
            st_pq -= cp ? qp << 16 : 0u;
            st_x += x_step + (cq ? x_q : 0u) + (cp ? x_p : 0u);
            st_y += y_step + (cq ? y_q : 0u) + (cp ? y_p : 0u);
            st_i += (uint32_t)BK;
        };
        auto setup_tile = [&](int number) {
            const Tile t = tile_of(number < tiles_total ? number : 0);   // (no tile: any; nothing of it is multiplied)
            tap_h = t.tap_h;
            tap_w = t.tap_w;
            tap_off = ((uint32_t)tap_h * (uint32_t)p.xsH + (uint32_t)tap_w * (uint32_t)p.xsW) * 4u;
#pragma unroll
            for (int ps = 0; ps < AP; ++ps) sa[ps] = (uint32_t)(t.m0 + ps * RPP < p.K ? t.m0 + ps * RPP : 0) * (uint32_t)p.wsRow * 4u;
#pragma unroll
            for (int ps = 0; ps < BP; ++ps) sb[ps] = (uint32_t)(t.n0 + ps * RPP < p.NPQ ? t.n0 + ps * RPP : 0) * (uint32_t)p.xsN * 4u;
            st_i = (uint32_t)(t.split * nsteps * BK + dl);
            const uint32_t n = magic_div(st_i, p.mRS);
            const uint32_t rem = st_i - n * (uint32_t)p.RS;
            const uint32_t pp = magic_div(rem, p.mS);
            const uint32_t qq = rem - pp * qn;
            st_pq = (pp << 16) | qq;
            st_x = n * sN + pp * sP + qq * sQ;
            st_y = n * dN + pp * dP + qq * dQ;
            put_offsets();
            get_offsets();
        };
        constexpr int NLD = 2 * (AP + BP), NCV = AP + BP;
        auto request = [&](auto set_c, int i) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            const int ps = i / 2, e = i % 2;
            if (ps < AP) {
                a_val[set][ps][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, a_off[e], sa[ps], 0));
            } else {
                b_val[set][ps - AP][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, b_off[e], sb[ps - AP], 0));
            }
        };
        SplitSeen seen;
        auto publish = [&](int it) { publish_seen(lds + Cfg::SEEN + ((it & 1) * Cfg::MOVERS + mw) * kSeenBytes, seen); };
        auto convert = [&](auto set_c, int ps) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            uint8_t *const dst = lds + set * STAGE + (ps < AP ? ps * RPP * ROW : Cfg::A_BYTES + (ps - AP) * RPP * ROW) + lrow * ROW + kp * 4;
            uint32_t h, m, l;
            if (ps < AP) split_pair(a_val[set][ps][0], a_val[set][ps][1], h, m, l, seen);
            else split_pair(b_val[set][ps - AP][0], b_val[set][ps - AP][1], h, m, l, seen);
            *reinterpret_cast<uint32_t *>(dst) = h;
            *reinterpret_cast<uint32_t *>(dst + PART) = m;
            *reinterpret_cast<uint32_t *>(dst + 2 * PART) = l;
        };
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        // one interval: see igconv_kernel_f32s.hpp
        auto interval = [&](auto set_c, auto other_c, int done) __attribute__((always_inline)) {
            advance();
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
        for (int ps = 0; ps < AP; ++ps) a_val[1][ps][0] = a_val[1][ps][1] = 0.f;
#pragma unroll
        for (int ps = 0; ps < BP; ++ps) b_val[1][ps][0] = b_val[1][ps][1] = 0.f;
        setup_tile(tile_number(0));
        int it = 1;
        for (;; ++it) {
            const int next = tile_number(it);
            for (int t = 0; t < nsteps; t += 2) {
                interval(S0{}, S1{}, t == 0 ? it - 2 : -1);
                interval(S1{}, S0{}, -1);
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
    float bvec[MB];   // (no bias in this pass: zeros, for the shared epilogue)
    load_bias<MB>(p, 0, l32, bvec);
    __builtin_amdgcn_s_setprio(2);
    mult.prime();
    for (int it = 0;; ++it) {
        const int number = tile_number(it);
        if (number >= tiles_total) break;
        const Tile t = tile_of(number);
        const int krow0 = t.m0 + wm * Cfg::TM, col0 = t.n0 + wn * Cfg::TN;
        mult.zero();
        mult.steps(nsteps);
        const uint32_t inexact = inexact_below<Cfg::MOVERS>(lds + Cfg::SEEN + (it & 1) * Cfg::MOVERS * kSeenBytes, nsteps * BK);
        if (__any(outside_split_range<MB, NB>(mult.acc, inexact))) {
            const int kb = t.split * nsteps * BK, ke = kb + nsteps * BK;
            wgrad_sums_in_fp32<Cfg>(p, mult.acc, krow0, col0, t.tap_h, t.tap_w, kb < p.CRS ? kb : p.CRS, ke < p.CRS ? ke : p.CRS, half, l32);
        }
        // (each range writes its own copy of the output, y_bytes long; the columns are channels, R*S elements apart, and
        // the tile's tap moves the base)
        const uint32_t ytap = (uint32_t)t.tap * 4u;
        const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(
            static_cast<char *>(p.y) + ((uint32_t)t.split * p.ySplitBytes + ytap), 0, p.y_bytes - ytap, kBufferWord3);
        store_tile<false, MB, NB, true>(p, ybuf, mult.acc, bvec, krow0, col0, half, l32);
    }
#endif
}

}  // namespace igc
#endif
