// bf16 convolution (forward, backward data) for any filter over tensors whose channels are contiguous, reading a filter
// that has been rewritten with the reduction's channel index innermost (launch_filter_taps_outer): both operands are
// then contiguous along the channels of a tap and go to LDS as they are loaded, as in the 1x1 kernel
// (igconv_kernel_bf16_pw.hpp), whose structure this is - moving and multiplying wavefronts, persistent workgroups, loads
// two steps ahead running on across the tile boundary.
//
// Reduction order: (32 channels, tap, channel), the order of the element-wise tap-major kernels that read the filter in
// place, with the same 16-index groups per MFMA: the same bits with and without the rewritten filter.  A step is two
// such units of 32 channels - in general two taps: four lanes of a row read 64 contiguous bytes of the one, four of the
// other - because one (8 MFMAs per wavefront) would be too short for its barrier.
// What it replaces loads 2-byte elements one by one and was bound by the number of loads: backward data of a 3x3 layer with
// stride 2, 32x256x28x28 -> 128x56x56, four phases of 43 us (the one of four taps) and
// less, now 13 and less; the layer with its 1x1 shortcut, forward and backward, 525 -> 225 us.
#ifndef IGCONV_KERNEL_BF16_TAPS_HPP_
#define IGCONV_KERNEL_BF16_TAPS_HPP_

#include "igconv_kernel.hpp"

namespace igc {

template <int BM_, int BN_, bool SWAP_>
struct Bf16TapsConfig {
    static constexpr int BM = BM_, BN = BN_, UNIT = 32;      // UNIT: channels per unit, two units per step
    static constexpr bool SWAP = SWAP_;
    static constexpr int THREADS = 512;
    static constexpr int ROW = 2 * UNIT * 2 + 16;            // an odd number of 16-byte units
    static constexpr int STAGE_BYTES = (BM + BN) * ROW;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
    static_assert(BM % 64 == 0 && BN % 64 == 0, "2 x 2 wavefronts of whole 32 x 32 blocks");
};

// `block`: the workgroup's number within its problem
template <class Cfg>
__device__ __forceinline__ void bf16_taps_body(const ConvKernelParams &p, uint32_t block) {
    constexpr int BM = Cfg::BM, BN = Cfg::BN, MB = BM / 64, NB = BN / 64, RB = Cfg::ROW;
    constexpr int NA = BM / 32, NBV = BN / 32;      // 16-byte loads per thread and step: rows tid/8 + 32 i
    __shared__ __attribute__((aligned(16))) uint8_t lds[Cfg::LDS_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool mover = wave_all >= 4;            // wavefronts 4-7 move, 0-3 multiply; both kinds number themselves 0-3
    const int wave = wave_all & 3, tid = (int)threadIdx.x & 255;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;

    const int tiles = p.tilesM * p.tilesN;
    const int xcd = (int)(block % 8u), slot = (int)(block / 8u);
    const int range_end = (xcd + 1) * p.tilesPerXcd < tiles ? (xcd + 1) * p.tilesPerXcd : tiles;
    int tile = xcd * p.tilesPerXcd + slot;
    if (tile >= range_end) return;

    const int units = p.ksteps;
    // steps per tile, an even number (the LDS stages alternate); what is added reads zeros; a backward-data phase that
    // meets no tap runs two steps of zeros
    const int steps = units > 4 ? ((units + 3) >> 2) << 1 : 2;

    if (mover) {
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        // loading role: 16-byte piece vec of the step (unit vec / 4), rows (filter rows / pixels) tid/8 + 32 i
        const int vec = tid & 7, row = tid >> 3;
        struct Rows {
            uint32_t a[NA];       // byte offset of the filter row, or the out-of-range marker
            uint32_t b[NBV];      // byte offset of the window origin (mod 2^32)
            u16x2 hw[NBV];        // its coordinates; 0x8000 in the row field: column beyond NPQ
        };
        auto tile_rows = [&](int t, Rows &o) {
            const bool live = t < range_end;
            const int m0 = (t % p.tilesM) * BM, n0 = (t / p.tilesM) * BN;
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int m = m0 + row + 32 * i;
                o.a[i] = live && m < p.K ? (uint32_t)m * (uint32_t)p.wsRow * 2u : kOutOfRange;
            }
#pragma unroll
            for (int i = 0; i < NBV; ++i) {
                const int j = n0 + row + 32 * i;
                const bool cv = live && j < p.NPQ;
                const uint32_t jj = cv ? (uint32_t)j : 0u;
                const uint32_t n = magic_div(jj, p.mPQ), rem = jj - n * (uint32_t)p.PQ;
                const uint32_t pp = magic_div(rem, p.mQ), qq = rem - pp * (uint32_t)p.Q;
                const int h0 = (int)pp * p.u - p.pad_h, w0 = (int)qq * p.v - p.pad_w;
                o.b[i] = (n * (uint32_t)p.xsN + (uint32_t)h0 * (uint32_t)p.xsH + (uint32_t)w0 * (uint32_t)p.xsW) * 2u;
                o.hw[i][1] = (uint16_t)(cv ? h0 : 0x8000);
                o.hw[i][0] = (uint16_t)w0;
            }
        };
        u16x2 hw_max;
        hw_max[1] = (uint16_t)(p.H - 1);
        hw_max[0] = (uint16_t)(p.W - 1);
        Rows cur, nxt;                         // of the current tile and of the next one
        u32x4 a0[NA], b0[NBV], a1[NA], b1[NBV];
        auto fetch_from = [&](int step, const Rows &o, u32x4 (&a)[NA], u32x4 (&b)[NBV]) __attribute__((always_inline)) {
            const uint32_t unit = (uint32_t)(2 * step + (vec >> 2));
            const uint32_t cc = magic_div(unit, p.mRS), tap = unit - cc * (uint32_t)p.RS;
            const uint32_t r = magic_div(tap, p.mS), sx = tap - r * (uint32_t)p.S;
            const uint32_t tr = p.flip ? (uint32_t)p.R - 1u - r : r, ts = p.flip ? (uint32_t)p.S - 1u - sx : sx;   // eq. 2 inverts the filter
            const uint32_t ch = cc * (uint32_t)Cfg::UNIT + (uint32_t)(vec & 3) * 8u;
            const bool live = unit < (uint32_t)units && ch < (uint32_t)p.C;
            const uint32_t ao = live ? ((uint32_t)p.wTap0 + r * (uint32_t)p.wsTapR + sx * (uint32_t)p.wsTapS + ch) * 2u : kOutOfRange;
            const uint32_t bo = (tr * (uint32_t)p.xsH + ts * (uint32_t)p.xsW + ch) * 2u;
            const u16x2 t2 = __builtin_bit_cast(u16x2, live ? (tr << 16) | ts : 0x80000000u);
#pragma unroll
            for (int i = 0; i < NA; ++i)
                a[i] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, (o.a[i] | ao) >= kOutOfRange ? kOutOfRange : o.a[i] + ao, 0, 0);
#pragma unroll
            for (int i = 0; i < NBV; ++i) {
                // (a dead unit of a dead column: 0x8000 + 0x8000 wraps to row 0 of the image's first column - a valid offset or
                // none, and such a column is never stored)
                const u16x2 hw = o.hw[i] + t2;
                const u16x2 cl = __builtin_elementwise_min(hw, hw_max);
                const bool ok = __builtin_bit_cast(uint32_t, cl) == __builtin_bit_cast(uint32_t, hw);
                b[i] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, ok ? o.b[i] + bo : kOutOfRange, 0, 0);
            }
        };
        auto stage = [&](int buf, const u32x4 (&a)[NA], const u32x4 (&b)[NBV]) __attribute__((always_inline)) {
            uint8_t *base = lds + buf * Cfg::STAGE_BYTES + row * RB + vec * 16;
#pragma unroll
            for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4 *>(base + 32 * i * RB) = a[i];
#pragma unroll
            for (int i = 0; i < NBV; ++i) *reinterpret_cast<u32x4 *>(base + (BM + 32 * i) * RB) = b[i];
        };
        // In step s the multipliers compute from LDS stage `at` while the movers put the loaded data of step s+1 into the
        // other stage and request step s+2 - of this tile, or step s+2-steps of the next one; one barrier per step.
        auto move = [&](int s, int at, u32x4 (&a_new)[NA], u32x4 (&b_new)[NBV], const u32x4 (&a_next)[NA],
                        const u32x4 (&b_next)[NBV]) __attribute__((always_inline)) {
            if (s + 2 < steps) fetch_from(s + 2, cur, a_new, b_new);
            else fetch_from(s + 2 - steps, nxt, a_new, b_new);
            stage(at ^ 1, a_next, b_next);
            __syncthreads();
        };
        tile_rows(tile, cur);
        fetch_from(0, cur, a0, b0);
        fetch_from(1, cur, a1, b1);
        stage(0, a0, b0);
        __syncthreads();
        for (; tile < range_end; tile += p.wgsPerXcd) {
            tile_rows(tile + p.wgsPerXcd, nxt);
            for (int s = 0; s < steps; s += 2) {
                move(s, 0, a0, b0, a1, b1);
                move(s + 1, 1, a1, b1, a0, b0);
            }
            cur = nxt;
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, kBufferWord3);
    f32x16 acc[MB][NB];
    auto multiply = [&](int at) __attribute__((always_inline)) {
        const uint8_t *a_base = lds + at * Cfg::STAGE_BYTES + (wm * (BM / 2) + l32) * RB + half * 16;
        const uint8_t *b_base = lds + at * Cfg::STAGE_BYTES + (BM + wn * (BN / 2) + l32) * RB + half * 16;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 av[MB], bv[NB];
#pragma unroll
            for (int i = 0; i < MB; ++i) av[i] = *reinterpret_cast<const bf16x8 *>(a_base + i * 32 * RB + ks * 32);
#pragma unroll
            for (int j = 0; j < NB; ++j) bv[j] = *reinterpret_cast<const bf16x8 *>(b_base + j * 32 * RB + ks * 32);
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if constexpr (Cfg::SWAP)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[j], av[i], acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
                }
        }
        __syncthreads();
    };
    __syncthreads();
    for (; tile < range_end; tile += p.wgsPerXcd) {
        const int m0 = (tile % p.tilesM) * BM, n0 = (tile / p.tilesM) * BN;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
        float bias[MB];
        load_bias<MB>(p, m0 + wm * (BM / 2), l32, bias);
        for (int s = 0; s < steps; s += 2) {
            multiply(0);
            multiply(1);
        }
        // (the movers are already on the next tile's first steps)
        store_tile<Cfg::SWAP, MB, NB>(p, ybuf, acc, bias, m0 + wm * (BM / 2), n0 + wn * (BN / 2), half, l32);
    }
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 4) void igconv_bf16_taps_kernel(const ConvKernelParams p) {
    bf16_taps_body<Cfg>(p, blockIdx.x);
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 4) void igconv_bf16_taps_phases_kernel(const ConvPhaseParams) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernel's name and signature only)
    uint32_t block;
    const ConvKernelParams p = phase_of_workgroup(&block);
    bf16_taps_body<Cfg>(p, block);
#endif
}

}  // namespace igc
#endif
