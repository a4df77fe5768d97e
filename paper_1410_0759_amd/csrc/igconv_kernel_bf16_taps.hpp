// bf16 convolution (forward, backward data) for any filter over tensors whose channels are contiguous, reading a filter
// that has been rewritten with the reduction's channel index innermost (launch_filter_taps_outer): both operands are
// then contiguous along the channels of a tap and go from global memory straight into LDS, 16 bytes per lane, without
// passing through registers.
//
// Reduction order: (32 channels, tap, channel), the order of the element-wise tap-major kernels that read the filter in
// place, with the same 16-index groups per MFMA: the same bits with and without the rewritten filter.  A step is one unit,
// 32 channels of one tap: 64 bytes of every row of the tile.
//
// What bounds it: pieces of 64 bytes from L2 (128-byte ones need another order of the sums) - 10 TB/s over the chip with the 128 x 256 tile at 256 -> 128x28x28,
// 5x5, 96 % of them hits, MFMAs busy for 60 % of the cycles; a 128 x 128 tile's step of 256 cycles of MFMAs asks for 16 KB, half as much again per product.  Hence
// the 128 x 256 tile for problems that fill the chip with it and have enough steps, and moving and multiplying wavefronts apart with a ring of stages
// in LDS - the one being read, the others complete or on their way: 80 KB per workgroup of the 128 x 128 tile and 72 of the
// 64 x 128 one, two of which share a compute unit's 160, 144 KB of the large one.  Persistent workgroups; the movers run on across the tile boundary, so that the next
// tile's first stages arrive while the finished tile is stored.
// Measured against the form before (steps of two units, requested two steps ahead into registers and written to LDS from
// there; branches around its loads made every step wait for those just issued), us with the filter's rewriting:
// backward data, 256 -> 128x28x28, 5x5, 128 images 230 -> 176 (930 TFLOP/s); 192 -> 320x27x27, 5x5, 12 images 62 -> 51; 128 ->
// 128x28x28, 5x5, 8 images 31 -> 26; forward, 128x56x56 -> 256, 3x3 stride 2, 32 images 33 -> 31, of which the filter 5.  644 random layers: 0.90 of the time
// on average, up to a tenth more with some channel counts that are odd multiples of eight (1x448x32x32 -> 216, 5x5, backward data 57.5 -> 64.5).
#ifndef IGCONV_KERNEL_BF16_TAPS_HPP_
#define IGCONV_KERNEL_BF16_TAPS_HPP_

#include "igconv_kernel.hpp"

namespace igc {

template <int BM_, int BN_, int STAGES_, bool SWAP_>
struct Bf16TapsConfig {
    static constexpr int BM = BM_, BN = BN_, UNIT = 32;      // UNIT: channels per step
    static constexpr int STAGES = STAGES_;
    static constexpr bool SWAP = SWAP_;
    static constexpr int THREADS = 512;
    static constexpr int ROW = UNIT * 2;                     // bytes; four 16-byte pieces
    static constexpr int STAGE_BYTES = (BM + BN) * ROW;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
    static constexpr int PER_CU = (160 * 1024) / LDS_BYTES < 2 ? 1 : 2;
    // 1 KB requests (16 rows) per mover and step
    static constexpr int LA = BM / 64, LB = BN / 64, LOADS = LA + LB;
    static_assert(BM % 64 == 0 && BN % 64 == 0, "2 x 2 wavefronts of whole 32 x 32 blocks");
    static_assert(STAGES >= 3 && LOADS * (STAGES - 2) < 64, "vmcnt is a 6-bit counter");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// `block`: the workgroup's number within its problem
template <class Cfg>
__device__ __forceinline__ void bf16_taps_body(const ConvKernelParams &p, uint32_t block) {
    constexpr int BM = Cfg::BM, BN = Cfg::BN, MB = BM / 64, NB = BN / 64, RB = Cfg::ROW, NS = Cfg::STAGES;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg::LDS_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool mover = wave_all >= 4;            // wavefronts 4-7 move, 0-3 multiply; both kinds number themselves 0-3
    const int wave = wave_all & 3;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;

    const int tiles = p.tilesM * p.tilesN;
    const int xcd = (int)(block % 8u), slot = (int)(block / 8u);
    const int range_end = (xcd + 1) * p.tilesPerXcd < tiles ? (xcd + 1) * p.tilesPerXcd : tiles;
    int tile = xcd * p.tilesPerXcd + slot;
    if (tile >= range_end) return;
    const int units = p.ksteps;              // steps per tile; none for a backward-data phase that meets no tap
    const int total = ((range_end - tile + p.wgsPerXcd - 1) / p.wgsPerXcd) * units;   // steps of this workgroup

    if (mover) {
        if (total == 0) return;              // (the multipliers meet no barrier either)
        const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
        const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
        // A request fills 16 rows: lane l writes slot l % 4 of row l / 4, which holds piece (l % 4) ^ (row / 4 % 4), so that the
        // 16-byte reads of one piece of 16 consecutive rows meet every bank once.  This wavefront's requests: rows
        // 16 (LA wave + i) of the filter tile, 16 (LB wave + i) of the pixels.
        const uint32_t piece = (uint32_t)((lane & 3) ^ (lane >> 4));
        const int row = lane >> 2;
        uint32_t a_off[Cfg::LA];       // byte offset of the piece in the filter row's first unit, or the out-of-range marker
        uint32_t b_off[Cfg::LB];       // of the piece in the window origin's first unit (mod 2^32)
        u16x2 b_hw[Cfg::LB];           // the origin's coordinates; 0x8000 in the row field: column beyond NPQ
        auto tile_rows = [&](int t) {
            const int m0 = (t % p.tilesM) * BM, n0 = (t / p.tilesM) * BN;
#pragma unroll
            for (int i = 0; i < Cfg::LA; ++i) {
                const int m = m0 + 16 * (Cfg::LA * wave + i) + row;
                a_off[i] = m < p.K ? (uint32_t)m * (uint32_t)p.wsRow * 2u + piece * 16u : kOutOfRange;
            }
#pragma unroll
            for (int i = 0; i < Cfg::LB; ++i) {
                const int j = n0 + 16 * (Cfg::LB * wave + i) + row;
                const bool cv = j < p.NPQ;
                const uint32_t jj = cv ? (uint32_t)j : 0u;
                const uint32_t n = magic_div(jj, p.mPQ), rem = jj - n * (uint32_t)p.PQ;
                const uint32_t pp = magic_div(rem, p.mQ), qq = rem - pp * (uint32_t)p.Q;
                const int h0 = (int)pp * p.u - p.pad_h, w0 = (int)qq * p.v - p.pad_w;
                b_off[i] = (n * (uint32_t)p.xsN + (uint32_t)h0 * (uint32_t)p.xsH + (uint32_t)w0 * (uint32_t)p.xsW) * 2u + piece * 16u;
                b_hw[i][1] = (uint16_t)(cv ? h0 : 0x8000);
                b_hw[i][0] = (uint16_t)w0;
            }
        };
        u16x2 hw_max;
        hw_max[1] = (uint16_t)(p.H - 1);
        hw_max[0] = (uint16_t)(p.W - 1);
        // the next step to request: its tap (row r, column sx, counted in the filter's order) and first channel
        int r = 0, sx = 0, c0 = 0, stage = 0, left = total;
        tile_rows(tile);
        auto request = [&]() __attribute__((always_inline)) {
            uint8_t *const dst = lds + stage * Cfg::STAGE_BYTES;
            stage = stage + 1 == NS ? 0 : stage + 1;
            const bool live = left > 0;       // (past the last step: requests that read nothing keep the counts alike)
            const uint32_t tr = (uint32_t)(p.flip ? p.R - 1 - r : r), ts = (uint32_t)(p.flip ? p.S - 1 - sx : sx);   // eq. 2 inverts the filter
            const uint32_t as = live ? (uint32_t)(p.wTap0 + r * p.wsTapR + sx * p.wsTapS + c0) * 2u : p.w_bytes;
            const uint32_t bo = (tr * (uint32_t)p.xsH + ts * (uint32_t)p.xsW + (uint32_t)c0) * 2u;
            const uint32_t bs = live ? 0u : p.x_bytes;
            const bool past = (int)piece * 8 >= p.C - c0;     // the last unit may end inside (C is a multiple of 8)
            const u16x2 t2 = __builtin_bit_cast(u16x2, (tr << 16) | ts);
#pragma unroll
            for (int i = 0; i < Cfg::LA; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void *)(dst + (Cfg::LA * wave + i) * 1024), 16,
                                                         past ? kOutOfRange : a_off[i], as, 0, 0);
#pragma unroll
            for (int i = 0; i < Cfg::LB; ++i) {
                const u16x2 hw = b_hw[i] + t2;
                const u16x2 cl = __builtin_elementwise_min(hw, hw_max);
                const bool ok = !past && __builtin_bit_cast(uint32_t, cl) == __builtin_bit_cast(uint32_t, hw);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void *)(dst + (BM / 16 + Cfg::LB * wave + i) * 1024), 16,
                                                         ok ? b_off[i] + bo : kOutOfRange, bs, 0, 0);
            }
            // the step after it; one tile after the other
            --left;
            if (++sx == p.S) {
                sx = 0;
                if (++r == p.R) {
                    r = 0;
                    c0 += Cfg::UNIT;
                    if (c0 >= p.C) {
                        c0 = 0;
                        tile += p.wgsPerXcd;
                        tile_rows(tile);      // (past the range: no request uses it)
                    }
                }
            }
        };
        // Barrier g gives away stage g and publishes stage g + 1: all requests but those of the NS - 2 steps after it have arrived.
        constexpr int later = Cfg::LOADS * (NS - 2);
        auto arrived = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70 | (later & 15) | ((later >> 4) << 14)); };
        auto barrier = [&]() { asm volatile("s_barrier" ::: "memory"); };
#pragma unroll
        for (int i = 0; i < NS - 1; ++i) request();
        arrived();                            // stage 0
        barrier();
        for (int g = 0; g < total; ++g) {
            request();                        // step g + NS - 1, where step g - 1 was
            arrived();                        // stage g + 1
            barrier();
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // nothing may be on its way into LDS when it is given away
        return;
    }
    const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, kBufferWord3);
    f32x16 acc[MB][NB];
    bf16x8 fa[2][MB], fb[2][NB];
    const uint32_t first = (uint32_t)(half ^ ((l32 >> 2) & 3)) * 16u;      // piece `half` of the lane's row; the second 16 channels: ^ 32
    const uint32_t a_base = (uint32_t)(wm * (BM / 2) + l32) * RB, b_base = (uint32_t)(BM + wn * (BN / 2) + l32) * RB;
    auto read = [&](int stage, auto ks) __attribute__((always_inline)) {
        constexpr int k = decltype(ks)::value;
        const uint8_t *const base = lds + stage * Cfg::STAGE_BYTES + (first ^ (k * 32u));
#pragma unroll
        for (int i = 0; i < MB; ++i) fa[k][i] = *reinterpret_cast<const bf16x8 *>(base + a_base + i * 32 * RB);
#pragma unroll
        for (int j = 0; j < NB; ++j) fb[k][j] = *reinterpret_cast<const bf16x8 *>(base + b_base + j * 32 * RB);
    };
    auto multiply = [&](auto ks) __attribute__((always_inline)) {
        constexpr int k = decltype(ks)::value;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (Cfg::SWAP)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[k][j], fa[k][i], acc[i][j], 0, 0, 0);
                else
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[k][i], fb[k][j], acc[i][j], 0, 0, 0);
            }
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    constexpr std::integral_constant<int, 0> k0;
    constexpr std::integral_constant<int, 1> k1;
    int stage = 0;
    if (total != 0) {
        barrier();
        read(0, k0);
    }
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
        for (int s = 0; s < units; ++s) {
            const int next = stage + 1 == NS ? 0 : stage + 1;
            read(stage, k1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(k0);
            __builtin_amdgcn_sched_barrier(0);
            barrier();                       // the stage is in registers; the next one is complete
            read(next, k0);                  // (after the workgroup's last step: a stage whose contents nobody uses)
            __builtin_amdgcn_sched_barrier(0);
            multiply(k1);
            __builtin_amdgcn_sched_barrier(0);
            stage = next;
        }
        // (the movers are already on the next tile's first steps)
        store_tile<Cfg::SWAP, MB, NB>(p, ybuf, acc, bias, m0 + wm * (BM / 2), n0 + wn * (BN / 2), half, l32);
    }
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 2 * Cfg::PER_CU) void igconv_bf16_taps_kernel(const ConvKernelParams p) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the host pass needs the kernel's name and signature only)
    bf16_taps_body<Cfg>(p, blockIdx.x);
#endif
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 2 * Cfg::PER_CU) void igconv_bf16_taps_phases_kernel(const ConvPhaseParams) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t block;
    const ConvKernelParams p = phase_of_workgroup(&block);
    bf16_taps_body<Cfg>(p, block);
#endif
}

}  // namespace igc
#endif
