// Forward pass of float layers with a short reduction - the first layer of a network on small images: one to four
// channels, 3x3 or 5x5 filters - on the vector units: a thread keeps KB output maps of PX pixels in registers and walks
// the window, the workgroup's filter rows in LDS.  A reduction of 27 indices is a single step of the matrix kernels, whose
// tile of 64 x 128, offset arithmetic per element, three barriers and epilogue through 32 x 32 blocks are then all of
// the time; here it is one round of window loads, the multiply-adds and the store.
//   1x3x32x32 -> 16, 3x3, bias and rectifier: 8.6 us (copy with the border written out, then a launch over it) -> 5.3;
//   128x3x32x32 -> 32, 3x3: 15.4 -> 9.8; 1x3x224x224 -> 64, 3x3: 12.5 -> 8.6.
// (A first form walked any filter size with the tap arithmetic per element: 6.4, and 2.5 times the instructions.)
// What bounds it: at small sizes the latency of that chain; at large ones the LDS reads of the filter (16 bytes for
// 4 * PX multiply-adds, hence two pixels and sixteen maps per thread) and the stores of y.
// Reduction order (c, r, s), a chain of fused multiply-adds (3x3: per channel).
#include "igconv_instantiate.hpp"
#include "igconv_kernel.hpp"

namespace igc {

constexpr int kFewChannels = 4;    // (LDS of the filter rows; see the rule in igconv_api.cpp)

template <int R, int S, int PX, int KB>
__global__ __launch_bounds__(256, 4) void igconv_few_channels_kernel(const ConvKernelParams p) {
    constexpr int T = R * S;
    __shared__ __attribute__((aligned(16))) float wl[kFewChannels * T * KB];   // [index][map]
    const int tid = (int)threadIdx.x;
    const int m0 = (int)blockIdx.y * KB;

    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.x), 0, p.x_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.w), 0, p.w_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, kBufferWord3);

    // filter rows to LDS, transposed; maps beyond K as zeros
    for (int k = tid >> 5; k < KB; k += 8)
        for (int e = tid & 31; e < p.CRS; e += 32)
            wl[e * KB + k] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, m0 + k < p.K ? (uint32_t)((m0 + k) * p.CRS + e) * 4u : kOutOfRange, 0, 0));
    // byte offsets of the window's elements in channel 0, the out-of-range marker for those in the border (they read zeros)
    uint32_t tap[PX][T], yoff[PX];
#pragma unroll
    for (int px = 0; px < PX; ++px) {
        const uint32_t j = blockIdx.x * (uint32_t)(256 * PX) + (uint32_t)(px * 256 + tid);
        const bool live = j < (uint32_t)p.NPQ;
        const uint32_t jj = live ? j : 0u;
        const uint32_t n = magic_div(jj, p.mPQ), rem = jj - n * (uint32_t)p.PQ;
        const uint32_t pp = magic_div(rem, p.mQ), qq = rem - pp * (uint32_t)p.Q;
        const int h0 = (int)pp * p.u - p.pad_h, w0 = (int)qq * p.v - p.pad_w;
        const uint32_t base = n * (uint32_t)p.xsN;
        yoff[px] = live ? (n * (uint32_t)p.ysN + pp * (uint32_t)p.ysP + qq * (uint32_t)p.ysQ) * 4u : kOutOfRange;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int h = h0 + (p.flip ? R - 1 - r : r);   // (eq. 2 walks the window backwards)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int w = w0 + (p.flip ? S - 1 - s : s);
                const bool in = live && (uint32_t)h < (uint32_t)p.H && (uint32_t)w < (uint32_t)p.W;
                tap[px][r * S + s] = in ? (base + (uint32_t)h * (uint32_t)p.xsH + (uint32_t)w * (uint32_t)p.xsW) * 4u : kOutOfRange;
            }
        }
    }
    auto request = [&](int c, float (&v)[T][PX]) __attribute__((always_inline)) {
        const uint32_t co = (uint32_t)c * (uint32_t)p.xsC * 4u;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int px = 0; px < PX; ++px)
                v[t][px] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, tap[px][t], co, 0));
    };
    float acc[PX][KB];
#pragma unroll
    for (int px = 0; px < PX; ++px)
#pragma unroll
        for (int k = 0; k < KB; ++k) acc[px][k] = 0.f;
    auto multiply = [&](int c, const float (&v)[T][PX]) __attribute__((always_inline)) {
        if constexpr (T == 9) {   // a channel's sum first, then added: shorter chains of roundings
#pragma unroll
            for (int q = 0; q < KB / 4; ++q) {
                float sum[PX][4];
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const f32x4 f = *reinterpret_cast<const f32x4 *>(&wl[(c * T + t) * KB + 4 * q]);
#pragma unroll
                    for (int px = 0; px < PX; ++px)
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[px][e] = t == 0 ? v[t][px] * f[e] : __builtin_fmaf(v[t][px], f[e], sum[px][e]);
                }
#pragma unroll
                for (int px = 0; px < PX; ++px)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[px][4 * q + e] += sum[px][e];
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {                  // (no registers for that)
#pragma unroll
            for (int t = 0; t < T; ++t) {
#pragma unroll
                for (int q = 0; q < KB / 4; ++q) {
                    const f32x4 f = *reinterpret_cast<const f32x4 *>(&wl[(c * T + t) * KB + 4 * q]);
#pragma unroll
                    for (int px = 0; px < PX; ++px)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[px][4 * q + e] = __builtin_fmaf(v[t][px], f[e], acc[px][4 * q + e]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    float v0[T][PX], v1[T][PX];
    request(0, v0);
    __syncthreads();
    for (int c = 0; c < p.C; c += 2) {
        if (c + 1 < p.C) request(c + 1, v1);
        multiply(c, v0);
        if (c + 1 >= p.C) break;
        if (c + 2 < p.C) request(c + 2, v0);
        multiply(c + 1, v1);
    }
    const bool use_beta = p.beta != 0.f, fused = p.bias != nullptr || p.act >= 0;
#pragma unroll
    for (int px = 0; px < PX; ++px)
#pragma unroll
        for (int b = 0; b < KB; b += 8) {
            float out[8];
            uint32_t off[8], row[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                out[k] = p.alpha * acc[px][b + k];
                off[k] = m0 + b + k < p.K ? yoff[px] : kOutOfRange;
                row[k] = few_channels_map_offset(m0 + b + k, p.K, (uint32_t)p.ysK * 4u);
            }
            if (use_beta) {
                float old[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) old[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ybuf, off[k], row[k], 0));
#pragma unroll
                for (int k = 0; k < 8; ++k) out[k] += p.beta * old[k];
            }
            if (fused) {
                if (p.bias != nullptr) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) out[k] += p.bias[m0 + b + k < p.K ? m0 + b + k : p.K - 1];
                }
                if (p.act == 0) activate<0>(out);
                else if (p.act == 1) activate<1>(out);
                else if (p.act == 2) activate<2>(out);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, out[k]), ybuf, off[k], row[k], 0);
        }
}

template <int R, int S, int PX, int KB>
static int launch_few(const ConvKernelParams &p, void *stream) {
    ConvKernelParams args = p;
    void *ptrs[] = {&args};
    const dim3 grid((unsigned)((p.NPQ + 256 * PX - 1) / (256 * PX)), (unsigned)((p.K + KB - 1) / KB));
    return (int)hipLaunchKernel((const void *)&igconv_few_channels_kernel<R, S, PX, KB>, grid, dim3(256), ptrs, 0, (hipStream_t)stream);
}

int launch_few_channels(const ConvKernelParams &p, int computeUnits, void *stream) {
    // One pixel and eight maps per thread while that does not fill the chip several times over; then fewer LDS reads per
    // multiply-add win: 131072 pixels x 32 maps, 3x3 9.8 and 10.7 us, 5x5 20.0 and 16.9; 200704 x 32, 3x3 16.6 and 15.1.
    const bool small = (long long)p.NPQ * p.K < (long long)computeUnits * 256 * (p.R == 3 ? 80 : 40);
    if (p.R == 3) return small ? launch_few<3, 3, 1, 8>(p, stream) : launch_few<3, 3, 2, 16>(p, stream);
    return small ? launch_few<5, 5, 1, 8>(p, stream) : launch_few<5, 5, 1, 16>(p, stream);
}

}  // namespace igc
