// fp32 kernels on the 16-bit matrix pipes, operands as two binary16 parts, with a staged image patch (igconv_kernel_f32h.hpp).
#include "igconv_kernel_f32h.hpp"

namespace igc {

// The filter as igconv_f32h_kernel reads it: a workgroup per (row block of 64 rows, chunk), a thread on two channels of a row.
// Bound by one round of loads and stores per workgroup, and by its launch.
__global__ __launch_bounds__(512) void igconv_split_filter_kernel(const float *w, uint8_t *out, HalvesChunk *table, int K, int C, int taps, int groups,
                                                                  uint32_t row_stride, uint32_t channel_stride, uint32_t w_bytes) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 64, CPT = 2;   // rows of a workgroup, channels of a thread
    __shared__ __attribute__((aligned(16))) uint32_t slots[8], counts[8], sums[8];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x, cb = chunk / groups, g = chunk - cb * groups;
    const int row = tid / (16 / CPT), sub = tid % (16 / CPT);
    const int k = blockIdx.y * BM + row;
    const int tap0 = halves_first_tap(g, taps);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(w), 0, w_bytes, kBufferWord3);
    float x[CPT][9];
#pragma unroll
    for (int e = 0; e < CPT; ++e) {   // (rows beyond K and channels beyond C are zero)
        const uint32_t off = k < K && cb * 16 + sub * CPT + e < C ? ((uint32_t)k * row_stride + (uint32_t)(cb * 16 + sub * CPT + e) * channel_stride + (uint32_t)tap0) * 4u : kOutOfRange;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, off + (uint32_t)q * 16u, 0, 0));
#pragma unroll
            for (int c = 0; c < 4; ++c) x[e][q * 4 + c] = v[c];
        }
        x[e][8] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wbuf, off + 32u, 0, 0));
    }
    HalvesSeen seen;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int e = 0; e < CPT; e += 2) {
            if (tap0 + t < 9 * g) x[e][t] = x[e + 1][t] = 0.f;   // (a tap that the group before has as well)
            look_at(seen, x[e][t], x[e + 1][t]);
        }
    publish_largest(reinterpret_cast<uint8_t *>(slots + wave), seen, lane);
    __syncthreads();
    uint32_t largest = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) largest = largest > slots[i] ? largest : slots[i];
    const HalvesScale sc = halves_scale((uint32_t)__builtin_amdgcn_readfirstlane((int)largest));
    uint32_t lossy = 0;
#pragma unroll
    for (int e = 0; e < CPT; ++e)
#pragma unroll
        for (int t = 0; t < 9; ++t) lossy += count_lossy(x[e][t], sc.below);
    float sum = 0.f;   // of the row's magnitudes: eight neighbouring threads have it
#pragma unroll
    for (int e = 0; e < CPT; ++e)
#pragma unroll
        for (int t = 0; t < 9; ++t) sum += __builtin_fabsf(x[e][t]) * sc.s;
    static_assert(16 / CPT == 8, "threads of a row");
#pragma unroll
    for (int d = 4; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    const uint32_t row_sum = wave_largest(__builtin_bit_cast(uint32_t, sum));   // (not negative: ordered like its bits)
    if (lanes_under(seen.smallest, far_below(sc.below)) != 0u) lossy |= kFarBelow;
    if (lane == 0) {
        counts[wave] = lossy;
        sums[wave] = row_sum;
    }
    uint8_t *const dst = out + ((size_t)blockIdx.y * gridDim.x + (size_t)chunk) * (9 * BM * 64) + (sub * CPT / 8) * (BM * 16) + row * 16 + sub * CPT % 8 * 2;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        uint32_t h, m;
        halves_pair(x[0][t], x[1][t], sc, h, m);
        *reinterpret_cast<uint32_t *>(dst + t * (BM * 64)) = h;
        *reinterpret_cast<uint32_t *>(dst + t * (BM * 64) + BM * 32) = m;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t n = 0, far = 0, most = 0;
        for (int i = 0; i < 8; ++i) {
            n += counts[i] & ~kFarBelow;
            far |= counts[i] & kFarBelow;
            most = most > sums[i] ? most : sums[i];
        }
        const float bound = __builtin_bit_cast(float, most) + 2.f;   // (rounded up; infinities and NaN, whose sums are multiplied again anyway: the largest)
        const uint32_t row_most = bound < 144.f * 32768.f ? (uint32_t)bound : 144u * 32768u;
        table[(size_t)blockIdx.y * gridDim.x + (size_t)chunk] = HalvesChunk{sc.e, (n < 144u ? n : 144u) | row_most << 8 | far};
    }
#endif
}

int launch_split_filter(const ConvKernelParams &p, void *out, void *stream) {
    const int groups = (p.RS + 8) / 9, chunks = (p.C + 15) / 16 * groups;
    uint8_t *const parts = static_cast<uint8_t *>(out);
    HalvesChunk *const table = reinterpret_cast<HalvesChunk *>(parts + (size_t)p.tilesM * (size_t)chunks * (size_t)(9 * 64 * 64));
    auto *const kernel = &igconv_split_filter_kernel;
    const float *w = static_cast<const float *>(p.w);
    int K = p.K, C = p.C, taps = p.RS, g = groups;
    uint32_t row_stride = (uint32_t)p.wsRow, channel_stride = (uint32_t)p.wsRed, w_bytes = p.w_bytes;
    uint8_t *o = parts;
    HalvesChunk *t = table;
    void *args[] = {&w, &o, &t, &K, &C, &taps, &g, &row_stride, &channel_stride, &w_bytes};
    return static_cast<int>(hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(chunks, p.tilesM), dim3(512), args, 0, static_cast<hipStream_t>(stream)));
}

template <class Cfg>
static int launch_f32h(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_f32h_kernel<Cfg>, "igconv_f32h_kernel", p, grid, Cfg::THREADS, stream);
}

//    name, BM, BN, WM, WN, patch pixels, channel-fastest tensors, patches in registers, one barrier per chunk
#define IGC_F32H_LIST(X) \
    X("f32 64x256x144 split patch halves", 64, 256, 1, 4, 640, false, 2, true) \
    X("f32 64x256x144 split patch halves swap", 64, 256, 1, 4, 640, true, 2, true) \
    X("f32 64x256x144 split patch halves, wide", 64, 256, 1, 4, 896, false, 2, false) \
    X("f32 64x256x144 split patch halves swap, wide", 64, 256, 1, 4, 896, true, 2, false) \
    X("f32 64x256x144 split patch halves, many taps", 64, 256, 1, 4, 896, false, 1, false) \
    X("f32 64x256x144 split patch halves swap, many taps", 64, 256, 1, 4, 896, true, 1, false)

#define IGC_F32H_INSTANTIATE(NAME, BM, BN, WM, WN, PIX, NHWC, SETS, WHOLE) \
    template __global__ void igconv_f32h_kernel<HalvesPatchConfig<BM, BN, WM, WN, PIX, NHWC, SETS, WHOLE>>(const ConvKernelParams);
IGC_F32H_LIST(IGC_F32H_INSTANTIATE)

#if !defined(__HIP_DEVICE_COMPILE__)
// (variants 7 and 8: operands as two binary16 parts, patch)
#define IGC_F32H_ROW(NAME, BM, BN, WM, WN, PIX, NHWC, SETS, WHOLE)                                            \
    {NAME, false, BM, BN, 144, NHWC, false, 3, 512, HalvesPatchConfig<BM, BN, WM, WN, PIX, NHWC, SETS, WHOLE>::LDS_BYTES, \
     &launch_f32h<HalvesPatchConfig<BM, BN, WM, WN, PIX, NHWC, SETS, WHOLE>>, SETS == 2 ? 7 : 8, false, PIX},
static const KernelInfo kRows[] = {IGC_F32H_LIST(IGC_F32H_ROW)};
const KernelGroup kGroupF32HalvesPatch = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#endif

}  // namespace igc
