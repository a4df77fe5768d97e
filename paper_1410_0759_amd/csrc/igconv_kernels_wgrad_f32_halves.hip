// fp32 backward-filter kernels on the 16-bit matrix pipes, every operand as two binary16 parts (igconv_kernel_wgrad_f32h.hpp,
// igconv_kernel_wgrad_f32h_rows.hpp).
#include "igconv_kernel_wgrad_f32h_rows.hpp"

namespace igc {

template <class Cfg>
static int launch_wgrad_f32h(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_wgrad_f32h_kernel<Cfg>, "igconv_wgrad_f32h_kernel", p, grid, Cfg::THREADS, stream);
}

template <class Cfg>
static int launch_wgrad_f32h_rows(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_wgrad_f32h_rows_kernel<Cfg>, "igconv_wgrad_f32h_rows_kernel", p, grid, Cfg::THREADS, stream);
}

// Parts of the kernels of variant 10 added up in order - eight runs of consecutive parts, as igconv_sum_parts_kernel - while the sums
// move to dw.  Four maps per thread.
__global__ __launch_bounds__(256) void igconv_sum_rows_kernel(const float4 *parts, float *out, WgradRowsPart part, int count, float alpha, float beta) {
    __shared__ float4 runs[8][32];
    const uint32_t el = threadIdx.x & 31u, g = threadIdx.x >> 5;
    const uint32_t e = blockIdx.x * 32u + el, stride = (uint32_t)part.tiles * (WgradRowsPart::kTileElems / 4);   // (a whole number of blocks)
    const int per = (count + 7) / 8, s0 = (int)g * per, s1 = min(count, s0 + per);
    float4 acc = {0.f, 0.f, 0.f, 0.f};
    auto add = [](float4 &a, const float4 &b) {
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
    };
    const float4 *src = parts + e;
    int s = s0;
    for (; s + 4 <= s1; s += 4) {
        const float4 a = src[(size_t)s * stride], b = src[(size_t)(s + 1) * stride], c = src[(size_t)(s + 2) * stride], d = src[(size_t)(s + 3) * stride];
        add(acc, a);
        add(acc, b);
        add(acc, c);
        add(acc, d);
    }
    for (; s < s1; ++s) add(acc, src[(size_t)s * stride]);
    runs[g][el] = acc;
    __syncthreads();
    if (g != 0) return;
    float4 sum = runs[0][el];
#pragma unroll
    for (int k = 1; k < 8; ++k) add(sum, runs[k][el]);
    // where they stand (igconv_kernel_wgrad_f32h_rows.hpp)
    const int lane = (int)(e & 63u), block = (int)(e >> 6);
    const int v4 = block & 3, mb = (block >> 2) & 1, t = (block >> 3) % 3, wave = (block / 24) % 3, tile = block / 72;
    const int unit = tile / part.tilesM, m0 = (tile - unit * part.tilesM) * 64;
    const int rg = unit / part.cblocks, c0 = (unit - rg * part.cblocks) * 32, groups = (part.S + 2) / 3, gr = rg / groups;
    const int r_first = gr * 3, s_first = (rg - gr * groups) * 3;
    const int row = part.flip ? 2 - wave : wave, tap = part.flip ? 2 - t : t;
    const int r = (r_first < part.R - 3 ? r_first : part.R - 3) + row, sx = (s_first < part.S - 3 ? s_first : part.S - 3) + tap;
    bool ours;
    const int c = wgrad_row(c0, lane & 31, part.C, &ours);
    if (!ours || r < r_first || sx < s_first) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = wgrad_row(m0 + mb * 32, v4 * 8 + (lane >> 5) * 4 + i, part.K, &ours);
        if (!ours) continue;
        float *const at = out + ((size_t)(k * part.C + c) * (size_t)part.R + (size_t)r) * (size_t)part.S + (size_t)sx;
        float v = alpha * (i == 0 ? sum.x : (i == 1 ? sum.y : (i == 2 ? sum.z : sum.w)));
        if (beta != 0.f) v += beta * *at;
        *at = v;
    }
}

//    name, channel-fastest tensors
#define IGC_WGRAD_F32H_LIST(X) \
    X("f32 64x64x128 wgrad halves", false) \
    X("f32 64x64x128 wgrad halves, channels innermost", true)

#define IGC_WGRAD_F32H_INSTANTIATE(NAME, NHWC) \
    template __global__ void igconv_wgrad_f32h_kernel<WgradHalvesConfig<NHWC>>(const ConvKernelParams);
IGC_WGRAD_F32H_LIST(IGC_WGRAD_F32H_INSTANTIATE)
#define IGC_WGRAD_F32H_ROWS_LIST(X) \
    X("f32 64x32x128 wgrad halves, three filter rows", false) \
    X("f32 64x32x128 wgrad halves, three filter rows, channels innermost", true)
#define IGC_WGRAD_F32H_ROWS_INSTANTIATE(NAME, NHWC) \
    template __global__ void igconv_wgrad_f32h_rows_kernel<WgradHalvesRowsConfig<NHWC>>(const ConvKernelParams);
IGC_WGRAD_F32H_ROWS_LIST(IGC_WGRAD_F32H_ROWS_INSTANTIATE)

#if !defined(__HIP_DEVICE_COMPILE__)
int launch_sum_rows(const float *parts, float *out, const WgradRowsPart &part, int count, float alpha, float beta, void *stream) {
    WgradRowsPart copy = part;
    void *argv[] = {&parts, &out, &copy, &count, &alpha, &beta};
    return static_cast<int>(hipLaunchKernel(reinterpret_cast<const void *>(&igconv_sum_rows_kernel), dim3((uint32_t)part.tiles * (WgradRowsPart::kTileElems / 128)),
                                            dim3(256), argv, 0, static_cast<hipStream_t>(stream)));
}
// (variant 9: operands as two binary16 parts, three taps of a filter row per tile)
#define IGC_WGRAD_F32H_ROW(NAME, NHWC)                                                                                  \
    {NAME, false, 64, 64, 128, NHWC, false, GATHER_WGRAD_TAP, 512, WgradHalvesConfig<NHWC>::LDS_BYTES, \
     &launch_wgrad_f32h<WgradHalvesConfig<NHWC>>, 9},
// (variant 10: the same with three filter rows by three taps per tile)
#define IGC_WGRAD_F32H_ROWS_ROW(NAME, NHWC)                                                                             \
    {NAME, false, 64, 32, 128, NHWC, false, GATHER_WGRAD_TAP, 512, WgradHalvesRowsConfig<NHWC>::LDS_BYTES, \
     &launch_wgrad_f32h_rows<WgradHalvesRowsConfig<NHWC>>, 10},
static const KernelInfo kRows[] = {IGC_WGRAD_F32H_LIST(IGC_WGRAD_F32H_ROW) IGC_WGRAD_F32H_ROWS_LIST(IGC_WGRAD_F32H_ROWS_ROW)};
const KernelGroup kGroupWgradF32Halves = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#endif

}  // namespace igc
