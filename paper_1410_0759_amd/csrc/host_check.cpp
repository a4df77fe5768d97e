// Driver for a build of the library's host tier (igconv_api.cpp: descriptors, validation, kernel choice, launch
// plans, workspace sizes, the address-reach check) under AddressSanitizer and UndefinedBehaviorSanitizer.  Runs
// without a GPU: it calls only entry points that end before the first launch - queries over a few thousand random
// layers in all three data types and both layouts, and every pass with null data pointers or contradictory
// descriptors, which must be refused.  A sanitizer report aborts the run; a wrong status code or a reach beyond an
// extent fails it.  Prints "host check ok".
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "igconv_api.cpp"   // (with what is internal to it: the choice of a kernel for lent space cannot be queried)

static unsigned long long state = 14100759ull;
static int draw(int lo, int hi) {   // uniform in lo..hi
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return (int)(lo + (long long)((state >> 33) % (unsigned long long)((long long)hi - lo + 1)));
}

#define REQUIRE(cond)                                                                  \
    do {                                                                               \
        if (!(cond)) {                                                                 \
            std::fprintf(stderr, "host check failed at line %d: %s (case %d)\n", __LINE__, #cond, it); \
            return 1;                                                                  \
        }                                                                              \
    } while (0)

int main() {
    igcHandle_t h = nullptr;
    int it = -1;
    REQUIRE(igcCreate(&h) == IGC_STATUS_SUCCESS);
    igcTensorDescriptor_t x, y, dx;
    igcFilterDescriptor_t w;
    igcConvolutionDescriptor_t c;
    REQUIRE(igcCreateTensorDescriptor(&x) == IGC_STATUS_SUCCESS && igcCreateTensorDescriptor(&y) == IGC_STATUS_SUCCESS &&
            igcCreateTensorDescriptor(&dx) == IGC_STATUS_SUCCESS && igcCreateFilterDescriptor(&w) == IGC_STATUS_SUCCESS &&
            igcCreateConvolutionDescriptor(&c) == IGC_STATUS_SUCCESS);
    const igcDataType types[3] = {IGC_DATA_FLOAT, IGC_DATA_BFLOAT16, IGC_DATA_DOUBLE};
    long long plans = 0;
    for (it = 0; it < 3000; ++it) {
        const bool big = it % 50 == 0;   // now and then a layer of realistic size
        const int N = big ? draw(16, 256) : draw(1, 5), C = big ? draw(3, 512) : draw(1, 70), K = big ? draw(16, 512) : draw(1, 200);
        const int R = draw(1, 11), S = draw(1, 11);
        const int pad_h = draw(0, R - 1), pad_w = draw(0, S - 1), u = draw(1, 4), v = draw(1, 4);
        const int H = draw(R > 2 * pad_h ? R - 2 * pad_h : 1, big ? 230 : 40), W = draw(S > 2 * pad_w ? S - 2 * pad_w : 1, big ? 230 : 40);
        const igcDataType dt = types[it % 3], odt = dt == IGC_DATA_DOUBLE ? IGC_DATA_DOUBLE : IGC_DATA_FLOAT;
        const bool nhwc = (it / 3) % 2 == 1;
        if (it % 97 == 0) REQUIRE(igcSetComputeUnits(h, draw(8, 400)) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetTensor4dDescriptor(x, dt, N, C, H, W, nhwc ? (long long)H * W * C : (long long)C * H * W, nhwc ? 1 : (long long)H * W,
                                         nhwc ? (long long)W * C : W, nhwc ? C : 1) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetTensor4dDescriptor(dx, odt, N, C, H, W, nhwc ? (long long)H * W * C : (long long)C * H * W, nhwc ? 1 : (long long)H * W,
                                         nhwc ? (long long)W * C : W, nhwc ? C : 1) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetFilter4dDescriptor(w, dt, K, C, R, S) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetConvolution2dDescriptor(c, pad_h, pad_w, u, v, it % 2 ? IGC_CONVOLUTION : IGC_CROSS_CORRELATION) == IGC_STATUS_SUCCESS);
        int n, k, p, q;
        REQUIRE(igcGetConvolution2dForwardOutputDim(c, x, w, &n, &k, &p, &q) == IGC_STATUS_SUCCESS);
        REQUIRE(n == N && k == K && p >= 1 && q >= 1);
        REQUIRE(igcSetTensor4dDescriptor(y, odt, n, k, p, q, nhwc ? (long long)p * q * k : (long long)k * p * q, nhwc ? 1 : (long long)p * q,
                                         nhwc ? (long long)q * k : q, nhwc ? k : 1) == IGC_STATUS_SUCCESS);
        igcConvolutionForwardPlan plan;
        const igcStatus st = igcGetConvolutionForwardPlan(h, x, w, c, y, &plan);
        REQUIRE(st == IGC_STATUS_SUCCESS || st == IGC_STATUS_NOT_SUPPORTED);
        if (st != IGC_STATUS_SUCCESS) continue;   // (extents of 2 GiB and more)
        ++plans;
        REQUIRE(plan.kernelId >= 0 && plan.kernelId < igcGetKernelCount() && igcGetKernelName(plan.kernelId) != nullptr);
        REQUIRE(plan.gridX >= 8 && plan.gridX % 8 == 0 && plan.threads % 64 == 0 && plan.ldsBytes <= 160 * 1024);
        size_t ws = 1, opt = 0;
        REQUIRE(igcGetConvolutionForwardWorkspaceSize(h, x, w, c, y, &ws) == IGC_STATUS_SUCCESS && ws == 0);
        REQUIRE(igcGetConvolutionForwardOptionalWorkspaceSize(h, x, w, c, y, &opt) == IGC_STATUS_SUCCESS);
        long long reach[3], extent[3];
        REQUIRE(igcGetConvolutionForwardAddressReach(h, x, w, c, y, reach, extent) == IGC_STATUS_SUCCESS);
        for (int i = 0; i < 3; ++i) REQUIRE(reach[i] > 0 && reach[i] <= extent[i] && extent[i] < (1ll << 31));
        // backward data and backward filter of the same layer (dy takes the inputs' type, dx / dw the output rule)
        igcTensorDescriptor_t dy = y;
        if (dt == IGC_DATA_BFLOAT16) {
            REQUIRE(igcCreateTensorDescriptor(&dy) == IGC_STATUS_SUCCESS);
            REQUIRE(igcSetTensor4dDescriptor(dy, dt, n, k, p, q, nhwc ? (long long)p * q * k : (long long)k * p * q, nhwc ? 1 : (long long)p * q,
                                             nhwc ? (long long)q * k : q, nhwc ? k : 1) == IGC_STATUS_SUCCESS);
        }
        size_t bd = 0, bf = 0;
        // (a float dx for bfloat16 inputs is twice the size of x: it may pass 2 GiB where x did not)
        const igcStatus sbd = igcGetConvolutionBackwardDataWorkspaceSize(h, w, dy, c, dx, &bd);
        REQUIRE(sbd == IGC_STATUS_SUCCESS || (sbd == IGC_STATUS_NOT_SUPPORTED && dt == IGC_DATA_BFLOAT16));
        if (sbd == IGC_STATUS_SUCCESS) {
            REQUIRE(igcGetConvolutionBackwardDataAddressReach(h, w, dy, c, dx, reach, extent) == IGC_STATUS_SUCCESS);
            for (int i = 0; i < 3; ++i) REQUIRE(reach[i] > 0 && reach[i] <= extent[i] && extent[i] < (1ll << 31));
        }
        igcFilterDescriptor_t dw = w;
        if (dt == IGC_DATA_BFLOAT16) {
            REQUIRE(igcCreateFilterDescriptor(&dw) == IGC_STATUS_SUCCESS);
            REQUIRE(igcSetFilter4dDescriptor(dw, IGC_DATA_FLOAT, K, C, R, S) == IGC_STATUS_SUCCESS);
        }
        const igcStatus sbf = igcGetConvolutionBackwardFilterWorkspaceSize(h, x, dy, c, dw, &bf);
        REQUIRE(sbf == IGC_STATUS_SUCCESS || (sbf == IGC_STATUS_NOT_SUPPORTED && dt == IGC_DATA_BFLOAT16));
        // every pass refuses null data pointers before anything else happens
        const float one = 1.f, zero = 0.f;
        const double one64 = 1.0, zero64 = 0.0;
        const void *al = dt == IGC_DATA_DOUBLE ? (const void *)&one64 : (const void *)&one;
        const void *be = dt == IGC_DATA_DOUBLE ? (const void *)&zero64 : (const void *)&zero;
        REQUIRE(igcConvolutionForward(h, al, x, nullptr, w, nullptr, c, nullptr, 0, be, y, nullptr) == IGC_STATUS_BAD_PARAM);
        REQUIRE(igcConvolutionBackwardData(h, al, w, nullptr, dy, nullptr, c, nullptr, 0, be, dx, nullptr) == IGC_STATUS_BAD_PARAM);
        REQUIRE(igcConvolutionBackwardFilter(h, al, x, nullptr, dy, nullptr, c, nullptr, 0, be, dw, nullptr) == IGC_STATUS_BAD_PARAM);
        // a y of the wrong size is refused by every query
        if (p > 1) {
            REQUIRE(igcSetTensor4dDescriptor(y, odt, n, k, p - 1, q, (long long)k * (p - 1) * q, (long long)(p - 1) * q, q, 1) == IGC_STATUS_SUCCESS);
            REQUIRE(igcGetConvolutionForwardPlan(h, x, w, c, y, &plan) == IGC_STATUS_BAD_PARAM);
        }
        if (dy != y) REQUIRE(igcDestroyTensorDescriptor(dy) == IGC_STATUS_SUCCESS);
        if (dw != w) REQUIRE(igcDestroyFilterDescriptor(dw) == IGC_STATUS_SUCCESS);
    }
    it = -2;
    REQUIRE(plans > 2500);
    // the division by multiply and shift, over divisors and numerators up to 2^31 - 1
    for (it = 0; it < 200000; ++it) {
        const unsigned d = (unsigned)draw(1, it % 2 ? 1 << 16 : 0x7fffffff), nn = (unsigned)draw(0, 0x7fffffff);
        unsigned mul = 0, shift = 0;
        REQUIRE(igcMagicDivisor(d, &mul, &shift) == IGC_STATUS_SUCCESS);
        REQUIRE(igcMagicDivide(nn, mul, shift) == nn / d);
    }
    // offsets of the few-channel epilogue, by the hardware's rule (vector offset against "size - scalar offset", modulo
    // 2^32): a map that exists is stored at its place, one that pads K to whole blocks of 8 or 16 nowhere
    for (it = 0; it < 200000; ++it) {
        const int K = draw(1, 70), block = it % 2 ? 8 : 16, N = draw(1, 3), PQ = draw(1, it % 5 ? 500 : 200000);
        const bool nhwc = it % 3 == 0;
        const unsigned ysK = nhwc ? 1u : (unsigned)PQ, ysN = (unsigned)K * (unsigned)PQ, size = ysN * (unsigned)N * 4u;
        for (int map = 0; map < (K + block - 1) / block * block; ++map) {
            const unsigned so = igc::few_channels_map_offset(map, K, ysK * 4u);
            REQUIRE(so <= size);
            REQUIRE(0x80000000u >= size - so);
            const unsigned last = ((unsigned)(N - 1) * ysN + (unsigned)(PQ - 1) * (nhwc ? (unsigned)K : 1u)) * 4u;   // the last pixel
            if (map < K) REQUIRE(last < size - so && so == (unsigned)map * ysK * 4u);
        }
    }
    // The split filter of the two-part float kernels is addressed with 32 bits and may be many times the filter: lent any room,
    // layers whose split filter is too large run elsewhere, those below it as before
    REQUIRE(igcSetComputeUnits(h, 256) == IGC_STATUS_SUCCESS);
    struct { int N, C, H, W, K, R, S, pad_h, pad_w; bool taken; } const rooms[] = {
        {359, 103570, 1, 1, 513, 2, 5, 1, 4, false},     // 2.1 GB of filter, 4.3 GB split
        {448, 116600, 1, 1, 449, 2, 5, 1, 4, false},
        {280, 1870000, 1, 1, 8, 3, 3, 2, 2, false},      // 0.5 GB, 4.3 GB
        {359, 52000, 1, 1, 513, 2, 5, 1, 4, false},      // 2.16 GB split: more than 2 GiB, less than 4
        {359, 50000, 1, 1, 513, 2, 5, 1, 4, true},       // 2.07 GB: less than 2 GiB
        {128, 64, 56, 56, 64, 3, 3, 1, 1, true}};
    for (it = 0; it < 6; ++it) {
        const auto &r = rooms[it];
        const int P = r.H + 2 * r.pad_h - r.R + 1, Q = r.W + 2 * r.pad_w - r.S + 1;
        REQUIRE(igcSetTensor4dDescriptor(x, IGC_DATA_FLOAT, r.N, r.C, r.H, r.W, (long long)r.C * r.H * r.W, r.H * r.W, r.W, 1) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetFilter4dDescriptor(w, IGC_DATA_FLOAT, r.K, r.C, r.R, r.S) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetConvolution2dDescriptor(c, r.pad_h, r.pad_w, 1, 1, IGC_CROSS_CORRELATION) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetTensor4dDescriptor(y, IGC_DATA_FLOAT, r.N, r.K, P, Q, (long long)r.K * P * Q, P * Q, Q, 1) == IGC_STATUS_SUCCESS);
        igc::Problem pr;
        REQUIRE(igc::validate(x, w, c, y, &pr) == IGC_STATUS_SUCCESS);
        pr.halves_room = (size_t)1 << 40;
        int id = -1;
        REQUIRE(igc::choose(h, pr, true, true, &id) == IGC_STATUS_SUCCESS);
        REQUIRE(igc::is_halves(*igc::kernel_info(id)) == r.taken);
    }
    // Backward filter, float: two binary16 parts of three filter rows per tile stand in for those of one row alone, never for the kernels that hold 24
    // bits of an operand; the query reports room for them where they run with it.  (kernel: variant with the room asked for, and with 64 MB more)
    struct { int N, C, H, W, K, R, S, pad, kernel, with_more; bool innermost; } const filters[] = {
        {23, 320, 14, 14, 144, 5, 5, 2, 4, 4, false}, {28, 64, 28, 28, 384, 3, 3, 0, 4, 4, false}, {24, 114, 37, 37, 50, 9, 9, 0, 4, 4, false},
        {13, 336, 18, 18, 112, 9, 9, 4, 4, 4, false}, {64, 256, 14, 14, 256, 3, 3, 1, 4, 4, false}, {34, 91, 45, 45, 11, 3, 3, 0, 4, 4, false},
        {89, 50, 16, 16, 11, 3, 3, 1, 0, 0, false}, {19, 312, 16, 16, 55, 3, 3, 1, 0, 0, false},
        {128, 64, 56, 56, 64, 3, 3, 1, 10, 10, false}, {128, 384, 13, 13, 256, 3, 3, 1, 10, 10, false}, {128, 96, 64, 64, 128, 9, 9, 0, 10, 10, false},
        {128, 64, 56, 56, 64, 3, 3, 1, 10, 10, true}};
    for (it = 0; it < 12; ++it) {
        const auto &r = filters[it];
        const int P = r.H + 2 * r.pad - r.R + 1, Q = r.W + 2 * r.pad - r.S + 1;
        auto set = [&](igcTensorDescriptor_t d, long long cc, long long hh, long long ww) {
            return igcSetTensor4dDescriptor(d, IGC_DATA_FLOAT, r.N, (int)cc, (int)hh, (int)ww, cc * hh * ww, r.innermost ? 1 : hh * ww, r.innermost ? ww * cc : ww, r.innermost ? cc : 1);
        };
        REQUIRE(set(x, r.C, r.H, r.W) == IGC_STATUS_SUCCESS && set(y, r.K, P, Q) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetFilter4dDescriptor(w, IGC_DATA_FLOAT, r.K, r.C, r.R, r.S) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetConvolution2dDescriptor(c, r.pad, r.pad, 1, 1, IGC_CROSS_CORRELATION) == IGC_STATUS_SUCCESS);
        size_t asked = 0;
        REQUIRE(igcGetConvolutionBackwardFilterWorkspaceSize(h, x, y, c, w, &asked) == IGC_STATUS_SUCCESS && asked <= (size_t)IGC_NOALLOC_SCRATCH_BYTES);
        for (size_t more : {(size_t)0, (size_t)64 << 20}) {
            igc::BackwardFilterProblem b;
            REQUIRE(igc::validate_backward_filter(x, y, c, w, &b) == IGC_STATUS_SUCCESS);
            igc::halves_backward_filter(h, &b, (long long)(asked + more), true);
            REQUIRE(igc::kernel_info(b.kernel_id)->variant == (more ? r.with_more : r.kernel));
        }
    }
    // ... and only where they count the pixels of the images with their borders in 31 bits (an image and its gradients, repeated by a stride of zero)
    for (it = 0; it < 2; ++it) {
        const int N = it ? 9200000 : 8000000;
        REQUIRE(igcSetTensor4dDescriptor(x, IGC_DATA_FLOAT, N, 128, 2, 58, 0, 116, 58, 1) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetTensor4dDescriptor(y, IGC_DATA_FLOAT, N, 512, 2, 58, 0, 116, 58, 1) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetFilter4dDescriptor(w, IGC_DATA_FLOAT, 512, 128, 3, 3) == IGC_STATUS_SUCCESS);
        REQUIRE(igcSetConvolution2dDescriptor(c, 1, 1, 1, 1, IGC_CROSS_CORRELATION) == IGC_STATUS_SUCCESS);
        igc::BackwardFilterProblem b;
        REQUIRE(igc::validate_backward_filter(x, y, c, w, &b) == IGC_STATUS_SUCCESS);
        igc::halves_backward_filter(h, &b, (long long)64 << 20, true);
        const igc::KernelInfo &ki = *igc::kernel_info(b.kernel_id);
        REQUIRE(ki.variant == (it ? 9 : 10));
        REQUIRE((long long)N * b.pr.kp.HpWp * b.pr.kp.Wp < (1ll << 31));
    }
    // Which kernels the layers of tests take that compare results alone.  (halved: tiles of an XCD's range that go as two halves)
    auto set_layer = [&](igcDataType in, bool innermost, int N, int C, int H, int W, int K, int R, int S, int pad_h, int pad_w, int stride) {
        const int P = (H + 2 * pad_h - R) / stride + 1, Q = (W + 2 * pad_w - S) / stride + 1;
        const igcDataType out = in == IGC_DATA_BFLOAT16 ? IGC_DATA_FLOAT : in;
        auto set = [&](igcTensorDescriptor_t d, igcDataType dt, bool last, long long cc, long long hh, long long ww) {
            return igcSetTensor4dDescriptor(d, dt, N, (int)cc, (int)hh, (int)ww, cc * hh * ww, last ? 1 : hh * ww, last ? ww * cc : ww, last ? cc : 1) == IGC_STATUS_SUCCESS;
        };
        // (16-bit gradients have their channels innermost)
        return set(x, in, innermost, C, H, W) && set(dx, out, innermost, C, H, W) && set(y, in, innermost || in == IGC_DATA_BFLOAT16, K, P, Q) &&
               igcSetFilter4dDescriptor(w, in, K, C, R, S) == IGC_STATUS_SUCCESS &&
               igcSetConvolution2dDescriptor(c, pad_h, pad_w, stride, stride, IGC_CROSS_CORRELATION) == IGC_STATUS_SUCCESS;
    };
    auto forward_kernel = [&](size_t halves_room, const igc::KernelInfo **ki) {   // tiles that go as halves
        igc::Problem pr;
        int id = -1;
        igcConvolutionForwardPlan plan;
        if (igc::validate(x, w, c, y, &pr) != IGC_STATUS_SUCCESS) return -1;
        pr.halves_room = halves_room;
        if (igc::choose(h, pr, true, true, &id) != IGC_STATUS_SUCCESS || igc::fill_plan(h, id, &pr, &plan) != IGC_STATUS_SUCCESS) return -1;
        *ki = igc::kernel_info(id);
        return (int)pr.kp.halvedPerXcd;
    };
    auto data_kernel = [&](bool filter_inner, size_t halves_room, const igc::KernelInfo **ki) {   // (of the phases that meet a tap: one kernel)
        igc::BackwardDataProblem b;
        std::vector<igc::PhaseLaunch> launches;
        if (igc::validate_backward_data(w, y, c, dx, &b) != IGC_STATUS_SUCCESS ||
            igc::plan_backward_data_phases(h, b, &launches, filter_inner, true, halves_room) != IGC_STATUS_SUCCESS) return -1;
        int halved = -1;
        for (const igc::PhaseLaunch &l : launches)
            if (!l.pr.zero_steps) {
                if (halved >= 0 && *ki != igc::kernel_info(l.id)) return -1;
                *ki = igc::kernel_info(l.id);
                halved = (int)l.pr.kp.halvedPerXcd;
            }
        return halved;
    };
    const igc::KernelInfo *ki = nullptr;
    for (it = 0; it < 12; ++it) {   // bfloat16 backward data: tiles of 128 x 256 on 8 compute units, smaller ones on 256 (test_backward_data_large_tiles)
        const int large[3][10] = {{40, 130, 30, 31, 72, 5, 5, 2, 2, 1}, {33, 256, 17, 16, 160, 3, 2, 1, 1, 1}, {16, 250, 32, 30, 520, 3, 3, 1, 1, 2}};
        const int *r = large[it / 4];
        REQUIRE(igcSetComputeUnits(h, it & 1 ? 256 : 8) == IGC_STATUS_SUCCESS);
        REQUIRE(set_layer(IGC_DATA_BFLOAT16, (it & 2) != 0, r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7], r[8], r[9]));
        REQUIRE(data_kernel(true, 0, &ki) >= 0);
        REQUIRE(ki->variant == 6 && ki->BN == (it & 1 ? 128 : 256));
    }
    for (it = 0; it < 6; ++it) {    // ... and not where a tile has few steps, alone or in one launch with other phases
        const int shorts[6][11] = {{41, 96, 56, 57, 256, 2, 2, 1, 1, 2, 128}, {68, 448, 32, 33, 64, 3, 3, 1, 1, 2, 128}, {66, 320, 28, 28, 208, 2, 2, 1, 1, 2, 128},
                                   {84, 416, 28, 28, 32, 3, 4, 1, 2, 1, 128}, {34, 224, 44, 44, 384, 2, 2, 0, 0, 2, 128},
                                   {128, 128, 28, 28, 256, 5, 5, 2, 2, 1, 256}};
        const int *r = shorts[it];
        REQUIRE(igcSetComputeUnits(h, 256) == IGC_STATUS_SUCCESS);
        REQUIRE(set_layer(IGC_DATA_BFLOAT16, true, r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7], r[8], r[9]));
        REQUIRE(data_kernel(true, 0, &ki) >= 0 && ki->variant == 6);
        REQUIRE(ki->BN == r[10]);
    }
    for (it = 0; it < 24; ++it) {   // double precision, forward and backward data (test_halved_tiles_f64)
        const int tiles[6][6] = {{3, 2, 75, 75, 10, 1}, {3, 2, 78, 78, 65, 8}, {5, 2, 70, 70, 64, 16}, {5, 2, 71, 71, 64, 0}, {15, 1, 66, 67, 9, 2}, {1, 3, 16, 97, 33, 4}};
        const int *r = tiles[it / 4];
        const bool data = it & 2;
        REQUIRE(igcSetComputeUnits(h, 256) == IGC_STATUS_SUCCESS);
        REQUIRE(set_layer(IGC_DATA_DOUBLE, it & 1, r[0], r[data ? 4 : 1], r[2], r[3], r[data ? 1 : 4], 3, 3, 1, 1, 1));
        REQUIRE((data ? data_kernel(false, 0, &ki) : forward_kernel(0, &ki)) == r[5]);
        REQUIRE(ki->f64 && ki->gmode == 14);
    }
    for (it = 0; it < 32; ++it) {   // float with more than nine taps, and the exchanged layer's backward data: one such tile on 16 compute units (test_halved_tiles)
        const int tiles[4][9] = {{4, 64, 15, 16, 96, 5, 5, 2, 2}, {7, 32, 20, 64, 40, 9, 9, 0, 0}, {17, 64, 1, 107, 60, 1, 21, 0, 10}, {16, 64, 12, 9, 130, 7, 2, 3, 1}};
        const int *r = tiles[it / 8];
        const bool data = it & 4;
        if (data && r[5] != r[6]) continue;
        REQUIRE(igcSetComputeUnits(h, it & 1 ? 16 : 8) == IGC_STATUS_SUCCESS);
        REQUIRE(set_layer(IGC_DATA_FLOAT, (it & 2) != 0, r[0], r[data ? 4 : 1], r[2], r[3], r[data ? 1 : 4], r[5], r[6], r[7], r[8], 1));
        REQUIRE((data ? data_kernel(false, (size_t)1 << 26, &ki) : forward_kernel((size_t)1 << 26, &ki)) == (it & 1));
        REQUIRE(ki->variant == 8);
    }
    for (it = 0; it < 2; ++it) {    // the same, three on 48 (test_a_half_tile_reads_its_own_columns)
        REQUIRE(igcSetComputeUnits(h, 48) == IGC_STATUS_SUCCESS);
        REQUIRE(set_layer(IGC_DATA_FLOAT, it, 8, 32, 20, 64, 40, 9, 9, 0, 0, 1));
        REQUIRE(forward_kernel((size_t)1 << 26, &ki) == 3 && ki->variant == 8);
    }
    for (it = 0; it < 12; ++it) {   // float, one tap, backward data: three parts from 32 maps on, where tiles are enough (test_backward_data_of_one_tap)
        const int taps[6][8] = {{40, 100, 31, 33, 31, 1, 0, 0}, {40, 100, 31, 33, 32, 1, 0, 4}, {40, 70, 31, 33, 33, 1, 0, 4},
                                {12, 300, 29, 31, 77, 1, 1, 4}, {24, 260, 41, 43, 65, 2, 0, 4}, {9, 40, 5, 7, 100, 1, 0, 0}};
        const int *r = taps[it / 2];
        REQUIRE(igcSetComputeUnits(h, 256) == IGC_STATUS_SUCCESS);
        REQUIRE(set_layer(IGC_DATA_FLOAT, it & 1, r[0], r[1], r[2], r[3], r[4], 1, 1, r[6], r[6], r[5]));
        REQUIRE(data_kernel(false, 0, &ki) >= 0 && ki->variant == r[7]);
    }
    it = -3;
    REQUIRE(igcDestroyTensorDescriptor(x) == IGC_STATUS_SUCCESS && igcDestroyTensorDescriptor(y) == IGC_STATUS_SUCCESS &&
            igcDestroyTensorDescriptor(dx) == IGC_STATUS_SUCCESS && igcDestroyFilterDescriptor(w) == IGC_STATUS_SUCCESS &&
            igcDestroyConvolutionDescriptor(c) == IGC_STATUS_SUCCESS && igcDestroy(h) == IGC_STATUS_SUCCESS);
    std::printf("host check ok (%lld plans)\n", plans);
    return 0;
}
