"""The bf16 kernels that read channel vectors of both operands, the filter rewritten with the channel index innermost:
same bits as the element-wise kernels that read the filter in place (no workspace), both against the oracle."""
import numpy as np
import pytest

from oracle import conv_oracle as oc
import workloads as wl

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _rnd(rng, shape, scale=1.0):
    return wl.round_to_bf16((rng.uniform(-1, 1, size=shape) * scale).astype(np.float32))


@pytest.mark.parametrize("layout", ["NHWC", "NCHW"])     # of dx; dy has its channels innermost
@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, S, pad, stride
    (3, 70, 15, 18, 40, 3, 3, (1, 1), (2, 2)),        # phases of four, two, two and one taps, a ragged last unit of channels
    (2, 130, 9, 10, 64, 1, 1, (0, 0), (2, 2)),        # phases without taps
    (2, 33, 14, 13, 8, 5, 5, (2, 2), (1, 1)),         # one unit per tap, most of it past the channels
    (1, 64, 12, 9, 136, 7, 2, (3, 0), (3, 1)),
    (2, 64, 8, 8, 72, 5, 3, (4, 2), (1, 1)),          # "full" border
])
def test_backward_data(prob, layout):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(3)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    dy = wl.with_layout(_rnd(rng, (N, K, P, Q)), "NHWC")
    w = _rnd(rng, (K, C, R, S), (K * R * S) ** -0.5)
    dx0 = rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32)
    for mode, alpha, beta in ((0, 1.0, 0.0), (1, 0.5, -1.5), (0, 1.0, 1.0)):
        print(prob, layout, mode, beta, flush=True)
        old = dx0 if beta else None
        want = oc.conv_backward_data(dy, w, (H, W), pad=pad, stride=stride, mode=mode, alpha=alpha, beta=beta, dx_old=old)
        got = gu.run_backward_data(dy, w, (H, W), pad, stride, mode, alpha, beta, old, "bf16", layout)
        assert gu.rel_err(got, want) <= gu.BOUND["bf16"]
        assert np.array_equal(got, gu.run_backward_data(dy, w, (H, W), pad, stride, mode, alpha, beta, old, "bf16", layout, workspace="none"))


@pytest.mark.parametrize("layout", ["NHWC", "NCHW"])     # of y
@pytest.mark.parametrize("prob", [
    (16, 72, 20, 20, 150, 5, 5, (2, 2), (1, 1)),
    (64, 64, 21, 19, 70, 7, 3, (3, 1), (2, 1)),
])
def test_forward(prob, layout):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(4)
    x, w = wl.with_layout(_rnd(rng, (N, C, H, W)), "NHWC"), _rnd(rng, (K, C, R, S), (C * R * S) ** -0.5)
    for mode in (0, 1):
        want = oc.conv_forward(x, w, pad=pad, stride=stride, mode=mode)
        g = gu.GpuConv(x, w, pad, stride, mode, dtype="bf16", y_layout=layout)
        assert g.plan().gatherMode == 1
        g.prefill(value=float("nan"))
        g.launch(1.0, 0.0)
        plain = g.result()
        assert g.lend_workspace() == w.size * 2
        print(prob, layout, mode, flush=True)
        g.prefill(value=float("nan"))
        g.launch(1.0, 0.0)
        got = g.result()
        g.ws.result()
        assert gu.rel_err(got, want) <= gu.BOUND["bf16"] and np.array_equal(got, plain)
        bias = rng.uniform(-1, 1, size=K).astype(np.float32)
        g.prefill(value=float("nan"))
        g.launch_fused(1.0, 0.0, bias, 1)
        assert gu.rel_err(g.result(), np.maximum(want + bias[None, :, None, None], 0.0)) <= gu.BOUND["bf16"]


@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, S, pad, stride: a small gradient in more than eight ranges, summed by the kernel that cuts the ranges into runs
    (24, 40, 28, 28, 72, 1, 1, (0, 0), (1, 1)),
    (16, 136, 20, 20, 8, 2, 2, (1, 0), (1, 1)),
    (40, 64, 30, 29, 24, 3, 1, (1, 0), (2, 1)),
])
def test_backward_filter_many_ranges(prob):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(5)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    x = wl.with_layout(_rnd(rng, (N, C, H, W)), "NHWC")
    dy = wl.with_layout(_rnd(rng, (N, K, P, Q)), "NHWC")
    dw0 = rng.uniform(-1, 1, size=(K, C, R, S)).astype(np.float32)
    for mode, alpha, beta in ((0, 1.0, 0.0), (1, 0.5, -1.5)):
        print(prob, mode, flush=True)
        want = oc.conv_backward_filter(x, dy, (R, S), pad=pad, stride=stride, mode=mode, alpha=alpha, beta=beta, dw_old=dw0 if beta else None)
        got, ws_bytes = gu.run_backward_filter(x, dy, (R, S), pad, stride, mode, alpha, beta, dw0 if beta else None, "bf16")
        assert ws_bytes > 8 * dw0.size * 4
        # (products of bfloat16 numbers are exact; sums of N*P*Q of them in float)
        assert gu.rel_err(got, want) <= gu.BOUND["bf16"]


@pytest.mark.parametrize("layout", ["NHWC", "NCHW"])     # of y
@pytest.mark.parametrize("prob", [
    # nine taps that no staged patch holds, more tiles than compute units (of which the handle is told 8)
    (16, 48, 32, 45, 70, 3, 3, (1, 1), (2, 2)),       # ragged rows and columns, half a unit of channels
    (40, 64, 29, 30, 136, 3, 3, (0, 1), (2, 2)),
    (24, 96, 40, 33, 24, 9, 1, (4, 0), (3, 2)),
])
def test_forward_nine_taps(prob, layout):
    import paper_1410_0759_amd as ig
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(6)
    x, w = wl.with_layout(_rnd(rng, (N, C, H, W)), "NHWC"), _rnd(rng, (K, C, R, S), (C * R * S) ** -0.5)
    bias = rng.uniform(-1, 1, size=K).astype(np.float32)
    for mode in (0, 1):
        print(prob, layout, mode, flush=True)
        want = oc.conv_forward(x, w, pad=pad, stride=stride, mode=mode)
        y0 = rng.uniform(-1, 1, size=want.shape).astype(np.float32)
        res = []
        for lent in (0, w.size * 2 - 2, w.size * 2):
            g = gu.GpuConv(x, w, pad, stride, mode, dtype="bf16", y_layout=layout)
            ig.set_compute_units(g.handle, 8)
            assert g.plan().gatherMode == 4
            if lent:
                g.lend_workspace(lent)
            g.prefill(y0, float("nan"))
            g.launch_fused(0.5, -1.5, bias, 1)
            res.append(g.result())
            if lent:
                g.ws.result()   # (guard bands)
            assert gu.rel_err(res[-1], np.maximum(0.5 * want - 1.5 * y0 + bias[None, :, None, None], 0.0)) <= gu.BOUND["bf16"]
        assert np.array_equal(res[0], res[1]) and not np.array_equal(res[0], res[2]), "the route under test did not run"


@pytest.mark.parametrize("layout", ["NHWC", "NCHW"])     # of dx
@pytest.mark.parametrize("prob", [
    # the 128 x 256 tile (the handle is told of 8 compute units), several tiles per workgroup
    (40, 130, 30, 31, 72, 5, 5, (2, 2), (1, 1)),      # ragged rows and columns, a ragged last unit of channels
    (33, 256, 17, 16, 160, 3, 2, (1, 1), (1, 1)),     # thirty steps per tile
    (16, 250, 32, 30, 520, 3, 3, (1, 1), (2, 2)),      # four stride phases, the last of one tap, in one launch
])
def test_backward_data_large_tiles(prob, layout):
    """(csrc/host_check.cpp requires that these layers take the large tile with 8 compute units, a smaller one with 256.)"""
    import torch
    import paper_1410_0759_amd as ig
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(7)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    dy, w = wl.with_layout(_rnd(rng, (N, K, P, Q)), "NHWC"), _rnd(rng, (K, C, R, S), (K * R * S) ** -0.5)
    want = oc.conv_backward_data(dy, w, (H, W), pad=pad, stride=stride)
    t = lambda a, lay: torch.from_numpy(np.ascontiguousarray(a)).to("cuda") if lay == "NCHW" else \
        torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 3, 1))).to("cuda").permute(0, 3, 1, 2)
    dyt, wt = t(dy, "NHWC").to(torch.bfloat16), t(w, "NCHW").to(torch.bfloat16)
    res = []
    for cus in (8, 256):
        h = ig.Handle()
        h.set_stream(torch.cuda.current_stream().cuda_stream)
        ig.set_compute_units(h, cus)
        dx = t(np.full((N, C, H, W), np.nan, np.float32), layout)
        wd = ig.FilterDescriptor().set(ig.IGC_DATA_BFLOAT16, K, C, R, S)
        cd = ig.ConvolutionDescriptor().set(pad[0], pad[1], stride[0], stride[1], ig.IGC_CROSS_CORRELATION)
        dyd, dxd = ig.tensor_descriptor_for(dyt), ig.tensor_descriptor_for(dx)
        n = ig.get_backward_data_workspace_size(h, wd, dyd, cd, dxd)
        assert n == w.size * 2
        ws = torch.empty(n // 4 + 4, device="cuda")
        print(prob, layout, cus, flush=True)
        ig.check(ig.convolution_backward_data(h, 1.0, wd, wt.data_ptr(), dyd, dyt.data_ptr(), cd, 0.0, dxd, dx.data_ptr(), ws.data_ptr(), n))
        res.append(dx.cpu().numpy())
        assert gu.rel_err(res[-1], want) <= gu.BOUND["bf16"]
    assert np.array_equal(res[0], res[1])      # (the same order of the sums in every tile)
