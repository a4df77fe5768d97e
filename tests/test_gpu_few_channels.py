"""Float forward pass with a short reduction on the vector units (at most four channels, 3x3 or 5x5): every form of the
kernel - one or two pixels per thread, eight or sixteen maps - at sizes around its blocks, against the oracle."""
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


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, pad, stride
    (1, 1, 3, 3, 1, 3, (0, 0), (1, 1)),           # one result
    (1, 3, 17, 15, 9, 3, (1, 1), (1, 1)),         # 255 pixels, a second block of maps with one
    (2, 4, 16, 8, 16, 3, (2, 0), (1, 1)),
    (1, 2, 5, 9, 7, 5, (4, 4), (1, 2)),           # windows mostly in the border
    (3, 3, 21, 11, 33, 5, (0, 2), (3, 1)),
    (37, 1, 30, 31, 40, 5, (0, 0), (1, 1)),       # unpadded
    (21, 3, 97, 101, 33, 3, (1, 1), (1, 1)),      # two pixels and sixteen maps per thread
    (11, 3, 90, 70, 50, 5, (2, 2), (1, 1)),       # sixteen maps
    (6, 2, 150, 128, 5, 5, (2, 1), (1, 1)),
])
def test_forward(prob, layout):
    gu = _gpu()
    N, C, H, W, K, R, pad, stride = prob
    rng = np.random.default_rng(21)
    x = wl.with_layout(rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32), layout)
    w = (rng.standard_normal(size=(K, C, R, R)) * (C * R * R) ** -0.5).astype(np.float32)
    bias = rng.uniform(-1, 1, size=K).astype(np.float32)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, R, stride[1], pad[1])
    y0 = rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32)
    # a chain of n fused multiply-adds: n roundings of at most half a unit of the sum of magnitudes
    magnitude = oc.conv_forward(np.abs(x), np.abs(w), pad=pad, stride=stride)
    bound = (C * R * R + 4) * 2.0 ** -24
    for mode in (0, 1):
        print(prob, layout, mode, flush=True)
        want = oc.conv_forward(x, w, pad=pad, stride=stride, mode=mode)
        g = gu.GpuConv(x, w, pad, stride, mode, y_layout=layout)
        g.prefill(value=float("nan"))
        g.launch(1.0, 0.0)
        got = g.result()
        mag = magnitude if mode == 0 else oc.conv_forward(np.abs(x), np.abs(w), pad=pad, stride=stride, mode=1)
        assert np.all(np.abs(got - want) <= bound * mag + 1e-37)
        g.prefill(y0)
        g.launch(0.5, -1.5)
        assert np.all(np.abs(g.result() - (0.5 * want - 1.5 * y0)) <= bound * mag + 2.0 ** -21)
        for act, fn in ((0, lambda v: 1 / (1 + np.exp(-v))), (1, lambda v: np.maximum(v, 0)), (2, np.tanh)):
            g.prefill(value=float("nan"))
            g.launch_fused(1.0, 0.0, bias, act)
            assert np.all(np.abs(g.result() - fn(want + bias[None, :, None, None])) <= bound * mag + 2.0 ** -21)
