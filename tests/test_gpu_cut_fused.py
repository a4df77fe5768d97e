"""A forward pass with bias and activation whose reduction is cut into ranges (few tiles, a lent workspace): the sum of
the ranges applies them."""
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
    # N, C, H, W, K, R, S, pad, stride
    (1, 256, 13, 13, 96, 3, 3, (1, 1), (1, 1)),      # results a multiple of four: vectors of four, up to 16 ranges
    (2, 512, 5, 5, 33, 5, 5, (2, 2), (1, 1)),        # 1650 results: one by one
    (1, 700, 1, 1, 7, 1, 1, (0, 0), (1, 1)),         # one pixel
    (3, 300, 9, 9, 1, 3, 3, (1, 1), (2, 2)),         # one map
])
def test_bias_and_activation(prob, layout):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    x, w = wl.random_problem(31, N, C, H, W, K, R, S)
    rng = np.random.default_rng(32)
    bias = rng.uniform(-1, 1, size=K).astype(np.float32)
    want = oc.conv_forward(x, w, pad=pad, stride=stride, mode=1)
    y0 = rng.uniform(-1, 1, size=want.shape).astype(np.float32)
    g = gu.GpuConv(x, w, pad, stride, 1, y_layout=layout)
    g.lend_workspace(6 * want.size * 4)
    b = bias[None, :, None, None]
    for act, fn in ((-1, lambda v: v), (0, lambda v: 1 / (1 + np.exp(-v))), (1, lambda v: np.maximum(v, 0)), (2, np.tanh)):
        print(prob, layout, act, flush=True)
        g.prefill(y0)
        g.launch_fused(0.5, -1.5, bias, act)
        got = g.result()
        g.ws.result()
        pre = 0.5 * want - 1.5 * y0 + b
        # (slopes of the activations are at most one; the float bound on the sums, a few units on the activation)
        assert np.abs(got - fn(pre)).max() <= gu.BOUND["f32"] * np.abs(want).max() + 2.0 ** -20
    g.prefill(y0)
    g.launch_fused(0.5, -1.5, None, 1)
    assert np.abs(g.result() - np.maximum(0.5 * want - 1.5 * y0, 0)).max() <= gu.BOUND["f32"] * np.abs(want).max() + 2.0 ** -20


@pytest.mark.parametrize("order", ["nkpq", "npqk", "knpq", "kpqn", "pqnk", "pkqn"])
@pytest.mark.parametrize("prob", [(2, 512, 5, 7, 36, 3, (1, 1)), (3, 300, 5, 5, 33, 3, (0, 1))])
def test_packed_orders_of_y(prob, order):
    """The map of an element follows from its place in y, whatever the order of the dimensions."""
    gu = _gpu()
    N, C, H, W, K, R, pad = prob
    x, w = wl.random_problem(33, N, C, H, W, K, R, R)
    rng = np.random.default_rng(34)
    bias = rng.uniform(-1, 1, size=K).astype(np.float32)
    want = oc.conv_forward(x, w, pad=pad, mode=1)
    y0 = rng.uniform(-1, 1, size=want.shape).astype(np.float32)
    sizes, strides, step = dict(zip("nkpq", want.shape)), {}, 1
    for d in reversed(order):
        strides[d], step = step, step * sizes[d]
    g = gu.GpuConv(x, w, pad, (1, 1), 1, y_strides=tuple(strides[d] for d in "nkpq"))
    print(prob, order, flush=True)
    plain = np.empty(0)
    for lent in (0, 4 * want.size * 4):
        if lent:
            g.lend_workspace(lent)
        g.prefill(y0)
        g.launch_fused(0.5, -1.5, bias, 2)
        got = g.result()
        assert np.abs(got - np.tanh(0.5 * want - 1.5 * y0 + bias[None, :, None, None])).max() <= gu.BOUND["f32"] * np.abs(want).max() + 2.0 ** -20
        plain = got if not lent else plain
    assert plain.size and not np.array_equal(got, plain)   # (the sums of the ranges round otherwise: the cut took place)
