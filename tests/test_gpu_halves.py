"""The kernels that write float operands as two binary16 numbers, scaled chunk by chunk: forward pass and backward data with a
lent workspace of the split filter's size.  On a handle told of eight compute units small problems take that route, several
tiles to a workgroup."""
import numpy as np
import pytest

import paper_1410_0759_amd as ig
from oracle import conv_oracle as oc
import workloads as wl
from tests.test_gpu_split import SMALL, _check, _planted, _same, _scaled

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _bytes(K, C, taps):
    return -(-K // 64) * -(-C // 16) * -(-taps // 9) * (9 * 64 * 64 + 8)


def _forward(gu, x, w, pad, stride, mode, layout, lent, alpha=1.0, beta=0.0, y0=None, bias=None, act=-1, units=8):
    g = gu.GpuConv(wl.with_layout(x, layout) if layout else x, w, pad, stride, mode, y_layout=layout or "NCHW")
    if units:
        ig.set_compute_units(g.handle, units)
    if lent:
        g.lend_workspace(lent)
    g.prefill(y0, float("nan"))
    g.launch_fused(alpha, beta, bias, act)
    got = g.result()
    if lent:
        g.ws.result()   # (guard bands)
    return got


def _backward_data(gu, dy, w, hw, pad, mode, layout, lent, alpha=1.0, beta=0.0, dx0=None):
    g = gu.GpuBackwardData(wl.with_layout(dy, layout), w, hw, pad, (1, 1), mode, "f32", layout, lent or "none")
    ig.set_compute_units(g.handle, 8)
    if dx0 is not None:
        g.out.prefill(old=dx0)
    else:
        g.out.prefill(value=float("nan"))
    g.launch(alpha, beta)
    g.ws.result()   # (guard bands)
    return g.out.result()


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, S, pad, stride
    (17, 48, 14, 13, 70, 3, 3, (1, 1), (1, 1)),       # nine taps, a barrier per chunk; ragged rows and columns
    (16, 100, 30, 17, 64, 3, 3, (0, 2), (2, 1)),     # channels: no whole blocks of 16
    (23, 48, 9, 40, 33, 1, 9, (0, 4), (1, 2)),        # nine taps in a row
    (9, 64, 5, 300, 65, 3, 3, (1, 1), (1, 1)),       # the wide patch
    (3, 32, 20, 64, 40, 9, 9, (0, 0), (1, 1)),       # tiles per image (two images' windows lie too far apart)
    (4, 36, 15, 16, 96, 5, 5, (2, 2), (1, 1)),       # 25 taps: the last group shares two with the one before
    (20, 48, 7, 31, 20, 1, 11, (0, 5), (1, 1)),       # eleven: shares seven
    (12, 64, 12, 14, 130, 7, 2, (3, 1), (1, 2)),
])
def test_forward(prob, layout):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    x, w = wl.random_problem(41, N, C, H, W, K, R, S)
    rng = np.random.default_rng(42)
    bias = rng.uniform(-1, 1, size=K).astype(np.float32)
    for mode in (0, 1):
        want = oc.conv_forward(x, w, pad=pad, stride=stride, mode=mode)
        y0 = rng.uniform(-1, 1, size=want.shape).astype(np.float32)
        print(prob, layout, mode, flush=True)
        # one byte less: another route, whose sums round otherwise
        plain = _forward(gu, x, w, pad, stride, mode, layout, 0)
        got = _forward(gu, x, w, pad, stride, mode, layout, _bytes(K, C, R * S))
        assert not np.array_equal(got, plain), "the route under test did not run"
        assert np.abs(got - want).max() <= gu.BOUND["f32"] * np.abs(want).max()
        # (as exact as the route without the workspace, which holds three parts of an operand: 1.25 allows for few results)
        assert np.linalg.norm(got - want) <= 1.25 * np.linalg.norm(plain - want)
        got = _forward(gu, x, w, pad, stride, mode, layout, _bytes(K, C, R * S), 0.5, -1.5, y0, bias, 1)
        pre = 0.5 * want - 1.5 * y0 + bias[None, :, None, None]
        assert np.abs(got - np.maximum(pre, 0)).max() <= gu.BOUND["f32"] * np.abs(want).max() + 2.0 ** -20


@pytest.mark.parametrize("order", ["nchw", "cnhw", "chwn"])
@pytest.mark.parametrize("images", [1, 7])
def test_channels_beyond_the_last(images, order):
    """53 channels, in blocks of 16: what is read in place of the missing ones, in tensors of any order, does not count."""
    gu = _gpu()
    K, C = 120, 53
    x, w = wl.random_problem(49, images, C, 60 - 5 * images, 81, K, 3, 3)
    where = {d: i for i, d in enumerate("nchw")}
    strided = np.ascontiguousarray(x.transpose([where[d] for d in order])).transpose([order.index(d) for d in "nchw"])
    print(images, order, flush=True)
    plain, got = (_forward(gu, strided, w, (1, 1), (1, 1), 1, None, n, units=8) for n in (0, _bytes(K, C, 9)))
    assert not np.array_equal(got, plain), "the route under test did not run"
    assert np.abs(got - oc.conv_forward(x, w, pad=(1, 1), mode=1)).max() <= gu.BOUND["f32"] * np.abs(got).max()


def test_room_for_the_split_filter_decides():
    gu = _gpu()
    x, w = wl.random_problem(43, 96, 64, 28, 28, 128, 3, 3)
    need = _bytes(128, 64, 9)
    plain, short, got = (_forward(gu, x, w, (1, 1), (1, 1), 1, "NCHW", n, units=0) for n in (0, need - 16, need))
    assert np.array_equal(plain, short) and not np.array_equal(plain, got)


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", [(17, 70, 14, 13, 48, 3, 3, (1, 1)), (3, 33, 20, 17, 68, 5, 5, (2, 1)), (2, 64, 24, 40, 32, 9, 9, (0, 0)),
                                  (23, 40, 9, 21, 48, 1, 11, (0, 5))])
def test_backward_data(prob, layout):
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    rng = np.random.default_rng(44)
    P, Q = H + 2 * pad[0] - R + 1, W + 2 * pad[1] - S + 1
    dy = rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32)
    w = (rng.standard_normal(size=(K, C, R, S)) * (K * R * S) ** -0.5).astype(np.float32)
    dx0 = rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32)
    for mode, alpha, beta in ((0, 1.0, 0.0), (1, 0.5, -1.5)):
        print(prob, layout, mode, flush=True)
        old = dx0 if beta else None
        want = oc.conv_backward_data(dy, w, (H, W), pad=pad, mode=mode, alpha=alpha, beta=beta, dx_old=old)
        plain = _backward_data(gu, dy, w, (H, W), pad, mode, layout, 0, alpha, beta, old)
        got = _backward_data(gu, dy, w, (H, W), pad, mode, layout, _bytes(C, K, R * S), alpha, beta, old)
        assert not np.array_equal(got, plain), "the route under test did not run"
        _same(got, want, (prob, layout, mode))
        assert np.linalg.norm(got - want) <= 1.25 * np.linalg.norm(plain - want)


PLANTED = [(12, 48, 14, 13, 70, 3, 3, (1, 1)), (4, 32, 15, 16, 70, 5, 5, (2, 2))]


@pytest.mark.parametrize("kind", ["inf", "nan", "huge", "tiny"])
@pytest.mark.parametrize("prob", PLANTED)
def test_values_outside_the_range(prob, kind):
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    rng = np.random.default_rng(45)
    x, w = wl.random_problem(46, N, C, H, W, K, R, S)
    for operand in (0, 1):
        a = [x, w]
        a[operand], other = _planted(a[operand], kind, rng)
        a[1 - operand] = a[1 - operand] * other
        print(prob, kind, operand, flush=True)
        got = _forward(gu, a[0], a[1], pad, (1, 1), 1, "NCHW", _bytes(K, C, R * S))
        _same(got, oc.conv_forward(a[0], a[1], pad=pad, mode=1), (prob, kind, operand))


@pytest.mark.parametrize("kind", [*SMALL, "channels", "wide range", "mostly zero"])
@pytest.mark.parametrize("prob", PLANTED)
def test_operands_of_unequal_size(prob, kind):
    """Rows, columns, channels or single operands far below the largest of their chunk."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    rng = np.random.default_rng(47)
    x, w = wl.random_problem(48, N, C, H, W, K, R, S)
    if kind in SMALL:
        sx, sw, rows, cols = SMALL[kind]
        x, w = _scaled(x, sx), _scaled(w, sw)
        w[3::7] = _scaled(w[3::7], rows)
        x[1, :, :5] = _scaled(x[1, :, :5], cols)
    elif kind == "channels":      # large operands of either side meet small ones of the other
        for c in range(C):
            x[:, c], w[:, c] = _scaled(x[:, c], 45 * (c % 2)), _scaled(w[:, c], 45 - 90 * (c % 2))
    elif kind == "wide range":
        x, w = (np.ldexp(a.astype(np.float64), rng.integers(-60, 1, size=a.shape)).astype(np.float32) for a in (x, w))
    else:
        x *= rng.random(size=x.shape) < 0.02
        x[:, :16] = 0
    print(prob, kind, flush=True)
    got = _forward(gu, x, w, pad, (1, 1), 1, "NCHW", _bytes(K, C, R * S))
    _check(got, oc.conv_forward(x, w, pad=pad, mode=1), oc.conv_forward(np.abs(x), np.abs(w), pad=pad, mode=1), w[0].size, (prob, kind))
