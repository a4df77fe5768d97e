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


def _backward_data(gu, dy, w, hw, pad, mode, layout, lent, alpha=1.0, beta=0.0, dx0=None, units=8):
    g = gu.GpuBackwardData(wl.with_layout(dy, layout), w, hw, pad, (1, 1), mode, "f32", layout, lent or "none")
    ig.set_compute_units(g.handle, units)
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
        # a little less: another route, whose sums round otherwise (or the one without any, whose order of sums the room can change too)
        plain = _forward(gu, x, w, pad, stride, mode, layout, 0)
        short = _forward(gu, x, w, pad, stride, mode, layout, _bytes(K, C, R * S) - 16)
        got = _forward(gu, x, w, pad, stride, mode, layout, _bytes(K, C, R * S))
        assert not np.array_equal(got, plain) and not np.array_equal(got, short), "the route under test did not run"
        assert np.abs(short - want).max() <= gu.BOUND["f32"] * np.abs(want).max()
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
        short = _backward_data(gu, dy, w, (H, W), pad, mode, layout, _bytes(C, K, R * S) - 16, alpha, beta, old)
        got = _backward_data(gu, dy, w, (H, W), pad, mode, layout, _bytes(C, K, R * S), alpha, beta, old)
        assert not np.array_equal(got, plain) and not np.array_equal(got, short), "the route under test did not run"
        _same(short, want, (prob, layout, mode))
        _same(got, want, (prob, layout, mode))
        assert np.linalg.norm(got - want) <= 1.25 * np.linalg.norm(plain - want)


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, S, pad: tiles for sixteen units, two per XCD; the last of an odd number goes as halves
    (4, 64, 15, 16, 96, 5, 5, (2, 2)),       # 8 tiles of 256 columns, all as halves
    (7, 32, 20, 64, 40, 9, 9, (0, 0)),       # 21, three to an image
    (17, 64, 1, 107, 60, 1, 21, (0, 10)),    # 8, the last one of 27 columns: nothing in its right half
    (16, 64, 12, 9, 130, 7, 2, (3, 1)),      # 24: two whole ones, then halves
], ids=str)
def test_halved_tiles(prob, layout):
    """(csrc/host_check.cpp requires that these layers take this route.)"""
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    rng = np.random.default_rng(50)
    for kind in (None, "inf", "nan", "tiny", "zeros"):
        x, w = wl.random_problem(51, N, C, H, W, K, R, S)
        if kind == "zeros":      # sums of zero beside operands far below the others
            x[:, 3::7], w[1::6], x[:, :, : H // 2] = 0, 0, 0
            x[:, 1, -1, -1] = 1e-14
        elif kind:
            x, other = _planted(x, kind, rng)
            w = w * other
        want = oc.conv_forward(x, w, pad=pad, mode=1)
        y0 = rng.uniform(-1, 1, size=want.shape).astype(np.float32)
        beta = -1.5 if kind is None else 0.0
        print(prob, layout, kind, flush=True)
        whole, got = (_forward(gu, x, w, pad, (1, 1), 1, layout, _bytes(K, C, R * S), 1.0, beta, y0, units=u) for u in (8, 16))
        _same(got, want + beta * y0 if beta else want, (prob, layout, kind))
        # (the products, their order and the exponents of the filter are the same; the patch's may differ)
        if kind is None:
            assert np.linalg.norm(got - want - beta * y0) <= 1.25 * np.linalg.norm(whole - want - beta * y0)
    wt = np.ascontiguousarray(w.transpose(1, 0, 2, 3)) if R == S else None
    if wt is not None:   # (the exchanged layer: as many rows and, but for the border, columns)
        dy = rng.uniform(-1, 1, size=(N, C, H + 2 * pad[0] - R + 1, W + 2 * pad[1] - S + 1)).astype(np.float32)
        dx = _backward_data(gu, dy, wt, (H, W), pad, 1, layout, _bytes(K, C, R * S), units=16)
        _same(dx, oc.conv_backward_data(dy, wt, (H, W), pad=pad, mode=1), (prob, layout, "data"))


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
def test_a_half_tile_reads_its_own_columns(layout):
    """What other tiles' pixels hold changes no bit of a tile's results: they are not among those whose largest sets its scale.  24 tiles of 256 output
    pixels, all as halves; a pixel of x that no window of the first tile has, but some of the 128 after it."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad = 8, 32, 20, 64, 40, 9, 9, (0, 0)
    x, w = wl.random_problem(76, N, C, H, W, K, R, S)
    large = x.copy()
    large[0, :, 13, 20] = 3e5
    print(layout, flush=True)
    got = [_forward(gu, a, w, pad, (1, 1), 1, layout, _bytes(K, C, R * S), units=48).transpose(1, 0, 2, 3).reshape(K, -1) for a in (x, large)]
    assert np.array_equal(got[0][:, :256], got[1][:, :256])
    assert np.abs(got[1][:, 256:384]).max() > 1e3 * np.abs(got[0]).max()


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


def _with_small_ones(kind, x, w, rng):
    """Operands of which some are far below the others: x is the gathered one (images x maps), w the filter's."""
    if kind.startswith("log-normal"):
        x = np.sign(x) * np.exp(3.0 * rng.standard_normal(size=x.shape))
    elif kind == "image scales":
        x = x * 10.0 ** (-4.0 * (np.arange(len(x)) % 4))[:, None, None, None]
    elif kind == "zero windows":
        x[:, :, : x.shape[2] // 2] = 0
        x[:, 1, -1, -1] = 1e-14
    elif kind == "one weight":
        w[-1, 0, 0, 0] = 1e-14
    elif kind == "one weight, filters of zeros":
        w[-1, 0, 0, 0] = 1e-30
        w[2::5], w[:, 3::7] = 0, 0
    if kind.endswith("maps of zeros"):
        x[:, 3::7], w[1::6] = 0, 0
        w[:, 2::5] = 0
    return x.astype(np.float32), w.astype(np.float32)


SMALL_ONES = ["log-normal", "log-normal, maps of zeros", "image scales", "zero windows", "one weight", "one weight, filters of zeros"]


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("kind", SMALL_ONES)
@pytest.mark.parametrize("prob", [(12, 48, 14, 13, 72, 3, 3, (1, 1), (1, 1)), (4, 36, 15, 16, 96, 5, 5, (2, 2), (1, 1)),
                                  (20, 48, 7, 31, 20, 1, 11, (0, 5), (1, 1)), (12, 64, 12, 14, 130, 7, 2, (3, 1), (1, 2))])
def test_sums_looked_at_again(prob, kind, layout):
    """Results that operands with something lost could have touched, a few of a tile or all: one by one, or the tile's together."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(61)
    for mode in (0, 1):
        x, w = wl.random_problem(62, N, C, H, W, K, R, S)
        x, w = _with_small_ones(kind, x, w, rng)
        print(prob, kind, layout, mode, flush=True)
        got = _forward(gu, x, w, pad, stride, mode, layout, _bytes(K, C, R * S))
        want, mag = (oc.conv_forward(a, b, pad=pad, stride=stride, mode=mode) for a, b in ((x, w), (np.abs(x), np.abs(w))))
        _check(got, want, mag, w[0].size, (prob, kind, layout, mode))
        if stride != (1, 1):
            continue
        P, Q = want.shape[2:]
        dy, w = _with_small_ones(kind, rng.uniform(-1, 1, size=(N, K, P, Q)), rng.standard_normal(size=(K, C, R, S)) * 0.1, rng)
        got = _backward_data(gu, dy, w, (H, W), pad, mode, layout, _bytes(C, K, R * S))
        want, mag = (oc.conv_backward_data(a, b, (H, W), pad=pad, mode=mode) for a, b in ((dy, w), (np.abs(dy), np.abs(w))))
        _check(got, want, mag, w[:, 0].size, (prob, kind, layout, mode, "backward data"))


def _microseconds(launch):
    """Best of several batches: what the device needs, not what else it does."""
    import torch
    best = float("inf")
    for _ in range(6):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(4):
            launch()
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 250)
    return best


@pytest.mark.parametrize("kind", ["one weight", "log-normal gradients", "log-normal gradients, maps of zeros"])
def test_a_few_small_operands_cost_little(kind):
    """128x64x56x56 -> 70, 3x3: one tiny weight in the block of rows that is not full, forward; gradients over many orders of magnitude,
    backward data.  (Multiplying every tile that holds a small operand again took 5.6, 4.8 and 5.4 times as long as without; now 1.0, 1.2 and 1.4.)"""
    gu = _gpu()
    N, C, H, K = 128, 64, 56, 70
    rng = np.random.default_rng(63)
    x = np.maximum(rng.standard_normal(size=(N, C, H, H), dtype=np.float32), 0)
    w = rng.standard_normal(size=(K, C, 3, 3), dtype=np.float32) * np.float32(0.06)
    dy = rng.standard_normal(size=(N, K, H, H), dtype=np.float32)
    times = []
    for small in (False, True):
        if small and kind == "one weight":
            w[69, 1, 1, 1] = 1e-12
        elif small:
            dy = np.copysign(np.exp(2.8 * rng.standard_normal(size=dy.shape, dtype=np.float32)), dy)
            if kind.endswith("zeros"):
                dy[:, 5::16], w[:, 5::16] = 0, 0
        if kind == "one weight":
            g = gu.GpuConv(x, w, (1, 1), (1, 1), 1)
            g.lend_workspace(_bytes(K, C, 9))
            g.prefill(None, 0.0)
            times.append(_microseconds(lambda: g.launch_fused(1.0, 0.0, None, -1)))
        else:
            g = gu.GpuBackwardData(dy, w, (H, H), (1, 1), (1, 1), 1, "f32", "NCHW", _bytes(C, K, 9))
            times.append(_microseconds(lambda: g.launch(1.0, 0.0)))
    print(kind, times, flush=True)
    assert times[1] <= 2.2 * times[0], times


def test_images_of_unequal_gradients():
    """128x384x13x13 -> 256, 3x3, backward data, tiles over three images: every other one's gradients 10^4 times smaller.  (6.5 times as long as
    without where every such tile was multiplied again with the fp32 instruction; now 2.2.)"""
    gu = _gpu()
    rng = np.random.default_rng(64)
    dy = rng.standard_normal(size=(128, 256, 13, 13), dtype=np.float32)
    w = rng.standard_normal(size=(256, 384, 3, 3), dtype=np.float32) * np.float32(0.02)
    times = []
    for small in (False, True):
        if small:
            dy[1::2] *= np.float32(1e-4)
        g = gu.GpuBackwardData(dy, w, (13, 13), (1, 1), (1, 1), 1, "f32", "NCHW", _bytes(384, 256, 9))
        times.append(_microseconds(lambda: g.launch(1.0, 0.0)))
    print(times, flush=True)
    assert times[1] <= 3.5 * times[0], times


# Operands that all have the same low bits: each of a sum's products loses on the same side.  A unit of an operand's last place is 2^-23 of it at most,
# the product left out 2^-22: 2^-21 of the sum of magnitudes.  The growing sum is rounded, by 2^-24 of it, at nine additions per chunk (five times the
# chunk's sum in all) and one of each chunk; three more for the small products, the scale and the result.
SAME_BITS = [1 + 2.0 ** -11, 1 + 3001 * 2.0 ** -23, 1 / 3, 0.1, 2.0 ** 14 - 2.0 ** -9]


@pytest.mark.parametrize("value", SAME_BITS)
@pytest.mark.parametrize("prob", PLANTED)
def test_operands_with_the_same_low_bits(prob, value):
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    x, w = (np.full(shape, value, np.float32) for shape in ((N, C, H, W), (K, C, R, S)))
    x[:, 1::2] *= 4     # (a power of two: the same bits)
    for sign in (1, -1):
        print(prob, value, sign, flush=True)
        got = _forward(gu, sign * x, w, pad, (1, 1), 1, "NCHW", _bytes(K, C, R * S))
        want = oc.conv_forward(sign * x, w, pad=pad, mode=1)
        chunks = -(-C // 16) * -(-(R * S) // 9)
        assert (np.abs(got - want) <= (2.0 ** -21 + (8 + chunks / 2) * 2.0 ** -24) * np.abs(want)).all()
