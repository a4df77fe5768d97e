"""The backward-filter kernel that writes float operands as two binary16 numbers.  On a handle told of eight compute units small
problems take that route, several (tile, range) pairs to a workgroup."""
import numpy as np
import pytest

import paper_1410_0759_amd as ig
from oracle import conv_oracle as oc
import workloads as wl
from tests.test_gpu_halves import SAME_BITS, _microseconds
from tests.test_gpu_split import SMALL, _check, _planted, _same, _scaled

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _problem(seed, N, C, H, W, K, R, S, pad, stride):
    rng = np.random.default_rng(seed)
    P, Q = (H + 2 * pad[0] - R) // stride[0] + 1, (W + 2 * pad[1] - S) // stride[1] + 1
    x = rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32)
    return x, (0.1 * rng.standard_normal(size=(N, K, P, Q))).astype(np.float32)


@pytest.fixture
def run(monkeypatch, capfd):
    def call(gu, x, dy, rs, pad, stride, mode=1, layout="NCHW", workspace="full", alpha=1.0, beta=0.0, old=None, units=8, kernel="wgrad halves"):
        g = gu.GpuBackwardFilter(wl.with_layout(x, layout) if layout else x, wl.with_layout(dy, layout) if layout else dy, rs, pad, stride, mode, "f32", workspace)
        if units:
            ig.set_compute_units(g.handle, units)
        if old is not None:
            g.out.prefill(old=old)
        else:
            g.out.prefill(value=float("nan"))
        monkeypatch.setenv("IGCONV_DEBUG", "1")
        capfd.readouterr()
        g.launch(alpha, beta)
        assert kernel in capfd.readouterr().err, "the route under test did not run"
        g.ws.result()   # (guard bands)
        return g.out.result()
    return call


PROBLEMS = [
    # N, C, H, W, K, R, S, pad, stride
    (12, 48, 14, 13, 70, 3, 3, (1, 1), (1, 1)),      # ragged rows; the last pair of units is half empty
    (40, 32, 11, 9, 64, 3, 3, (1, 1), (1, 1)),       # shortest output rows: the longest patch
    (9, 33, 40, 31, 45, 5, 4, (2, 1), (2, 1)),       # four taps in a row: the second three share two; vertical stride
    (6, 96, 20, 24, 8, 3, 7, (1, 3), (1, 1)),        # eight maps
    (5, 40, 30, 40, 130, 1, 5, (0, 2), (1, 1)),      # one filter row
    (3, 25, 40, 60, 72, 9, 9, (0, 0), (1, 1)),       # channels: the last block has the last eight again
    (1, 32, 30, 300, 64, 3, 3, (1, 1), (1, 1)),      # rows longer than two chunks
]


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", PROBLEMS)
def test_backward_filter(prob, layout, run):
    gu = _gpu()
    *dims, pad, stride = prob
    rs = dims[5:]
    x, dy = _problem(51, *prob)
    rng = np.random.default_rng(52)
    for mode, alpha, beta, workspace in ((1, 1.0, 0.0, "full"), (0, 0.5, -1.5, "full"), (0, 1.0, 0.0, "none"), (1, 0.5, -1.5, "none")):
        print(prob, layout, mode, workspace, flush=True)
        old = rng.uniform(-1, 1, size=(dims[4], dims[1], *rs)).astype(np.float32) if beta else None
        want = oc.conv_backward_filter(x, dy, rs, pad=pad, stride=stride, mode=mode, alpha=alpha, beta=beta, dw_old=old)
        got = run(gu, x, dy, rs, pad, stride, mode, layout, workspace, alpha, beta, old)
        assert np.abs(got - want).max() <= gu.BOUND["f32"] * np.abs(want).max()
        if beta == 0.0:   # (1.3e-7 and twice the chains' roundings: see halves_backward_filter in igconv_api.cpp)
            assert np.linalg.norm(got - want) <= (1.5e-7 + 1.3e-8 * (dy.size / dims[4]) ** 0.5) * np.linalg.norm(want)


def test_every_compute_unit(run):
    """All of the chip: ranges of a few chunks, hundreds of parts."""
    gu = _gpu()
    x, dy = _problem(53, 24, 32, 40, 41, 64, 5, 5, (2, 2), (1, 1))
    want = oc.conv_backward_filter(x, dy, (5, 5), pad=(2, 2), stride=(1, 1), mode=1)
    got = run(gu, x, dy, (5, 5), (2, 2), (1, 1), units=0)
    assert np.abs(got - want).max() <= gu.BOUND["f32"] * np.abs(want).max()


PLANTED = [(12, 48, 14, 13, 70, 3, 3, (1, 1), (1, 1)), (9, 33, 40, 31, 45, 5, 4, (2, 1), (2, 1))]


@pytest.mark.parametrize("kind", ["inf", "nan", "huge", "tiny"])
@pytest.mark.parametrize("prob", PLANTED)
def test_values_outside_the_range(prob, kind, run):
    gu = _gpu()
    *dims, pad, stride = prob
    rng = np.random.default_rng(54)
    x, dy = _problem(55, *prob)
    for operand in (0, 1):
        a = [x, dy]
        a[operand], other = _planted(a[operand], kind, rng)
        a[1 - operand] = a[1 - operand] * other
        print(prob, kind, operand, flush=True)
        got = run(gu, a[0], a[1], dims[5:], pad, stride)
        _same(got, oc.conv_backward_filter(a[0], a[1], dims[5:], pad=pad, stride=stride, mode=1), (prob, kind, operand))


@pytest.mark.parametrize("kind", [*SMALL, "images", "drift", "wide range", "mostly zero"])
@pytest.mark.parametrize("prob", PLANTED)
def test_operands_of_unequal_size(prob, kind, run):
    """Maps, channels, images or single operands far below the largest of their chunk, or of another chunk of the range."""
    gu = _gpu()
    *dims, pad, stride = prob
    rng = np.random.default_rng(56)
    x, dy = _problem(57, *prob)
    if kind in SMALL:
        sx, sy, rows, cols = SMALL[kind]
        x, dy = _scaled(x, sx), _scaled(dy, sy)
        dy[:, 3::7] = _scaled(dy[:, 3::7], rows)
        x[:, :5] = _scaled(x[:, :5], cols)
    elif kind == "images":      # exponents that leave what a range may span, up and down
        for n in range(dims[0]):
            x[n], dy[n] = _scaled(x[n], 60 - 30 * (n % 5)), _scaled(dy[n], 10 * (n % 3) - 60)
    elif kind == "drift":       # sums scaled again from image to image
        for n in range(dims[0]):
            x[n] = _scaled(x[n], (n * 5) % 17)
    elif kind == "wide range":
        x, dy = (np.ldexp(a.astype(np.float64), rng.integers(-60, 1, size=a.shape)).astype(np.float32) for a in (x, dy))
    else:
        x *= rng.random(size=x.shape) < 0.02
        x[0], dy[-1] = 0, 0
    print(prob, kind, flush=True)
    got = run(gu, x, dy, dims[5:], pad, stride)
    want = oc.conv_backward_filter(x, dy, dims[5:], pad=pad, stride=stride, mode=1)
    magnitude = oc.conv_backward_filter(np.abs(x), np.abs(dy), dims[5:], pad=pad, stride=stride, mode=1)
    _check(got, want, magnitude, dy.size // dims[4], (prob, kind))


@pytest.mark.parametrize("order", ["cnhw", "chwn", "whcn", "hnwc"])
def test_tensors_of_any_order(order, run):
    """Both operands in other orders than the two usual ones, x cut out of a larger tensor: the same sums as packed."""
    gu = _gpu()
    prob = (12, 48, 14, 13, 70, 3, 3, (1, 1), (1, 1))
    x, dy = _problem(60, *prob)
    where = {d: i for i, d in enumerate("nchw")}
    placed = lambda a: np.ascontiguousarray(a.transpose([where[d] for d in order])).transpose([order.index(d) for d in "nchw"])
    larger = np.zeros((13, 51, 15, 16), np.float32)
    larger[:12, 2:50, :14, 1:14] = x
    cut = placed(larger)[:12, 2:50, :14, 1:14]
    print(order, flush=True)
    want = run(gu, x, dy, (3, 3), (1, 1), (1, 1), layout="NHWC" if order[-1] == "c" else "NCHW")
    assert np.array_equal(run(gu, cut, placed(dy), (3, 3), (1, 1), (1, 1), layout=None), want)


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("kind", ["log-normal", "log-normal, maps of zeros", "image scales", "one gradient", "falling", "rising"])
@pytest.mark.parametrize("prob", [PROBLEMS[0], PROBLEMS[2], PROBLEMS[5]])
def test_sums_looked_at_again(prob, kind, layout, run):
    """Results that operands with something lost could have touched, a few of a range or all; ranges whose chunks differ by more than sums can
    be multiplied up or down."""
    gu = _gpu()
    *dims, pad, stride = prob
    rng = np.random.default_rng(71)
    x, dy = _problem(72, *prob)
    dy = dy.astype(np.float64)
    n = np.arange(dims[0])
    if kind.startswith("log-normal"):
        dy = np.sign(dy) * np.exp(3.0 * rng.standard_normal(size=dy.shape))
    elif kind == "image scales":
        dy = dy * 10.0 ** (-4.0 * (n % 4))[:, None, None, None]
    elif kind == "one gradient":
        dy[0, 0, 0, 0] = 1e-14
    else:
        dy = dy * 2.0 ** (-33.0 * (n if kind == "falling" else n[::-1]) / len(n) * 3)[:, None, None, None]
    if kind.endswith("maps of zeros"):
        dy[:, 1::6], x[:, 2::5] = 0, 0
    dy = dy.astype(np.float32)
    for mode, workspace in ((0, "full"), (1, "none")):
        print(prob, kind, layout, mode, workspace, flush=True)
        got = run(gu, x, dy, dims[5:], pad, stride, mode, layout, workspace)
        want, mag = (oc.conv_backward_filter(a, b, dims[5:], pad=pad, stride=stride, mode=mode) for a, b in ((x, dy), (np.abs(x), np.abs(dy))))
        _check(got, want, mag, dy.size // dims[4], (prob, kind, layout, mode))


@pytest.mark.parametrize("kind", ["one gradient, a map of zeros", "log-normal gradients, maps of zeros", "image scales"])
def test_a_few_small_operands_cost_little(kind):
    """128x64x56x56 -> 64, 3x3.  (Multiplying every range that holds a small operand again took 5.2, 5.3 and 5.2 times as long as without; now
    1.2, 1.0 and 1.6.)"""
    gu = _gpu()
    rng = np.random.default_rng(73)
    x = np.maximum(rng.standard_normal(size=(128, 64, 56, 56), dtype=np.float32), 0)
    dy = rng.standard_normal(size=x.shape, dtype=np.float32)
    times = []
    for small in (False, True):
        if small and kind == "one gradient, a map of zeros":
            dy[:, 3, 5, 5], dy[:, 9] = 1e-11, 0
        elif small and kind == "image scales":
            dy *= (np.float32(10) ** (np.arange(128) * 5 % 13 * -1.0).astype(np.float32))[:, None, None, None]
        elif small:
            dy = np.copysign(np.exp(2 * rng.standard_normal(size=dy.shape, dtype=np.float32)), dy)
            dy[:, 5::16], x[:, 5::16] = 0, 0
        g = gu.GpuBackwardFilter(x, dy, (3, 3), (1, 1), (1, 1), 1, "f32", "full")
        times.append(_microseconds(lambda: g.launch(1.0, 0.0)))
    print(kind, times, flush=True)
    assert times[1] <= 2.2 * times[0], times


@pytest.mark.parametrize("value", SAME_BITS)
@pytest.mark.parametrize("prob", PLANTED)
def test_operands_with_the_same_low_bits(prob, value, run):
    """As in the forward pass: 2^-21 of the sum of magnitudes, and 2^-24 of the growing sum per addition of sixteen pixels' products; the two halves',
    the small products', the scale's and the parts' (of up to 24 ranges on eight compute units, half of the sum on average)."""
    gu = _gpu()
    *dims, pad, stride = prob
    x, dy = _problem(74, *prob)
    x[:], dy[:] = np.float32(value), np.float32(value)
    print(prob, value, flush=True)
    got = run(gu, x, dy, dims[5:], pad, stride)
    want = oc.conv_backward_filter(x, dy, dims[5:], pad=pad, stride=stride, mode=1)
    assert (np.abs(got - want) <= (2.0 ** -21 + (dy.size / dims[4] / 32 + 16) * 2.0 ** -24) * np.abs(want)).all()


ROWS = [
    # N, C, H, W, K, R, S, pad, stride: three filter rows and taps per tile
    (10, 40, 20, 57, 70, 3, 3, (1, 1), (1, 1)),      # long rows: chunks keep to one image
    (12, 33, 21, 13, 45, 5, 4, (2, 1), (1, 1)),      # five rows and four taps: the second three share one and two
    (30, 25, 18, 23, 8, 7, 7, (3, 3), (1, 1)),       # eight maps, the last eight channels again; three groups of rows and of taps
    (40, 64, 9, 9, 130, 3, 3, (1, 1), (1, 1)),       # shortest rows, two images and more per chunk; ragged third block of maps
    (1, 32, 150, 58, 64, 6, 3, (0, 1), (1, 1)),      # one image
    (64, 40, 6, 11, 24, 3, 5, (1, 2), (1, 1)),       # images of 66 pixels
]


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", ROWS)
def test_three_filter_rows(prob, layout, monkeypatch, capfd):
    """With room for every range, for two, for none, and a workspace off the 16-byte boundary; several tiles and chains of sums per workgroup."""
    import torch
    gu = _gpu()
    *dims, pad, stride = prob
    N, C, H, W, K, R, S = dims
    x, dy = _problem(61, *prob)
    rng = np.random.default_rng(62)
    old = rng.uniform(-1, 1, size=(K, C, R, S)).astype(np.float32)
    h = ig.Handle()
    h.set_stream(torch.cuda.current_stream().cuda_stream)
    ig.set_compute_units(h, 8)
    put = lambda a: torch.from_numpy(a).cuda() if layout == "NCHW" else torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 3, 1))).cuda().permute(0, 3, 1, 2)
    xt, dyt = put(x), put(dy)
    xd, dyd = ig.tensor_descriptor_for(xt), ig.tensor_descriptor_for(dyt)
    wd = ig.FilterDescriptor().set(ig.IGC_DATA_FLOAT, K, C, R, S)
    monkeypatch.setenv("IGCONV_DEBUG", "1")
    for mode in (ig.IGC_CONVOLUTION, ig.IGC_CROSS_CORRELATION):
        cd = ig.ConvolutionDescriptor().set(*pad, *stride, mode)
        full = ig.get_backward_filter_workspace_size(h, xd, dyd, cd, wd)
        tiles = -(-K // 64) * -(-C // 32) * -(-R // 3) * -(-S // 3)
        for room, offset, alpha, beta in ((full, 0, 0.5, -1.5), (2 * tiles * 18432 * 4, 0, 1.0, 0.0), (0, 0, 0.5, -1.5), (full, 4, 1.0, 0.0)):
            ws = torch.full((full // 4 + tiles * 18432 * 2 + 8,), float("nan"), device="cuda")
            dw = torch.from_numpy(old if beta else np.full_like(old, np.nan)).cuda()
            capfd.readouterr()
            ig.check(ig.convolution_backward_filter(h, alpha, xd, xt.data_ptr(), dyd, dyt.data_ptr(), cd, beta, wd, dw.data_ptr(),
                                                    ws.data_ptr() + offset if room else 0, room))
            torch.cuda.synchronize()
            err = capfd.readouterr().err
            print(prob, layout, mode, room, offset, err, flush=True)
            assert "three filter rows" in err or room != full or offset, err      # (with less room another kernel may be chosen)
            assert torch.isnan(ws[(room + offset + 3) // 4:]).all()       # (nothing beyond the room lent)
            want = oc.conv_backward_filter(x, dy, (R, S), pad=pad, stride=stride, mode=mode, alpha=alpha, beta=beta, dw_old=old if beta else None)
            got = dw.cpu().numpy()
            assert np.abs(got - want).max() <= gu.BOUND["f32"] * np.abs(want).max()
            if beta == 0.0:
                assert np.linalg.norm(got - want) <= (1.5e-7 + 1.3e-8 * (dy.size / K) ** 0.5) * np.linalg.norm(want)


@pytest.mark.parametrize("kind", ["inf", "nan", "huge", "tiny", "images", "drift", "wide range", "mostly zero"])
@pytest.mark.parametrize("prob", ROWS[:4:3])
def test_three_filter_rows_outside_the_range(prob, kind, run):
    """Values that one exponent does not hold, in either operand: chunks of one image and of several."""
    gu = _gpu()
    *dims, pad, stride = prob
    rng = np.random.default_rng(77)
    for operand in (0, 1):
        a = list(_problem(78, *prob))
        if kind == "images":      # exponents that leave what a range may span, up and down
            for n in range(dims[0]):
                a[operand][n], a[1 - operand][n] = _scaled(a[operand][n], 60 - 30 * (n % 5)), _scaled(a[1 - operand][n], 10 * (n % 3) - 60)
        elif kind == "drift":       # sums scaled again from image to image
            for n in range(dims[0]):
                a[operand][n] = _scaled(a[operand][n], (n * 5) % 17)
        elif kind == "wide range":
            a[operand] = np.ldexp(a[operand].astype(np.float64), rng.integers(-60, 1, size=a[operand].shape)).astype(np.float32)
        elif kind == "mostly zero":
            a[operand] *= rng.random(size=a[operand].shape) < 0.02
            a[operand][0], a[operand][1, 1, -1, -1] = 0, 1e-14
        else:
            a[operand], other = _planted(a[operand], kind, rng)
            a[1 - operand] = a[1 - operand] * other
        print(prob, kind, operand, flush=True)
        got = run(gu, a[0], a[1], dims[5:], pad, stride, workspace=8 << 20, kernel="three filter rows")
        want = oc.conv_backward_filter(a[0], a[1], dims[5:], pad=pad, stride=stride, mode=1)
        _same(got, want, (prob, kind, operand))
        if kind in ("images", "drift", "wide range", "mostly zero"):
            magnitude = oc.conv_backward_filter(np.abs(a[0]), np.abs(a[1]), dims[5:], pad=pad, stride=stride, mode=1)
            _check(got, want, magnitude, a[1].size // dims[4], (prob, kind, operand))


@pytest.mark.parametrize("prob", [
    # with three bfloat16 parts, with the fp32 instruction
    (34, 91, 45, 45, 11, 3, 3, (0, 0), (1, 1)), (89, 50, 16, 16, 11, 3, 3, (1, 1), (1, 1)),
], ids=str)
def test_products_of_24_bits_where_three_rows_would_be_faster(prob):
    """One gradient that is not zero: every result is one product, rounded (2^-24) after what three parts leave out (2^-25).  Two binary16 parts leave up to 2^-22."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    x, dy = _problem(75, *prob)
    n, p, q = N // 2, H // 2, W // 2
    one = dy[n, :, p, q].astype(np.float64)
    dy[:] = 0
    dy[n, :, p, q] = one
    g = gu.GpuBackwardFilter(x, dy, (R, S), pad, stride, 1, "f32", "full")
    g.out.prefill(value=float("nan"))
    print(prob, g.asked, flush=True)
    g.launch(1.0, 0.0)
    want = one[:, None, None, None] * x[n][:, p - pad[0]:p - pad[0] + R, q - pad[1]:q - pad[1] + S].astype(np.float64)
    assert np.abs(g.out.result() / want - 1).max() <= 2.0 ** -23
