"""The kernels that write float operands as sums of three bfloat16 numbers, outside the range where that is exact:
infinities and NaN, values that round to infinity, values whose parts are bfloat16 denormals.  Inside it the parity tests
(every kernel of the table, both backward passes) compare them with the oracle like any other kernel."""
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


def _planted(a, kind, rng):
    """`a` with a few elements replaced, or scaled as a whole; the other operand's scale that keeps results in range."""
    a = a.copy()
    flat = a.reshape(-1)
    at = rng.choice(flat.size, size=min(6, flat.size), replace=False)
    if kind == "inf":
        flat[at[:3]], flat[at[3:]] = np.inf, -np.inf
    elif kind == "nan":
        flat[at] = np.nan
    elif kind == "huge":      # rounds to infinity in bfloat16, finite in float
        flat[at] = np.float32(3.4e38)
        return a, np.float32(2.0 ** -20)
    elif kind == "tiny":      # the second and third parts are below bfloat16's smallest denormal
        return a * np.float32(2.0 ** -115), np.float32(1.0)
    return a, np.float32(1.0)


def _same(got, want, kind):
    """Infinities and NaN where the oracle has them; elsewhere the float bound, relative to the largest finite value."""
    with np.errstate(over="ignore"):
        want32 = want.astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(want32)), kind
    inf = np.isinf(want32)
    assert np.array_equal(got[inf], want32[inf]), kind
    fin = np.isfinite(want32)
    big = np.abs(want[fin]).max()
    # (results near the smallest normal float: one unit of the denormal grid)
    assert np.abs(got[fin].astype(np.float64) - want[fin]).max() <= 2e-5 * big + 1.5e-45, kind


@pytest.mark.parametrize("kind", ["inf", "nan", "huge", "tiny"])
@pytest.mark.parametrize("swap", [False, True])
def test_forward_outside_the_split_range(kind, swap):
    import paper_1410_0759_amd as ig
    gu = _gpu()
    rng = np.random.default_rng(7)
    for kid, name in enumerate(ig.kernel_names()):
        if "split" not in name or "wgrad" in name or ("swap" in name) != swap:
            continue
        pad = (0, 0) if "nopad" in name else (1, 1)
        x, w = wl.random_problem(11, 2, 48 if "patch" in name else 20, 11, 13, 70, 3, 3)
        x, ws = _planted(x, kind, rng)
        x, w = wl.with_layout(x, "NHWC" if swap else "NCHW"), w * ws
        want = oc.conv_forward(x, w, pad=pad, mode=1)
        print(kind, name, flush=True)
        got, plan = gu.run(x, w, pad, (1, 1), 1, y_layout="NHWC" if swap else "NCHW", kernel=kid)
        assert plan.kernelId == kid
        _same(got, want, (kind, name))


@pytest.mark.parametrize("kind", ["plain", "inf", "nan", "huge", "tiny"])
@pytest.mark.parametrize("prob", [(16, 130, 32, 32, 24, 5, 5, 2), (20, 130, 24, 24, 24, 9, 9, 4)])
def test_backward_data_outside_the_split_range(kind, prob):
    """Sizes at which the general route runs on the split kernels (a compute unit's worth of tiles; more than 63 taps too)."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    rng = np.random.default_rng(8)
    P, Q = H + 2 * pad - R + 1, W + 2 * pad - S + 1
    dy = rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32)
    w = (rng.standard_normal(size=(K, C, R, S)) * (K * R * S) ** -0.5).astype(np.float32)
    dy, ws = _planted(dy, kind, rng)
    w = w * ws
    want = oc.conv_backward_data(dy, w, (H, W), pad=(pad, pad), mode=0)
    print(kind, prob, flush=True)
    _same(gu.run_backward_data(dy, w, (H, W), (pad, pad), (1, 1), 0, workspace="none"), want, kind)


@pytest.mark.parametrize("kind", ["plain", "inf", "nan", "huge", "tiny"])
@pytest.mark.parametrize("prob", [(4, 100, 15, 14, 70, 3, 3, (1, 1), (1, 1)), (3, 70, 9, 17, 130, 5, 2, (2, 0), (2, 1)),
                                  (2, 33, 8, 8, 33, 1, 1, (0, 0), (1, 1)), (2, 130, 6, 5, 140, 3, 3, (1, 1), (1, 2)),
                                  (4, 100, 15, 14, 64, 3, 3, (1, 1), (1, 1)), (3, 128, 8, 8, 120, 1, 1, (0, 0), (1, 1))])
def test_backward_filter_outside_the_split_range(kind, prob):
    """Every tile shape of the split kernels - by the least padding of K and C: 96 x 128 twice, (the fp32 kernel's 64 x 64),
    96 x 64 run as 128 x 64, 64 x 128, 128 x 128 - with and without a cut reduction."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(9)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    x = rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32)
    dy, xs = _planted(rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32), kind, rng)
    x = x * xs
    want = oc.conv_backward_filter(x, dy, (R, S), pad=pad, stride=stride, mode=1)
    for workspace in ("full", "none"):
        print(kind, prob, workspace, flush=True)
        _same(gu.run_backward_filter(x, dy, (R, S), pad, stride, 1, workspace=workspace)[0], want, kind)


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", [(40, 96, 14, 13, 32, 3, 3, (1, 1)), (20, 70, 28, 28, 16, 3, 3, (2, 1)), (24, 130, 12, 16, 48, 1, 9, (0, 3)),
                                  (9, 64, 40, 40, 80, 3, 3, (0, 2))])
def test_backward_data_from_a_staged_patch(prob, layout):
    """Unit stride and nine taps at sizes where backward data runs from a staged patch of dy: both filter orders, ragged
    tiles, one to five chunks of channels, borders on either side."""
    gu = _gpu()
    N, C, H, W, K, R, S, pad = prob
    rng = np.random.default_rng(10)
    P, Q = H + 2 * pad[0] - R + 1, W + 2 * pad[1] - S + 1
    dy = wl.with_layout(rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32), layout)
    w = (rng.standard_normal(size=(K, C, R, S)) * (K * R * S) ** -0.5).astype(np.float32)
    dx0 = rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32)
    for mode, alpha, beta in ((0, 1.0, 0.0), (1, 0.5, -1.5)):
        print(prob, layout, mode, flush=True)
        want = oc.conv_backward_data(dy, w, (H, W), pad=pad, mode=mode, alpha=alpha, beta=beta, dx_old=dx0 if beta else None)
        got = gu.run_backward_data(dy, w, (H, W), pad, (1, 1), mode, alpha, beta, dx0 if beta else None, "f32", layout)
        _same(got, want, (prob, layout, mode))


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("kind", ["plain", "inf", "tiny"])
@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, S, pad, stride: the phases that meet a tap run in one launch when there are two to four of them
    (3, 33, 15, 18, 20, 3, 3, (1, 1), (2, 2)),        # four phases of one to four taps
    (2, 140, 9, 11, 30, 1, 3, (0, 1), (2, 2)),        # two phases with taps, two without
    (5, 101, 7, 23, 13, 2, 5, (1, 0), (1, 3)),        # three
    (1, 65, 33, 6, 40, 4, 1, (3, 0), (4, 1)),         # four of one tap
    (2, 129, 13, 12, 9, 5, 4, (2, 1), (3, 2)),        # six: one launch each
])
def test_strided_backward_data(prob, kind, layout):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    rng = np.random.default_rng(12)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    dy, ws = _planted(rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32), kind, rng)
    dy = wl.with_layout(dy, layout)
    w = (rng.standard_normal(size=(K, C, R, S)) * (K * R * S) ** -0.5).astype(np.float32) * ws
    dx0 = rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32)
    for mode, alpha, beta in ((0, 1.0, 0.0), (1, 0.5, 1.0)) if kind == "plain" else ((0, 1.0, 0.0),):
        for workspace in ("full", "none"):
            print(prob, kind, layout, mode, workspace, flush=True)
            old = dx0 if beta else None
            want = oc.conv_backward_data(dy, w, (H, W), pad=pad, stride=stride, mode=mode, alpha=alpha, beta=beta, dx_old=old)
            _same(gu.run_backward_data(dy, w, (H, W), pad, stride, mode, alpha, beta, old, "f32", layout, workspace=workspace), want, kind)


# Operands so small that the second and third parts leave bfloat16's range, where the results do not show it: multiplied
# by large ones, or beside rows or columns of ordinary size.
# kind -> (scale of all of one operand, of all of the other one, of some rows of the product, of some of its columns)
SMALL = {
    "116 and 40": (-116, 40, 0, 0), "120 and 50": (-120, 50, 0, 0), "125 and 60": (-125, 60, 0, 0),
    "50 and 120": (50, -120, 0, 0), "denormal": (-140, 20, 0, 0), "denormal and large": (-146, 110, 0, 0),
    "rows": (0, 0, -120, 0), "rows at the bottom": (0, 0, -125, 0), "columns": (0, 0, 0, -120), "columns at the bottom": (0, 0, 0, -125),
    "rows and columns": (0, 0, -60, -62), "denormal rows": (0, 0, -140, 0),
}


def _scaled(a, exponent):
    """a * 2^exponent, rounded once (float holds the powers down to 2^-149 only)."""
    return np.ldexp(a.astype(np.float64), exponent).astype(np.float32)


def _check(got, want, magnitude, terms, what):
    """Sums of `terms` products: as many roundings of half a unit of the sum of magnitudes, or of the denormal grid."""
    err = np.abs(got - want)
    bad = err > (terms + 8) * 2.0 ** -24 * magnitude + terms * 2.0 ** -149
    assert not bad.any(), (what, int(bad.sum()), float((err / np.maximum(magnitude, 2.0 ** -149)).max()))


@pytest.mark.parametrize("kind", SMALL)
@pytest.mark.parametrize("swap", [False, True])
def test_forward_with_small_operands(kind, swap):
    import paper_1410_0759_amd as ig
    gu = _gpu()
    sx, sw, rows, cols = SMALL[kind]
    for kid, name in enumerate(ig.kernel_names()):
        if "split" not in name or "wgrad" in name or ("swap" in name) != swap:
            continue
        pad = (0, 0) if "nopad" in name else (1, 1)
        x, w = wl.random_problem(11, 2, 48 if "patch" in name else 20, 11, 13, 70, 3, 3)
        x, w = _scaled(x, sx), _scaled(w, sw)
        w[3::7] = _scaled(w[3::7], rows)              # maps
        x[1, :, :5] = _scaled(x[1, :, :5], cols)      # pixels
        x = wl.with_layout(x, "NHWC" if swap else "NCHW")
        print(kind, name, flush=True)
        got, plan = gu.run(x, w, pad, (1, 1), 1, y_layout="NHWC" if swap else "NCHW", kernel=kid)
        assert plan.kernelId == kid
        _check(got, oc.conv_forward(x, w, pad=pad, mode=1), oc.conv_forward(np.abs(x), np.abs(w), pad=pad, mode=1), w[0].size, (kind, name))


@pytest.mark.parametrize("kind", SMALL)
@pytest.mark.parametrize("prob", [(16, 130, 32, 32, 24, 5, 5, (2, 2), (1, 1)),     # the general route
                                  (40, 96, 14, 13, 32, 3, 3, (1, 1), (1, 1)),      # a staged patch of dy
                                  (5, 101, 15, 23, 13, 3, 3, (1, 1), (2, 2))])     # four phases in one launch
def test_backward_data_with_small_operands(prob, kind):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    sy, sw, rows, cols = SMALL[kind]
    rng = np.random.default_rng(13)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    dy = _scaled(rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32), sy)
    w = _scaled((rng.standard_normal(size=(K, C, R, S)) * (K * R * S) ** -0.5).astype(np.float32), sw)
    w[:, 3::7] = _scaled(w[:, 3::7], rows)
    dy[1, :, :5] = _scaled(dy[1, :, :5], cols)
    print(kind, prob, flush=True)
    got = gu.run_backward_data(dy, w, (H, W), pad, stride, 0, workspace="none")
    want, mag = (oc.conv_backward_data(a, b, (H, W), pad=pad, stride=stride, mode=0) for a, b in ((dy, w), (np.abs(dy), np.abs(w))))
    _check(got, want, mag, K * R * S, (kind, prob))


@pytest.mark.parametrize("kind", SMALL)
@pytest.mark.parametrize("prob", [(4, 100, 15, 14, 64, 3, 3, (1, 1), (1, 1)),      # 64 x 128 tiles
                                  (3, 70, 9, 17, 130, 5, 2, (2, 0), (2, 1)),       # 96 x 128
                                  (2, 33, 6, 5, 128, 3, 3, (1, 1), (1, 2)),        # 128 x 64
                                  (3, 128, 8, 8, 120, 1, 1, (0, 0), (1, 1))])      # 128 x 128
def test_backward_filter_with_small_operands(prob, kind):
    gu = _gpu()
    N, C, H, W, K, R, S, pad, stride = prob
    sy, sx, rows, cols = SMALL[kind]
    rng = np.random.default_rng(14)
    P, Q = oc.output_dim(H, R, stride[0], pad[0]), oc.output_dim(W, S, stride[1], pad[1])
    x = _scaled(rng.uniform(-1, 1, size=(N, C, H, W)).astype(np.float32), sx)
    dy = _scaled(rng.uniform(-1, 1, size=(N, K, P, Q)).astype(np.float32), sy)
    dy[:, 3::7] = _scaled(dy[:, 3::7], rows)
    x[:, 2::5] = _scaled(x[:, 2::5], cols)
    want, mag = (oc.conv_backward_filter(a, b, (R, S), pad=pad, stride=stride, mode=1) for a, b in ((x, dy), (np.abs(x), np.abs(dy))))
    for workspace in ("full", "none"):
        print(kind, prob, workspace, flush=True)
        got = gu.run_backward_filter(x, dy, (R, S), pad, stride, 1, workspace=workspace)[0]
        _check(got, want, mag, N * P * Q, (kind, prob, workspace))
