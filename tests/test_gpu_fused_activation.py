"""Sigmoid and tanh of the fused forward pass over the whole range of their argument: the filter passes x through (one tap
of one channel is 1), so that the argument is known exactly, on every kind of kernel that applies them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _arguments(n):
    rng = np.random.default_rng(41)
    ends = [0.0, -0.0, 1e-45, -1e-38, 87.0, -87.0, -87.2, -87.4, -88.0, -88.6, 88.6, 200.0, -200.0, np.inf, -np.inf, np.nan]
    v = np.concatenate([np.array(ends), rng.choice([-1, 1], size=n - len(ends)) * np.exp(rng.uniform(np.log(1e-4), np.log(100.0), size=n - len(ends)))])
    return rng.permutation(v).astype(np.float32)


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
@pytest.mark.parametrize("prob", [
    # N, C, H, W, K, R, workspace
    (1, 1, 60, 70, 5, 3, 0),          # few channels on the vector units
    (2, 5, 40, 60, 40, 1, 0),         # matrix kernels
    (40, 64, 20, 20, 64, 3, 0),       # ... operands in parts, a staged patch
    (1, 512, 7, 9, 64, 3, 1 << 20),   # a reduction cut into ranges: the sum applies it
])
def test_sigmoid_and_tanh(prob, layout):
    import workloads as wl
    gu = _gpu()
    N, C, H, W, K, R, workspace = prob
    x = np.zeros((N, C, H, W), dtype=np.float32)
    x[:, 0] = _arguments(N * H * W).reshape(N, H, W)
    w = np.zeros((K, C, R, R), dtype=np.float32)
    w[:, 0, R // 2, R // 2] = 1.0
    if R > 1:   # (a tap of zero times an infinity or NaN is NaN: finite values only)
        x = np.nan_to_num(x, nan=0.5, posinf=150.0, neginf=-150.0)
    g = gu.GpuConv(wl.with_layout(x, layout), w, (R // 2, R // 2), (1, 1), 1, y_layout=layout)
    if workspace:
        g.lend_workspace(workspace)
    v = np.broadcast_to(x[:, :1].astype(np.float64), (N, K, H, W))
    with np.errstate(over="ignore"):
        for act, want in ((0, 1.0 / (1.0 + np.exp(-v))), (2, np.tanh(v))):
            g.prefill(value=float("nan"))
            print(prob, layout, act, flush=True)
            g.launch_fused(1.0, 0.0, None, act)
            got = g.result()
            assert np.array_equal(np.isnan(got), np.isnan(want))
            ok = ~np.isnan(want)
            err = np.abs(got - want)[ok]
            if act == 0:
                # exp: half a unit of x * log2(e) (|x| * 2^-24 of the result), log2(e) as a float (off by 1.34e-8 = 0.23 * 2^-24
                # of itself: another 0.23 |x| * 2^-24) and one unit of its own, the addition, the quotient; beyond 88.7 exp(-x) is infinite and the result 0 instead of less than 2^-127
                bound = np.where(v < -88.7, 2.0 ** -127, (1.23 * np.minimum(np.abs(v), 100.0) + 5.0) * 2.0 ** -24 * want + 2.0 ** -149)[ok]
            else:
                bound = np.full(err.shape, 4 * 2.0 ** -24)   # (the same through (1 - e) / (1 + e), where e * |x| < 1)
            assert np.all(err <= bound), (act, float((err / bound).max()), v[ok][np.argmax(err / bound)])
