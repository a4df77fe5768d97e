"""Performance cases: what programs that use this library have it do, through its public entry points.

A case is one pass of a layer (or of one of the other functions) as a training or serving program makes it: the
program holds device buffers, descriptors, a handle and workspaces of the sizes the library's queries report, and calls
the entry points in the order of the layer's forward and backward pass.  Every output the calls leave is returned.

Kinds of pass:
  forward   convolution with bias and rectifier fused into its epilogue (serving)
  train     forward (bias and activation), activation backward, bias gradient, filter gradient and, unless the layer is
            the first of its network, data gradient.  With a `shortcut` a 1x1 convolution over the same input is added
            to the layer (forward accumulates into y, backward data into dx: alpha/beta form).
              float: activation fused, its backward pass from y.  double: bias and activation as separate calls (not fused
              there).  bfloat16: x, w, dy in 16 bits, results float; dy is what the program rounded to 16 bits.
  pool      pooling forward and backward
  softmax   softmax forward and backward
  pointwise layout change, activation forward and backward
"""
import math
import random

import torch

import paper_1410_0759_amd as ig

_DT = {"f32": (ig.IGC_DATA_FLOAT, torch.float32), "bf16": (ig.IGC_DATA_BFLOAT16, torch.bfloat16),
       "f64": (ig.IGC_DATA_DOUBLE, torch.float64)}
_ACT = {"none": ig.IGC_ACTIVATION_IDENTITY, "sigmoid": ig.IGC_ACTIVATION_SIGMOID, "relu": ig.IGC_ACTIVATION_RELU,
        "tanh": ig.IGC_ACTIVATION_TANH}


def _conv(name, kind, dtype, layout, N, C, H, W, K, R, S, pad, stride, act, data_grad=True, shortcut=False, flip=False):
    return {"name": name, "kind": kind, "dtype": dtype, "layout": layout, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R,
            "S": S, "pad_h": pad[0], "pad_w": pad[1], "u": stride[0], "v": stride[1], "act": act, "data_grad": data_grad,
            "shortcut": shortcut, "flip": flip}


def listed():
    return [
        # one small image through a small first layer: the latency of a call
        _conv("tiny_forward", "forward", "f32", "NCHW", 1, 3, 32, 32, 16, 3, 3, (1, 1), (1, 1), "relu"),
        # the last layers of a deep network at a serving mini-batch
        _conv("serving_7x7", "forward", "f32", "NCHW", 4, 512, 7, 7, 512, 3, 3, (1, 1), (1, 1), "relu"),
        # first layer of a large-filter network: three channels, 11x11 taps, stride 4; no gradient of the images
        _conv("first_layer_11x11", "train", "f32", "NCHW", 64, 3, 227, 227, 96, 11, 11, (0, 0), (4, 4), "tanh", data_grad=False),
        # the ordinary 3x3 layer of a training mini-batch
        _conv("mid_3x3", "train", "f32", "NCHW", 128, 64, 56, 56, 64, 3, 3, (1, 1), (1, 1), "tanh"),
        # a deep 3x3 layer on small images with a 1x1 shortcut added to it (y and dx accumulate)
        _conv("deep_3x3_shortcut", "train", "f32", "NCHW", 128, 384, 13, 13, 256, 3, 3, (1, 1), (1, 1), "tanh", shortcut=True),
        # the largest: second layer of the paper's layer collection, 9x9 taps without a border
        _conv("table2_9x9", "train", "f32", "NCHW", 128, 96, 64, 64, 128, 9, 9, (0, 0), (1, 1), "tanh"),
        # nothing divides: odd channels, odd image, stride 2, a ragged mini-batch at the end of an epoch, eq. 2's flipped filter
        _conv("ragged_stride2", "train", "f32", "NCHW", 37, 101, 29, 31, 77, 3, 3, (1, 1), (2, 2), "tanh", flip=True),
        # bfloat16, channels innermost: the ordinary 3x3 layer
        _conv("bf16_3x3", "train", "bf16", "NHWC", 32, 512, 14, 14, 512, 3, 3, (1, 1), (1, 1), "relu"),
        # bfloat16, channels innermost: the layer that halves the image, with its 1x1 shortcut
        _conv("bf16_halving_shortcut", "train", "bf16", "NHWC", 32, 128, 56, 56, 256, 3, 3, (1, 1), (2, 2), "relu", shortcut=True),
        # double precision
        _conv("f64_mid_3x3", "train", "f64", "NCHW", 32, 64, 56, 56, 64, 3, 3, (1, 1), (1, 1), "tanh"),
        # overlapping 3x3 maximum pooling after a rectifier (many equal zeros)
        {"name": "pool_max_3x3", "kind": "pool", "dtype": "f32", "layout": "NCHW", "mode": "max", "N": 128, "C": 96, "H": 55,
         "W": 55, "win": 3, "pad": 0, "stride": 2},
        # per-pixel classification over 21 classes
        {"name": "softmax_pixels", "kind": "softmax", "dtype": "f32", "layout": "NCHW", "mode": "channel", "N": 32, "C": 21,
         "H": 128, "W": 128},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_MAX_FLOPS = 2.4e12     # about the largest listed case's
_MAX_FLOPS_SLOW = 1.0e11   # for double precision and for 16-bit layers


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["forward", "train", "train", "train", "train", "pool", "softmax", "pointwise"])
    if kind == "pool":
        win = rng.choice([2, 3, 3, 5])
        return {"kind": "pool", "dtype": "f32", "layout": rng.choice(["NCHW", "NCHW", "NHWC"]), "mode": rng.choice(["max", "max", "average"]),
                "N": _log_int(rng, 1, 128), "C": _log_int(rng, 3, 256), "H": _log_int(rng, 7, 60), "W": _log_int(rng, 7, 60),
                "win": win, "pad": rng.choice([0, 0, 1]), "stride": rng.choice([1, 2, 2, 3]) if win > 2 else 2}
    if kind == "softmax":
        mode = rng.choice(["channel", "instance"])
        hw = (_log_int(rng, 4, 128), _log_int(rng, 4, 128)) if mode == "channel" else (1, 1)
        return {"kind": "softmax", "dtype": "f32", "layout": "NCHW", "mode": mode, "N": _log_int(rng, 1, 32) if mode == "channel" else
                _log_int(rng, 1, 512), "C": _log_int(rng, 2, 64) if mode == "channel" else _log_int(rng, 10, 4000), "H": hw[0], "W": hw[1]}
    if kind == "pointwise":
        return {"kind": "pointwise", "dtype": rng.choice(["f32", "f32", "f64"]), "layout": rng.choice(["NCHW", "NHWC"]),
                "act": rng.choice(["relu", "tanh", "sigmoid"]), "N": _log_int(rng, 1, 64), "C": _log_int(rng, 3, 256),
                "H": _log_int(rng, 5, 60), "W": _log_int(rng, 5, 60)}
    while True:
        dtype = rng.choice(["f32", "f32", "f32", "bf16", "f64"])
        if kind == "forward":
            dtype = rng.choice(["f32", "f32", "bf16"])
        H = _log_int(rng, 7, 128)
        W = max(5, min(160, int(H * rng.choice([1.0, 1.0, rng.uniform(0.7, 1.4)]))))
        R = rng.choice([1, 3, 3, 3, 5, 7, 9])
        S = rng.choice([R, R, R, R + 2])
        stride = rng.choice([1, 1, 1, 2])
        if R == 1:
            S, pad = 1, (0, 0)
        else:
            pad = rng.choice([(R // 2, S // 2), (R // 2, S // 2), (0, 0)])
        if H + 2 * pad[0] < R or W + 2 * pad[1] < S:
            continue
        C, K = _log_int(rng, 1, 512), _log_int(rng, 8, 512)
        if rng.random() < 0.6:      # most layers have channels in eights or more
            q = rng.choice([8, 16, 32])
            C, K = max(q, C // q * q), max(q, K // q * q)
        case = _conv("", kind, dtype, "NHWC" if dtype == "bf16" else rng.choice(["NCHW", "NCHW", "NCHW", "NHWC"]),
                     _log_int(rng, 1, 8 if kind == "forward" else 128), C, H, W, K, R, S, pad, (stride, stride),
                     "relu" if kind == "forward" or dtype == "bf16" else rng.choice(["tanh", "sigmoid"]),
                     data_grad=rng.random() < 0.8, shortcut=kind == "train" and R % 2 == 1 and S == R and pad == (R // 2, R // 2) and rng.random() < 0.3,
                     flip=rng.random() < 0.2)
        del case["name"]
        w = work(case)
        if w["flops"] <= (_MAX_FLOPS if dtype == "f32" else _MAX_FLOPS_SLOW) and w["bytes"] <= 1.5e9:
            return case


# ---------------------------------------------------------------------------------------------- shapes
def _out(case):
    if case["kind"] == "pool":
        o = lambda n: (n + 2 * case["pad"] - case["win"]) // case["stride"] + 1
        return o(case["H"]), o(case["W"])
    return ((case["H"] + 2 * case["pad_h"] - case["R"]) // case["u"] + 1, (case["W"] + 2 * case["pad_w"] - case["S"]) // case["v"] + 1)


def work(case):
    """Bytes: each input read once, each output written once.  Flops: 2 per multiply-add, zero border counted."""
    k = case["kind"]
    e = {"f32": 4, "bf16": 2, "f64": 8}[case["dtype"]]
    nx = case["N"] * case["C"] * case["H"] * case["W"]
    if k == "pool":
        P, Q = _out(case)
        ny = case["N"] * case["C"] * P * Q
        # x; y; dy and dx (the backward pass takes its maximum from x: read once)
        return {"bytes": e * (2 * nx + 2 * ny), "flops": 2 * ny * case["win"] ** 2}
    if k == "softmax":
        return {"bytes": e * 4 * nx, "flops": 8 * nx}
    if k == "pointwise":
        return {"bytes": e * 5 * nx, "flops": 8 * nx}
    P, Q = _out(case)
    ny = case["N"] * case["K"] * P * Q
    taps = case["R"] * case["S"] + (1 if case["shortcut"] else 0)
    nw = case["K"] * case["C"] * taps
    eo = 8 if case["dtype"] == "f64" else 4
    passes, b = 1, e * (nx + nw) + eo * (ny + case["K"])
    if k == "train":
        passes = 3 if case["data_grad"] else 2
        b += e * ny + eo * (nw + case["K"]) + (eo * nx if case["data_grad"] else 0)
    return {"bytes": b, "flops": 2 * ny * case["C"] * taps * passes}


# ---------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _memory(t, layout):
    """The same logical (N,C,H,W) tensor with its memory in the given order."""
    return t.contiguous() if layout == "NCHW" else t.permute(0, 2, 3, 1).contiguous().permute(0, 3, 1, 2)


def _empty(shape, layout, dtype):
    if layout == "NCHW":
        return torch.empty(shape, dtype=dtype, device="cuda")
    n, c, h, w = shape
    return torch.empty((n, h, w, c), dtype=dtype, device="cuda").permute(0, 3, 1, 2)


def _rounded(t, dtype):
    return t.to(torch.bfloat16) if dtype == "bf16" else t.to(_DT[dtype][1])


def _inputs(case, seed):
    """The arrays a pass reads, in their data type (logical NCHW / KCRS)."""
    g = _gen(seed)
    d = torch.float64 if case["dtype"] == "f64" else torch.float32
    xs = (case["N"], case["C"], case["H"], case["W"])
    uni = lambda s: torch.rand(s, generator=g, device="cuda", dtype=d) * 2 - 1
    nrm = lambda s, std: torch.randn(s, generator=g, device="cuda", dtype=d) * std
    k = case["kind"]
    if k == "pool":      # feature maps after a rectifier
        P, Q = _out(case)
        return {"x": torch.relu(nrm(xs, 1.0)), "dy": nrm((xs[0], xs[1], P, Q), 0.1)}
    if k in ("softmax", "pointwise"):
        return {"x": nrm(xs, 2.0), "dy": nrm(xs, 0.1)}
    C, K, R, S = case["C"], case["K"], case["R"], case["S"]
    P, Q = _out(case)
    a = {"x": _rounded(uni(xs) if C > 4 else (uni(xs) + 1) / 2, case["dtype"]),     # images lie in [0, 1]
         "w": _rounded(nrm((K, C, R, S), math.sqrt(2.0 / (C * R * S))), case["dtype"]), "bias": nrm((K,), 0.1)}
    if case["shortcut"]:
        a["w1"] = _rounded(nrm((K, C, 1, 1), math.sqrt(1.0 / C)), case["dtype"])
    if case["kind"] == "train":
        a["dy"] = _rounded(nrm((case["N"], K, P, Q), 0.1), case["dtype"])
    return a


# ---------------------------------------------------------------------------------------------- state
class _Workspace:
    """Device memory of the largest size the layer's queries report."""

    def __init__(self, sizes):
        self.bytes = max(sizes)
        self.buf = torch.empty((self.bytes + 3) // 4, dtype=torch.float32, device="cuda") if self.bytes else None
        self.ptr = self.buf.data_ptr() if self.bytes else 0


def prepare(case, seed):
    s = {"case": case, "handle": ig.Handle()}
    s["handle"].set_stream(torch.cuda.current_stream().cuda_stream)
    a = _inputs(case, seed)
    lay = case["layout"]
    k = case["kind"]
    desc = ig.tensor_descriptor_for
    if k in ("pool", "softmax", "pointwise"):
        s["x"], s["dy"] = _memory(a["x"], lay), _memory(a["dy"], lay)
        s["y"] = _empty(s["dy"].shape, lay, s["x"].dtype)
        s["dx"] = _empty(s["x"].shape, lay, s["x"].dtype)
        if k == "pool":
            s["pool"] = ig.PoolingDescriptor().set(ig.IGC_POOLING_MAX if case["mode"] == "max" else ig.IGC_POOLING_AVERAGE, case["win"],
                                                   case["win"], case["pad"], case["pad"], case["stride"], case["stride"])
        if k == "pointwise":
            s["t"] = _empty(s["x"].shape, "NHWC" if lay == "NCHW" else "NCHW", s["x"].dtype)
            s["td"] = desc(s["t"])
            s["y"], s["dx"] = torch.empty_like(s["t"]), torch.empty_like(s["t"])
            s["dy"] = _memory(a["dy"], "NHWC" if lay == "NCHW" else "NCHW")
        s["xd"], s["dyd"], s["yd"], s["dxd"] = desc(s["x"]), desc(s["dy"]), desc(s["y"]), desc(s["dx"])
        return s

    dt, tt = _DT[case["dtype"]]
    ot = torch.float64 if case["dtype"] == "f64" else torch.float32
    odt = ig.IGC_DATA_DOUBLE if case["dtype"] == "f64" else ig.IGC_DATA_FLOAT
    C, K, R, S = case["C"], case["K"], case["R"], case["S"]
    P, Q = _out(case)
    h = s["handle"]
    s["x"], s["w"], s["bias"] = _memory(a["x"], lay), a["w"].contiguous(), a["bias"].to(ot)
    s["y"] = _empty((case["N"], K, P, Q), lay, ot)
    s["xd"], s["yd"] = desc(s["x"]), desc(s["y"])
    mode = ig.IGC_CONVOLUTION if case["flip"] else ig.IGC_CROSS_CORRELATION
    s["branches"] = [(ig.FilterDescriptor().set(dt, K, C, R, S), s["w"],
                      ig.ConvolutionDescriptor().set(case["pad_h"], case["pad_w"], case["u"], case["v"], mode))]
    if case["shortcut"]:
        s["w1"] = a["w1"].contiguous()
        s["branches"].append((ig.FilterDescriptor().set(dt, K, C, 1, 1), s["w1"], ig.ConvolutionDescriptor().set(0, 0, case["u"], case["v"], mode)))
    sizes = [ig.get_optional_workspace_size(h, s["xd"], wd, cd, s["yd"]) for wd, _, cd in s["branches"]]
    s["bd"] = ig.TensorDescriptor().set(odt, 1, K, 1, 1, (K, 1, 1, 1))
    if case["kind"] == "train":
        s["dy"] = _memory(a["dy"], lay)
        s["dyd"] = desc(s["dy"])
        s["dz"] = s["dy"] if case["dtype"] == "bf16" else torch.empty_like(s["y"])
        s["dzd"] = desc(s["dz"])
        s["db"] = torch.empty(K, dtype=ot, device="cuda")
        s["dw"] = [torch.empty(w.shape, dtype=ot, device="cuda") for _, w, _ in s["branches"]]
        s["dwd"] = [ig.FilterDescriptor().set(odt, *w.shape) for _, w, _ in s["branches"]]
        sizes.append(ig.get_backward_bias_workspace_size(h, s["dzd"], s["bd"]))
        sizes += [ig.get_backward_filter_workspace_size(h, s["xd"], s["dzd"], cd, dwd) for (_, _, cd), dwd in zip(s["branches"], s["dwd"])]
        if case["data_grad"]:
            s["dx"] = _empty(s["x"].shape, lay, ot)
            s["dxd"] = desc(s["dx"])
            sizes += [ig.get_backward_data_workspace_size(h, wd, s["dzd"], cd, s["dxd"]) for wd, _, cd in s["branches"]]
    s["ws"] = _Workspace(sizes)
    return s


# ---------------------------------------------------------------------------------------------- the pass
def run(s):
    case, h = s["case"], s["handle"]
    k, ok = case["kind"], ig.check
    x, y = s["x"].data_ptr(), s["y"].data_ptr()
    if k == "pool":
        ok(ig.pooling_forward(h, s["pool"], 1.0, s["xd"], x, 0.0, s["yd"], y))
        ok(ig.pooling_backward(h, s["pool"], 1.0, s["dyd"], s["dy"].data_ptr(), s["xd"], x, 0.0, s["dxd"], s["dx"].data_ptr()))
        return {"y": s["y"], "dx": s["dx"]}
    if k == "softmax":
        mode = ig.IGC_SOFTMAX_MODE_CHANNEL if case["mode"] == "channel" else ig.IGC_SOFTMAX_MODE_INSTANCE
        ok(ig.softmax_forward(h, mode, 1.0, s["xd"], x, 0.0, s["yd"], y))
        ok(ig.softmax_backward(h, mode, 1.0, s["yd"], y, s["dyd"], s["dy"].data_ptr(), 0.0, s["dxd"], s["dx"].data_ptr()))
        return {"y": s["y"], "dx": s["dx"]}
    if k == "pointwise":
        m, t = _ACT[case["act"]], s["t"].data_ptr()
        ok(ig.transform_tensor(h, 1.0, s["xd"], x, 0.0, s["td"], t))
        ok(ig.activation_forward(h, m, 1.0, s["td"], t, 0.0, s["yd"], y))
        ok(ig.activation_backward(h, m, 1.0, s["yd"], y, s["dyd"], s["dy"].data_ptr(), s["td"], t, 0.0, s["dxd"], s["dx"].data_ptr()))
        return {"t": s["t"], "y": s["y"], "dx": s["dx"]}

    ws, wsb, act = s["ws"].ptr, s["ws"].bytes, _ACT[case["act"]]
    wd, w, cd = s["branches"][0]
    beta = 0.0
    if case["shortcut"]:
        wd1, w1, cd1 = s["branches"][1]
        ok(ig.convolution_forward(h, 1.0, s["xd"], x, wd1, w1.data_ptr(), cd1, 0.0, s["yd"], y, ws, wsb))
        beta = 1.0
    if case["dtype"] == "f64":
        ok(ig.convolution_forward(h, 1.0, s["xd"], x, wd, w.data_ptr(), cd, beta, s["yd"], y, ws, wsb))
        ok(ig.add_tensor(h, 1.0, s["bd"], s["bias"].data_ptr(), 1.0, s["yd"], y))
        ok(ig.activation_forward(h, act, 1.0, s["yd"], y, 0.0, s["yd"], y))
    else:
        ok(ig.convolution_bias_activation_forward(h, 1.0, s["xd"], x, wd, w.data_ptr(), cd, beta, s["bias"].data_ptr(), act, s["yd"], y, ws, wsb))
    if k == "forward":
        return {"y": s["y"]}
    dz = s["dz"].data_ptr()
    if case["dtype"] != "bf16":     # (sigmoid and tanh: the derivative comes from y)
        ok(ig.activation_backward(h, act, 1.0, s["yd"], y, s["dyd"], s["dy"].data_ptr(), s["yd"], y, 0.0, s["dzd"], dz))
    ok(ig.convolution_backward_bias(h, 1.0, s["dzd"], dz, 0.0, s["bd"], s["db"].data_ptr(), ws, wsb))
    out = {"y": s["y"], "db": s["db"], "dw": s["dw"]}
    for i, (wd, w, cd) in enumerate(s["branches"]):
        ok(ig.convolution_backward_filter(h, 1.0, s["xd"], x, s["dzd"], dz, cd, 0.0, s["dwd"][i], s["dw"][i].data_ptr(), ws, wsb))
        if case["data_grad"]:
            ok(ig.convolution_backward_data(h, 1.0, wd, w.data_ptr(), s["dzd"], dz, cd, 1.0 if i else 0.0, s["dxd"], s["dx"].data_ptr(), ws, wsb))
    if case["data_grad"]:
        out["dx"] = s["dx"]
    return out


# ---------------------------------------------------------------------------------------------- what is right
def tolerance(case):
    """Four times what the same sums in another order (this library's kernels forced one after the other, or the 64-bit
    result) differ by.  float convolutions: 32-bit sums; bfloat16 inputs are summed in 32 bits as well; the rectifier of a
    16-bit layer is the last step of y, so nothing is amplified."""
    if case["dtype"] == "f64":
        return {"rel": 1e-13, "max": 1e-10}
    if case["kind"] == "pool" and case["mode"] == "max":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 1e-5, "max": 2e-4}


def _conv64(x, w, pad, stride, flip, shape):
    """Convolution in 64 bits, tap by tap (each tap is a matrix product)."""
    N, K, P, Q = shape
    y = torch.zeros((N, K, P * Q), dtype=torch.float64, device=x.device)
    for r, s, patch in _patches(x, w.shape[2], w.shape[3], pad, stride, flip, P, Q):
        y += torch.matmul(w[:, :, r, s].contiguous(), patch)
    return y.reshape(shape)


def _window(r, s, R, S, stride, flip, P, Q):
    tr, ts = (R - 1 - r, S - 1 - s) if flip else (r, s)
    return slice(tr, tr + stride[0] * (P - 1) + 1, stride[0]), slice(ts, ts + stride[1] * (Q - 1) + 1, stride[1])


def _patches(x, R, S, pad, stride, flip, P, Q):
    xp = torch.nn.functional.pad(x, (pad[1], pad[1], pad[0], pad[0]))
    for r in range(R):
        for s in range(S):
            a, b = _window(r, s, R, S, stride, flip, P, Q)
            yield r, s, xp[:, :, a, b].reshape(x.shape[0], x.shape[1], P * Q)


def _softmax64(x, dim):
    e = torch.exp(x - x.amax(dim, keepdim=True))
    return e / e.sum(dim, keepdim=True)


def exact(case, seed):
    a = {n: t.double() for n, t in _inputs(case, seed).items()}
    k = case["kind"]
    if k == "softmax":
        dim = 1 if case["mode"] == "channel" else (1, 2, 3)
        y = _softmax64(a["x"], dim)
        return {"y": y, "dx": y * (a["dy"] - (a["dy"] * y).sum(dim, keepdim=True))}
    if k == "pointwise":
        x = a["x"]
        y = {"relu": torch.relu, "tanh": torch.tanh, "sigmoid": torch.sigmoid}[case["act"]](x)
        d = {"relu": (x > 0).double(), "tanh": 1 - y * y, "sigmoid": y * (1 - y)}[case["act"]]
        return {"t": x, "y": y, "dx": a["dy"] * d}
    if k == "pool":
        return _pool64(case, a["x"], a["dy"])
    if work(case)["flops"] > 5e12:
        return None
    pad, stride, flip = (case["pad_h"], case["pad_w"]), (case["u"], case["v"]), case["flip"]
    P, Q = _out(case)
    shape = (case["N"], case["K"], P, Q)
    z = _conv64(a["x"], a["w"], pad, stride, flip, shape)
    if case["shortcut"]:
        z += _conv64(a["x"], a["w1"], (0, 0), stride, flip, shape)
    y = {"relu": torch.relu, "tanh": torch.tanh, "sigmoid": torch.sigmoid}[case["act"]](z + a["bias"][None, :, None, None])
    if k == "forward":
        return {"y": y}
    dz = a["dy"]
    if case["dtype"] != "bf16":
        dz = dz * ((1 - y * y) if case["act"] == "tanh" else y * (1 - y))
    out = {"y": y, "db": dz.sum((0, 2, 3)), "dw": []}
    rows = dz.reshape(shape[0], shape[1], P * Q).permute(1, 0, 2).reshape(shape[1], -1)
    dx = torch.zeros_like(a["x"])
    for w, pd in [(a["w"], pad)] + ([(a["w1"], (0, 0))] if case["shortcut"] else []):
        R, S = w.shape[2:]
        dw = torch.empty_like(w)
        for r, s, patch in _patches(a["x"], R, S, pd, stride, flip, P, Q):
            dw[:, :, r, s] = rows @ patch.permute(1, 0, 2).reshape(case["C"], -1).t()
        out["dw"].append(dw)
        if case["data_grad"]:
            full = torch.zeros((case["N"], case["C"], case["H"] + 2 * pd[0], case["W"] + 2 * pd[1]), dtype=torch.float64, device=dz.device)
            for r in range(R):
                for s in range(S):
                    sl = _window(r, s, R, S, stride, flip, P, Q)
                    full[:, :, sl[0], sl[1]] += torch.matmul(w[:, :, r, s].t().contiguous(), dz.reshape(shape[0], shape[1], -1)).reshape(
                        case["N"], case["C"], P, Q)
            dx += full[:, :, pd[0]:pd[0] + case["H"], pd[1]:pd[1] + case["W"]]
    if case["data_grad"]:
        out["dx"] = dx
    return out


def _pool64(case, x, dy):
    P, Q = _out(case)
    win, pad, st = case["win"], case["pad"], (case["stride"], case["stride"])
    big = case["mode"] == "max"
    xp = torch.nn.functional.pad(x, (pad,) * 4, value=-math.inf if big else 0.0)
    inside = torch.nn.functional.pad(torch.ones_like(x[:1, :1]), (pad,) * 4)
    taps = [_window(r, s, win, win, st, False, P, Q) for r in range(win) for s in range(win)]
    full = torch.zeros_like(xp)
    if big:     # the first of equal maxima in scan order
        best = torch.full(dy.shape, -math.inf, dtype=torch.float64, device=x.device)
        where = torch.zeros(dy.shape, dtype=torch.int16, device=x.device)
        for i, (a, b) in enumerate(taps):
            more = xp[:, :, a, b] > best
            best = torch.where(more, xp[:, :, a, b], best)
            where = torch.where(more, torch.full_like(where, i), where)
        for i, (a, b) in enumerate(taps):
            full[:, :, a, b] += torch.where(where == i, dy, torch.zeros_like(dy))
        y = best
    else:
        count = sum(inside[:, :, a, b] for a, b in taps)
        y = sum(xp[:, :, a, b] for a, b in taps) / count
        for a, b in taps:
            full[:, :, a, b] += dy / count
    return {"y": y, "dx": full[:, :, pad:pad + case["H"], pad:pad + case["W"]]}
