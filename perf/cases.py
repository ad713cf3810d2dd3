"""Performance cases: the fixed-point layers and whole forwards that programs call this library for.

Every case is a plain dict.  prepare() makes what a program holds before the call (seeded integer tensors on the
GPU, a prepared Chain, a captured graph), run() is one pass through the public entry points of
paper_2202_05239_amd.binding, exact() the same integers in 64-bit torch.  The arithmetic is integer from end to end,
so every output has exactly one right value.
"""
import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2202_05239_amd import binding, workloads

NETS = {"resnet18": workloads.config3, "resnet50": workloads.config4, "resnet50_private": workloads.resnet50_private_fl,
        "mobilenet_v1": workloads.mobilenet_v1_forward, "mobilenet_v2": workloads.mobilenet_v2_forward}


def listed():
    return [
        # the smallest call: one GEMM of a single small layer, nothing but latency
        dict(name="gemm_256x64x64", kind="gemm", M=256, K=64, N=64, x_type="u8", y_type="u8", fl_x=4, fl_w=7, fl_y=4),
        # the classifier of ResNet-50 on a serving batch: pooled features to raw 32-bit logits
        dict(name="gemm_classifier", kind="gemm", M=64, K=2048, N=1000, x_type="u8", y_type="s32", fl_x=5, fl_w=8, fl_y=5),
        # one ResNet-18 style 3x3 layer called on its own
        dict(name="conv3x3_b32", kind="conv", B=32, H=56, W=56, Cin=64, Cout=64, k=3, stride=1, x_type="u8", y_type="u8",
             res="", dual=False, fl_x=5, fl_w=8, fl_y=5),
        # a layer of a network with widths that are no multiples of anything, on images of odd sizes, signed activations
        dict(name="conv3x3_ragged", kind="conv", B=9, H=37, W=53, Cin=42, Cout=70, k=3, stride=2, x_type="s8", y_type="s8",
             res="", dual=False, fl_x=4, fl_w=7, fl_y=4),
        # the layer that closes a bottleneck block: residual in, one output format per child
        dict(name="conv1x1_res_dual", kind="conv", B=64, H=14, W=14, Cin=256, Cout=1024, k=1, stride=1, x_type="u8", y_type="u8",
             res="u8", dual=True, fl_x=5, fl_w=8, fl_y=5),
        # the depthwise layer of a MobileNetV2 block
        dict(name="dwconv3x3_b64", kind="dwconv", B=64, H=56, W=56, C=144, stride=1, x_type="u8", y_type="u8", fl_x=5, fl_w=6, fl_y=5),
        # float images to the network's 8-bit input codes
        dict(name="input_codes_b64", kind="codes", n=64 * 224 * 224 * 3, fl=5, signed=True),
        # one image through ResNet-50, captured once: a service that answers requests one by one
        dict(name="resnet50_b1", kind="net", net="resnet50", batch=1, hw=224, streams=1, graph=True),
        # a small serving batch, every block output in two formats
        dict(name="resnet50_private_b16", kind="net", net="resnet50_private", batch=16, hw=224, streams=1, graph=False),
        # ResNet-18 at its evaluation batch
        dict(name="resnet18_b64", kind="net", net="resnet18", batch=64, hw=224, streams=1, graph=False),
        # a mobile network on a batch that divides by nothing
        dict(name="mobilenet_v2_b27", kind="net", net="mobilenet_v2", batch=27, hw=224, streams=1, graph=False),
        # the throughput run: ResNet-50 at batch 256, both halves of the batch side by side, captured
        dict(name="resnet50_b256", kind="net", net="resnet50", batch=256, hw=224, streams=2, graph=True),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _width(rng, lo, hi):
    """A channel count: mostly a multiple of 16 or 8, as networks have them, otherwise any number."""
    n, u = _log(rng, lo, hi), rng.random()
    step = 16 if u < 0.5 else 8 if u < 0.75 else 1
    return max(step, n // step * step)


def _formats(rng):
    fl_x, fl_w = rng.randint(3, 6), rng.randint(6, 9)
    return dict(fl_x=fl_x, fl_w=fl_w, fl_y=rng.randint(3, 6))


def draw(rng):
    u = rng.random()
    x_type = rng.choice(("u8", "u8", "s8"))
    if u < 0.15:
        return dict(kind="gemm", M=_log(rng, 1, 4096), K=_width(rng, 16, 4096), N=_width(rng, 10, 4096), x_type=x_type,
                    y_type=rng.choice(("u8", "s8", "s32")), **_formats(rng))
    if u < 0.40:
        while True:
            c = dict(kind="conv", B=_log(rng, 1, 128), H=_log(rng, 7, 112), W=_log(rng, 7, 112), Cin=_width(rng, 8, 512),
                     Cout=_width(rng, 8, 1024), k=rng.choice((1, 1, 3, 3, 3, 5)), stride=rng.choice((1, 1, 2)), x_type=x_type,
                     y_type=rng.choice(("u8", "u8", "s8")), res=rng.choice(("", "", "u8", "s8")), dual=rng.random() < 0.2, **_formats(rng))
            w = work(c)
            if w["flops"] < 6e10 and w["bytes"] < 2e8:
                return c
    if u < 0.50:
        return dict(kind="dwconv", B=_log(rng, 1, 64), H=_log(rng, 7, 112), W=_log(rng, 7, 112), C=_width(rng, 16, 512),
                    stride=rng.choice((1, 2)), x_type=x_type, y_type=rng.choice(("u8", "u8", "s8")), **_formats(rng))
    if u < 0.60:
        return dict(kind="codes", n=_log(rng, 1000, 256 * 224 * 224 * 3), fl=rng.randint(3, 7), signed=rng.random() < 0.5)
    return dict(kind="net", net=rng.choice(sorted(NETS)), batch=_log(rng, 1, 192), hw=rng.choice((96, 128, 160, 192, 199, 224)),
                streams=rng.choice((1, 1, 2)), graph=rng.random() < 0.5)


def _out(n, k, stride, pad):
    return (n + 2 * pad - k) // stride + 1


def _operands(case, seed):
    """What the single layers take, as numpy arrays: x, w, bias, residual, and the quantisation record."""
    rng = np.random.default_rng([seed, 1])
    kind = case["kind"]
    q = SimpleNamespace(fl_x=case["fl_x"], fl_w=case["fl_w"], fl_y=case["fl_y"], x_type=case["x_type"], y_type=case["y_type"],
                        clip_lo=0 if case["y_type"] != "s8" else -127, clip_hi=255 if case["y_type"] != "s8" else 127)
    if kind == "gemm":
        xs, ws, n, K = (case["M"], case["K"]), (case["N"], case["K"]), case["N"], case["K"]
    elif kind == "conv":
        k = case["k"]
        xs, ws, n, K = (case["B"], case["H"], case["W"], case["Cin"]), (case["Cout"], k, k, case["Cin"]), case["Cout"], k * k * case["Cin"]
    else:
        xs, ws, n, K = (case["B"], case["H"], case["W"], case["C"]), (3, 3, case["C"]), case["C"], 9
    # post-ReLU activations are half-normal codes, linear ones normal
    x = rng.standard_normal(xs, dtype=np.float32) * np.float32(2.0 ** case["fl_x"])
    x = np.clip(np.rint(np.abs(x)), 0, 255).astype(np.uint8) if case["x_type"] == "u8" else np.clip(np.rint(x), -127, 127).astype(np.int8)
    w = workloads.draw_weight(rng, ws, math.sqrt(2.0 / K), case["fl_w"])
    bias = workloads.draw_bias(rng, n, case["fl_x"] + case["fl_w"])
    res = None
    if kind == "conv":
        pad = case["k"] // 2
        ys = (case["B"], _out(case["H"], case["k"], case["stride"], pad), _out(case["W"], case["k"], case["stride"], pad), n)
        if case["res"]:
            q.res_type, q.fl_res = case["res"], case["fl_y"]
            res = rng.integers(0, 128, ys).astype(np.uint8) if case["res"] == "u8" else rng.integers(-127, 128, ys).astype(np.int8)
        if case["dual"]:
            q.fl_y2, q.clip_lo2, q.clip_hi2, q.y2_type = case["fl_y"] - 1, q.clip_lo, q.clip_hi, case["y_type"]
    return x, w, bias, res, q


def _images(case, seed):
    return np.random.default_rng([seed, 2]).standard_normal(case["n"], dtype=np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "net":
        x, net = NETS[case["net"]](seed=seed, batch=case["batch"], hw=case["hw"])
        chain = binding.Chain(net, streams=case["streams"]).prepare(case["batch"])
        x = torch.from_numpy(x).cuda()
        out = torch.empty((case["batch"],) + chain.out_shape, dtype=chain.out_dtype, device="cuda")
        graph = chain.capture(x, out) if case["graph"] else None
        return dict(kind=kind, chain=chain, x=x, out=out, graph=graph)
    if kind == "codes":
        x = torch.from_numpy(_images(case, seed)).cuda()
        out = torch.empty(case["n"], dtype=torch.int8 if case["signed"] else torch.uint8, device="cuda")
        return dict(kind=kind, x=x, out=out, fl=case["fl"], signed=case["signed"])
    x, w, bias, res, q = _operands(case, seed)
    x, w, bias, res = (None if a is None else torch.from_numpy(a).cuda() for a in (x, w, bias, res))
    dtype = binding.TORCH_DTYPE[case["y_type"]]
    st = dict(kind=kind, x=x, w=w, bias=bias, res=res, q=q, y2=None)
    if kind == "gemm":
        ys = (case["M"], case["N"])
    else:
        k, stride = (case["k"] if kind == "conv" else 3), case["stride"]
        st["stride"], st["pad"] = (stride, stride), (k // 2, k // 2)
        ys = (case["B"], _out(case["H"], k, stride, k // 2), _out(case["W"], k, stride, k // 2), bias.numel())
        if kind == "conv" and case["dual"]:
            st["y2"] = torch.empty(ys, dtype=dtype, device="cuda")
    st["y"] = torch.empty(ys, dtype=dtype, device="cuda")
    return st


def run(state):
    s = state
    if s["kind"] == "net":
        if s["graph"] is None:
            return s["chain"].run(s["x"], s["out"])
        s["graph"].replay()
        return s["out"]
    if s["kind"] == "codes":
        return binding.f8_fix_quant_code(s["x"], s["fl"], s["signed"], out=s["out"])
    if s["kind"] == "gemm":
        return binding.f8_gemm_fixed(s["x"], s["w"], s["bias"], s["y"], s["q"])
    if s["kind"] == "dwconv":
        return binding.f8_dwconv_fixed(s["x"], s["w"], s["bias"], s["y"], s["q"], s["stride"], s["pad"])
    if s["y2"] is not None:
        return binding.f8_conv2d_fixed_dual(s["x"], s["w"], s["bias"], s["y"], s["y2"], s["q"], s["stride"], s["pad"], s["res"])
    return binding.f8_conv2d_fixed(s["x"], s["w"], s["bias"], s["y"], s["q"], s["stride"], s["pad"], s["res"])


@functools.lru_cache(maxsize=None)
def _net_size(name, hw):
    """(multiply-accumulates and input bytes of an image, bytes of the weights and biases)."""
    x, net = NETS[name](seed=1, batch=1, hw=hw)
    weights = sum((0 if L.w is None else L.w.nbytes) + (0 if L.bias is None else L.bias.nbytes) for L in net.layers)
    return net.macs_per_image, x.nbytes, weights


def work(case):
    kind = case["kind"]
    if kind == "net":
        macs, image, weights = _net_size(case["net"], case["hw"])
        return {"bytes": case["batch"] * (image + 4 * 1000) + weights, "flops": 2 * macs * case["batch"]}
    if kind == "codes":
        return {"bytes": 5 * case["n"], "flops": 0}
    if kind == "gemm":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": M * K + N * K + 4 * N + M * N * (4 if case["y_type"] == "s32" else 1), "flops": 2 * M * K * N}
    k, stride = (case["k"] if kind == "conv" else 3), case["stride"]
    P, Q = _out(case["H"], k, stride, k // 2), _out(case["W"], k, stride, k // 2)
    M = case["B"] * P * Q
    # a strided 1x1 layer reads only the pixels that it uses
    pixels = M if k < stride else case["B"] * case["H"] * case["W"]
    if kind == "dwconv":
        return {"bytes": (pixels + M) * case["C"] + 13 * case["C"], "flops": 18 * M * case["C"]}
    K, N = k * k * case["Cin"], case["Cout"]
    outs = 1 + bool(case["res"]) + bool(case["dual"])
    return {"bytes": pixels * case["Cin"] + outs * M * N + N * K + 4 * N, "flops": 2 * M * K * N}


def tolerance(case):
    return "exact"


# ---- the same integers in 64-bit torch (every value below 2^53, so float64 holds them exactly) ----

def _shift_round(a, s):
    return torch.floor((a + 2.0 ** (s - 1)) * 2.0 ** -s) if s >= 1 else a * 2.0 ** -s


def _window(x, r, s, stride, P, Q):
    return x[:, r:r + (P - 1) * stride + 1:stride, s:s + (Q - 1) * stride + 1:stride]


def _layer(x, w, bias, L, res, depthwise, R, S, stride, pad):
    """x [B][H][W][C] float64 on the GPU; returns the accumulator [B][P][Q][N] with bias and residual."""
    B, H, W, C = x.shape
    P, Q = _out(H, R, stride, pad), _out(W, S, stride, pad)
    if pad:
        x = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    acc = None
    for r in range(R):
        for s in range(S):
            t = _window(x, r, s, stride, P, Q)
            t = t * w[r, s] if depthwise else torch.mm(t.reshape(B * P * Q, C), w[:, r, s, :].t().contiguous())
            acc = t if acc is None else acc.add_(t)
    acc = acc.reshape(B, P, Q, -1)
    if bias is not None:
        acc = acc + bias
    if res is not None:
        acc = acc + _shift_round(res, L.fl_res - L.fl_x - L.fl_w)
    return acc


def _requant(acc, s, lo, hi):
    return _shift_round(acc, s).clamp_(lo, hi)


def _net_exact(x, net, out):
    consts = [None if L.w is None else (torch.from_numpy(L.w).cuda().double(), None if L.bias is None else torch.from_numpy(L.bias).cuda().double())
              for L in net.layers]
    last = {}
    for i, L in enumerate(net.layers):
        last[L.src] = i
        if L.res >= 0:
            last[L.res] = i
    step = 16
    for b in range(0, x.shape[0], step):
        t = {0: torch.from_numpy(x[b:b + step]).cuda().double()}
        for i, L in enumerate(net.layers):
            v = t[L.src]
            if L.op == "maxpool":
                P, Q = L.out_hw
                p = torch.nn.functional.pad(v, (0, 0, L.pad, L.pad, L.pad, L.pad), value=-1e9)
                y = None
                for r in range(L.R):
                    for s in range(L.S):
                        u = _window(p, r, s, L.stride, P, Q)
                        y = u if y is None else torch.maximum(y, u)
            elif L.op == "gpool":
                y = _requant(v.sum(dim=(1, 2), keepdim=True), L.fl_x + L.fl_w - L.fl_y, L.clip_lo, L.clip_hi)
            else:
                w, bias = consts[i]
                acc = _layer(v, w, bias, L, t[L.res] if L.res >= 0 else None, L.op == "dwconv", L.R, L.S, L.stride, L.pad)
                y = acc if L.y_type == "s32" else _requant(acc, L.fl_x + L.fl_w - L.fl_y, L.clip_lo, L.clip_hi)
                if L.dst2 > 0:
                    t[L.dst2] = _requant(acc, L.fl_x + L.fl_w - L.fl_y2, L.clip_lo2, L.clip_hi2)
            t[L.dst] = y
            for k in [k for k in t if last.get(k, len(net.layers)) <= i]:
                del t[k]
        out[b:b + step] = t[net.layers[-1].dst]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "net":
        x, net = NETS[case["net"]](seed=seed, batch=case["batch"], hw=case["hw"])
        L = net.layers[-1]
        return _net_exact(x, net, torch.empty((case["batch"],) + tuple(L.out_hw) + (L.Cout,), dtype=torch.float64, device="cuda")).long()
    if kind == "codes":
        v = torch.from_numpy(_images(case, seed)).cuda().double() * 2.0 ** case["fl"]
        v = v.clamp_(-127, 127) if case["signed"] else v.clamp_(0, 255)
        return torch.floor(v + 0.5).long()
    x, w, bias, res, q = _operands(case, seed)
    x, w, bias, res = (None if a is None else torch.from_numpy(a).cuda().double() for a in (x, w, bias, res))
    if kind == "gemm":
        acc = torch.mm(x, w.t().contiguous()) + bias
    else:
        k = case["k"] if kind == "conv" else 3
        acc = _layer(x, w, bias, q, res, kind == "dwconv", k, k, case["stride"], k // 2)
    if case["y_type"] == "s32":
        return acc.long()
    s = q.fl_x + q.fl_w - q.fl_y
    y = _requant(acc, s, q.clip_lo, q.clip_hi).long()
    if kind == "conv" and case["dual"]:
        return y, _requant(acc, s + 1, q.clip_lo2, q.clip_hi2).long()
    return y
