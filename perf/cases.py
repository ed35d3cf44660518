"""Performance cases of the masked linear layer, its schedules and its quantizers.

Each case is a dict of plain values.  Its ``kind`` names the public entry
points that a pass goes through:

  linear    masked_linear on activation codes
  conv      masked_conv3x3 on an NHWC image
  schedule  run_schedule over blocks of layers, several denoising steps
  act       quantize_activations_batch over the inputs of a block
  layer     fp32 activations -> codes (and low-rank branch) -> masked_linear
  weights   the offline path: quantize_weights, the packers, weight_colsums

``block`` names the layer shapes of a transformer or UNet block (the ones
that inputs.py's workloads have), ``weights`` the stored copies that the
caller keeps: "rows", "packed", or "all" (rows, packed and bit planes).
"""
from __future__ import annotations

import torch

import paper_2608_03057_amd as tasq

DEV = "cuda:0"

# (N, K) of the linear layers of one block, in order.
BLOCKS = {
    "pixart": [(3456, 1152), (1152, 1152), (4608, 1152), (1152, 4608)],
    "sana": [(6720, 2240), (2240, 2240), (11200, 2240), (2240, 5600)],
}
# The UNet block: (tokens, N, K) of its linears at two resolutions, then one
# 3x3 conv (H, W, C, N).
UNET_LINEARS = [(4096, 1920, 640), (4096, 640, 640), (4096, 5120, 640), (4096, 640, 2560),
                (1024, 3840, 1280), (1024, 1280, 1280), (1024, 10240, 1280),
                (1024, 1280, 5120)]
UNET_CONV = (32, 32, 1280, 1280)

# Output widths of the blocks' layers; drawn sizes come from these as well.
WIDTHS = [640, 1152, 1280, 1920, 2240, 3456, 3840, 4608, 5120, 5600, 6720, 10240, 11200]


def listed():
    return [
        # One projection of a 256-token image (256x256 pixels): the smallest
        # GEMM call, where latency counts.
        dict(name="linear_256", kind="linear", M=256, N=1152, K=1152, b=6, weights="rows",
             bias=False),
        # QKV projection of a 1024-pixel image pair, weight kept as it is
        # stored.
        dict(name="linear_8192", kind="linear", M=8192, N=3456, K=1152, b=5, weights="rows",
             bias=False),
        # The widest layer of the DiT blocks (GLU up projection at four
        # images), weight kept in the packed order.
        dict(name="linear_packed_4096", kind="linear", M=4096, N=11200, K=2240, b=7,
             weights="packed", bias=True),
        # Sizes that divide nothing: text tokens through an odd-sized layer.
        dict(name="linear_ragged", kind="linear", M=777, N=1111, K=1153, b=5, weights="rows",
             bias=True),
        # Few tokens in flight (an embedding or modulation layer, a small
        # batch): a weight stream, every stored copy at hand.
        dict(name="linear_few_tokens", kind="linear", M=16, N=4608, K=1152, b=4, weights="all",
             bias=True),
        # The UNet's 3x3 conv at 32x32 pixels with its split-K workspace.
        dict(name="conv_32x32", kind="conv", H=32, W=32, C=1280, N=1280, b=4, bias=True),
        # A UNet block (linears at two resolutions and a conv) over a
        # distilled model's four steps, one stage per step.
        dict(name="schedule_unet", kind="schedule", block="unet", blocks=1, M=0, S=4, T=4,
             b_lo=4, b_hi=8, weights="rows"),
        # The whole 28-block model at two 1024-pixel images, 20 steps in four
        # stages: the benchmark workload.
        dict(name="schedule_28_blocks", kind="schedule", block="pixart", blocks=28, M=8192, S=4,
             T=20, b_lo=2, b_hi=8, weights="rows"),
        # The same model with 16 tokens in flight: bit-plane streams.
        dict(name="schedule_16_tokens", kind="schedule", block="pixart", blocks=28, M=16, S=4,
             T=20, b_lo=2, b_hi=8, weights="all"),
        # Activation quantizer over the inputs of one transformer block.
        dict(name="act_block", kind="act", block="pixart", M=8192),
        # One whole layer from fp32 activations: quantizer fused with the
        # low-rank down projection, then the GEMM with zero point and branch.
        dict(name="layer_lowrank", kind="layer", M=4096, N=2240, K=2240, b=6, rank=32,
             weights="rows", bias=True),
        # Preparing one layer's stored weight from its fp32 weight.
        dict(name="weights_4608", kind="weights", N=4608, K=1152),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _width(rng):
    """A layer width: one of the blocks' (half of the time), a multiple of 16
    or any size."""
    r = rng.random()
    if r < 0.5:
        return rng.choice(WIDTHS)
    n = _log_int(rng, 96, 8192)
    return n if r > 0.8 else max(16, n // 16 * 16)


def draw(rng):
    r = rng.random()
    if r < 0.40:
        return dict(kind="linear", M=_log_int(rng, 1, 16384), N=_width(rng), K=_width(rng),
                    b=rng.randint(1, 8), weights=rng.choice(["rows", "packed", "all"]),
                    bias=rng.random() < 0.5)
    if r < 0.50:
        return dict(kind="conv", H=_log_int(rng, 8, 128), W=_log_int(rng, 8, 128),
                    C=rng.choice([4, 64, 320, 640, 1280, _log_int(rng, 3, 1280)]),
                    N=rng.choice([320, 640, 1280, _log_int(rng, 3, 1280)]),
                    b=rng.randint(2, 8), bias=rng.random() < 0.5)
    if r < 0.70:
        S = rng.randint(1, 5)
        return dict(kind="schedule", block=rng.choice(["pixart", "pixart", "sana"]),
                    blocks=_log_int(rng, 1, 20), M=_log_int(rng, 1, 8192), S=S,
                    T=rng.randint(S, 8), b_lo=2, b_hi=8, weights=rng.choice(["rows", "all"]))
    if r < 0.80:
        return dict(kind="act", block=rng.choice(["pixart", "sana"]), M=_log_int(rng, 1, 8192))
    if r < 0.92:
        return dict(kind="layer", M=_log_int(rng, 1, 8192), N=_width(rng), K=_width(rng),
                    b=rng.randint(2, 8), rank=rng.choice([0, 16, 32]),
                    weights=rng.choice(["rows", "packed"]), bias=rng.random() < 0.5)
    return dict(kind="weights", N=_width(rng), K=_width(rng))


# ------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _codes(g, *shape):
    """int8 codes as a symmetric quantizer leaves them: a bell of standard
    deviation 32, clipped."""
    return torch.randn(shape, generator=g, device=DEV).mul_(32).round_().clamp_(-127, 127).to(
        torch.int8)


def _acts(g, M, K):
    """fp32 activations with a few large channels."""
    x = torch.randn((M, K), generator=g, device=DEV)
    x[:, ::61] *= 24.0
    return x


def _real_weights(g, N, K):
    """fp32 weights whose spread and offset differ by output channel."""
    sigma = torch.rand((N, 1), generator=g, device=DEV) * 0.04 + 0.01
    mu = torch.rand((N, 1), generator=g, device=DEV) * 0.01 - 0.005
    return torch.randn((N, K), generator=g, device=DEV) * sigma + mu


def _scales(g, N):
    return torch.rand(N, generator=g, device=DEV) * 9e-3 + 1e-3


def _bias(g, N, wanted):
    return torch.rand(N, generator=g, device=DEV) * 2 - 1 if wanted else None


def _copies(W, kind):
    """(rows, packed, planes) of the stored copies that the caller keeps."""
    packed = tasq.pack_weights(W) if kind in ("packed", "all") else None
    planes = tasq.pack_planes(W) if kind == "all" and W.dim() == 2 else None
    return (None if kind == "packed" else W), packed, planes


def _shapes(case):
    """[(M, N, K)] of a block's linears, repeated over the blocks."""
    if case["block"] == "unet":
        return UNET_LINEARS * case["blocks"]
    return [(case["M"], N, K) for N, K in BLOCKS[case["block"]]] * case["blocks"]


def _table(case, seed, L):
    g = torch.Generator().manual_seed(int(seed))
    return torch.randint(case["b_lo"], case["b_hi"] + 1, (L, case["S"]), generator=g,
                         dtype=torch.uint8)


SX = 0.02


def prepare(case, seed):
    g = _gen(seed)
    k = case["kind"]
    s = dict(case=case)
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        s["X"] = _codes(g, M, K)
        s["W"], s["packed"], s["planes"] = _copies(_codes(g, N, K), case["weights"])
        s["sw"], s["bias"] = _scales(g, N), _bias(g, N, case["bias"])
        s["y"] = torch.empty((M, N), device=DEV)
        ws = tasq.workspace_bytes(M, N, K)
        s["ws"] = torch.empty(ws, dtype=torch.uint8, device=DEV) if ws else None
    elif k == "conv":
        H, Wd, C, N = case["H"], case["W"], case["C"], case["N"]
        s["X"], s["W"] = _codes(g, H, Wd, C), _codes(g, N, 3, 3, C)
        s["sw"], s["bias"] = _scales(g, N), _bias(g, N, case["bias"])
        s["y"] = torch.empty((H, Wd, N), device=DEV)
        ws = tasq.workspace_bytes(H * Wd, N, 9 * C)
        s["ws"] = torch.empty(ws, dtype=torch.uint8, device=DEV) if ws else None
    elif k == "schedule":
        layers, keep = [], []
        shapes = _shapes(case)
        conv = UNET_CONV if case["block"] == "unet" else None
        sizes = [M * N for M, N, _ in shapes] + ([conv[0] * conv[1] * conv[3]] if conv else [])
        s["y"] = torch.empty(sum(sizes), device=DEV)
        outs = torch.split(s["y"], sizes)
        for (M, N, K), y in zip(shapes, outs):
            X, W = _codes(g, M, K), _codes(g, N, K)
            W, packed, planes = _copies(W, case["weights"])
            sw = _scales(g, N)
            layers.append(tasq.make_layer(X, W, SX, sw, y=y, packed=packed, planes=planes))
            keep.append((X, W, packed, planes, sw))
        if conv:
            H, Wd, C, N = conv
            X, W, sw = _codes(g, H, Wd, C), _codes(g, N, 3, 3, C), _scales(g, N)
            layers.append(tasq.make_layer(X, W, SX, sw, y=outs[-1]))
            keep.append((X, W, None, None, sw))
        s["layers"], s["keep"] = layers, keep
        s["table"] = _table(case, seed, len(layers))
        s["ws"] = torch.empty(tasq.schedule_workspace_bytes(layers), dtype=torch.uint8,
                              device=DEV)
    elif k == "act":
        Ks = [K for _, K in BLOCKS[case["block"]]]
        s["xs"] = [_acts(g, case["M"], K) for K in Ks]
        s["outs"] = [torch.empty(x.shape, dtype=torch.int8, device=DEV) for x in s["xs"]]
        s["params"] = [torch.empty(1028, device=DEV) for _ in Ks]
    elif k == "layer":
        M, N, K, r = case["M"], case["N"], case["K"], case["rank"]
        s["x"] = _acts(g, M, K)
        W = _codes(g, N, K)
        s["colsums"] = tasq.weight_colsums(W)
        s["W"], s["packed"], _ = _copies(W, case["weights"])
        s["sw"], s["bias"] = _scales(g, N), _bias(g, N, case["bias"])
        if r:
            s["down"] = (torch.randn((r, K), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
            s["up"] = (torch.randn((N, r), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
            s["T"] = torch.empty((M, r), device=DEV)
        s["codes"] = torch.empty((M, K), dtype=torch.int8, device=DEV)
        s["params"] = torch.empty(1028, device=DEV)
        s["y"] = torch.empty((M, N), device=DEV)
    elif k == "weights":
        s["W"] = _real_weights(g, case["N"], case["K"])
    else:
        raise ValueError(k)
    return s


# --------------------------------------------------------------------- pass

def run(s):
    case = s["case"]
    k = case["kind"]
    if k == "linear":
        return tasq.masked_linear(s["X"], s["W"], SX, s["sw"], case["b"], s["bias"],
                                  want_acc=False, y=s["y"], packed=s["packed"],
                                  planes=s["planes"], workspace=s["ws"])[1]
    if k == "conv":
        return tasq.masked_conv3x3(s["X"], s["W"], SX, s["sw"], case["b"], s["bias"],
                                   want_acc=False, y=s["y"], workspace=s["ws"])[1]
    if k == "schedule":
        tasq.run_schedule(s["layers"], s["table"], case["S"], case["T"], 0, case["T"],
                          workspace=s["ws"])
        return s["y"]
    if k == "act":
        outs, params = tasq.quantize_activations_batch(s["xs"], s["outs"], s["params"])
        # The scale and the zero point; the rest of a buffer is scratch.
        return {"codes": outs, "scale": [p[:2] for p in params]}
    if k == "layer":
        if case["rank"]:
            X, act, T = tasq.quantize_activations_lowrank(s["x"], s["down"], s["codes"],
                                                          s["params"], s["T"])
            lowrank = (T, s["up"])
        else:
            X, act = tasq.quantize_activations(s["x"], s["codes"], s["params"])
            lowrank = None
        y = tasq.masked_linear(X, s["W"], 1.0, s["sw"], case["b"], s["bias"], want_acc=False,
                               y=s["y"], packed=s["packed"], act=act, colsums=s["colsums"],
                               lowrank=lowrank)[1]
        return {"y": y, "codes": X, "scale": act[:2]}
    Q, alpha, z, sw = tasq.quantize_weights(s["W"])
    return {"codes": Q, "alpha": alpha, "z": z, "sw": sw, "packed": tasq.pack_weights(Q),
            "planes": tasq.pack_planes(Q), "colsums": tasq.weight_colsums(Q)}


# --------------------------------------------------------------------- work

def _linear_work(M, N, K, w_bytes=None):
    return dict(bytes=M * K + (N * K if w_bytes is None else w_bytes) + 4.0 * M * N,
                flops=2.0 * M * N * K)


def work(case):
    k = case["kind"]
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        # With the planes at hand only the top b of 8 bits need be read.
        share = case["b"] / 8 if case["weights"] == "all" else 1.0
        return _linear_work(M, N, K, N * K * share)
    if k == "conv":
        px, C, N = case["H"] * case["W"], case["C"], case["N"]
        return dict(bytes=px * C + 9.0 * C * N + 4.0 * px * N, flops=18.0 * px * C * N)
    if k == "schedule":
        out = dict(bytes=0.0, flops=0.0)
        shapes = _shapes(case)
        for M, N, K in shapes:
            # About the mean share of the bits where the planes are kept.
            share = (case["b_lo"] + case["b_hi"]) / 16 if (
                case["weights"] == "all" and M <= 64) else 1.0
            w = _linear_work(M, N, K, N * K * share)
            out["bytes"] += w["bytes"]
            out["flops"] += w["flops"]
        if case["block"] == "unet":
            H, Wd, C, N = UNET_CONV
            out["bytes"] += H * Wd * C + 9.0 * C * N + 4.0 * H * Wd * N
            out["flops"] += 18.0 * H * Wd * C * N
        return {n: v * case["T"] for n, v in out.items()}
    if k == "act":
        n = sum(case["M"] * K for _, K in BLOCKS[case["block"]])
        return dict(bytes=5.0 * n, flops=0.0)
    if k == "layer":
        M, N, K, r = case["M"], case["N"], case["K"], case["rank"]
        return dict(bytes=5.0 * M * K + N * K + 4.0 * M * N + 2.0 * r * (N + K),
                    flops=2.0 * M * N * K + 2.0 * M * r * (N + K))
    N, K = case["N"], case["K"]
    # fp32 weight in; codes, packed codes, planes and the sums out.
    return dict(bytes=4.0 * N * K + N * K + tasq.packed_weight_bytes(N, K) +
                tasq.planes_bytes(N, K) + 44.0 * N, flops=0.0)


def tolerance(case):
    k = case["kind"]
    if k in ("act", "weights"):
        # Codes, scales and layouts are decided in IEEE single precision.
        return "exact"
    if k == "layer":
        # The low-rank branch sums in fp32 and enters as two bfloat16 parts:
        # 4.3e-7 off the 64-bit result, 6e-8 without it.
        return {"rel": 1.8e-6, "max": 4e-5}
    # Exact int32 sums, then at most four fp32 roundings per output: 4.3e-8
    # off the 64-bit result.
    return {"rel": 1.8e-7, "max": 2e-6}


# -------------------------------------------------------------------- exact

def _masked64(W, b):
    step = 2.0 ** (8 - b)
    return torch.floor(W.reshape(W.shape[0], -1).to(torch.float64) / step) * step


def _linear64(X, W, b, sx, sw, bias):
    acc = X.reshape(X.shape[0], -1).to(torch.float64) @ _masked64(W, b).T
    y = acc * (sx * sw.to(torch.float64))
    return y if bias is None else y + bias.to(torch.float64)


def _conv64(X, W, b, sx, sw, bias):
    H, Wd, C = X.shape
    pad = torch.zeros((H + 2, Wd + 2, C), dtype=torch.float64, device=X.device)
    pad[1:-1, 1:-1] = X.to(torch.float64)
    Wb = _masked64(W, b).reshape(W.shape[0], 3, 3, C)
    acc = 0
    for r in range(3):
        for c in range(3):
            acc = acc + pad[r:r + H, c:c + Wd].reshape(H * Wd, C) @ Wb[:, r, c].T
    y = acc * (sx * sw.to(torch.float64))
    y = y if bias is None else y + bias.to(torch.float64)
    return y.reshape(H, Wd, -1)


def _act64(x):
    """(codes, alpha, z) of fp32 activations: the codes as the quantizer's
    single-precision definition gives them, on the CPU."""
    x = x.cpu()
    lo, hi = x.min(), x.max()
    if bool(hi == lo):
        alpha, z = torch.tensor(1.0), -lo
    else:
        alpha = (hi - lo) / 255.0
        z = -lo / alpha
    codes = torch.clamp(torch.round(x / alpha + z), 0, 255) - 128
    return codes.to(torch.float64).to(DEV), float(alpha), float(z)


def _scale64(x):
    lo, hi = x.min().double(), x.max().double()
    alpha = (hi - lo) / 255.0 if bool(hi > lo) else torch.ones_like(hi)
    return torch.stack([alpha, -lo / alpha])


def exact(case, seed):
    """Outputs in 64-bit arithmetic; integer outputs have none."""
    k = case["kind"]
    g = _gen(seed)
    if k == "linear":
        N, K = case["N"], case["K"]
        X, W = _codes(g, case["M"], K), _codes(g, N, K)
        return _linear64(X, W, case["b"], SX, _scales(g, N), _bias(g, N, case["bias"]))
    if k == "conv":
        X = _codes(g, case["H"], case["W"], case["C"])
        W = _codes(g, case["N"], 3, 3, case["C"])
        return _conv64(X, W, case["b"], SX, _scales(g, case["N"]),
                       _bias(g, case["N"], case["bias"]))
    if k == "schedule":
        shapes = _shapes(case)
        L = len(shapes) + (1 if case["block"] == "unet" else 0)
        last = _table(case, seed, L)[:, ((case["T"] - 1) * case["S"]) // case["T"]].tolist()
        ys = []
        for (M, N, K), b in zip(shapes, last):
            X, W = _codes(g, M, K), _codes(g, N, K)
            ys.append(_linear64(X, W, b, SX, _scales(g, N), None).reshape(-1))
        if case["block"] == "unet":
            H, Wd, C, N = UNET_CONV
            X, W = _codes(g, H, Wd, C), _codes(g, N, 3, 3, C)
            ys.append(_conv64(X, W, last[-1], SX, _scales(g, N), None).reshape(-1))
        return torch.cat(ys)
    if k == "act":
        xs = [_acts(g, case["M"], K) for _, K in BLOCKS[case["block"]]]
        return {"codes": [None] * len(xs), "scale": [_scale64(x) for x in xs]}
    if k == "layer":
        M, N, K, r = case["M"], case["N"], case["K"], case["rank"]
        x, W = _acts(g, M, K), _codes(g, N, K)
        sw, bias = _scales(g, N), _bias(g, N, case["bias"])
        Q, alpha, z = _act64(x)
        Wb = _masked64(W, case["b"])
        y = alpha * sw.to(torch.float64) * (Q @ Wb.T + (128.0 - z) * Wb.sum(1))
        if bias is not None:
            y = y + bias.to(torch.float64)
        if r:
            down = (torch.randn((r, K), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
            up = (torch.randn((N, r), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
            y = y + (x.to(torch.bfloat16).to(torch.float64) @ down.to(torch.float64).T) @ (
                up.to(torch.float64).T)
        return {"y": y, "codes": None, "scale": _scale64(x)}
    W = _real_weights(g, case["N"], case["K"]).to(torch.float64)
    lo, hi = W.min(1).values, W.max(1).values
    alpha = torch.where(hi > lo, (hi - lo) / 256.0, torch.ones_like(lo))
    return {"codes": None, "alpha": alpha, "z": -lo / alpha, "sw": alpha * 256.0 / 255.0,
            "packed": None, "planes": None, "colsums": None}
