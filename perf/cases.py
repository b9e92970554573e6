"""The work that programs have this library do, as cases that can be timed: decode steps and prefills of a decoder
layer's quantized linears (W8A8 and W4A8), the MLP block with its fused quantizers, the rotated W4A8 configuration, and
the offline preparation of weights.

A case is a dict of plain values.  `kind` names the program, the other entries its sizes:
  linear    one ql_w8a8_linear / ql_w4a8_linear call: x [M,K] fp16 -> y [M,N] fp16
  layer     DecoderLayerLinears.forward: qkv, o, gate+up, SwiGLU + quantizer, down (hidden d, MLP width F)
  mlp       RMSNorm + quantizer, gate+up GEMM, SwiGLU + quantizer, down GEMM
  rotated   the enhanced W4A8 configuration: SmoothQuant vector + Hadamard rotation + quantizer, then the GEMM
  prepare   offline: calibration maximum, SmoothQuant scales, transformed weight quantization
`graph` marks calls that a serving loop replays from a captured HIP graph (decode steps); the others are plain calls.
Hidden sizes are those of the benchmark's two decoder layers (d 1536 / F 6144 and d 4096 / F 11008); drawn cases take
any size between and around them.
"""
import math

import torch

from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd.layer import DecoderLayerLinears

DEV = "cuda"
GROUP = 128
EPS = 1e-5
MOST_OPS = 1.4e12        # a drawn case multiplies at most this much (the largest listed one: 1.65e12)


def listed():
    return [
        # The smallest call: one token through the O projection of the small model, called directly.
        dict(name="linear_m1_w8_small", kind="linear", M=1, K=1536, N=1536, bits=8, bias=True),
        # Decode steps: one sequence in int8, a batch of eight in int4, replayed from a graph.
        dict(name="layer_m1_w8", kind="layer", M=1, d=4096, F=11008, bits=8, graph=True),
        dict(name="layer_m8_w4", kind="layer", M=8, d=4096, F=11008, bits=4, graph=True),
        # A decode batch of 32 through the longest K.
        dict(name="linear_m32_w8_down", kind="linear", M=32, K=11008, N=4096, bits=8, bias=False),
        # A short prompt of odd length through the fused QKV projection.
        dict(name="linear_m197_w8_qkv", kind="linear", M=197, K=4096, N=12288, bits=8, bias=True),
        # A prefill chunk of 512 tokens in int4.
        dict(name="linear_m512_w4_down", kind="linear", M=512, K=11008, N=4096, bits=4, bias=False),
        # The MLP of the small model on a ragged prompt, normalisation and activation fused into the quantizers.
        dict(name="mlp_m1900_w8_small", kind="mlp", M=1900, d=1536, F=6144, bits=8),
        # The benchmark's prefill: 4096 tokens through the layer.
        dict(name="layer_m4096_w8", kind="layer", M=4096, d=4096, F=11008, bits=8, graph=False),
        # The same prompt through the widest projection in int4.
        dict(name="linear_m4096_w4_gate_up", kind="linear", M=4096, K=4096, N=22016, bits=4, bias=False),
        # Long prefill: 16384 tokens through the down projection.
        dict(name="linear_m16384_w8_down", kind="linear", M=16384, K=11008, N=4096, bits=8, bias=False),
        # The enhanced W4A8 configuration on a prompt of odd length.
        dict(name="rotated_m3001_w4", kind="rotated", M=3001, K=4096, N=4096, bits=4, smooth=True),
        # Weights of that configuration, prepared when a model is loaded.
        dict(name="prepare_w4_down", kind="prepare", M=512, K=11008, N=4096, bits=4),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _multiple(rng, lo, hi, step):
    return max(step, _log_uniform(rng, lo, hi) // step * step)


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "linear", "layer", "layer", "mlp", "rotated", "prepare"])
    bits = rng.choice([8, 4])
    if kind == "linear":
        K = _multiple(rng, 1024, 12288, 128 if bits == 4 else 64)
        N = _log_uniform(rng, 1024, 24576)
        if rng.random() < 0.7:
            N = max(64, N // 64 * 64)
        M = _log_uniform(rng, 1, min(16384, MOST_OPS / (2.0 * N * K)))
        return dict(kind=kind, M=M, K=K, N=N, bits=bits, bias=rng.random() < 0.5)
    if kind in ("layer", "mlp"):
        d = _multiple(rng, 1024, 5120, 128)
        F = max(256, int(d * rng.uniform(2.5, 4.0)) // 128 * 128)
        width = 4.0 * d * d + 3.0 * d * F
        M = _log_uniform(rng, 1, min(8192, MOST_OPS / (2.0 * width)))
        c = dict(kind=kind, M=M, d=d, F=F, bits=bits)
        if kind == "layer":
            c["graph"] = M <= 64
        return c
    if kind == "rotated":
        K, N = _multiple(rng, 1024, 12288, 128), _multiple(rng, 1024, 16384, 64)
        M = _log_uniform(rng, 64, min(8192, MOST_OPS / (2.0 * N * K)))
        return dict(kind=kind, M=M, K=K, N=N, bits=bits, smooth=rng.random() < 0.5)
    return dict(kind=kind, M=_log_uniform(rng, 64, 2048), K=_multiple(rng, 1024, 12288, 128), N=_multiple(rng, 1024, 12288, 32), bits=bits)


# ---- inputs

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _activations(g, M, K):
    """fp16 N(0,1) with 1 % of the channels amplified 20 times, as activations of decoder layers have them."""
    x = torch.randn((M, K), generator=g, device=DEV, dtype=torch.float32)
    loud = torch.randperm(K, generator=g, device=DEV)[: max(1, round(0.01 * K))]
    x[:, loud] *= 20.0
    return x.half()


def _weights(g, N, K):
    return (torch.randn((N, K), generator=g, device=DEV, dtype=torch.float32) * 0.02).half()


def _bias(g, N):
    return (torch.randn(N, generator=g, device=DEV, dtype=torch.float32) * 0.01).half()


def _hidden_gain(g, K):
    return (1.0 + 0.1 * torch.randn(K, generator=g, device=DEV, dtype=torch.float32)).half()


def _inputs(c, seed):
    """Everything random of a case, the same for prepare() and exact()."""
    g = _generator(seed)
    if c["kind"] == "layer":
        d, F = c["d"], c["F"]
        w = {"qkv": _weights(g, 3 * d, d), "o": _weights(g, d, d), "gate_up": _weights(g, 2 * F, d), "down": _weights(g, d, F)}
        return {"x": _activations(g, c["M"], d), "w": w, "bias": {k: _bias(g, v.shape[0]) for k, v in w.items()}}
    if c["kind"] == "mlp":
        d, F = c["d"], c["F"]
        return {"x": _activations(g, c["M"], d), "gamma": _hidden_gain(g, d), "w_gu": _weights(g, 2 * F, d), "w_down": _weights(g, d, F)}
    i = {"x": _activations(g, c["M"], c["K"]), "w": _weights(g, c["N"], c["K"])}
    if c["kind"] == "linear":
        i["bias"] = _bias(g, c["N"]) if c["bias"] else None
    return i


def _bytes(n):
    return torch.empty(int(n), dtype=torch.uint8, device=DEV)


def _quantized(w, bits):
    """Kernel-layout blob and (int8) channel scales of fp16 weights."""
    N, K = w.shape
    group = 0 if bits == 8 else GROUP
    _, sb, kb = ql.ql_weight_bytes(N, K, bits, group)
    scales, kern = _bytes(sb), _bytes(kb)
    ql.ql_quant_weight(w, bits, group, None, scales, kern)
    return kern, scales.view(torch.float32) if bits == 8 else None


def _output(M, N):
    """[M,N] fp16 whose row stride is the next multiple of 8."""
    return torch.empty((M, (N + 7) // 8 * 8), dtype=torch.float16, device=DEV)[:, :N]


def _gemm(s, which, xq, sx, M, K, N, y):
    kern, sw = s[which]
    if s["bits"] == 8:
        ql.ql_w8a8_gemm(xq, sx, M, K, kern, sw, None, N, y, s["ws"])
    else:
        ql.ql_w4a8_gemm(xq, sx, M, K, kern, GROUP, None, N, y, s["ws"])


def prepare(c, seed):
    i = _inputs(c, seed)
    kind, M, bits = c["kind"], c["M"], c["bits"]
    s = {"kind": kind, "M": M, "bits": bits, "x": i["x"]}
    if kind == "linear":
        K, N = c["K"], c["N"]
        s.update(N=N, bias=i["bias"], y=_output(M, N), ws=_bytes(ql.ql_workspace_bytes(M, N, K, bits)))
        s["kern"], s["sw"] = _quantized(i["w"], bits)
    elif kind == "layer":
        w = i["w"]
        s["layer"] = layer = DecoderLayerLinears(w["qkv"], w["o"], w["gate_up"], w["down"], bits, M, i["bias"])
        s["graph"] = None
        if c["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                layer.forward(s["x"])
            torch.cuda.current_stream().wait_stream(side)
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                s["y"] = layer.forward(s["x"])
    elif kind == "mlp":
        d, F = c["d"], c["F"]
        s.update(d=d, F=F, gamma=i["gamma"], gu=_quantized(i["w_gu"], bits), down=_quantized(i["w_down"], bits))
        s.update(xq=_bytes(ql.ql_act_kernel_bytes(M, d)), sx=torch.empty(M, device=DEV), y_gu=_output(M, 2 * F),
                 hq=_bytes(ql.ql_act_kernel_bytes(M, F)), sh=torch.empty(M, device=DEV), y=_output(M, d),
                 ws=_bytes(max(ql.ql_workspace_bytes(M, 2 * F, d, bits), ql.ql_workspace_bytes(M, d, F, bits))))
    elif kind == "rotated":
        K, N = c["K"], c["N"]
        group = 0 if bits == 8 else GROUP
        block = ql.ql_hadamard_block(K)
        smooth = inv = None
        if c["smooth"]:
            xmax = torch.zeros(K, device=DEV)
            smooth, inv = torch.empty(K, device=DEV), torch.empty(K, device=DEV)
            ql.ql_smooth_calibrate(i["x"], xmax)
            ql.ql_smooth_scales(xmax, i["w"], 0.5, smooth, inv)
        _, sb, kb = ql.ql_weight_bytes(N, K, bits, group)
        scales, kern = _bytes(sb), _bytes(kb)
        ql.ql_quant_weight_transformed(i["w"], bits, group, smooth, block, torch.empty((N, K), device=DEV), None, scales, kern)
        s.update(K=K, N=N, block=block, inv=inv, w=(kern, scales.view(torch.float32) if bits == 8 else None), y=_output(M, N),
                 xq=_bytes(ql.ql_act_kernel_bytes(M, K)), sx=torch.empty(M, device=DEV), ws=_bytes(ql.ql_workspace_bytes(M, N, K, bits)))
    else:
        K, N = c["K"], c["N"]
        s["group"] = group = 0 if bits == 8 else GROUP
        cb, sb, kb = ql.ql_weight_bytes(N, K, bits, group)
        s.update(w=i["w"], block=ql.ql_hadamard_block(K), xmax=torch.zeros(K, device=DEV), smooth=torch.empty(K, device=DEV),
                 inv=torch.empty(K, device=DEV), w32=torch.empty((N, K), device=DEV), canon=_bytes(cb), scales=_bytes(sb), kern=_bytes(kb))
    return s


def run(s):
    kind, M, x = s["kind"], s["M"], s["x"]
    if kind == "linear":
        if s["bits"] == 8:
            ql.ql_w8a8_linear(x, s["kern"], s["sw"], s["bias"], s["N"], s["y"], s["ws"])
        else:
            ql.ql_w4a8_linear(x, s["kern"], GROUP, s["bias"], s["N"], s["y"], s["ws"])
        return s["y"]
    if kind == "layer":
        if s["graph"] is None:
            return s["layer"].forward(x)
        s["graph"].replay()
        return s["y"]
    if kind == "mlp":
        d, F = s["d"], s["F"]
        ql.ql_quant_act_rmsnorm(x, s["gamma"], EPS, None, s["xq"], s["sx"])
        _gemm(s, "gu", s["xq"], s["sx"], M, d, 2 * F, s["y_gu"])
        ql.ql_quant_act_swiglu(s["y_gu"], None, s["hq"], s["sh"])
        _gemm(s, "down", s["hq"], s["sh"], M, F, d, s["y"])
        return s["y"]
    if kind == "rotated":
        ql.ql_quant_act_per_token_transformed(x, s["inv"], s["block"], None, s["xq"], s["sx"])
        _gemm(s, "w", s["xq"], s["sx"], M, s["K"], s["N"], s["y"])
        return {"sx": s["sx"], "y": s["y"]}
    ql.ql_smooth_calibrate(x, s["xmax"])
    ql.ql_smooth_scales(s["xmax"], s["w"], 0.5, s["smooth"], s["inv"])
    ql.ql_quant_weight_transformed(s["w"], s["bits"], s["group"], s["smooth"], s["block"], s["w32"], s["canon"], s["scales"], s["kern"])
    scales = s["scales"].view(torch.float32 if s["bits"] == 8 else torch.float16)
    return {"smooth": s["smooth"], "inv_smooth": s["inv"], "codes": s["canon"], "scales": scales}


# ---- what a pass cannot do without

def _weight_bytes(N, K, bits):
    return N * K + 4 * N if bits == 8 else N * K / 2 + 2 * N * K / GROUP


def work(c):
    M, bits = c["M"], c["bits"]
    if c["kind"] in ("linear", "rotated"):
        K, N = c["K"], c["N"]
        return {"bytes": 2 * M * K + _weight_bytes(N, K, bits) + 2 * M * N, "flops": 2.0 * M * N * K}
    if c["kind"] == "prepare":
        K, N = c["K"], c["N"]
        codes = N * K if bits == 8 else N * K / 2
        return {"bytes": 2 * N * K + 2 * M * K + 2 * codes + 12 * K + (_weight_bytes(N, K, bits) - codes) * 2, "flops": N * K}
    d, F = c["d"], c["F"]
    mats = [(2 * F, d), (d, F)] if c["kind"] == "mlp" else [(3 * d, d), (d, d), (2 * F, d), (d, F)]
    # the outputs of the inner projections are stored: they are returned by public calls
    inner = 2 * M * 2 * F if c["kind"] == "mlp" else 2 * M * (3 * d + d + 2 * F)
    return {"bytes": 2 * M * d + inner + 2 * M * d + sum(_weight_bytes(n, k, bits) for n, k in mats),
            "flops": sum(2.0 * M * n * k for n, k in mats)}


# ---- the same in 64 bits, from the definition: integer decisions in fp32 as documented, everything else in float64

def _over(a, b):
    """a / b as one IEEE division (torch turns division by a plain number, and of one, into a product)."""
    a, b = (t if torch.is_tensor(t) else torch.full_like(o, t) for t, o in ((a, b), (b, a)))
    return a / b


def _codes(v32):
    """Per-token int8 codes (as float64) and scales of fp32 values."""
    amax = v32.abs().amax(dim=1, keepdim=True)
    zero = amax == 0
    sx = torch.where(zero, torch.ones_like(amax), _over(amax, 127.0))
    inv = torch.where(zero, torch.zeros_like(amax), _over(127.0, amax))
    return torch.clamp(torch.round(v32 * inv), -127, 127).double(), sx


def _weights64(w32, bits):
    """Dequantized weights in float64."""
    N, K = w32.shape
    if bits == 8:
        s = _over(w32.abs().amax(dim=1, keepdim=True), 127.0)
        s = torch.where(s == 0, torch.ones_like(s), s)
        return torch.clamp(torch.round(w32 / s), -127, 127).double() * s.double()
    g = w32.view(N, K // GROUP, GROUP)
    s = _over(g.abs().amax(dim=2, keepdim=True), 7.0).half().float()
    s = torch.where(s == 0, torch.ones_like(s), s)
    return (torch.clamp(torch.round(g / s), -7, 7).double() * s.double()).view(N, K)


def _linear64(v32, w32, bits, bias=None):
    q, sx = _codes(v32)
    y = torch.matmul(q, _weights64(w32, bits).t()) * sx.double()
    return y if bias is None else y + bias.double()


def _hadamard(v32, block):
    """Block Hadamard transform of the last dimension in fp32, stages 1, 2, 4, ... in order."""
    rows, K = v32.shape
    h = 1
    while h < block:
        v = v32.view(rows, K // (2 * h), 2, h)
        v32 = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), dim=2).view(rows, K)
        h *= 2
    return v32 * (1.0 / math.sqrt(block))


def _swiglu(y_gu, F):
    gate, up = y_gu[:, :F].double(), y_gu[:, F:].double()
    return (gate / (1.0 + torch.exp(-gate)) * up).float()


def _smooth64(x, w):
    xm, wm = x.float().abs().amax(dim=0).double(), w.float().abs().amax(dim=0).double()
    return torch.where((xm > 0) & (wm > 0), torch.sqrt(xm) / torch.sqrt(wm.clamp_min(1e-300)), torch.ones_like(xm))


def exact(c, seed):
    i = _inputs(c, seed)
    kind, bits, x = c["kind"], c["bits"], i["x"]
    if kind == "linear":
        return _linear64(x.float(), i["w"].float(), bits, i["bias"])
    if kind == "layer":   # the projections' outputs are fp16 by definition: each next step starts from them
        d, F, b = c["d"], c["F"], i["bias"]
        w = {k: v.float() for k, v in i["w"].items()}
        y = _linear64(x.float(), w["qkv"], bits, b["qkv"]).half()[:, :d]
        y = _linear64(y.float(), w["o"], bits, b["o"]).half()
        y = _linear64(y.float(), w["gate_up"], bits, b["gate_up"]).half()
        return _linear64(_swiglu(y, F), w["down"], bits, b["down"])
    if kind == "mlp":
        x64 = x.double()
        h = (x64 * torch.rsqrt((x64 * x64).mean(dim=1, keepdim=True) + EPS) * i["gamma"].double()).float()
        y = _linear64(h, i["w_gu"].float(), bits).half()
        return _linear64(_swiglu(y, c["F"]), i["w_down"].float(), bits)
    K = c["K"]
    block = min(K & -K, 4096)
    w32, x32 = i["w"].float(), x.float()
    if kind == "rotated":
        if c["smooth"]:
            s = _smooth64(x, i["w"]).float()
            w32, x32 = w32 * s, x32 * _over(1.0, s)
        w32, x32 = _hadamard(w32, block), _hadamard(x32, block)
        return {"sx": _codes(x32)[1].view(-1).double(), "y": _linear64(x32, w32, bits)}
    s = _smooth64(x, i["w"])
    t = _hadamard(w32 * s.float(), block)
    if bits == 8:
        scales = t.double().abs().amax(dim=1) / 127.0
    else:
        scales = t.double().view(c["N"], K // GROUP, GROUP).abs().amax(dim=2) / 7.0
    return {"smooth": s, "inv_smooth": 1.0 / s, "codes": None, "scales": scales.view(-1)}


def tolerance(c):
    # One fp16 rounding of the output either way.  In chained linears such a rounding can move int8 codes of the next
    # one; in the rotated and prepared cases a last bit of the SmoothQuant vector can.
    if c["kind"] in ("layer", "mlp"):
        return {"rel": 4e-3, "max": 0.1}
    if c["kind"] == "prepare":
        return {"rel": 2e-4, "max": 0.01, "differ": 1e-4}
    if c["kind"] == "rotated":
        return {"rel": 2e-3, "max": 0.05}
    return {"rel": 5e-4, "max": 0.01}
