"""The work that a program does with this framework, as cases that can be timed.

A case is one call chain of the public Python entry points on one linear of a
diffusion transformer, or on the data that leads to it:

  w8a8       layer.route on an INT8 layer: smooth + per-token quantization,
             INT8 GEMM, dequantization and bias
  modulated  layer.route_modulated: the same behind the adaLN modulation of a
             transformer block (QKV and FFN-up inputs)
  protected  layer.route on a layer kept in bf16
  q8_0, q4_k layer.route on a GGUF weight-only layer
  profile    one calibration batch of one layer: per-channel absmax and the
             fragility statistics
  encode     one layer's weights into the format a checkpoint keeps: "w8a8"
             (smoothing factors, then int8 codes and scales), "q8_0", "q4_k"

M is tokens, K input channels, N output channels. The widths 4096, 12288 and
16384, the 4608 tokens (4096 image + 512 text) and the 64 x 256 -> 512 layer
are those of bench.py and the tests; the other sizes are generic."""
from __future__ import annotations

import math

import torch

from paper_2606_12280_amd import layer, ops
from paper_2606_12280_amd.fragility import Profile

DEV = "cuda:0"
LINEAR = ("w8a8", "modulated", "protected", "q8_0", "q4_k")
EPS = 1e-6
ALPHA = 0.5
MAX_MNK = 4608 * 4096 * 16384    # the largest listed GEMM
MAX_WEIGHTS = 24576 * 4096       # the largest listed weight
MAX_TOKENS = 4608


def listed() -> list[dict]:
    return [
        # the smallest call: the tests' and the smoke run's tiny layer, where
        # launches and the host path are the time
        {"name": "tiny_w8a8", "op": "w8a8", "M": 64, "N": 512, "K": 256, "bias": True},
        # one conditioning vector (the timestep embedding) to a block's six
        # modulation vectors: every step, every block, one row
        {"name": "modulation_w8a8", "op": "w8a8", "M": 1, "N": 24576, "K": 4096, "bias": True},
        # a text prompt alone through a square projection: ragged token count
        {"name": "text_w8a8", "op": "w8a8", "M": 333, "N": 4096, "K": 4096, "bias": True},
        # QKV of a smaller model whose width is an odd multiple of 64: ragged
        # in every size
        {"name": "odd_qkv_modulated", "op": "modulated", "M": 1117, "N": 8640, "K": 2880,
         "bias": True},
        # FFN up at the full token count, behind its modulation
        {"name": "ffn_up_modulated", "op": "modulated", "M": 4608, "N": 16384, "K": 4096,
         "bias": True},
        # FFN down kept in bf16: the most fragile layers
        {"name": "ffn_down_protected", "op": "protected", "M": 4608, "N": 4096, "K": 16384,
         "bias": True},
        # the output projection of every image and text token to its patch of
        # 64 values, usually kept in bf16
        {"name": "patch_out_protected", "op": "protected", "M": 4608, "N": 64, "K": 4096,
         "bias": True},
        # a short prompt through a Q8_0 QKV projection
        {"name": "prompt_q8_0", "op": "q8_0", "M": 154, "N": 12288, "K": 4096, "bias": True},
        # a 512 x 512 image (1024 tokens) with 256 text tokens through a Q4_K
        # FFN up, no bias
        {"name": "ffn_up_q4_k", "op": "q4_k", "M": 1280, "N": 16384, "K": 4096, "bias": False},
        # calibration: one batch of one layer's input
        {"name": "calibrate", "op": "profile", "M": 4608, "K": 4096},
        # preparing a checkpoint, one layer: INT8 with smoothing ...
        {"name": "encode_w8a8", "op": "encode", "fmt": "w8a8", "N": 16384, "K": 4096},
        # ... and Q4_K
        {"name": "encode_q4_k", "op": "encode", "fmt": "q4_k", "N": 4096, "K": 16384},
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng) -> dict:
    """A case of the listed kinds: sizes over the whole range on a log scale,
    K any multiple of 64 (256 for Q4_K), N and M any integer."""
    kind = rng.choice(["w8a8", "w8a8", "modulated", "protected", "q8_0", "q4_k", "profile",
                       "encode"])
    fmt = rng.choice(["w8a8", "q8_0", "q4_k"]) if kind == "encode" else None
    step = 256 if "q4_k" in (kind, fmt) else 64
    k_max = 8192 if kind == "modulated" else 16384
    K = step * _log_int(rng, 256 // step, k_max // step)
    if kind == "profile":
        return {"op": kind, "M": _log_int(rng, 64, MAX_TOKENS), "K": K}
    N = _log_int(rng, 64, min(24576, MAX_WEIGHTS // K))
    if rng.random() < 0.5:
        N = (N + 63) // 64 * 64  # layers are mostly multiples of 64 wide
    N = min(N, MAX_WEIGHTS // K)
    if kind == "encode":
        return {"op": kind, "fmt": fmt, "N": N, "K": K}
    M = _log_int(rng, 1, min(MAX_TOKENS, MAX_MNK // (N * K)))
    return {"op": kind, "M": M, "N": N, "K": K, "bias": rng.random() < 0.75}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _activations(g, M: int, K: int, gelu: bool) -> torch.Tensor:
    """Plain linears: N(0, 1) with 1% of the channels x 20. FFN-down inputs:
    GELU(N(0, 1.5)) times a log-normal scale per channel."""
    z = torch.randn(M, K, generator=g, device=DEV)
    if gelu:
        c = torch.exp(1.5 * torch.randn(K, generator=g, device=DEV))
        return (torch.nn.functional.gelu(1.5 * z) * c).to(torch.bfloat16)
    n_out = max(1, round(0.01 * K))
    z[:, torch.randperm(K, generator=g, device=DEV)[:n_out]] *= 20.0
    return z.to(torch.bfloat16)


def _inputs(case: dict, seed: int) -> dict:
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    d = {}
    N, K, M = case.get("N"), case["K"], case.get("M")
    if M is not None:
        d["X"] = _activations(g, M, K, gelu=N is not None and K > N and M > 1
                              and case["op"] != "modulated")
    if N is not None:
        d["W"] = (0.02 * torch.randn(N, K, generator=g, device=DEV)).to(torch.bfloat16)
        d["bias"] = ((0.01 * torch.randn(N, generator=g, device=DEV)).to(torch.bfloat16)
                     if case.get("bias") else None)
    if case["op"] == "modulated":
        d["shift"] = (0.2 * torch.randn(K, generator=g, device=DEV)).to(torch.bfloat16)
        d["scale"] = (0.2 * torch.randn(K, generator=g, device=DEV)).to(torch.bfloat16)
    if case["op"] in ("w8a8", "modulated") or case.get("fmt") == "w8a8":
        # per-channel activation absmax of an earlier calibration pass
        u = torch.rand(K, generator=g, device=DEV)
        s = 3.0 + 2.0 * u
        s[torch.randperm(K, generator=g, device=DEV)[:max(1, round(0.01 * K))]] *= 20.0
        d["act_absmax"] = s
    return d


def prepare(case: dict, seed: int) -> dict:
    d = _inputs(case, seed)
    op = case["op"]
    st = {"op": op}
    if op in LINEAR:
        W, b = d["W"], d["bias"]
        if op in ("w8a8", "modulated"):
            lam = ops.w8a8_smooth_factors(d["act_absmax"], W, ALPHA)
            st["lay"] = layer.prepare_linear(W, b, lam, protected=False)
        elif op == "protected":
            st["lay"] = layer.prepare_linear(W, b, None, protected=True)
        elif op == "q8_0":
            st["lay"] = layer.prepare_q8_0(W, b)
        else:
            st["lay"] = layer.prepare_q4_k(W, b)
        st["X"] = d["X"]
        st["ws"] = layer.Workspace(DEV)
        if op == "modulated":
            st["shift"], st["scale"] = d["shift"], d["scale"]
    elif op == "profile":
        st["X"] = d["X"]
        st["absmax"] = torch.zeros(case["K"], dtype=torch.float32, device=DEV)
        st["prof"] = Profile(1, 1, DEV)
    else:
        st["fmt"], st["W"] = case["fmt"], d["W"]
        st["act_absmax"] = d.get("act_absmax")
    return st


def run(st: dict):
    op = st["op"]
    if op == "modulated":
        return layer.route_modulated(st["lay"], st["X"], st["shift"], st["scale"], EPS,
                                     ws=st["ws"])
    if op in LINEAR:
        return layer.route(st["lay"], st["X"], ws=st["ws"])
    if op == "profile":
        ops.w8a8_act_absmax(st["X"], st["absmax"])
        st["prof"].record(0, 0, st["X"])
        return {"absmax": st["absmax"], "stats": st["prof"].stats}
    if st["fmt"] == "w8a8":
        lam = ops.w8a8_smooth_factors(st["act_absmax"], st["W"], ALPHA)
        lay = layer.prepare_linear(st["W"], None, lam, protected=False)
        return {"lambda": lam, "inv_lambda": lay.inv_lambda, "w_scale": lay.w_scale,
                "Wq": lay.Wq}
    if st["fmt"] == "q8_0":
        lay = layer.prepare_q8_0(st["W"], None)
        return {"qs": lay.q8_qs, "d": lay.q8_d}
    q = layer.prepare_q4_k(st["W"], None).q4k
    return {"qs": q.qs, "scales": q.scales, "d": q.d, "dmin": q.dmin}


# --------------------------------------------------------------------------
# what a pass cannot do without, and what it should give
# --------------------------------------------------------------------------

def _code_bytes(fmt: str, N: int, K: int) -> float:
    """One layer's weights in a format, scales included."""
    return {"w8a8": N * K + 4 * N + 4 * K, "modulated": N * K + 4 * N + 4 * K,
            "protected": 2 * N * K, "q8_0": N * K * 8.5 / 8, "q4_k": N * K * 4.5 / 8}[fmt]


def work(case: dict) -> dict:
    op, K = case["op"], case["K"]
    M, N = case.get("M"), case.get("N")
    if op == "profile":
        return {"bytes": 2 * M * K + 8 * K + 32, "flops": 9 * M * K}
    if op == "encode":
        stats = 8 * K if case["fmt"] == "w8a8" else 0  # absmax in, factors out
        return {"bytes": 2 * N * K + _code_bytes(case["fmt"], N, K) + stats, "flops": 4 * N * K}
    b = 2 * M * K + _code_bytes(op, N, K) + 2 * M * N + (2 * N if case["bias"] else 0)
    if op == "modulated":
        b += 4 * K
    return {"bytes": b, "flops": 2 * M * N * K}


def tolerance(case: dict):
    """Codes, scales and int32 sums are defined operation by operation, so
    INT8 layers and every encoder give the same bits. bf16 products summed in
    binary32 differ by the order of the sum, which moves a few outputs to the
    next bf16 value (2e-5 to 8.5e-5 and one bf16 step, 2^-7, against the same
    sums in two halves of K). The fragility statistics are binary64 sums."""
    op = case["op"]
    if op in ("protected", "q8_0", "q4_k"):
        return {"rel": 3.5e-4, "max": 0.032}
    if op == "profile":
        return {"rel": 1e-12, "max": 1e-11}
    return "exact"


# --------------------------------------------------------------------------
# the same results in 64 bits, by plain torch
# --------------------------------------------------------------------------

def _quantize64(v: torch.Tensor):
    """Per-row symmetric codes of v (binary64) and their scales."""
    a = v.abs().amax(dim=1, keepdim=True)
    s = a / 127.0
    return torch.round(v * (127.0 / a)).clamp_(-127, 127), s


def _lambda64(act_absmax: torch.Tensor, W: torch.Tensor) -> torch.Tensor:
    return act_absmax.double() ** ALPHA / W.abs().amax(dim=0).double() ** (1.0 - ALPHA)


def _gguf64(fmt: str, W: torch.Tensor) -> torch.Tensor:
    """The bf16 weights that a GGUF layer multiplies with (binary32 steps, as
    the formats define them), as binary64."""
    N, K = W.shape
    w = W.float()
    if fmt == "q8_0":
        w = w.view(N, K // 32, 32)
        amax = w.abs().amax(dim=2, keepdim=True)
        d = (amax / 127.0).clamp(max=65504.0).half().float()
        inv = torch.where(d != 0, 1.0 / d, torch.zeros_like(d))
        q = torch.round(w * inv).clamp(-127, 127)
        return (d * q).view(N, K).to(torch.bfloat16).double()
    w = w.view(N, K // 256, 8, 32)
    lo = w.amin(dim=3, keepdim=True).clamp(max=0.0)
    hi = w.amax(dim=3, keepdim=True)
    a, b = (hi - lo) / 15.0, -lo
    d = (a.amax(dim=2, keepdim=True).clamp(min=0.0) / 63.0).clamp(max=65504.0).half().float()
    dm = (b.amax(dim=2, keepdim=True).clamp(min=0.0) / 63.0).clamp(max=65504.0).half().float()
    sc = torch.round(a * torch.where(d != 0, 1.0 / d, 0.0)).clamp(max=63.0)
    mn = torch.round(b * torch.where(dm != 0, 1.0 / dm, 0.0)).clamp(max=63.0)
    s, o = d * sc, dm * mn
    q = torch.round((w + o) * torch.where(s != 0, 1.0 / s, 0.0)).clamp(0.0, 15.0)
    return (s * q - o).view(N, K).to(torch.bfloat16).double()


def exact(case: dict, seed: int):
    d = _inputs(case, seed)
    op = case["op"]
    if op == "profile":
        x = d["X"].double()
        mean = x.mean()
        c = x - mean
        m2 = (c * c).mean()
        stats = torch.stack([x.abs().max(), mean, m2.sqrt(), (c ** 4).mean() / (m2 * m2)])
        return {"absmax": x.abs().amax(dim=0), "stats": stats.view(1, 1, 4)}
    W = d["W"]
    if op == "encode":
        N, K = W.shape
        if case["fmt"] == "w8a8":
            lam = _lambda64(d["act_absmax"], W)
            w_scale = (W.double() * lam).abs().amax(dim=1) / 127.0
            return {"lambda": lam, "inv_lambda": 1.0 / lam, "w_scale": w_scale, "Wq": None}
        if case["fmt"] == "q8_0":
            return {"qs": None, "d": W.double().view(N, K // 32, 32).abs().amax(dim=2) / 127.0}
        w = W.double().view(N, K // 256, 8, 32)
        lo = w.amin(dim=3).clamp(max=0.0)
        return {"qs": None, "scales": None,
                "d": ((w.amax(dim=3) - lo) / 15.0).amax(dim=2).clamp(min=0.0) / 63.0,
                "dmin": (-lo).amax(dim=2) / 63.0}
    b = d["bias"].double() if d["bias"] is not None else 0.0
    x = d["X"].double()
    if op == "protected":
        return x @ W.double().t() + b
    if op in ("q8_0", "q4_k"):
        return x @ _gguf64(op, W).t() + b
    lam = _lambda64(d["act_absmax"], W)
    if op == "modulated":
        x = x - x.mean(dim=1, keepdim=True)
        x = x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + EPS)
        x = x * (1.0 + d["scale"].double()) + d["shift"].double()
        x = x.to(torch.bfloat16).double()  # the modulated tensor is a bf16 tensor
    xq, xs = _quantize64(x / lam)
    wq, ws = _quantize64(W.double() * lam)
    return (xq @ wq.t()) * (xs * ws.t()) + b
