"""Timed cases of the 2:4 sparse linear-layer path: what a program that deploys a compressed vision transformer has this
package do, through its public classes and functions.

Kinds of case
  linear   a linear layer at inference (`SparseLinear.forward`): on the int8 path the fp16 or fp32 activations are quantised
           with the scale of this tensor and multiplied; on the fp16 path they are multiplied as they are.
  step     the same with the weight preparation in front of it (`SparseLinear.prepare_weights` + `forward`): bench.py's step.
  block    the four linear layers of an encoder block with calibrated scales, chained in int8 (`EncoderBlockLinears.forward`).
           Attention and normalisation are the caller's own kernels and are left out: the attention output is in hand.
  patch    a patch embedding from images to tokens (`SparsePatchEmbed.forward`).
  weights  fp32 weights to what the GEMM reads, as a model is loaded: `prepare_weights` for int8 and fp16; for int4 the pair-wise
           4:8 storage (prune, quantise, compress) and from it the packed int8 2:4 operand.

Sizes are those of synth.CONFIGS, the report and the tests.  Activations ~ N(0, 1) (the second feed-forward layer: GELU of
that), weights ~ N(0, 0.02), biases ~ N(0, 0.01), as in synth.py, made on the GPU from the seed.
"""
import math

import torch

from paper_2305_10727_amd import gpusq as G
from paper_2305_10727_amd.pipeline import EncoderBlockLinears, SparseLinear, SparsePatchEmbed

_DTYPES = {"f16": torch.float16, "f32": torch.float32, "i8": torch.int8}


def _linear(name, M, K, N, precision="int8", gelu=False, x="f16", out="f16", dist="normal", kind="linear"):
    return dict(name=name, kind=kind, M=M, K=K, N=N, precision=precision, gelu=gelu, x=x, out=out, dist=dist)


def listed():
    return [
        # one image, the narrowest layer in use: launches and host time
        _linear("tiny layer, batch 1", 197, 192, 768),
        # one image through an encoder block of ViT-B: the latency of a chain of small launches
        dict(name="ViT-B block, batch 1", kind="block", M=197, D=768, hidden=3072),
        # the classifier of 1000 classes for a batch of 64: few rows, a width that is no multiple of a tile
        _linear("classifier, batch 64, fp16", 64, 768, 1000, precision="fp16"),
        # odd rows, a K that ends inside a K step, int8 output for a layer that follows
        _linear("ragged layer, int8 out", 333, 1040, 520, gelu=True, out="i8"),
        # the benchmark: ViT-B's first feed-forward layer at batch 64 with its weight preparation
        _linear("ViT-B fc1, batch 64, step", 64 * 197, 768, 3072, gelu=True, kind="step"),
        # the same layer on the fp16 path, weights in hand
        _linear("ViT-B fc1, batch 64, fp16", 64 * 197, 768, 3072, precision="fp16", gelu=True),
        # the second feed-forward layer: long K, skewed activations
        _linear("ViT-B fc2, batch 128", 128 * 197, 3072, 768, dist="gelu_normal"),
        # a batch through the linear layers of a block of Swin-B's third stage
        dict(name="Swin-B block, batch 64", kind="block", M=64 * 196, D=512, hidden=2048),
        # images to tokens: 16 x 16 patches on the int8 path, 14 x 14 patches on the fp16 path
        dict(name="patches 16, batch 64", kind="patch", B=64, C=3, H=224, W=224, P=16, D=768, precision="int8"),
        dict(name="patches 14, batch 256, fp16", kind="patch", B=256, C=3, H=224, W=224, P=14, D=1280, precision="fp16"),
        # a model with int4 weights is prepared: ViT-H's first feed-forward layer
        dict(name="ViT-H fc1 weights, int4", kind="weights", N=5120, K=1280, format="int4"),
        # a large batch through the widest layer: throughput
        _linear("ViT-H fc1, batch 256", 256 * 257, 1280, 5120, gelu=True),
    ]


# what the largest listed case costs: a drawn case stays below it (an fp16 product counts twice, its matrix rate is half)
_MAX_OPS = 256 * 257 * 1280 * 5120
_MAX_BYTES = 256 * 257 * 2 * (1280 + 5120)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _multiple(rng, lo, hi, of):
    return max(of, _log_int(rng, lo, hi) // of * of)


def draw(rng):
    kind = rng.choice(("linear",) * 8 + ("step", "step") + ("block",) * 4 + ("patch",) * 3 + ("weights",) * 3)
    precision = rng.choice(("int8", "int8", "fp16"))
    if kind in ("linear", "step"):
        # widths are whole multiples of 64 in most models, of 16 (K) and 4 (N) at the least
        K = _multiple(rng, 64, 5120, rng.choice((64, 64, 64, 16)))
        N = _multiple(rng, 64, 5120, rng.choice((64, 64, 64, 4)))
        x = "f16" if precision == "fp16" else rng.choice(("f16", "f16", "f16", "f32"))
        cap = min(256 * 257, _MAX_OPS // (K * N * (2 if precision == "fp16" else 1)), _MAX_BYTES // (K * (4 if x == "f32" else 2) + 2 * N))
        gelu = rng.random() < 0.4
        return dict(kind=kind, M=_log_int(rng, 1, cap), K=K, N=N, precision=precision, gelu=gelu, x=x,
                    out="f16" if precision == "fp16" else rng.choice(("f16", "f16", "f16", "i8")),
                    dist="gelu_normal" if not gelu and rng.random() < 0.3 else "normal")
    if kind == "block":
        D = _multiple(rng, 192, 1280, 64)
        cap = min(128 * 257, _MAX_OPS // (12 * D * D))
        return dict(kind="block", M=_log_int(rng, 1, cap), D=D, hidden=4 * D)
    if kind == "patch":
        P = rng.choice((16, 16, 14))
        D = _multiple(rng, 192, 1280, 64)
        H, W = P * rng.randint(8, 24), P * rng.randint(8, 24)
        cap = 256 * 224 * 224 // (H * W)
        return dict(kind="patch", B=_log_int(rng, 1, cap), C=3, H=H, W=W, P=P, D=D, precision=precision)
    fmt = rng.choice(("int8", "fp16", "int4"))
    of = 8 if fmt == "int4" else 4
    return dict(kind="weights", N=_multiple(rng, 192, 5120, rng.choice((64, 64, 4))), K=_multiple(rng, 192, 5120, rng.choice((64, 64, of))),
                format=fmt)


# ---------------------------------------------------------------------------------------------------- what is in hand
class _Inputs:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, shape, sigma=1.0, dtype=torch.float32):
        x = torch.randn(shape, generator=self.g, device="cuda", dtype=dtype)
        return x if sigma == 1.0 else x.mul_(sigma)

    def activations(self, M, K, dtype, dist):
        x = self.normal((M, K), dtype=dtype)
        return torch.nn.functional.gelu(x) if dist == "gelu_normal" else x

    def weights(self, *shape):
        return self.normal(shape, 0.02)

    def bias(self, N):
        return self.normal((N,), 0.01)


def _scalar(v):
    return torch.full((1,), v, dtype=torch.float32, device="cuda")


def prepare(case, seed):
    kind, r = case["kind"], _Inputs(seed)
    if kind in ("linear", "step"):
        M, K, N = case["M"], case["K"], case["N"]
        lin = SparseLinear(M, K, N, case["precision"], gelu=case["gelu"], bias=True, out_dtype=_DTYPES[case["out"]], x_dtype=_DTYPES[case["x"]])
        W = r.weights(N, K)
        if kind == "linear":
            lin.prepare_weights(W)
            W = None
        # outputs have a deviation of about 0.02 sqrt(K)
        out_scale = _scalar(4 * 0.02 * math.sqrt(K) / 127) if case["out"] == "i8" else None
        return dict(kind=kind, lin=lin, W=W, X=r.activations(M, K, _DTYPES[case["x"]], case["dist"]), bias=r.bias(N), out_scale=out_scale)
    if kind == "block":
        M, D, hidden = case["M"], case["D"], case["hidden"]
        gain = 0.02 * math.sqrt(D)  # of a layer with D inputs
        # calibrated scales: four deviations on 127 codes; the attention output is such that the next layer's input has deviation 1
        scales = {"x": 4 / 127, "qkv": 4 * gain / 127, "attn": 1 / (gain * 31), "h": 4 / 127, "g": 4 * gain / 127}
        block = EncoderBlockLinears(M, D, hidden, {k: _scalar(v) for k, v in scales.items()})
        block.prepare_weights(r.weights(3 * D, D), r.weights(D, D), r.weights(hidden, D), r.weights(D, hidden))
        block.proj.Xq.copy_(r.normal((M, D), 31.0).round_().clamp_(-127, 127))
        return dict(kind=kind, block=block, x=r.normal((M, D), dtype=torch.float16), biases=tuple(r.bias(n) for n in (3 * D, D, hidden, D)))
    if kind == "patch":
        B, C, H, W, P, D = (case[k] for k in "BCHWPD")
        embed = SparsePatchEmbed(B, C, H, W, P, D, case["precision"])
        embed.prepare_weights(r.weights(D, C, P, P))
        return dict(kind=kind, embed=embed, img=r.normal((B, C, H, W), dtype=torch.float16), bias=r.bias(D))
    return dict(kind=kind, format=case["format"], W=r.weights(case["N"], case["K"]))


def _attention_elsewhere(qkv, out):
    pass


# --------------------------------------------------------------------------------------------------------- one pass
def run(state):
    kind = state["kind"]
    if kind == "linear":
        return state["lin"].forward(state["X"], state["bias"], state["out_scale"])
    if kind == "step":
        lin = state["lin"]
        lin.prepare_weights(state["W"], intermediates=False)
        y = lin.forward(state["X"], state["bias"], state["out_scale"])
        return {"packed": lin.packed, "y": y}
    if kind == "block":
        block = state["block"]
        y = block.forward(state["x"], state["biases"], _attention_elsewhere)
        return {"qkv": block.qkv.Y, "proj": block.proj.Y, "hidden": block.fc1.Y, "y": y}
    if kind == "patch":
        return state["embed"].forward(state["img"], state["bias"])
    W = state["W"]
    if state["format"] == "int4":
        codes, scale = G.quantize_rows_int4(G.prune_4to8_pairs(W, one_per_group=True))
        values4, meta4 = G.compress_int4(codes)
        values8, meta8 = G.int4_to_sparse_int8(values4, meta4, W.shape[1])
        return {"values": values4, "meta": meta4, "scale": scale, "packed": G.pack(values8, meta8, W.shape[1])}
    return {k: v for k, v in G.prepare_weights(W, torch.int8 if state["format"] == "int8" else torch.float16).items() if v is not None}


# ------------------------------------------------------------------------------------------ what it cannot do without
def _packed(N, K, e):
    """kept values and 2-bit positions"""
    return N * K * e / 2 + N * K / 8


def work(case):
    """flops: of the kept half of the weights (one multiply and one add each)"""
    kind = case["kind"]
    if kind in ("linear", "step"):
        M, K, N = case["M"], case["K"], case["N"]
        int8 = case["precision"] == "int8"
        weights = _packed(N, K, 1 if int8 else 2) + N * (8 if int8 else 4)
        size = M * K * (4 if case["x"] == "f32" else 2) + M * N * (1 if case["out"] == "i8" else 2) + weights
        return {"bytes": size + (4 * N * K if kind == "step" else 0), "flops": M * N * K}
    if kind == "block":
        M, D, hidden = case["M"], case["D"], case["hidden"]
        n, weights = 5 * D + hidden, 4 * D * D + 2 * D * hidden
        # in: x (fp16), attention output (int8); out: qkv and hidden codes (int8), proj and y (fp16)
        return {"bytes": M * (2 * D + D + 3 * D + hidden + 4 * D) + _packed(1, weights, 1) + 8 * n, "flops": M * weights}
    if kind == "patch":
        B, C, H, W, P, D = (case[k] for k in "BCHWPD")
        M, K = B * (H // P) * (W // P), C * P * P
        int8 = case["precision"] == "int8"
        return {"bytes": 2 * B * C * H * W + 2 * M * D + _packed(D, K, 1 if int8 else 2) + 8 * D, "flops": M * D * K}
    N, K = case["N"], case["K"]
    out = {"int8": _packed(N, K, 1) + 4 * N, "fp16": _packed(N, K, 2), "int4": N * K * 2.5 / 8 + 4 * N + _packed(N, K, 1)}[case["format"]]
    return {"bytes": 4 * N * K + out, "flops": N * K}


def tolerance(case):
    """Codes, packed weights and the int8 path's linear outputs are defined bit by bit.  GELU is right to one unit in the last
    place of fp16 (a code of its result may then fall on the other side of a tie), an fp16 product to the order of its fp32
    sums and one rounding to fp16."""
    kind = case["kind"]
    if kind == "weights" or (kind in ("linear", "step") and case["precision"] == "int8" and not case["gelu"]):
        return "exact"
    if kind == "patch" and case["precision"] == "int8":
        return "exact"
    if kind == "block":
        return {"rel": 1e-3, "max": 1e-2, "differ": 2e-3}  # fc2 multiplies the codes of GELU
    if kind in ("linear", "step") and case["out"] == "i8":
        return {"rel": 5e-4, "max": 2e-3, "differ": 2e-3}
    return {"rel": 5e-4, "max": 2e-3}
