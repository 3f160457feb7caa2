"""What is measured: the calls a training or inference program makes of this package, over their real range.

Kinds of case
  attention      one attention call, forward alone (inference) or forward and backward (training), through
                 the torch.autograd front end or, with front="binding", through the C ABI's binding on
                 preallocated outputs and workspace
  layer_norm     layer_norm forward and backward over M tokens of width D
  bias_gelu      bias_gelu forward and backward over M tokens of width F
  encoder_layer  one pre-norm encoder layer, forward and backward, from layer_norm, attention_qkvpacked and
                 bias_gelu_linear; the other matrix products are torch's

Values follow the package's synthetic recipe: q, k, v and gradients N(0,1), normalisation gains
1 + 0.1 N(0,1) and biases 0.1 N(0,1), pre-activations 1.5 N(0,1).  Softmax scale is 1/sqrt(d).
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

import paper_2309_16669_amd as av
from paper_2309_16669_amd import autograd as ag

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16}


def _attention(name, B, H, N, d=64, dtype="bf16", causal=False, packed=False, train=True, front="autograd"):
    c = {"kind": "attention", "B": B, "H": H, "N": N, "d": d, "dtype": dtype, "causal": causal, "packed": packed,
         "train": train, "front": front}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the text encoder on one caption of 77 tokens, as when a query is embedded to search videos: the
        # smallest call, all launch and latency
        _attention("caption_infer", 1, 8, 77, causal=True, train=False),
        # one 16-frame clip at 224 x 224 (8 x 14 x 14 tokens) through a ViT-B layer: features of one video
        _attention("clip_infer", 1, 12, 1568, dtype="f16", packed=True, train=False),
        # fine-tuning with two clips of 4 frames (784 tokens and a class token) of a 16-head encoder per GPU
        _attention("clips_cls_train", 2, 16, 785, packed=True),
        # the ViT-B video training batch: 32 clips of 1568 tokens, outputs and workspace kept by the program
        _attention("vitb_batch_train", 32, 12, 1568, front="binding"),
        # 16 frames at 336 x 336 (8 x 21 x 21 tokens), ViT-L heads, fp16 as under automatic mixed precision
        _attention("vitl_336_train", 4, 16, 3528, dtype="f16", packed=True),
        # ViT-H-width heads of 80 channels
        _attention("vith_d80_train", 8, 16, 1568, d=80),
        # a text-encoder layer on the 2048 captions of a contrastive batch
        _attention("text_77_train", 2048, 8, 77, causal=True, packed=True),
        # temporal half of a divided space/time layer: one problem of 16 frames per position of 32 clips
        _attention("temporal_16_train", 32 * 196, 12, 16),
        # its spatial half: one problem of 14 x 14 tokens per frame of 32 clips of 8 frames
        _attention("spatial_196_train", 32 * 8, 12, 196, packed=True),
        # normalisation in front of attention and MLP on the training batch's tokens
        {"name": "layer_norm_train", "kind": "layer_norm", "M": 32 * 1568, "D": 768, "dtype": "bf16"},
        # the MLP's bias + GELU on the same tokens
        {"name": "bias_gelu_train", "kind": "bias_gelu", "M": 32 * 1568, "F": 3072, "dtype": "bf16"},
        # a whole ViT-B layer at the shape of the memory profile: 16 videos of 784 tokens
        {"name": "encoder_layer_train", "kind": "encoder_layer", "B": 16, "N": 784, "H": 12, "d": 64, "dtype": "bf16"},
    ]


# no drawn case costs more than these: elements of one tensor of the temporal batch, and the operations of
# the video training batch
MOST_ELEMENTS = 32 * 196 * 12 * 16 * 64
MOST_FLOPS = 14.0 * 32 * 12 * 1568 ** 2 * 64


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_attention(rng, n_lo, n_hi, b_hi, causal):
    d = rng.choice((64, 64, 64, 80))
    H = rng.choice((6, 8, 12, 16))
    N = _log_int(rng, n_lo, n_hi)
    train = rng.random() < 0.75
    most = int(min(b_hi, MOST_ELEMENTS / (N * H * d), MOST_FLOPS / (14.0 * H * N * N * d)))
    B = _log_int(rng, 1, max(1, most))
    return _attention(None, B, H, N, d, rng.choice(("bf16", "bf16", "f16")), causal, rng.random() < 0.5, train,
                      rng.choice(("autograd", "autograd", "binding")))


def draw(rng):
    pick = rng.random()
    if pick < 0.30:   # joint space-time attention: 2 to 32 frames at 224 or 336, with or without a class token
        return _draw_attention(rng, 392, 3600, 64, False)
    if pick < 0.45:   # text
        return _draw_attention(rng, 33, 128, 4096, True)
    if pick < 0.60:   # spatial attention of one frame
        return _draw_attention(rng, 49, 600, 1024, False)
    if pick < 0.70:   # temporal attention
        return _draw_attention(rng, 2, 32, 20000, False)
    if pick < 0.82:
        return {"kind": "layer_norm", "M": _log_int(rng, 77, 64000), "D": 8 * rng.randint(32, 160),
                "dtype": rng.choice(("bf16", "f16"))}
    if pick < 0.94:
        return {"kind": "bias_gelu", "M": _log_int(rng, 77, 50000), "F": 8 * rng.randint(128, 400),
                "dtype": rng.choice(("bf16", "f16"))}
    N = _log_int(rng, 77, 1600)
    return {"kind": "encoder_layer", "B": _log_int(rng, 1, max(1, 12000 // N)), "N": N, "H": rng.choice((8, 12)), "d": 64,
            "dtype": "bf16"}


class State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = DTYPES[case["dtype"]]

    def normal(*shape, mul=1.0, add=0.0, dtype=dt):
        # drawn in slices, so that no fp32 copy of a large tensor is ever held
        out = torch.empty(shape, dtype=dtype, device="cuda")
        flat = out.view(-1)
        for i in range(0, flat.numel(), 1 << 24):
            part = flat[i:i + (1 << 24)]
            part.copy_(torch.randn(part.numel(), generator=gen, device="cuda").mul_(mul).add_(add))
        return out

    s = State()
    s.case = case
    kind = case["kind"]
    if kind == "attention":
        B, H, N, d = (case[k] for k in ("B", "H", "N", "d"))
        s.scale = 1.0 / math.sqrt(d)
        s.qkv = normal(B, N, 3, H, d) if case["packed"] else None
        s.q, s.k, s.v = (None, None, None) if case["packed"] else (normal(B, N, H, d) for _ in range(3))
        s.dO = normal(B, N, H, d) if case["train"] else None
        if case["front"] == "binding":
            s.first = s.qkv if case["packed"] else s.q
            s.o = torch.empty((B, N, H, d), dtype=dt, device="cuda")
            s.lse = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
            if case["train"]:
                s.grads = tuple(torch.empty_like(t) for t in ((s.qkv,) if case["packed"] else (s.q, s.k, s.v)))
                s.ws = torch.empty(av.attn_bwd_workspace_bytes(B, H, N, d), dtype=torch.uint8, device="cuda")
        elif case["train"]:
            s.leaves = [t.requires_grad_() for t in ((s.qkv,) if case["packed"] else (s.q, s.k, s.v))]
    elif kind == "layer_norm":
        M, D = case["M"], case["D"]
        s.x = normal(M, D).requires_grad_()
        s.gamma = normal(D, mul=0.1, add=1.0, dtype=torch.float32).requires_grad_()
        s.beta = normal(D, mul=0.1, dtype=torch.float32).requires_grad_()
        s.dy = normal(M, D)
    elif kind == "bias_gelu":
        M, W = case["M"], case["F"]
        s.x = normal(M, W, mul=1.5).requires_grad_()
        s.bias = normal(W, mul=0.1, dtype=torch.float32).requires_grad_()
        s.dy = normal(M, W)
    else:
        B, N, H, d = (case[k] for k in ("B", "N", "H", "d"))
        W = H * d
        s.x = normal(B, N, W).requires_grad_()
        s.dy = normal(B, N, W)
        one = dict(mul=0.1, add=1.0, dtype=torch.float32)
        zero = dict(mul=0.1, dtype=torch.float32)
        s.par = {
            "g1": normal(W, **one), "b1": normal(W, **zero), "g2": normal(W, **one), "b2": normal(W, **zero),
            "wqkv": normal(3 * W, W, mul=W ** -0.5), "bqkv": normal(3 * W, mul=0.1),
            "wo": normal(W, W, mul=W ** -0.5), "bo": normal(W, mul=0.1),
            "w1": normal(4 * W, W, mul=W ** -0.5), "c1": normal(4 * W, **zero),
            "w2": normal(W, 4 * W, mul=(4 * W) ** -0.5), "c2": normal(W, mul=0.1),
        }
        for p in s.par.values():
            p.requires_grad_()
        s.leaves = [s.x, *s.par.values()]
    return s


def _run_attention(s):
    c = s.case
    if c["front"] == "binding":
        av.attn_fwd_ex(s.first, s.k, s.v, s.o, s.lse, s.scale, c["causal"])
        if not c["train"]:
            return {"o": s.o, "lse": s.lse}
        dq, dk, dv = (s.grads[0], None, None) if c["packed"] else s.grads
        av.attn_bwd_ex(s.first, s.k, s.v, s.o, s.lse, s.dO, dq, dk, dv, s.scale, s.ws, c["causal"])
        return {"o": s.o, "lse": s.lse, "grads": s.grads}

    def call():
        if c["packed"]:
            return ag.attention_qkvpacked(s.qkv, causal=c["causal"])
        return ag.attention(s.q, s.k, s.v, causal=c["causal"])

    if not c["train"]:
        with torch.no_grad():
            return {"o": call()}
    o = call()
    return {"o": o.detach(), "grads": torch.autograd.grad(o, s.leaves, s.dO)}


def _run_layer(s):
    c, p = s.case, s.par
    B, N, H, d = (c[k] for k in ("B", "N", "H", "d"))
    W = H * d
    qkv = F.linear(ag.layer_norm(s.x, p["g1"], p["b1"]), p["wqkv"], p["bqkv"])
    o = ag.attention_qkvpacked(qkv.view(B, N, 3, H, d))
    x1 = s.x + F.linear(o.view(B, N, W), p["wo"], p["bo"])
    h = F.linear(ag.layer_norm(x1, p["g2"], p["b2"]), p["w1"])
    y = x1 + ag.bias_gelu_linear(h, p["c1"], p["w2"], p["c2"])
    return {"y": y.detach(), "grads": torch.autograd.grad(y, s.leaves, s.dy)}


def run(state):
    kind = state.case["kind"]
    if kind == "attention":
        return _run_attention(state)
    if kind == "encoder_layer":
        return _run_layer(state)
    if kind == "layer_norm":
        y = ag.layer_norm(state.x, state.gamma, state.beta)
        leaves = (state.x, state.gamma, state.beta)
    else:
        y = ag.bias_gelu(state.x, state.bias)
        leaves = (state.x, state.bias)
    return {"y": y.detach(), "grads": torch.autograd.grad(y, leaves, state.dy)}


def work(case):
    kind = case["kind"]
    if kind == "attention":
        B, H, N, d = (case[k] for k in ("B", "H", "N", "d"))
        tensor, lse = 2 * B * H * N * d, 4 * B * H * N
        pairs = B * H * (N * (N + 1) // 2 if case["causal"] else N * N)
        # forward: q, k, v in, o out (and LSE where it is handed over); backward: q, k, v, o, dO, LSE in, dq, dk, dv out
        if not case["train"]:
            return {"bytes": 4 * tensor + (lse if case["front"] == "binding" else 0), "flops": 4 * d * pairs}
        return {"bytes": 12 * tensor + 2 * lse, "flops": 14 * d * pairs}
    if kind == "layer_norm":
        M, D = case["M"], case["D"]
        # x in, y out, mean and 1/sigma out; x, dy and the two in, dx out; gain, bias and their gradients
        return {"bytes": 10 * M * D + 16 * M + 5 * 4 * D, "flops": 24 * M * D}
    if kind == "bias_gelu":
        M, W = case["M"], case["F"]
        return {"bytes": 10 * M * W + 3 * 4 * W, "flops": 50 * M * W}
    B, N, H, d = (case[k] for k in ("B", "N", "H", "d"))
    W, T = H * d, B * N
    weights = 12 * W * W
    # matrix products: forward, input gradient and weight gradient; attention as above.  Bytes: x, dy in, y, dx out,
    # weights in, their gradients out, and what is kept between the passes once out and once in
    kept = 2 * T * W * (1 + 1 + 3 + 1 + 1 + 1 + 4)
    return {"bytes": 2 * 4 * T * W + 2 * 3 * weights + 2 * kept, "flops": 3 * 2 * T * weights + 14 * B * H * N * N * d}


def tolerance(case):
    # Four times the largest error of any output measured against the same path in 64 bits (2-norm, and largest element over
    # the result's rms or over itself).  What sets it: the rounding of results to the 16-bit format, of the softmax weights
    # and of dS before they enter a product, and of o before it enters the row sums of dO o o.
    bf16 = case["dtype"] == "bf16"
    kind = case["kind"]
    if kind == "attention":
        if case["N"] < 4:   # dS cancels almost completely over two or three keys
            # measured 3.8e-3, 5.6e-2 in bf16; 4.7e-4, 4.3e-3 in fp16
            return {"rel": 1.5e-2, "max": 2.2e-1} if bf16 else {"rel": 1.9e-3, "max": 1.8e-2}
        # measured 3.0e-3, 3.1e-2 in bf16; 3.7e-4, 4.2e-3 in fp16 (4 <= N <= 3528, d = 64 and 80, causal and not)
        return {"rel": 1.2e-2, "max": 1.3e-1} if bf16 else {"rel": 1.5e-3, "max": 1.7e-2}
    if kind == "encoder_layer":   # measured 5.9e-3, 4.1e-2 over the output and the 13 gradients
        return {"rel": 2.4e-2, "max": 1.7e-1}
    # one rounding of y and dx: measured 1.7e-3, 3.9e-3 in bf16; 2.1e-4, 4.9e-4 in fp16
    return {"rel": 6.8e-3, "max": 1.6e-2} if bf16 else {"rel": 8.4e-4, "max": 2.0e-3}
