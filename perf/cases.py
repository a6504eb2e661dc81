"""The work a program gives this framework, as cases that can be timed and compared.

A case is one pass of one MoHGE layer through the public layer object (`MoHGELayer`): a forward
pass, or a training step (forward, both auxiliary losses, backward).  `listed()` names the cases
that stand for the use of the layer from a single decoded token to the largest prefill; `draw()`
gives further ones of the same ranges.  The layer shapes are the ones `synth.WORKLOADS` names plus
generic ones with odd sizes; inputs are drawn on the GPU with the distributions `synth` states
(x, dy ~ N(0, 1), weights ~ N(0, 0.02^2), Zipf-shaped logit bias where routing is skewed).
"""
from __future__ import annotations

import math

import torch

import paper_2604_23108_amd as M

# Layer shapes: hidden size, groups x experts per group, widths, groups and experts kept per token,
# selection over all kept groups ("global") or inside each ("group").  The largest single-GPU share
# (decode and skewed prefill), the mid-sized layer (prefill and training), the three layer shapes of
# the paper's architecture table, and two generic ones: a hidden size and a group size that are no
# powers of two, and many experts in few wide groups.
SHAPES = {
    "large": dict(d=4096, groups=4, experts=16, d_ff="768,1024,1536,2048", k_groups=2, k_experts=4, select="group"),
    "mid": dict(d=2048, groups=3, experts=8, d_ff="512,1024,1536", k_groups=2, k_experts=4, select="group"),
    "paper_1b": dict(d=1024, groups=8, experts=4, d_ff="256,320,384,512,640,768,832,896", k_groups=3, k_experts=6,
                     select="global"),
    "paper_3b": dict(d=1024, groups=8, experts=8, d_ff="384,512,640,768,896,1024,1152,1280", k_groups=3, k_experts=6,
                     select="global"),
    "paper_14b": dict(d=1024, groups=8, experts=16, d_ff="640,768,896,1024,1152,1280,1408,1536", k_groups=3,
                      k_experts=6, select="global"),
    "odd": dict(d=1344, groups=5, experts=5, d_ff="192,448,704,960,1216", k_groups=2, k_experts=4, select="group"),
    "wide": dict(d=2560, groups=2, experts=32, d_ff="1088,1728", k_groups=2, k_experts=6, select="global"),
}


def _case(shape: str, T: int, **kw) -> dict:
    c = dict(SHAPES[shape], T=T, dtype="bf16", weights="bf16", step="forward", skew=0.0, shared=0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a unit-sized fp32 layer, launches and latency only
        dict(_case("large", 64, d=128, groups=3, experts=4, d_ff="64,128,256", k_groups=2, k_experts=2,
                   dtype="f32"), name="f32_tiny"),
        # a full layer in fp32, as one runs it to check a model's numerics
        dict(_case("paper_1b", 512, dtype="f32"), name="f32_layer"),
        # one token of one sequence: interactive decoding
        dict(_case("large", 1), name="decode_1"),
        # a decode step of 32 sequences: every touched expert's weights are streamed once
        dict(_case("large", 32), name="decode_32"),
        # the same with quantised expert weights, at batch sizes a server sees between those two
        dict(_case("large", 32, weights="fp8"), name="decode_32_fp8"),
        dict(_case("large", 7, weights="mxfp4"), name="decode_7_mxfp4"),
        # a serving step beyond decode size (many sequences, or a few with speculative tokens):
        # a handful of rows per expert, all weights touched
        dict(_case("large", 160), name="batch_160"),
        # prefill of an odd number of tokens through a layer of the paper with its two shared experts
        dict(_case("paper_3b", 1531, shared=640), name="prefill_1531_shared"),
        # a mid-sized prefill
        dict(_case("mid", 4096), name="prefill_4096"),
        # the largest prefill, token counts per expert ranging over more than a factor of ten
        dict(_case("large", 16384, skew=2.0), name="prefill_16384_skewed"),
        # a training step of a small micro-batch of odd size
        dict(_case("paper_1b", 777, step="train"), name="train_777"),
        # a training step of a full micro-batch
        dict(_case("mid", 8192, step="train"), name="train_8192"),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "decode", "decode", "batch", "batch", "prefill", "prefill", "train"])
    shape = rng.choice(sorted(SHAPES))
    if kind == "f32":
        c = _case(rng.choice(["paper_1b", "odd", "mid"]), _log_int(rng, 9, 512), dtype="f32")
    elif kind == "decode":
        c = _case(shape, rng.randint(1, 32), weights=rng.choice(["bf16", "bf16", "fp8", "mxfp4"]))
    elif kind == "batch":
        c = _case(shape, _log_int(rng, 33, 1024))
    elif kind == "prefill":
        c = _case(shape, _log_int(rng, 1024, 16384), skew=rng.choice([0.0, 0.0, 1.0, 2.0]),
                  shared=rng.choice([0, 0, 0, 320, 640]))
    else:
        c = _case(shape if shape != "large" else "mid", _log_int(rng, 200, 8192), step="train",
                  skew=rng.choice([0.0, 0.0, 1.0]))
    if rng.random() < 0.25:
        c["select"] = "global" if c["select"] == "group" else "group"
    # no drawn case costs more than the largest listed one of its kind
    most = {"f32": listed()[1], "train": listed()[-1]}.get(kind, listed()[9])
    while work(c)["flops"] > work(most)["flops"]:
        c["T"] = c["T"] * 3 // 4
    return c


def _widths(case):
    return [int(f) for f in case["d_ff"].split(",")]


def work(case):
    T, d, ke, ff = case["T"], case["d"], case["k_experts"], _widths(case)
    train = case["step"] == "train"
    n_e, outs = case["groups"] * case["experts"], case["groups"] * (case["experts"] + 1)
    f_mean = sum(ff) / len(ff)
    # every token's pairs through an expert of average width, the router's logits, shared experts;
    # the backward pass costs twice the forward
    flops = 6.0 * T * ke * d * f_mean + 2.0 * T * d * outs + 6.0 * T * 2 * d * case["shared"]
    if train:
        flops *= 3
    # weights of the experts that T uniformly routed tokens are expected to touch
    touched = n_e * (1.0 - (1.0 - ke / n_e) ** T)
    elt = 2.0 if case["dtype"] == "bf16" else 4.0
    # stored weights: FP8 codes and one fp32 scale per row, MXFP4 codes and a byte per 32
    per_weight = {"bf16": elt, "fp8": 1.0, "mxfp4": 0.5 + 1.0 / 32}[case["weights"]]
    expert = 3 * d * f_mean * per_weight + ((2 * f_mean + d) * 4 if case["weights"] == "fp8" else 0)
    shared = 2 * 3 * d * case["shared"] * elt
    bytes_ = touched * expert + shared + 4.0 * outs * d + 2.0 * T * d * elt + T * (case["k_experts"] * 8.0)
    if train:
        # dy read, dx written, all weight gradients written
        bytes_ += 2.0 * T * d * elt + n_e * 3 * d * f_mean * elt + 4.0 * outs * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # Four times the error measured against the same layer in float64 (on the routing taken): bf16 forward
    # 2.9e-3 (largest 0.016 of the rms), with gradients 4.0e-3 (0.035).  fp32 is 2e-7 with sums over 64
    # lanes; a running sum over 1024 terms is expected at 1e-6 (2^-24 sqrt(1024) / sqrt(3)).  `differ` is
    # for expert ids of tokens whose selection keys tie within the fp32 error of a logit.
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5, "differ": 1e-4}
    if case["step"] == "train":
        return {"rel": 1.6e-2, "max": 0.14, "differ": 1e-4}
    return {"rel": 1.2e-2, "max": 0.065, "differ": 1e-4}


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    bf = case["dtype"] == "bf16"
    dt = torch.bfloat16 if bf else torch.float32
    T, d, N, ff = case["T"], case["d"], case["experts"], _widths(case)

    def normal(*shape, scale=1.0, dtype=dt):
        t = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
        return t.mul_(scale).to(dtype)

    train = case["step"] == "train"
    s = _State()
    s.x = normal(T, d)
    w_group = normal(case["groups"], d, scale=0.02, dtype=torch.float32)
    w_expert = normal(case["groups"] * N, d, scale=0.02, dtype=torch.float32)
    w13 = [normal(N, 2 * f, d, scale=0.02) for f in ff]
    w2 = [normal(N, d, f, scale=0.02) for f in ff]
    bias = None
    if case["skew"] > 0:
        ranks = torch.stack([torch.randperm(N, generator=gen, device="cuda") for _ in ff]).float() + 1.0
        bias = (-case["skew"] * 1.1 * ranks.log()).reshape(-1).contiguous()
    cfg = M.Config(T=T, d=d, n_groups=case["groups"], experts_per_group=N, d_ff=ff, k_groups=case["k_groups"],
                   k_experts=case["k_experts"],
                   select_mode=M.SELECT_GLOBAL if case["select"] == "global" else M.SELECT_PER_GROUP,
                   dtype=M.BF16 if bf else M.F32)
    shared = None
    if case["shared"]:
        f = case["shared"]
        shared = M.SharedExperts(T, d, normal(2, 2 * f, d, scale=0.02), normal(2, d, f, scale=0.02), dtype=cfg.dtype,
                                 backward=train)
    s.layer = M.MoHGELayer(cfg, w_group, w_expert, w13, w2, bias, training=train, backward=train, shared=shared)
    if case["weights"] == "fp8":
        s.layer.use_fp8_weights()
    elif case["weights"] == "mxfp4":
        s.layer.use_mxfp4_weights()
    s.dy = normal(T, d) if train else None
    return s


def run(state):
    L = state.layer
    y = L.forward(state.x)
    out = {"y": y, "expert_idx": L.expert_idx, "gates": L.gates}
    if state.dy is not None:
        out.update(dx=L.backward(state.x, state.dy), losses=L.losses, dw13=L.dw13, dw2=L.dw2, dw_group=L.dw_group,
                   dw_expert=L.dw_expert)
    return out
