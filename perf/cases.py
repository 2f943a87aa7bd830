"""Performance cases of the rank layer: what a serving program has this library do, over the range of sizes it meets.

A serving step hands one EP rank's MoE layer a batch of anything from a few decode tokens to a 65 536-token prefill, lets
the policy pick the precision (or forces it), and calls the layer (`kind` "layer"), a pipeline of layers that encodes the
next layer's weights beside the current one's GEMMs ("pipeline"), the entry points one by one ("stages"), or the weight
encoder alone ("encode").  Shapes are those of the repository's workloads (Kimi-VL-A3B: 64 experts, top-6, 8 local,
H 2048, I 1408; Qwen3-VL-30B-A3B: 128 experts, top-8, 16 local, H 2048, I 768; the tiny layer: 8 experts, top-2, H 256,
I 128) and generic ones with odd multiples of 128.  Inputs are drawn on the GPU with the distributions of the
repository's synthetic workloads: x ~ N(0,1), weights ~ N(0,0.02), logits N(0,1) plus, for vision tokens, a Zipf bias
towards the experts of rank 0 (the "hot" rank; every other rank is a "cold" one).

Fields of a case: kind; shape E, k, D, H, I; T (tokens); rank (0 hot); vision (share of vision tokens); zipf (exponent;
0: +2 on experts 0 and 1, the tiny layer's recipe); prec "policy" | "bf16" | "fp4"; encode "main" | "side" |
"speculative" (where a layer call puts the weight encoding; "side" is the binding's default).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2604_19503_amd as R
from paper_2604_19503_amd.binding import default_config

KIMI = dict(E=64, k=6, D=8, H=2048, I=1408, vision=0.75, zipf=1.1)
QWEN = dict(E=128, k=8, D=8, H=2048, I=768, vision=0.80, zipf=1.2)
TINY = dict(E=8, k=2, D=1, H=256, I=128, vision=0.5, zipf=0.0)

FORCE = {"policy": R.FORCE_NONE, "bf16": R.BF16, "fp4": R.FP4}
ENCODE = {"main": 0, "side": 1, "speculative": 3}
BETA = 0.5


def _layer(name, shape, T, prec="policy", encode="side", rank=0, kind="layer"):
    return dict(shape, name=name, kind=kind, T=T, prec=prec, encode=encode, rank=rank)


def listed():
    return [
        # a decode step: a couple of dozen sequences, one token each; the LB gate keeps it in BF16
        _layer("kimi_decode_24", KIMI, 24),
        # a busy decode batch on the many-expert model
        _layer("qwen_decode_192", QWEN, 192),
        # the smallest complete layer, all experts on one rank (the smoke workload), FP4 path
        _layer("tiny_512_fp4", TINY, 512, prec="fp4"),
        # a chunk of a chunked prefill, not a round number of tokens, still below the gate
        _layer("kimi_chunk_1000", KIMI, 1000),
        # a short prefill just above the gate: the hot rank switches to FP4
        _layer("qwen_prefill_3001", QWEN, 3001),
        # an odd layer shape (H and I odd multiples of 128) at an odd batch size, BF16
        _layer("ragged_5003_bf16", dict(E=32, k=4, D=4, H=1152, I=640, vision=0.6, zipf=1.1), 5003, prec="bf16"),
        # a full prefill batch seen by a rank without load: the policy leaves it in BF16
        _layer("kimi_cold_16384", KIMI, 16384, rank=5),
        # the benchmark's headline: the same batch on the hot rank, FP4 by policy, encoders ahead of the decision
        _layer("kimi_hot_16384", KIMI, 16384, encode="speculative"),
        # the all-BF16 baseline of the same layer
        _layer("kimi_bf16_16384", KIMI, 16384, prec="bf16"),
        # a program that calls the entry points one by one, FP4
        _layer("qwen_stages_8192_fp4", QWEN, 8192, prec="fp4", encode="main", kind="stages"),
        # the largest: two layers of distinct weights in a pipeline, each encoding the other's weights beside its GEMMs
        _layer("qwen_pipeline_65536_fp4", QWEN, 65536, prec="fp4", kind="pipeline"),
        # the precision transformation of one layer's experts alone
        _layer("kimi_encode", KIMI, 1, prec="fp4", kind="encode"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.choice(["kimi", "qwen", "kimi", "qwen", "tiny", "odd"])
    kind = rng.choice(["layer"] * 7 + ["stages", "stages", "encode"])
    if what == "tiny":
        shape, T = dict(TINY), _log_int(rng, 1, 4096)
    elif what == "odd":
        E, D, k = rng.choice([(8, 2, 2), (16, 2, 2), (32, 4, 4), (64, 8, 6), (48, 4, 4), (256, 8, 8)])
        shape = dict(E=E, D=D, k=k, H=128 * rng.randint(3, 24), I=128 * rng.randint(1, 12), vision=rng.choice([0.5, 0.6, 0.85]), zipf=1.1)
        T = _log_int(rng, 1, 16384)
    else:
        shape, T = dict(KIMI if what == "kimi" else QWEN), _log_int(rng, 1, 65536 if kind == "layer" else 16384)
    case = dict(shape, kind=kind, T=T, rank=rng.choice([0, 0, shape["D"] - 1]), prec=rng.choice(["policy", "policy", "policy", "bf16", "fp4"]),
                encode=rng.choice(["main", "side", "side", "speculative"]))
    if kind == "stages":
        case.update(prec=rng.choice(["bf16", "fp4"]), encode="main")
    if kind == "encode":
        case.update(T=1, prec="fp4", encode="main", rank=0, E=rng.randint(1, 64), D=1, k=1)
    return case


# ---------------------------------------------------------------------------------------------- inputs
def _logits(case, is_vision, gen):
    E, T = case["E"], case["T"]
    lg = torch.randn((T, E), generator=gen, device="cuda")
    if case["zipf"] == 0.0:
        lg[:, :2] += 2.0 * is_vision.to(torch.float32)[:, None]
        return lg
    nl = E // case["D"]
    z = torch.empty(E, device="cuda")                    # Zipf ranks: 1..nl on rank 0's experts, the rest behind them
    z[:nl] = 1.0 + torch.randperm(nl, generator=gen, device="cuda").float()
    z[nl:] = nl + 1.0 + torch.randperm(E - nl, generator=gen, device="cuda").float()
    p = z ** -case["zipf"]
    bias = BETA * torch.log(E * p / p.sum())
    return lg.addcmul_(is_vision.to(torch.float32)[:, None], bias[None, :])


def _randn_bf16(shape, std, gen):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(torch.bfloat16)


class _State:
    pass


def prepare(case, seed):
    """Tokens, logits, weights, the context, and the caller's buffers (rows that a call leaves unwritten hold zeros)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 7919 + 17)
    E, k, D, H, I, T = (case[n] for n in ("E", "k", "D", "H", "I", "T"))
    nl = E // D
    s = _State()
    s.case = case
    s.cfg = default_config(T, E, k, D, H, I)
    s.ctx = R.Context(s.cfg)
    n_layers = 2 if case["kind"] == "pipeline" else 1
    s.weights = [(_randn_bf16((nl, 2 * I, H), 0.02, gen), _randn_bf16((nl, H, I), 0.02, gen)) for _ in range(n_layers)]
    if case["kind"] == "encode":
        s.buf = R.WeightBuffers(s.cfg)
        for t in (s.buf.w13_s, s.buf.w2_s):
            t.zero_()
        return s
    s.is_vision = torch.zeros(T, dtype=torch.uint8, device="cuda")
    s.is_vision[torch.randperm(T, generator=gen, device="cuda")[: int(round(case["vision"] * T))]] = 1
    s.x = _randn_bf16((T, H), 1.0, gen)
    s.logits = [_logits(case, s.is_vision, gen) for _ in range(n_layers)]
    s.buf = b = R.LayerBuffers(s.cfg, T)
    for t in (b.row_to_assign, b.assign_to_row, b.out, b.w13_s, b.w2_s, b.x_s):
        t.zero_()
    if case["kind"] == "stages":
        for t in (b.x_perm, b.x_q, b.y_rows):
            t.zero_()
        return s
    force = FORCE[case["prec"]]
    if case["kind"] == "layer":
        s.io = s.ctx.make_io(s.logits[0], s.is_vision, s.x, *s.weights[0], b, case["rank"], force=force, overlap=ENCODE[case["encode"]])
        return s
    # pipeline: two layers alternate between a pair of FP4 weight buffers; the first layer's weights are encoded up front
    pair = [R.WeightBuffers(s.cfg), R.WeightBuffers(s.cfg)]
    s.outs = [torch.zeros((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    s.ios = []
    for i in (0, 1):
        io = s.ctx.make_io(s.logits[i], s.is_vision, s.x, *s.weights[i], b, case["rank"], force=force, overlap=4)
        io.out = s.outs[i].data_ptr()
        s.ctx.use_weight_buffers(io, pair[i])
        s.ctx.set_prefetch(io, *s.weights[1 - i], pair[1 - i], 0)
        s.ios.append(io)
    s.ctx.quantize_experts_fp4(*s.weights[0], pair[0])
    return s


def run(s):
    kind, b = s.case["kind"], s.buf
    if kind == "encode":
        s.ctx.quantize_experts_fp4(*s.weights[0], b)
        return [b.w13_q, b.w13_s, b.w2_q, b.w2_s]
    if kind == "layer":
        prec = s.ctx.layer_forward(s.io)
        return [b.out, b.topk_ids, b.topk_w, b.expert_cnt, b.expert_vis, b.rank_load, b.rank_vis, b.expert_offsets, b.row_to_assign,
                b.assign_to_row, prec, s.io.ib_global]
    if kind == "pipeline":
        for io in s.ios:
            s.ctx.layer_forward(io)
        return [s.outs[0], s.outs[1], b.topk_ids, b.topk_w, b.expert_cnt, b.expert_vis, b.expert_offsets, b.assign_to_row]
    prec = FORCE[s.case["prec"]]
    s.ctx.route_stats(s.logits[0], s.is_vision, b)
    plan, ib, _ = s.ctx.select_precision(b, s.case["T"], force=prec)
    rows = [b.x_perm]
    if prec == R.FP4:
        s.ctx.quantize_experts_fp4(*s.weights[0], b)
        rows = [b.x_q, b.x_s, b.w13_q, b.w13_s, b.w2_q, b.w2_s]
    s.ctx.permute(s.x, b, s.case["rank"], prec)
    s.ctx.grouped_moe_ffn(prec, *s.weights[0], b)
    s.ctx.combine(b)
    return [b.out, b.y_rows, b.topk_ids, b.topk_w, b.expert_cnt, b.expert_vis, b.expert_offsets, b.row_to_assign, b.assign_to_row, plan, ib] + rows


# ---------------------------------------------------------------------------------------------- work
@functools.lru_cache(maxsize=None)
def _routing(E, k, D, T, rank, vision, zipf):
    """(rows on the rank per token, share of tokens with a local expert, local experts with a row), estimated on up to
    4096 tokens of the same distribution."""
    n, nl = min(T, 4096), E // D
    rng = np.random.default_rng(5)
    lg = rng.standard_normal((n, E))
    vis = rng.random(n) < vision
    if zipf == 0.0:
        lg[vis, :2] += 2.0
    else:
        p = np.arange(1, E + 1, dtype=np.float64) ** -zipf
        p /= p.sum()
        lg[vis] += BETA * np.log(E * p)
    top = np.argpartition(-lg, k - 1, axis=1)[:, :k]
    mine = top // nl == rank
    return mine.sum() / n, mine.any(axis=1).mean(), len(np.unique(top[mine]))


def work(case):
    E, k, D, H, I, T = (case[n] for n in ("E", "k", "D", "H", "I", "T"))
    nl = E // D
    n_weights = 3 * H * I
    codes = 0.5 + 1.0 / 32
    if case["kind"] == "encode":
        return {"bytes": nl * n_weights * (2 + codes), "flops": 0}
    per_token, share, active = _routing(E, k, D, T, case["rank"], case["vision"], case["zipf"])
    rows = per_token * T
    flops = 6.0 * rows * H * I
    # logits, flags, routing results and the permutation's tables; tokens in, tokens out
    b = T * (4 * E + 1 + 8 * k + 4 * k) + 4 * rows + 2 * H * T * share + 2 * H * T
    if case["kind"] == "stages":                       # the permuted rows and the expert outputs are results here
        fp4 = case["prec"] == "fp4"
        b += rows * H * (codes if fp4 else 2) + rows * H * 2 + (nl * n_weights * (2 + codes) if fp4 else active * n_weights * 2)
    else:
        b += active * n_weights * 2
    n = 2 if case["kind"] == "pipeline" else 1
    return {"bytes": n * b, "flops": n * flops}


def tolerance(case):
    """Integers, codes and scales are exact (no "differ").  BF16 results: two correct implementations differ by output
    roundings (2^-9 relative each, rms) and by boundary flips of the BF16 intermediate; on the FP4 path a flip moves an
    intermediate value by a whole E2M1 step, which the repository's end-to-end bound puts at 4e-3 in the norm."""
    if case["kind"] == "encode":
        return "exact"
    return {"rel": 5e-3, "max": 0.03 if case["prec"] == "bf16" else 0.1}
