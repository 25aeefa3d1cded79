"""What a user of this library has it do, as cases that can be timed and compared.

One pass is a call (or the chain of calls) that a serving or evaluation program makes through the public Python
entry points, on weights that it laid out once and on activations that are new each time:

  layer    moe_layer_forward through MoELayer: gate, routing, expert FFNs, combine, dense branch of Residual-MoE
  block    moe_decode_block_forward: one decode step of a whole decoder block with its key/value cache
  stages   moe_gate, moe_dispatch, moe_expert_ffn, moe_combine as calls of their own: what a program with an
           exchange between devices around the expert FFNs uses

Shapes are those of the benchmark (workloads/configs.py) and of the model family that they belong to: hidden sizes
1024, 2048 and 4096 with d_ffn = 4 d_model, 32 to 128 experts, decode batches up to 256 tokens and prefill batches up
to 16384, plus the small fp32 layers that tests and comparisons use.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2201_05596_amd as moe

WEIGHT_STD = 0.02        # gate, expert, dense-branch weights, as in workloads/generate.py
BIAS_STD = 0.02
ZIPF = 1.5               # gate bias of skewed routing: ZIPF * ln(1 / (e + 1))
LARGEST_S = 2.9e-3       # estimated time of the largest listed case (`estimate` below); drawn cases stay below it


def _capacity(c):
    return max(1, math.ceil(c["capacity_factor"] * c["top_k"] * c["T"] / c["E"] - 1e-9))


def _case(kind, T, d, E, top_k=1, cf=1.0, dtype="bf16", residual=False, skewed=False, packed=True, f=None, heads=0, max_len=0):
    return {"kind": kind, "T": T, "d_model": d, "d_ffn": f if f else 4 * d, "E": E, "top_k": top_k, "capacity_factor": cf,
            "dtype": dtype, "residual": residual, "skewed": skewed, "packed": packed and dtype == "bf16", "heads": heads,
            "max_len": max_len}


def listed():
    named = {
        # the fp32 layer of the smallest configuration: launches and host work are all there is to it
        "tiny_fp32": _case("layer", 256, 64, 8, dtype="f32"),
        # an fp32 layer of ordinary size, as evaluated next to fp32 training code
        "fp32_top2": _case("layer", 1536, 512, 8, top_k=2, cf=1.25, dtype="f32"),
        # one sequence decoding on a 350M+MoE-128 layer: the latency of a single user's token
        "decode_1": _case("layer", 1, 1024, 128, cf=2.0),
        # a small decode batch on a Residual-MoE layer (1.3B+PR-MoE-64): few rows in the experts and in the dense branch
        "decode_residual_16": _case("layer", 16, 2048, 64, cf=2.0, residual=True),
        # the decode batch of the benchmark on a 1.3B+MoE-128 layer
        "decode_64": _case("layer", 64, 2048, 128, cf=2.0),
        # the same decode step with the rest of the decoder block: 16 heads, sequences at all positions of a 2048 cache
        "block_64": _case("block", 64, 2048, 128, cf=2.0, heads=16, max_len=2048),
        # a ragged chunk of a prefill, top-2, on weights as the checkpoint holds them
        "chunk_777_plain": _case("layer", 777, 1024, 128, top_k=2, cf=1.25, packed=False),
        # prefill of 8 x 1024 tokens on a 350M+MoE-128 layer
        "prefill_128": _case("layer", 8192, 1024, 128),
        # the same tokens on the two layer kinds of 350M+PR-MoE-32/64
        "prefill_residual_32": _case("layer", 8192, 1024, 32, residual=True),
        "prefill_residual_64": _case("layer", 8192, 1024, 64, residual=True),
        # one GPU's share of a 6.7B-class model: top-2 with a few experts at capacity and many with a handful of rows
        "prefill_skewed": _case("layer", 16384, 4096, 64, top_k=2, cf=1.25, skewed=True),
        # the steps called one by one on an odd number of tokens
        "stages_4001": _case("stages", 4001, 1024, 32, top_k=2),
    }
    return [dict(c, name=n) for n, c in named.items()]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.choice(["fp32", "decode", "decode", "prefill", "prefill", "prefill", "stages", "block"])
    top_k = rng.choice([1, 1, 2])
    residual = rng.random() < 0.4
    if what == "fp32":
        c = _case("layer", _log_int(rng, 1, 2048), rng.choice([64, 128, 200, 256, 512]), rng.choice([4, 8, 16, 31]), top_k,
                  rng.choice([1.0, 1.25, 2.0]), "f32", residual)
    elif what in ("decode", "block"):
        c = _case("layer", _log_int(rng, 1, 256), rng.choice([1024, 2048]), rng.choice([32, 64, 128]), top_k,
                  rng.choice([1.0, 2.0, 4.0]), residual=residual, skewed=rng.random() < 0.3, packed=rng.random() < 0.8)
        if what == "block":
            c.update(kind="block", heads=c["d_model"] // rng.choice([64, 128]), max_len=_log_int(rng, 128, 2048))
    else:
        d = rng.choice([1000, 1024, 1024, 2048, 4096])
        E = rng.choice([16, 32, 40, 64] if d == 4096 else [16, 32, 40, 64, 128])
        c = _case("layer", _log_int(rng, 257, 16384), d, E, top_k, rng.choice([1.0, 1.25, 1.5]), residual=residual,
                  skewed=rng.random() < 0.3, packed=rng.random() < 0.8)
        if what == "stages":
            c.update(kind="stages", residual=False)
    while estimate(c) > LARGEST_S and c["T"] > 1:
        c["T"] = int(c["T"] * 0.7)
    return c


def _rows(c):
    """Rows that the experts keep, for activations and gate weights of the distributions that prepare() draws from."""
    r = np.random.RandomState(0)
    logits = r.standard_normal((c["T"], c["E"])) * (WEIGHT_STD * math.sqrt(c["d_model"]))
    if c["skewed"]:
        logits += ZIPF * np.log(1.0 / (np.arange(c["E"]) + 1.0))
    chosen = np.argsort(-logits, axis=1)[:, :c["top_k"]]
    return np.minimum(np.bincount(chosen.reshape(-1), minlength=c["E"]), _capacity(c))


def work(c):
    """Every weight of an expert that has a row, and of the dense parts, read once; activations read and written once."""
    T, d, f, E, k = c["T"], c["d_model"], c["d_ffn"], c["E"], c["top_k"]
    el = 4 if c["dtype"] == "f32" else 2
    rows = _rows(c)
    kept, touched = int(rows.sum()), int((rows > 0).sum())
    ffn = (2 * d * f + f + d) * el
    nbytes = touched * ffn + 2 * T * d * el + d * E * 4
    flops = 4 * d * f * kept + 2 * T * d * E
    if c["residual"]:
        nbytes += ffn
        flops += 4 * d * f * T
    if c["kind"] == "stages":          # the sorted rows and the expert outputs are results of calls of their own
        nbytes += 4 * kept * d * el
    if c["kind"] == "block":           # positions are uniform over the cache
        nbytes += 4 * d * d * el + T * d * c["max_len"] * el
        flops += 8 * T * d * d + 2 * T * d * c["max_len"]
    return {"bytes": nbytes, "flops": flops}


def estimate(c):
    """Seconds that a pass takes at most, roughly: keeps drawn cases below the largest listed one."""
    w = work(c)
    return max(w["bytes"] / 5e12, w["flops"] / (5e12 if c["dtype"] == "f32" else 0.6e15))


def tolerance(c):
    """About four times the distance to the same layer in 64 bits (out of bf16 layers: rel 2.9e-3, max 2.3e-2; of fp32
    ones: rel 9.5e-7, max 7e-6; fp32 logits and gate weights of either: rel 4e-7).  An expert may change where two logits
    are equal to within their rounding; in the decoder block, whose gate reads activations that were rounded to bf16 on
    the way, that can show as a token's whole expert output (logits move by up to 3.5e-3 with the cache in another order)."""
    if c["dtype"] == "f32":
        return {"rel": 4e-6, "max": 3e-5, "differ": 2e-3}
    return {"rel": 1e-2, "max": 0.3 if c["kind"] == "block" else 9e-2, "differ": 2e-3}


def _normal(shape, std, dtype, gen):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    for part in out if out.dim() == 3 else [out]:      # one expert at a time: no large fp32 temporary
        part.normal_(0.0, std, generator=gen)
    return out


def prepare(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    T, d, f, E, k, C = c["T"], c["d_model"], c["d_ffn"], c["E"], c["top_k"], _capacity(c)
    el, f32, i32 = torch.float32 if c["dtype"] == "f32" else torch.bfloat16, torch.float32, torch.int32

    def empty(*shape, dtype=el):
        return torch.empty(shape, dtype=dtype, device="cuda")

    x = _normal((T, d), 1.0, el, gen)
    Wg = _normal((d, E), WEIGHT_STD, f32, gen)
    bg = None
    if c["skewed"]:
        bg = (ZIPF * torch.log(1.0 / (torch.arange(E, dtype=torch.float64) + 1.0))).to(f32).cuda()

    def ffn_weight(*shape):            # inference weights: laid out once for the matrix cores where the program asks for it
        w = _normal(shape, WEIGHT_STD, el, gen)
        return moe.moe_pack_weights(w) if c["packed"] and c["kind"] != "layer" else w

    w = dict(W1=ffn_weight(E, d, f), b1=_normal((E, f), BIAS_STD, el, gen), W2=ffn_weight(E, f, d), b2=_normal((E, d), BIAS_STD, el, gen))
    if c["residual"]:
        w.update(Wd1=ffn_weight(d, f), bd1=_normal((f,), BIAS_STD, el, gen), Wd2=ffn_weight(f, d), bd2=_normal((d,), BIAS_STD, el, gen))
    if c["kind"] == "layer":
        return {"layer": moe.MoELayer(T, d, f, E, k, C, c["dtype"], Wg, bg, pack_weights=c["packed"], **w), "x": x}

    gate = moe.moe_pack_gate(Wg) if c["packed"] else None
    flags = (moe.MOE_FLAG_PACKED_WEIGHTS if c["packed"] else 0) | (moe.MOE_FLAG_PACKED_GATE if gate is not None else 0)
    Wg = Wg if gate is None else gate
    shape = moe.make_shape(T, d, f, E, k, C, c["dtype"], c["residual"], flags)
    if c["kind"] == "stages":
        return {"shape": shape, "x": x, "Wg": Wg, "bg": bg, "w": w, "logits": empty(T, E, dtype=f32),
                "expert_idx": empty(T, k, dtype=i32), "slot_idx": empty(T, k, dtype=i32), "gate_w": empty(T, k, dtype=f32),
                "expert_rows": empty(E, dtype=i32), "slot_token": empty(E, C, dtype=i32), "xe": empty(E, C, d),
                "ye": empty(E, C, d), "out": empty(T, d), "ws": moe.alloc_workspace(shape)}
    H, L = c["heads"], c["max_len"]
    block = moe.MoeBlockShape(H, L)

    def gain(mean):
        return torch.randn((d,), generator=gen, device="cuda", dtype=f32) * 0.1 + mean

    w.update(Wg=Wg, bg=bg, ln1_gamma=gain(1.0), ln1_beta=gain(0.0), ln2_gamma=gain(1.0), ln2_beta=gain(0.0),
             Wqkv=_normal((d, 3 * d), 4 * WEIGHT_STD, el, gen), bqkv=_normal((3 * d,), BIAS_STD, el, gen),
             Wo=_normal((d, d), WEIGHT_STD, el, gen), bo=_normal((d,), BIAS_STD, el, gen))
    return {"shape": shape, "block": block, "weights": w, "x": x, "out": empty(T, d), "logits": empty(T, E, dtype=f32),
            "k_cache": _normal((T, H, L * (d // H)), 1.0, el, gen).view(T, H, L, d // H),
            "v_cache": _normal((T, H, L * (d // H)), 1.0, el, gen).view(T, H, L, d // H),
            "pos": torch.randint(0, L, (T,), generator=gen, device="cuda").to(i32),
            "ws": torch.empty(moe.moe_decode_block_workspace_bytes(shape, block), dtype=torch.uint8, device="cuda")}


def run(s):
    if "layer" in s:
        out = s["layer"](s["x"])
        return dict(s["layer"].routing, out=out)
    if "block" in s:
        moe.moe_decode_block_forward(s["shape"], s["block"], s["weights"], s["x"], s["k_cache"], s["v_cache"], s["pos"],
                                     s["out"], None, None, s["logits"], s["ws"])
        return {n: s[n] for n in ("out", "logits", "k_cache", "v_cache")}
    sh, w = s["shape"], s["w"]
    moe.moe_gate(sh, s["x"], s["Wg"], s["bg"], s["logits"], s["expert_idx"], s["slot_idx"], s["gate_w"], s["expert_rows"],
                 s["slot_token"], s["ws"])
    moe.moe_dispatch(sh, s["x"], s["slot_token"], s["expert_rows"], s["xe"])
    moe.moe_expert_ffn(sh, s["xe"], s["expert_rows"], w["W1"], w["b1"], w["W2"], w["b2"], s["ye"], s["ws"])
    moe.moe_combine(sh, s["ye"], s["expert_idx"], s["slot_idx"], s["gate_w"], None, s["out"])
    return {n: s[n] for n in ("logits", "expert_idx", "slot_idx", "gate_w", "expert_rows", "slot_token", "out")}
