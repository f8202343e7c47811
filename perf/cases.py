"""The work that a training program has this library do, as cases that can be timed and compared.

One pass is what one device does for one attention layer (or for one micro-batch, where the work lists are refilled):
forward and backward over a pack of variable-length sequences on the device's share of the heads.  The packs stand for the
mixed-length batches that the library schedules: the five configurations and the 4096-token workload of
`hspmd_workloads`, and generic packs of the same kinds at other sizes.

A case is a dict of plain values:
  path       "step"   packed offsets + refill of the plan + forward + backward: a micro-batch's first layer, as in bench.py
             "layer"  forward + backward on a plan that is kept: every other layer of the micro-batch
             "fwd"    forward alone: evaluation, and the recomputed forward of a checkpointed layer
             "rope"   rotation of q and k, forward, backward that turns dQ and dK back; the unrotated q and k are views into one
                      projection output
             "ring"   one rank of context-parallel attention: the rank's last chunk of every sequence meets all `chunks`
                      key/value chunks (refill of the block plans, block forwards, merges, block backwards)
  mix        how the pack's lengths are drawn until `tokens` are reached (the last sequence is cut to fit):
             "fixed" (lo = hi = the length), "list" (text of lengths), "lognormal" (mu_len, sigma, lo, hi),
             "uniform" (lo, hi), "bimodal" (70 % in [lo, hi], 30 % in [lo2, hi2])
  pack       the seed of the lengths (the same pack for every seed of the values)
  heads, kv_heads, head_dim, grads ("f32" or "bf16"), scale (of the N(0, 1) values)
  fused      q, k and v are views into one fused projection output
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2504_20490_amd as A

ROPE_BASE = 10000.0


def _case(name, path, mix, tokens, heads, kv_heads, head_dim, grads="bf16", scale=1.0, pack=1, fused=False, **more):
    return dict({"name": name, "path": path, "mix": mix, "tokens": tokens, "heads": heads, "kv_heads": kv_heads,
                 "head_dim": head_dim, "grads": grads, "scale": scale, "pack": pack, "fused": fused}, **more)


def listed():
    return [
        # the smallest pack of the repository's configurations: nothing but latency, launches and host work
        _case("tiny_step", "step", "list", 192, 2, 2, 64, "f32", lengths="17,64,111"),
        # a small micro-batch on a small share of the heads (wide tensor parallelism), ragged lengths
        _case("small_layer", "layer", "lognormal", 2053, 8, 8, 128, mu_len=512, sigma=0.8, lo=16, hi=2048, pack=2),
        # short sequences only (instruction tuning), the narrow head: many items of one or two tiles
        _case("short_step", "step", "uniform", 16384, 16, 16, 64, lo=32, hi=512, pack=3, fused=True),
        # evaluation / recomputed forward of a few ordinary sequences, grouped KV heads
        _case("prefill_fwd", "fwd", "lognormal", 6001, 32, 8, 128, mu_len=1500, sigma=0.7, lo=64, hi=4096, pack=4, fused=True),
        # 8 x 2048, the dense-batch equivalent
        _case("uniform_layer", "layer", "fixed", 16384, 32, 32, 128, "f32", lo=2048, hi=2048),
        # log-normal lengths filled to 16384 tokens
        _case("mixed16k_step", "step", "list", 16384, 32, 32, 128, "f32",
              lengths="311,627,1059,8192,896,2008,846,1128,262,1055"),
        # 24 of 40 heads (an uneven 3:2 split), 32768 tokens: the headline workload
        _case("asym32k_step", "step", "list", 32768, 24, 24, 128, "f32", lengths="1851,8713,1898,4207,450,4813,10836"),
        # long-tail bimodal pack with grouped KV heads: the largest
        _case("bimodal64k_step", "step", "list", 65536, 32, 8, 128, "f32", 1.0 / math.sqrt(128.0),
              lengths="1358,315,1290,1206,1104,29082,327,18500,2034,1608,1898,1986,1517,3311"),
        # 8 x 4096, 16 of 64 heads of a hidden-6656 model: head_dim 104 lies between the tile widths
        _case("dim104_layer", "layer", "fixed", 32768, 16, 16, 104, lo=4096, hi=4096),
        # one long document on a small share of the heads
        _case("long_layer", "layer", "fixed", 16001, 5, 5, 128, lo=16001, hi=16001),
        # rotary embedding around the attention, grouped KV heads
        _case("rope_layer", "rope", "lognormal", 8192, 32, 8, 128, mu_len=1024, sigma=1.0, lo=32, hi=8192, pack=5),
        # context parallelism over 4 devices on the headline pack: the last (heaviest) rank
        _case("ring4_step", "ring", "list", 32768, 24, 24, 128, "f32", lengths="1851,8713,1898,4207,450,4813,10836", chunks=4),
    ]


# visible pairs x heads x (head_dim / 128) that a drawn case may have: half of the largest listed one's
_MOST = 1.0e10


def draw(rng):
    """One more case of the same ranges: 192 to 65536 tokens, 1 to 40 heads, any path and mix."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    path = rng.choice(["step", "step", "layer", "layer", "fwd", "rope", "ring"])
    while True:
        tokens = log(192, 65536)
        kv_heads = rng.randint(1, 8) if rng.random() < 0.5 else rng.choice([8, 12, 16, 24, 32, 40])
        group = rng.choice([1, 1, 1, 2, 4]) if kv_heads <= 10 else 1
        head_dim = rng.choice([128, 128, 128, 64, 104, 96, 80])
        case = {"path": path, "tokens": tokens, "heads": kv_heads * group, "kv_heads": kv_heads, "head_dim": head_dim,
                "grads": "f32" if path == "ring" else rng.choice(["f32", "bf16"]),
                "scale": rng.choice([1.0, 1.0, 1.0 / math.sqrt(128.0)]), "pack": rng.randrange(1 << 20)}
        mix = rng.choice(["lognormal", "lognormal", "uniform", "fixed", "bimodal"])
        case["mix"] = mix
        if mix == "lognormal":
            case.update(mu_len=log(128, 2048), sigma=round(rng.uniform(0.5, 1.2), 3), lo=16, hi=16384)
        elif mix == "uniform":
            lo = log(16, 1024)
            case.update(lo=lo, hi=lo * rng.randint(2, 16))
        elif mix == "fixed":
            length = log(128, 16384)
            case.update(lo=length, hi=length)
        else:
            case.update(lo=128, hi=2048, lo2=log(2048, 16384), hi2=24576)
        if path == "ring":
            case["chunks"] = rng.choice([2, 3, 4, 8])
        case["fused"] = path in ("step", "layer", "fwd") and rng.random() < 0.5
        if _pairs(_lengths(case)) * case["heads"] * head_dim / 128.0 <= _MOST:
            return case


def _lengths(case):
    if case["mix"] == "list":
        return [int(x) for x in case["lengths"].split(",")]
    rng = random.Random(case["pack"])
    out, left = [], case["tokens"]
    while left > 0:
        if case["mix"] == "lognormal":
            n = int(math.exp(math.log(case["mu_len"]) + case["sigma"] * rng.gauss(0.0, 1.0)) + 0.5)
            n = min(max(n, case["lo"]), case["hi"])
        elif case["mix"] == "bimodal" and rng.random() >= 0.7:
            n = rng.randint(case["lo2"], case["hi2"])
        else:
            n = rng.randint(case["lo"], case["hi"])
        out.append(min(n, left))
        left -= out[-1]
    return out


def _pairs(lengths):
    """Visible (query, key) pairs per head."""
    return sum(n * (n + 1) // 2 for n in lengths)


def _ring_edges(case, lengths):
    return [[n * c // case["chunks"] for c in range(case["chunks"] + 1)] for n in lengths]


def work(case):
    """Matrix products over the visible pairs (2 in the forward, 5 in the backward), every tensor read and written once."""
    lengths = _lengths(case)
    hq, hkv, d, T = case["heads"], case["kv_heads"], case["head_dim"], sum(_lengths(case))
    g = 4 if case["grads"] == "f32" else 2
    pairs, Tq, forward = _pairs(lengths), T, 2
    if case["path"] == "ring":
        edges = _ring_edges(case, lengths)
        Tq = sum(e[-1] - e[-2] for e in edges)
        pairs = sum((e[-1] - e[-2]) * (e[-1] + e[-2] + 1) // 2 for e in edges)
    product = 2 * d * pairs * hq
    q_side, kv_side, lse = Tq * hq * d, T * hkv * d, 4 * Tq * hq
    nbytes = 2 * q_side + 2 * 2 * kv_side + 2 * q_side + lse          # q, k, v in; o, lse out
    products = forward
    if case["path"] != "fwd":
        products += 5
        nbytes += (2 + 2 + 2) * q_side + 2 * 2 * kv_side + lse        # q, o, dO, k, v, lse in
        nbytes += g * q_side + 2 * g * kv_side                        # dQ, dK, dV out
    if case["path"] == "rope":
        nbytes += 2 * 2 * (T * hq * d + T * hkv * d)                  # q, k rotated once
    return {"bytes": nbytes, "flops": products * product}


def tolerance(case):
    """bf16 inputs and operands, fp32 accumulation.  Against the same formulas in fp64 on the same bf16 inputs the listed
    cases' outputs are off by rel 1.6e-3 to 2.6e-3 (2-norm) and in single elements by up to 0.2 of the larger of the
    tensor's root mean square and the value (the first tokens of a sequence, whose weights of order one carry a whole bf16
    rounding, in tensors whose other rows are small); four times that is stated."""
    return {"rel": 1e-2, "max": 0.8}


def _values(gen, shape, scale):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    return (x if scale == 1.0 else x.mul_(scale)).to(torch.bfloat16)


def prepare(case, seed):
    """Inputs on the device, output tensors, workspace, and the plan(s) that the program keeps."""
    lengths = _lengths(case)
    T, hq, hkv, d = sum(lengths), case["heads"], case["kv_heads"], case["head_dim"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    grad = torch.float32 if case["grads"] == "f32" else torch.bfloat16
    s = {"path": case["path"], "lengths": lengths, "grad": A.GRAD_F32 if case["grads"] == "f32" else A.GRAD_BF16}
    empty = lambda *shape, dtype: torch.empty(*shape, dtype=dtype, device="cuda")
    if case["path"] == "ring":
        return _prepare_ring(case, lengths, gen, s)
    if case["path"] == "rope":
        both = _values(gen, (T, hq + hkv, d), case["scale"])
        s["q"], s["k"], s["v"] = both[:, :hq], both[:, hq:], _values(gen, (T, hkv, d), case["scale"])
        s["q_rot"], s["k_rot"] = empty(T, hq, d, dtype=torch.bfloat16), empty(T, hkv, d, dtype=torch.bfloat16)
        s["positions"] = max(lengths)
        s["table"] = empty(s["positions"], d // 2, 2, dtype=torch.float32)
        A.rope_table(s["table"], s["positions"], d, ROPE_BASE)
    elif case["fused"]:
        fused = _values(gen, (T, hq + 2 * hkv, d), case["scale"])
        s["q"], s["k"], s["v"] = fused[:, :hq], fused[:, hq:hq + hkv], fused[:, hq + hkv:]
    else:
        s["q"] = _values(gen, (T, hq, d), case["scale"])
        s["k"], s["v"] = _values(gen, (T, hkv, d), case["scale"]), _values(gen, (T, hkv, d), case["scale"])
    cu, _, _ = A.build_cu_seqlens(lengths)
    s["plan"] = A.Plan(cu, hq, hkv, d)
    s["o"], s["lse"] = empty(T, hq, d, dtype=torch.bfloat16), empty(hq, T, dtype=torch.float32)
    if case["path"] != "fwd":
        s["do"] = _values(gen, (T, hq, d), case["scale"])
        s["dq"], s["dk"], s["dv"] = (empty(T, h, d, dtype=grad) for h in (hq, hkv, hkv))
        s["ws"] = empty(s["plan"].bwd_workspace_bytes(), dtype=torch.uint8)
    return s


def _prepare_ring(case, lengths, gen, s):
    n, hq, hkv, d = case["chunks"], case["heads"], case["kv_heads"], case["head_dim"]
    edges = _ring_edges(case, lengths)
    cu = lambda sizes: np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    sizes = [[e[c + 1] - e[c] for e in edges] for c in range(n)]
    starts = [[e[c] for e in edges] for c in range(n)]
    empty = lambda *shape, dtype=torch.float32: torch.empty(*shape, dtype=dtype, device="cuda")
    tq = sum(sizes[-1])
    s["q"], s["do"] = _values(gen, (tq, hq, d), case["scale"]), _values(gen, (tq, hq, d), case["scale"])
    s["kv"] = [tuple(_values(gen, (sum(sizes[c]), hkv, d), case["scale"]) for _ in range(2)) for c in range(n)]
    s["geometry"] = [(cu(sizes[-1]), cu(sizes[c]), starts[-1], starts[c]) for c in range(n)]
    s["plans"] = [A.BlockPlan(*g, hq, hkv, d) for g in s["geometry"]]
    s["o_acc"], s["o_part"] = empty(tq, hq, d), empty(tq, hq, d)
    s["lse"], s["lse_part"] = empty(hq, tq), empty(hq, tq)
    s["o"] = empty(tq, hq, d, dtype=torch.bfloat16)
    s["dq"] = empty(tq, hq, d)
    s["dkv"] = [tuple(torch.empty(x.shape, dtype=torch.float32, device="cuda") for x in pair) for pair in s["kv"]]
    s["ws"] = empty(s["plans"][0].bwd_workspace_bytes(), dtype=torch.uint8)
    return s


def run(s):
    """One pass; the outputs are the state's own buffers."""
    path = s["path"]
    if path == "ring":
        return _run_ring(s)
    plan = s["plan"]
    if path == "step":
        cu, _, _ = A.build_cu_seqlens(s["lengths"])
        plan.update(cu)
    if path == "rope":
        A.rope_qk(plan, s["q"], s["k"], s["q_rot"], s["k_rot"], s["table"], s["positions"])
        A.attn_varlen_fwd(plan, s["q_rot"], s["k_rot"], s["v"], s["o"], s["lse"])
        A.attn_varlen_bwd_rope(plan, s["q_rot"], s["k_rot"], s["v"], s["o"], s["lse"], s["do"], s["dq"], s["dk"], s["dv"],
                               s["ws"], s["table"], s["positions"], grad_dtype=s["grad"])
    else:
        A.attn_varlen_fwd(plan, s["q"], s["k"], s["v"], s["o"], s["lse"])
        if path == "fwd":
            return {"o": s["o"], "lse": s["lse"]}
        A.attn_varlen_bwd(plan, s["q"], s["k"], s["v"], s["o"], s["lse"], s["do"], s["dq"], s["dk"], s["dv"], s["ws"],
                          grad_dtype=s["grad"])
    return {name: s[name] for name in ("o", "lse", "dq", "dk", "dv")}


def _run_ring(s):
    plans, n = s["plans"], len(s["plans"])
    for plan, geometry in zip(plans, s["geometry"]):
        plan.update(*geometry)
    for c, plan in enumerate(plans):
        k, v = s["kv"][c]
        if c == 0:
            A.attn_block_fwd(plan, s["q"], k, v, s["o_acc"], s["lse"])
            continue
        A.attn_block_fwd(plan, s["q"], k, v, s["o_part"], s["lse_part"])
        A.attn_merge(s["o_acc"], s["lse"], s["o_part"], s["lse_part"], s["o_acc"], s["lse"], s["o"] if c == n - 1 else None)
    for c, plan in enumerate(plans):
        k, v = s["kv"][c]
        A.attn_block_bwd(plan, s["q"], k, v, s["o"], s["lse"], s["do"], s["dq"], s["dkv"][c][0], s["dkv"][c][1], s["ws"],
                         dq_accumulate=c > 0, reuse_statistics=c > 0)
    return {"o": s["o"], "lse": s["lse"], "dq": s["dq"], "dkv": s["dkv"]}
