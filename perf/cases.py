"""What a user of the library has it do, as cases whose time and results can be measured.

A case is one pass over a packed batch through the public entry points of paper_2510_10620_amd: the attention
forward, the forward and backward of a training step, one device's share of a plan (partial slots, their merge and the
share's backward), or the block instructions that move and reduce data around them.  Lengths, masks, head counts and
block sizes are those of the package's workloads and benchmark, the small shapes those of its tests.
"""
import math

import numpy as np
import torch

import paper_2510_10620_amd as P
from paper_2510_10620_amd import workloads as W

# Fields of a case.
#   do      "fwd": attention forward (inference, or the recomputation of a checkpointed layer);
#           "step": forward and backward (one attention layer of a training step);
#           "share": forward into partial slots, merge, backward with the global O and LSE (one device of a plan);
#           "move": Blockwise Copy into a block buffer, merge of partial outputs, sum of gradient partials, delta
#   dist    "equal" (sequences of `median` tokens), "lognormal" or "uniform" (workloads.draw_lengths), "list" (`lens`)
#   mask    a mask family of workloads.MaskSpec with its window / sink (causal_blockwise: mask blocks of 256 tokens);
#           rows "window": the table has WINDOW rows and no range array is used
_BASE = dict(do="step", dist="lognormal", lens="", tokens=65536, median=2048, lo=512, hi=32768, len_seed=2, mask="causal",
             window=0, sink=0, rows="ranges", block=1024, hq=32, hkv=8, d=128, dtype="bf16", shares=8)


def _case(name, **kw):
    c = dict(_BASE, name=name)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: 512 tokens, one head, fp32; all latency
        _case("tiny_f32", dist="list", lens="128,384", block=64, hq=1, hkv=1, d=64, dtype="f32"),
        # a handful of short ragged sequences in bf16, one of a single token: latency and launches again
        _case("small_ragged", dist="list", lens="300,77,1000,1,130", block=128, hq=4, hkv=2),
        # fp32 training of an ordinary batch (debugging, reference runs)
        _case("f32_batch", tokens=8192, hi=8192, median=1024, lo=64, hq=8, hkv=2, d=64, dtype="f32", block=512),
        # bf16 with heads of 64, an ordinary batch
        _case("d64_batch", tokens=16384, hi=16384, hq=16, hkv=4, d=64),
        # many equal short sequences
        _case("short_1024", dist="equal", median=1024),
        # the benchmark's batch: causal, log-normal lengths
        _case("causal_varlen"),
        # the same batch on one rank of an 8-way tensor-parallel group
        _case("tp_shard", hq=4, hkv=1),
        # sliding window given by two numbers (WINDOW rows)
        _case("sliding_window", dist="uniform", tokens=131072, lo=8192, hi=65536, len_seed=3, mask="window", window=4096, rows="window"),
        # mask blocks of 256 tokens with a window of two and a sink block: per-token range arrays
        _case("causal_blockwise", dist="uniform", tokens=131072, lo=8192, hi=65536, len_seed=6, mask="causal_blockwise", window=2, sink=1),
        # one document of the largest length with a five-token sequence beside it, forward only
        _case("long_forward", do="fwd", dist="list", lens="131067,5", tokens=131072),
        # one device's eighth of the computation blocks of a plan over 262 144 tokens, in four divisions
        _case("plan_share", do="share", tokens=262144, lo=1024, hi=131072, median=8192, len_seed=5, block=2048),
        # the data movement of an iteration: Q blocks into a block buffer, four divisions' partial outputs merged,
        # two gradient partials summed, delta
        _case("block_moves", do="move"),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "f32", "d64", "bf16", "bf16", "bf16", "masked", "masked", "fwd", "share", "move"])
    heads = {"small": [(4, 2), (8, 2), (1, 1), (6, 3)], "f32": [(1, 1), (4, 2), (8, 2), (4, 4)], "d64": [(16, 4), (8, 2), (4, 4), (8, 1)]}
    hq, hkv = rng.choice(heads.get(kind, [(32, 8), (32, 8), (16, 4), (8, 2), (4, 1), (24, 6), (16, 16)]))
    c = dict(_BASE, hq=hq, hkv=hkv, len_seed=rng.randrange(1 << 20))
    if kind == "small":
        n = rng.randrange(1, 7)
        c.update(dist="list", lens=",".join(str(_loguniform(rng, 1, 1500)) for _ in range(n)), block=rng.choice([64, 128, 256, 1024]),
                 do=rng.choice(["fwd", "step"]))
    elif kind == "f32":
        c.update(tokens=_loguniform(rng, 256, 8192), lo=16, dtype="f32", d=rng.choice([32, 64, 64, 128]), block=rng.choice([64, 256, 512, 1024]),
                 do=rng.choice(["fwd", "step"]))
        c.update(hi=c["tokens"], median=max(32, c["tokens"] // rng.choice([2, 4, 8])))
    elif kind == "d64":
        c.update(tokens=_loguniform(rng, 512, 16384), lo=16, d=rng.choice([32, 64, 64]), block=rng.choice([128, 512, 1024]),
                 do=rng.choice(["fwd", "step"]))
        c.update(hi=c["tokens"], median=max(64, c["tokens"] // rng.choice([2, 4, 8])))
    elif kind in ("bf16", "fwd", "share", "move"):
        c.update(do={"bf16": "step"}.get(kind, kind), tokens=_loguniform(rng, 2048, 98304), lo=rng.choice([64, 512, 1024]),
                 median=_loguniform(rng, 512, 8192), block=rng.choice([256, 512, 1024, 2048, 4096]))
        if kind == "bf16" and rng.random() < 0.3:
            c.update(dist="equal", median=_loguniform(rng, 256, 4096))
        if kind == "share":
            c.update(shares=rng.choice([2, 4, 8]))
    else:
        c.update(dist="uniform", tokens=_loguniform(rng, 8192, 131072), lo=512, mask=rng.choice(["window", "lambda", "causal_blockwise", "shared_question"]),
                 block=rng.choice([512, 1024, 2048]), do=rng.choice(["step", "step", "fwd"]))
        c.update(hi=max(1024, c["tokens"] // 2))
        if c["mask"] == "window":
            c.update(window=_loguniform(rng, 128, 8192), rows=rng.choice(["window", "ranges"]))
        elif c["mask"] == "lambda":
            c.update(window=_loguniform(rng, 128, 8192), sink=_loguniform(rng, 1, 256), rows=rng.choice(["window", "ranges"]))
        elif c["mask"] == "causal_blockwise":
            c.update(window=rng.randrange(1, 9), sink=1)
    return c


def _lengths(c):
    if c["dist"] == "list":
        return [int(x) for x in c["lens"].split(",")]
    if c["dist"] == "equal":
        n = max(1, c["tokens"] // c["median"])
        return [c["median"]] * n
    return W.draw_lengths(c["tokens"], c["dist"], c["lo"], c["hi"], seed=c["len_seed"], median=c["median"])


def _tables(c):
    """(cu_seqlens, range arrays or None, the batch's block table)"""
    cu = W.cu_from_lengths(_lengths(c))
    spec = W.MaskSpec(c["mask"], window=c["window"], sink=c["sink"])
    if c["rows"] == "window":
        return cu, None, P.dcp_build_block_table_window(cu, c["block"], c["window"], c["sink"])
    ranges = W.attn_ranges(spec, cu)
    return cu, ranges, P.dcp_build_block_table(cu, c["block"], ranges)


def _share(c, table):
    """The table rows of one device of `shares` and the partial slot of each, in four divisions."""
    rows = table[W.deal_share(len(table), c["shares"], 205, 0)]
    slot, n_slots, _ = W.deal_divisions(rows[:, 0], 4, 305)
    return rows, slot, n_slots


def _randn(gen, shape, scale, dtype):
    return (torch.randn(shape, device="cuda", generator=gen, dtype=torch.float32) * scale).to(dtype)


def prepare(case, seed):
    c = case
    cu, ranges, table = _tables(c)
    T, hq, hkv, d = int(cu[-1]), c["hq"], c["hkv"], c["d"]
    dtype, code = (torch.bfloat16, P.DCP_BF16) if c["dtype"] == "bf16" else (torch.float32, P.DCP_F32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = dict(do=c["do"], scale=1.0 / math.sqrt(d))
    s["rg"] = torch.from_numpy(np.ascontiguousarray(ranges)).cuda() if ranges is not None and (table[:, 2] == P.DCP_MASK_RANGES).any() else None
    scale_in = 1.0 / math.sqrt(d)
    s["q"], s["k"], s["v"] = _randn(gen, (T, hq, d), scale_in, dtype), _randn(gen, (T, hkv, d), scale_in, dtype), _randn(gen, (T, hkv, d), scale_in, dtype)
    s["out"], s["lse"] = torch.empty_like(s["q"]), torch.empty((hq, T), dtype=torch.float32, device="cuda")

    def plan_of(rows, slot=None, n_slots=0):
        plan = P.dcp_plan_create(cu, c["block"], rows, slot, n_slots)
        if c["rows"] == "window":
            P.dcp_plan_set_window(plan, c["window"], c["sink"])
        P.dcp_plan_prepare(plan, hq, hkv, d, code)
        return plan

    if c["do"] == "share" or c["do"] == "move":
        # the global O and LSE that the backward of a share uses come from the whole table
        P.dcp_block_attn_fwd(plan_of(table), s["q"], s["k"], s["v"], s["out"], s["lse"], s["scale"], s["rg"])
        if c["do"] == "share":
            table, slot, n_slots = _share(c, table)
        else:
            slot, n_slots, _ = W.deal_divisions(table[:, 0], 4, 305)
        s["plan"] = plan_of(table, slot, n_slots)
        s["o_part"] = torch.zeros((n_slots, c["block"], hq, d), dtype=dtype, device="cuda")
        s["lse_part"] = torch.zeros((n_slots, hq, c["block"]), dtype=torch.float32, device="cuda")
        s["out_m"], s["lse_m"] = torch.empty_like(s["out"]), torch.empty_like(s["lse"])
    else:
        s["plan"] = plan_of(table)
    if c["do"] != "fwd":
        s["do_"] = _randn(gen, (T, hq, d), 1.0, dtype)
        s["dq"], s["dk"], s["dv"] = torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])
        s["ws"] = torch.empty(max(256, P.dcp_bwd_workspace_bytes(s["plan"], hq, hkv, d, code)), dtype=torch.uint8, device="cuda")
    if c["do"] == "move":
        P.dcp_block_attn_fwd(s["plan"], s["q"], s["k"], s["v"], s["o_part"], s["lse_part"], s["scale"], s["rg"])
        start, length = s["plan"].export("BLK_START"), s["plan"].export("BLK_LEN")
        slots = np.random.default_rng(c["len_seed"]).permutation(len(start)).astype(np.int32)
        s["list"] = P.CopyList(np.stack([start, slots * c["block"], length], axis=1), T, len(start) * c["block"])
        s["buf"] = torch.zeros((len(start) * c["block"], hq, d), dtype=dtype, device="cuda")
        P.dcp_blockwise_copy(s["list"], s["q"], s["buf"])
        s["buf"].zero_()
        s["delta"] = torch.empty((hq, T), dtype=torch.float32, device="cuda")
    return s


def run(state):
    s = state
    if s["do"] == "fwd" or s["do"] == "step":
        P.dcp_block_attn_fwd(s["plan"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["scale"], s["rg"])
        if s["do"] == "fwd":
            return {"out": s["out"], "lse": s["lse"]}
        P.dcp_block_attn_bwd(s["plan"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["do_"], s["dq"], s["dk"], s["dv"], s["scale"], s["ws"], s["rg"])
        return {"out": s["out"], "lse": s["lse"], "dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}
    if s["do"] == "share":
        P.dcp_block_attn_fwd(s["plan"], s["q"], s["k"], s["v"], s["o_part"], s["lse_part"], s["scale"], s["rg"])
        P.dcp_merge_partials(s["plan"], s["o_part"], s["lse_part"], s["out_m"], s["lse_m"])
        P.dcp_block_attn_bwd(s["plan"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["do_"], s["dq"], s["dk"], s["dv"], s["scale"], s["ws"], s["rg"])
        return {"out": s["out_m"], "lse": s["lse_m"], "dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}
    P.dcp_blockwise_copy(s["list"], s["q"], s["buf"])
    P.dcp_merge_partials(s["plan"], s["o_part"], s["lse_part"], s["out_m"], s["lse_m"])
    P.dcp_sum_partials([s["do_"], s["q"]], s["dq"])
    P.dcp_bwd_delta(s["out"], s["do_"], s["delta"])
    return {"buf": s["buf"], "out": s["out_m"], "lse": s["lse_m"], "dq": s["dq"], "delta": s["delta"]}


def work(case):
    c = case
    cu, ranges, table = _tables(c)
    T, e = int(cu[-1]), 2 if c["dtype"] == "bf16" else 4
    row_q, row_kv, row_l = c["hq"] * c["d"] * e, c["hkv"] * c["d"] * e, c["hq"] * 4
    length = np.diff(cu).astype(np.int64)
    blocks = -(-length // c["block"])
    blk_len = np.concatenate([np.minimum(c["block"], n - c["block"] * np.arange(b)) for n, b in zip(length, blocks)])
    if c["do"] == "move":
        slot, n_slots, slot_q = W.deal_divisions(table[:, 0], 4, 305)
        parts = int(blk_len[slot_q].sum())
        # copy; merge; sum of two; delta from O and dO
        moved = 2 * T * row_q + (parts + T) * (row_q + row_l) + 3 * T * row_q + 2 * T * row_q + T * row_l
        return {"bytes": moved, "flops": 2.0 * parts * c["hq"] * c["d"] + 3.0 * T * c["hq"] * c["d"]}
    q_rows = kv_rows = T
    merged = 0
    if c["do"] == "share":
        table, slot, n_slots = _share(c, table)
        q_rows, kv_rows = int(blk_len[np.unique(table[:, 0])].sum()), int(blk_len[np.unique(table[:, 1])].sum())
        merged = 2 * int(sum(blk_len[q] for q in dict(zip(slot.tolist(), table[:, 0].tolist())).values())) * (row_q + row_l)
    count = P.dcp_count_pairs_window(cu, c["block"], table, c["window"], c["sink"]) if c["rows"] == "window" else P.dcp_count_pairs(cu, c["block"], table, ranges)
    pairs = float(count.sum())
    # q, k, v in; O and LSE out; and dO in, dQ, dK, dV out (a share's backward also reads the global O and LSE)
    moved = q_rows * row_q + 2 * kv_rows * row_kv + T * (row_q + row_l) + merged
    if c["do"] != "fwd":
        moved += q_rows * row_q + T * row_q + 2 * T * row_kv
    if c["do"] == "share":
        moved += q_rows * (row_q + row_l)
    return {"bytes": float(moved), "flops": (4 if c["do"] == "fwd" else 14) * pairs * c["hq"] * c["d"]}


def tolerance(case):
    # four times the distance of the outputs from the same attention in 64 bits: 2.5e-3 (single values 0.1) in bf16,
    # 1.8e-6 (7e-5) in fp32, the gradients of K and V the farthest
    return {"rel": 1e-2, "max": 0.4} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 4e-4}
