"""The bf16 kernels whose waves split the other side, the fp32 kernels of 16 rows a workgroup, and the rule that takes a launch to
them, against the fp64 oracle: rows and blocks around their 32-row tiles and 128-row work items, walks of one tile and of more than 64, every mask kind, slots and strided
inputs, in batches small enough for one backward launch, for two, and with heads enough for the kernels that share their tiles
(test_gpu_forms.py asserts form by form what runs).
Bounds: those of the I/O type in helpers.TOL."""
import numpy as np
import pytest

from paper_2510_10620_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 33, 63, 65, 127, 129, 257, 640]
ALL = ("out", "lse", "dq", "dk", "dv")


def _launches(g):
    """(results of the backward, dQ launches of their own)"""
    import paper_2510_10620_amd as P
    P.dcp_profile_enable(True)
    grads = g.backward()
    n = P.dcp_profile_read("dq")[1]
    P.dcp_profile_enable(False)
    return grads, n


def _run(name, lens, B, heads, d, spec, seed, window_rows=False, slots=False, strided=False, dtype="bf16"):
    import torch
    w = W.custom_workload(name, lens, B, heads[0], heads[1], d, dtype, spec, seed=seed, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    ref = H.oracle_full(w, tensors, table)
    t, window = table.copy(), None
    if window_rows:
        t[t[:, 2] == W.MASK_RANGES, 2] = W.MASK_WINDOW
        window = (spec.window, spec.sink)
    slot, n_slots = (None, 0)
    if slots:
        slot, n_slots, _ = W.deal_divisions(table[:, 0], 3, 5)
    g = H.GpuRun(w, tensors, t, slot, n_slots, window=window)
    if strided:
        hq, hkv = heads
        fused = torch.cat([g.q, g.k, g.v], dim=1).contiguous()
        g.q, g.k, g.v = fused[:, :hq], fused[:, hq:hq + hkv], fused[:, hq + hkv:]
    out, lse = g.forward()
    (dq, dk, dv), own_dq = _launches(g)
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), ref, ALL, f"{name} D{d} B{B} {heads} {spec.kind}")
    return own_dq


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,heads,launches", [(64, (2, 1), None), (66, (2, 1), 1), (512, (2, 1), 1), (512, (16, 4), 2), (64, (64, 64), 2)],
                         ids=["short-blocks", "one", "one-long-blocks", "two", "shared"])
@pytest.mark.parametrize("spec,window_rows", [(W.MaskSpec("causal"), False), (W.MaskSpec("lambda", window=70, sink=9), False),
                                              (W.MaskSpec("lambda", window=70, sink=9), True)], ids=["causal", "ranges", "window"])
def test_tile_edges(d, B, heads, launches, spec, window_rows):
    own_dq = _run("edges", EDGES, B, heads, d, spec, 81, window_rows)   # (blocks of 64: one launch or two, as D and the mask have it)
    assert launches is None or own_dq == launches - 1, "the batch is meant for the other number of backward launches"


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,heads,launches", [(64, (1, 1), 1), (512, (8, 8), 2), (64, (32, 32), 2)], ids=["one", "two", "many"])
@pytest.mark.parametrize("spec,window_rows", [(W.MaskSpec("causal"), False), (W.MaskSpec("lambda", window=70, sink=9), False),
                                              (W.MaskSpec("lambda", window=70, sink=9), True)], ids=["causal", "ranges", "window"])
def test_tile_edges_f32(d, B, heads, launches, spec, window_rows):
    """16 rows a workgroup in all but D 32, whose two-launch batches take 32 in the forward and dQ."""
    own_dq = _run("edges", EDGES, B, heads, d, spec, 85, window_rows, dtype="f32")
    assert own_dq == launches - 1, "the batch is meant for the other number of backward launches"


@pytest.mark.parametrize("d", [32, 64, 128])
def test_f32_long_walks_slots_and_strides(d):
    _run("long", [2300, 33], 2304, (4, 1), d, W.MaskSpec("causal"), 86, dtype="f32")
    _run("slots", [300, 700, 1], 128, (4, 2), d, W.MaskSpec("causal_blockwise", window=2, sink=1, mblock=64), 87, slots=True, strided=True, dtype="f32")


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("spec", [W.MaskSpec("causal"), W.MaskSpec("shared_question")], ids=lambda s: s.kind)
def test_long_walks_few_heads(d, spec):
    """Blocks of more than 64 query tiles, eight query heads to a KV head: dK/dV walks them 64 at a time."""
    _run("long", [2300, 33], 2304, (8, 1), d, spec, 82)


@pytest.mark.parametrize("d", [32, 64, 128])
def test_slots_strides_and_a_row_without_keys(d):
    """Partial slots with their merge, q / k / v as views of one projection, three mask blocks."""
    _run("slots", [300, 700, 1], 128, (4, 2), d, W.MaskSpec("causal_blockwise", window=2, sink=1, mblock=64), 83, slots=True, strided=True)


@pytest.mark.parametrize("d", [64, 128])
def test_prepared_for_other_heads(d):
    """A plan made ready for 128 query heads (D = 128: cut dK/dV items, which the split kernels do not take) serves two: on that list where
    none may be created (the entry point that allocates nothing), else on their own."""
    import paper_2510_10620_amd as P
    w = W.custom_workload("prep", [1300, 200], 128, 2, 2, d, "bf16", W.MaskSpec("causal"), seed=84, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    ref = H.oracle_full(w, tensors, table)
    for hq in (2, 128):
        g = H.GpuRun(w, tensors, table)
        P.dcp_plan_prepare(g.plan, hq, 2, d, P.DCP_BF16)
        out, lse = g.forward()
        grads = [g.torch.full_like(x, float("nan")) for x in (g.q, g.k, g.v)]
        P.dcp_block_attn_bwd_static(g.plan, g.q, g.k, g.v, g.out, g.lse, g.dout, *grads, w.softmax_scale, g.ranges)
        g.torch.cuda.synchronize()
        for dq, dk, dv in ([H.from_torch(x) for x in grads], g.backward()):
            H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), ref, ALL, f"prepared for {hq} D{d}")


@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("bf16", 64), ("bf16", 128), ("f32", 32), ("f32", 64), ("f32", 128)])
def test_gradients_over_the_inputs(dtype, d):
    """dQ over O, dK over K and dV over V in a batch that is small enough for one backward launch takes two, which allow it."""
    import paper_2510_10620_amd as P
    w = W.custom_workload("inplace", [300, 77, 33], 128, 4, 2, d, dtype, W.MaskSpec("causal"), seed=88, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    ref = H.oracle_full(w, tensors, table)
    for dq_over, dkv_over in [(True, False), (False, True), (True, True)]:
        g = H.GpuRun(w, tensors, table)
        g.forward()
        dq = g.out if dq_over else g.q.new_full(g.q.shape, float("nan"))
        dk, dv = (g.k, g.v) if dkv_over else (g.k.new_full(g.k.shape, float("nan")), g.v.new_full(g.v.shape, float("nan")))
        ws = g.torch.empty(max(256, P.dcp_bwd_workspace_bytes(g.plan, w.hq, w.hkv, d, P.DCP_BF16 if dtype == "bf16" else P.DCP_F32)),
                           dtype=g.torch.uint8, device="cuda")
        P.dcp_profile_enable(True)
        P.dcp_block_attn_bwd(g.plan, g.q, g.k, g.v, g.out, g.lse, g.dout, dq, dk, dv, w.softmax_scale, ws, g.ranges)
        own_dq = P.dcp_profile_read("dq")[1]
        P.dcp_profile_enable(False)
        assert own_dq == 1
        H.check(w, dict(dq=H.from_torch(dq), dk=H.from_torch(dk), dv=H.from_torch(dv)), ref, ("dq", "dk", "dv"), f"in place {dtype} D{d}")
