"""The fp32 MFMA kernels at the sizes where they can go wrong, against the fp64 oracle: rows and blocks around their
32-row tiles and 128-row work items, units with fewer tiles than a workgroup has waves, every head dimension, mask kind
and memory layout.  Bounds: those of fp32 I/O in helpers.TOL."""
import pytest

from paper_2510_10620_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 127, 129, 257, 300]


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,heads,spec", [
    (64, (2, 1), W.MaskSpec("causal")), (96, (3, 3), W.MaskSpec("lambda", window=70, sink=9)), (512, (4, 2), W.MaskSpec("shared_question")),
    (33, (2, 2), W.MaskSpec("window", window=40))], ids=lambda x: getattr(x, "kind", None))
def test_f32_tiles(d, B, heads, spec):
    w = W.custom_workload("f32", LENS, B, heads[0], heads[1], d, "f32", spec, seed=61, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    ref = H.oracle_full(w, tensors, table)
    window = (spec.window, spec.sink) if spec.kind == "window" else None
    t = table.copy()
    if window:
        t[t[:, 2] == W.MASK_RANGES, 2] = W.MASK_WINDOW   # no range array: two numbers
    g = H.GpuRun(w, tensors, t, window=window)
    out, lse = g.forward()
    dq, dk, dv = g.backward()
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), ref, ("out", "lse", "dq", "dk", "dv"), f"f32 D{d} B{B} {spec.kind}")


def test_f32_partial_slots_and_empty_rows():
    """Divisions into partial slots with their merge, and a table that leaves query blocks and keys without partners."""
    w = W.custom_workload("f32s", [150, 260], 64, 4, 2, 64, "f32", W.MaskSpec("causal"), seed=62, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    table = table[::2]
    slot, n_slots, _ = W.deal_divisions(table[:, 0], 2, 5)
    ref = H.oracle_full(w, tensors, table)
    g = H.GpuRun(w, tensors, table, slot, n_slots)
    out, lse = g.forward()
    dq, dk, dv = g.backward()
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), ref, ("out", "lse", "dq", "dk", "dv"), "f32 slots")


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 32), ("bf16", 64), ("f32", 128)])
def test_selector_and_token_strides(dtype, d):
    """MFMA by name stays refused outside bf16 with D = 128, and token strides past the 32-bit offsets of the kernels for
    these shapes (2^24 elements) run on the thread-per-row family: its results, bit for bit."""
    import torch
    import paper_2510_10620_amd as P
    w = W.custom_workload("far", [3], 64, 1, 1, d, dtype, W.MaskSpec("causal"), seed=65, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    with pytest.raises(P.DcpError) as ei:
        H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_MFMA).forward()
    assert ei.value.status == P.DCP_ERR_UNSUPPORTED
    ref = H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)
    far = H.GpuRun(w, tensors, table)
    k = torch.empty(2 * ((1 << 24) + 8) + d, dtype=far.k.dtype, device="cuda").as_strided((3, 1, d), ((1 << 24) + 8, d, 1))
    k.copy_(far.k)
    far.k = k
    for a, b in zip(ref.forward() + ref.backward(), far.forward() + far.backward()):
        assert (a == b).all()


@pytest.mark.parametrize("dtype,d", [("f32", 32), ("bf16", 64)])
def test_largest_block_size_under_a_mask(dtype, d):
    """Blocks as long as an int allows (one per sequence) in a table with per-token ranges, whose bounds the backward
    works out block by block."""
    import torch
    import paper_2510_10620_amd as P
    B = 2 ** 31 - 1
    w = W.custom_workload("blocks", [150, 33], B, 2, 1, d, dtype, W.MaskSpec("window", window=3), seed=71, input_scale=0.5)
    tensors, table = W.make_tensors(w), P.dcp_build_block_table(w.cu_seqlens, B, w.ranges)
    assert (table[:, 2] == W.MASK_RANGES).all()
    fast, slow = H.GpuRun(w, tensors, table), H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)
    ref = slow.forward() + slow.backward()
    got = fast.forward()
    outs = [torch.full_like(x, float("nan")) for x in (fast.q, fast.k, fast.v)]
    code = P.DCP_BF16 if dtype == "bf16" else P.DCP_F32
    ws = torch.full((P.dcp_bwd_workspace_bytes(fast.plan, 2, 1, d, code),), 0x7f, dtype=torch.uint8, device="cuda")   # bounds left as they are hide every tile
    P.dcp_block_attn_bwd(fast.plan, fast.q, fast.k, fast.v, fast.out, fast.lse, fast.dout, *outs, w.softmax_scale, ws, fast.ranges)
    torch.cuda.synchronize()
    got += tuple(H.from_torch(x) for x in outs)
    names = ("out", "lse", "dq", "dk", "dv")
    H.check(w, dict(zip(names, got)), dict(zip(names, ref)), names, f"block size {B}")


@pytest.mark.parametrize("dtype,d,hq,hkv", [("f32", 32, 4, 2), ("f32", 64, 4, 2), ("f32", 128, 4, 1), ("bf16", 32, 4, 2)])
@pytest.mark.parametrize("slots", [False, True])
def test_many_short_sequences_take_the_thread_per_row_kernels(dtype, d, hq, hkv, slots):
    """3 000 sequences of 1 to 3 tokens, where the MFMA kernels took up to 20 times as long: AUTO gives the bits of the
    thread-per-row kernels, and the right results."""
    import numpy as np
    import paper_2510_10620_amd as P
    lens = [1 + i % 3 for i in range(3000)]
    w = W.custom_workload("short", lens, 64, hq, hkv, d, dtype, W.MaskSpec("causal"), seed=75, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    slot, n_slots, _ = W.deal_divisions(table[:, 0], 2, 5) if slots else (None, 0, None)
    auto, rows = (H.GpuRun(w, tensors, table, slot, n_slots, impl) for impl in (P.DCP_IMPL_AUTO, P.DCP_IMPL_SCALAR))
    ref = rows.forward() + rows.backward()
    got = auto.forward() + auto.backward()
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    names = ("out", "lse", "dq", "dk", "dv")
    H.check(w, dict(zip(names, got)), H.oracle_full(w, tensors, table), names, f"short {dtype} D{d}")
