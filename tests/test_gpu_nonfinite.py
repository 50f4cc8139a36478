"""Values that are not finite, in the kernels for fp32 and for heads of 32 and 64: rows that the backward leaves out, and Inf / NaN
in the inputs, which may reach only the pairs that are visible."""
import numpy as np
import pytest

from paper_2510_10620_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 32), ("bf16", 64)]


@pytest.mark.parametrize("dtype,d", SHAPES)
@pytest.mark.parametrize("spec", [W.MaskSpec("causal"), W.MaskSpec("lambda", window=70, sink=9)], ids=lambda s: s.kind)
def test_rows_switched_off_by_their_lse(dtype, d, spec):
    """Query rows whose LSE is -inf (or NaN) contribute nothing to the backward though the table lists keys that they
    see: the gradients are those of dO = 0 in these rows, to the bit (P times 0 and 0 times dP are both 0)."""
    w = W.custom_workload("off", [150, 33, 260], 64, 4, 2, d, dtype, spec, seed=67, input_scale=0.5)
    g = H.GpuRun(w, W.make_tensors(w), H.oracle_table(w))
    g.forward_only()
    off = [0, 5, 40, 149, 150, 182, 183, 300, 442]
    lse, lse_off, dout = g.lse, g.lse.clone(), g.dout
    lse_off[:, off[:-2]] = float("-inf")
    lse_off[1, off[-2:]] = float("nan")
    g.dout = dout.clone()
    g.dout[off[:-2]] = 0
    g.dout[off[-2:], 1] = 0
    want = g.backward(lse=lse)
    g.dout = dout
    for name, a, b in zip(("dq", "dk", "dv"), g.backward(lse=lse_off), want):
        assert (a == b).all(), name


def _same(a, b, w, label):
    """Inf and NaN at the same places, the finite values within the bounds of helpers.TOL."""
    assert (np.isnan(a) == np.isnan(b)).all(), f"{label}: NaN at {np.argwhere(np.isnan(a) != np.isnan(b))[:4].tolist()}, .."
    inf = np.isinf(b)
    assert (np.isinf(a) == inf).all() and (a[inf] == b[inf]).all(), f"{label}: Inf at {np.argwhere(np.isinf(a) != inf)[:4].tolist()}, .."
    fin = np.isfinite(b)
    a, b, tol = a[fin], b[fin], H.TOL[w.dtype]["lse" if label.endswith("lse") else "o"]
    assert (np.abs(a - b) <= tol + 2.0 ** -7 * np.abs(b)).all() if fin.any() else True, label


PLANT = {   # tensor -> (token, head, column or all, value); tokens of the second and third sequence too
    "v": [(40, 0, 3, "inf"), (100, 1, 5, "nan"), (170, 0, None, "-inf"), (290, 1, 0, "inf"), (442, 0, 7, "nan")],
    "k": [(100, 0, 2, "nan"), (149, 1, None, "nan"), (330, 1, 4, "inf")],
    "q": [(60, 1, 0, "inf"), (176, 3, None, "nan"), (310, 0, 1, "-inf")],
    "dout": [(47, 0, 2, "inf"), (120, 3, None, "nan"), (250, 2, 6, "-inf")],
    "out": [(47, 1, 2, "nan"), (120, 2, 1, "inf"), (400, 0, None, "-inf")]}


@pytest.mark.parametrize("dtype,d", SHAPES)
@pytest.mark.parametrize("spec", [W.MaskSpec("causal"), W.MaskSpec("lambda", window=70, sink=9)], ids=lambda s: s.kind)
def test_inf_and_nan_reach_visible_pairs_only(dtype, d, spec):
    """Against the thread-per-row kernels, which pass over every pair that is not visible.  One tensor at a time; the
    backward of both is given the same O and LSE, and LSE 1 in rows whose own is not finite, so that none is off."""
    import torch
    import paper_2510_10620_amd as P
    w = W.custom_workload("nonfinite", [150, 33, 260], 64, 4, 2, d, dtype, spec, seed=68, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    for name, plants in PLANT.items():
        fast, slow = H.GpuRun(w, tensors, table), H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)
        def plant(x):
            for tok, head, col, value in plants:
                x[tok, head, slice(None) if col is None else col] = float(value)
        if name != "out":
            for g in (fast, slow):
                plant(getattr(g, name))
        ref = slow.forward()
        for a, b, n in zip(fast.forward(), ref, ("out", "lse")):
            _same(a, b, w, f"{name} planted, {n}")
        out, lse = slow.out.clone(), slow.lse.clone()
        if name == "out":
            plant(out)
        lse[~torch.isfinite(lse)] = 1.0
        for a, b, n in zip(fast.backward(out, lse), slow.backward(out, lse), ("dq", "dk", "dv")):
            _same(a, b, w, f"{name} planted, {n}")


@pytest.mark.parametrize("dtype,d", SHAPES)
def test_values_near_the_largest(dtype, d):
    """V of 1e38: the running maximum is raised lazily, so weights of 2^7 meet V before the division by their sum; O is
    finite all the same.  One key beyond the first tiles outweighs the others."""
    w = W.custom_workload("large", [300], 512, 1, 1, d, dtype, W.MaskSpec("causal"), seed=74)
    g = H.GpuRun(w, W.make_tensors(w), H.oracle_table(w))
    g.q.fill_(1.0)
    g.k.zero_()
    g.k[261] = 7 * np.log(2) / np.sqrt(d)
    g.v.fill_(1e38)
    out, _ = g.forward()
    assert (np.abs(out / 1e38 - 1) <= (1e-5 if dtype == "f32" else 2.0 ** -7)).all()


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("heads,form", [(16, 1), (128, 0)], ids=["split", "shared"])
def test_inf_and_nan_in_a_large_narrow_batch(d, heads, form):
    """dK/dV whose waves split the other side, and the kernel that shares a tile among them."""
    import torch
    import paper_2510_10620_amd as P
    w = W.custom_workload("nonfinite_l", [700, 129] + [40] * 57, 128, heads, heads, d, "bf16", W.MaskSpec("causal"), seed=73, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    assert P.dcp_plan_export_forms(H.GpuRun(w, tensors, table).plan, heads, heads, d, P.DCP_BF16)["dkv"] == form
    fast, slow = H.GpuRun(w, tensors, table), H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)
    for g in (fast, slow):
        g.v[40, 3, 1], g.v[650, 5], g.q[300, 7, 2], g.dout[820, 15, 9] = float("inf"), float("nan"), float("inf"), float("nan")
    ref = slow.forward()
    for a, b, n in zip(fast.forward(), ref, ("out", "lse")):
        _same(a, b, w, n)
    lse = torch.where(torch.isfinite(slow.lse), slow.lse, 1.0)
    for a, b, n in zip(fast.backward(slow.out, lse), slow.backward(slow.out, lse), ("dq", "dk", "dv")):
        _same(a, b, w, n)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64)])
def test_inf_in_partial_slots_and_block_buffers(dtype, d):
    """The same through partial slots and permuted block buffers (rows live elsewhere than their packed index says)."""
    import torch
    import paper_2510_10620_amd as P
    w = W.custom_workload("nonfinite_b", [150, 33, 260], 64, 4, 2, d, dtype, W.MaskSpec("causal"), seed=69, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    slot, n_slots, _ = W.deal_divisions(table[:, 0], 2, 5)
    nb, B, got = 9, w.block_size, []
    assert sum(-(-n // B) for n in (150, 33, 260)) == nb
    rng = np.random.default_rng(5)
    qs, ks = rng.permutation(nb).astype(np.int32), rng.permutation(nb).astype(np.int32)
    for impl in (P.DCP_IMPL_AUTO, P.DCP_IMPL_SCALAR):
        g = H.GpuRun(w, tensors, table, slot, n_slots, impl)
        P.dcp_plan_set_block_buffers(g.plan, qs, nb, ks, nb)
        start, length = g.plan.export("BLK_START"), g.plan.export("BLK_LEN")
        def buf(x, slots):
            y = torch.zeros((nb * B,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda")
            for b in range(nb):
                y[slots[b] * B:slots[b] * B + length[b]] = x[start[b]:start[b] + length[b]]
            return y
        g.v[40, 0, 3] = float("inf")
        g.v[300, 1] = float("nan")
        q, k, v, do = buf(g.q, qs), buf(g.k, ks), buf(g.v, ks), buf(g.dout, qs)
        o_part = torch.zeros((n_slots, B, w.hq, d), dtype=q.dtype, device="cuda")
        lse_part = torch.zeros((n_slots, w.hq, B), device="cuda")
        P.dcp_block_attn_fwd(g.plan, q, k, v, o_part, lse_part, w.softmax_scale, None, impl)
        out, lse = torch.zeros_like(q), torch.full((w.hq, nb * B), 1.0, device="cuda")
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        ws = torch.empty(max(256, P.dcp_bwd_workspace_bytes(g.plan, w.hq, w.hkv, d, P.DCP_BF16 if dtype == "bf16" else P.DCP_F32)),
                         dtype=torch.uint8, device="cuda")
        P.dcp_block_attn_bwd(g.plan, q, k, v, out, lse, do, dq, dk, dv, w.softmax_scale, ws, None, impl)
        torch.cuda.synchronize()
        got.append([H.from_torch(x) for x in (o_part, lse_part, dq, dk, dv)])
    for a, b, n in zip(got[0], got[1], ("o_part", "lse", "dq", "dk", "dv")):
        _same(a, b, w, n)
