"""The fp32 kernels that multiply in bf16 parts (D 32 and 64): one group of waves and several, odd head groups, ragged and one-token
sequences, against the fp64 oracle; values of every size, whose last bits are in the third part; Inf and NaN, which have no parts; block
buffers, partial slots, strides, gradients over the inputs and rows that are off."""
import numpy as np
import pytest

import paper_2510_10620_amd as P
from paper_2510_10620_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

EQ, MIXED = [161] * 10 + [1, 33], [1100, 127, 65, 31]
SPECS = {"causal": W.MaskSpec("causal"), "lambda": W.MaskSpec("lambda", window=70, sink=9)}
# D, lengths, block size, heads, groups of every kernel
CASES = [(32, EQ, 512, (15, 5), 1), (32, MIXED, 512, (18, 6), 2), (32, [900, 257, 129, 65, 33, 1], 512, (16, 4), 2),
         (64, EQ, 512, (15, 5), 1), (64, MIXED, 512, (18, 6), 2), (64, [1500], 512, (16, 4), 2),
         (64, EQ + EQ, 512, (15, 5), 1)]
NAMES = ("out", "lse", "dq", "dk", "dv")


def _run(case, mask, spread=False, scale=0.5, exponents=()):
    d, lens, B, (hq, hkv), groups = case
    w = W.custom_workload("parts", lens, B, hq, hkv, d, "f32", SPECS[mask], seed=96, input_scale=scale)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    if spread:   # magnitudes over 2^-20 .. 1
        rng = np.random.default_rng(7)
        tensors = {k: (v * np.exp2(-20 * rng.random(v.shape))).astype(v.dtype) if isinstance(v, np.ndarray) and v.dtype == np.float32 else v
                   for k, v in tensors.items()}
    for n, e in exponents:
        tensors[n] = np.ldexp(tensors[n], e)
    g = H.GpuRun(w, tensors, table)
    forms = P.dcp_plan_export_forms(g.plan, hq, hkv, d, P.DCP_F32)
    assert (forms["fwd"], forms["dq"]) == (P.DCP_FORM_SHARED, P.DCP_FORM_SHARED)
    assert case is CASES[3] or forms["dkv"] == P.DCP_FORM_SHARED
    assert P.dcp_plan_export_part_groups(g.plan, hq, hkv, d) == (groups,) * 3
    return w, tensors, table, g


@pytest.mark.parametrize("mask", list(SPECS))
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"D{c[0]}-{len(c[1])}-{c[3][0]}x{c[3][1]}-g{c[4]}")
def test_results(case, mask):
    w, tensors, table, g = _run(case, mask)
    out, lse = g.forward()
    dq, dk, dv = g.backward()
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), H.oracle_full(w, tensors, table), NAMES, str(case))


@pytest.mark.parametrize("case", [CASES[2], CASES[5]], ids=["D32", "D64"])
def test_all_bits_of_the_inputs_count(case):
    """With the third parts of one operand left out, each product would be off by up to 2^-17 of it, 2^-19 in the mean square; fp32 sums of
    this length are off by 2^-22 of the norm or less.  The gradients see P = 2^(s - lse2): LSE and lse2 (here 8 to 16) are rounded once each,
    by up to 2^-21, which puts all of a row's weights off by up to 2 x 2^-21 ln 2 = 2^-20.5."""
    w, tensors, table, g = _run(case, "causal", spread=True)
    got = dict(zip(NAMES, g.forward() + g.backward()))
    ref = H.oracle_full(w, tensors, table)
    for n in NAMES:
        a, b = got[n].astype(np.float64), np.asarray(ref[n])
        assert np.linalg.norm(a - b) <= (2.0 ** -20 if n[0] == "d" else 2.0 ** -21) * np.linalg.norm(b), n


@pytest.mark.parametrize("exponents", [(("dout", -112),), (("v", -118),), (("k", -118),), (("q", -118),), (("q", 60), ("k", -60), ("dout", -100)),
                                       (("q", 100), ("k", -100)), (("q", -100), ("k", 100)), (("v", 114),), (("dout", 100),)],
                         ids=lambda x: "-".join(f"{n}{e}" for n, e in x))
@pytest.mark.parametrize("case", [CASES[0], CASES[1], CASES[3], CASES[4]], ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_numbers_of_any_size_keep_their_bits(case, exponents):
    """An operand, or the dS that comes of it, down to 2^-140: parts that ended at bf16's smallest number would leave it fewer than 10 bits; or up
    to 2^116, which overflows in the parts and is worked out again.  The bounds are those of test_all_bits_of_the_inputs_count; what is new is that results of 2^-126 and less are rounded to 2^-149."""
    w, tensors, table, g = _run(case, "causal", exponents=exponents)
    got = dict(zip(NAMES, g.forward() + g.backward()))
    ref = H.oracle_full(w, tensors, table)
    for n in NAMES:
        a, b = got[n].astype(np.float64), np.asarray(ref[n])
        bound = (2.0 ** -20 if n[0] == "d" else 2.0 ** -21) * np.linalg.norm(b) + 2.0 ** -149 * np.sqrt(b.size)
        assert np.linalg.norm(a - b) <= bound, (n, np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("mask", list(SPECS))
@pytest.mark.parametrize("case", [CASES[0], CASES[1], CASES[3], CASES[4]], ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_inf_in_k(case, mask):
    """Against the thread-per-row kernels: where q is negative in that column the score is -Inf, the key has weight 0 and the row is finite.
    3.4e38 is finite, its first part is not (q is small enough for finite scores)."""
    from tests.test_gpu_nonfinite import _same
    w, tensors, table, fast = _run(case, mask, scale=0.1)
    slow = H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)
    for g in (fast, slow):
        g.k[w.total_tokens // 3, 0, 5], g.k[w.total_tokens // 2, w.hkv - 1, 2] = float("inf"), 3.4e38
    for a, b, n in zip(fast.forward(), slow.forward(), ("out", "lse")):
        _same(a, b, w, n)
    assert np.isfinite(H.from_torch(slow.out)).any() and not np.isfinite(H.from_torch(slow.out)).all()


@pytest.mark.parametrize("case", [CASES[1], CASES[4]], ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_lse_of_repaired_rows(case):
    """Several groups of waves, and every row but the first of a sequence is worked out again: the second key of each sequence is Inf where q is
    negative, so its weight is 0.  A row's LSE is that of its other keys, whichever group repairs it."""
    import torch
    from tests.test_gpu_nonfinite import _same
    w, tensors, table, fast = _run(case, "causal")
    slow = H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)
    second = torch.as_tensor(w.cu_seqlens[:-1].astype(np.int64) + 1).cuda()
    for g in (fast, slow):
        g.q[:, :, 5] = -g.q[:, :, 5].abs() - 0.1
        g.k[second, :, 5] = float("inf")
    out, lse = slow.forward()
    assert np.isfinite(lse).all()
    for _ in range(4):
        for a, b, n in zip(fast.forward(), (out, lse), ("out", "lse")):
            _same(a, b, w, n)


@pytest.mark.parametrize("d,mask,lens,B,heads", [(32, "causal", [1500], 64, (6, 3)), (32, "lambda", [1030, 7], 1024, (8, 8)), (64, "causal", [2050, 33], 64, (4, 4)),
                                                 (64, "lambda", [2050, 33], 1024, (6, 3))], ids=["D32-causal", "D32-ranges", "D64-causal", "D64-ranges"])
def test_dkv_in_parts_behind_32_rows_on_the_fp32_pipe(d, mask, lens, B, heads):
    """Few long walks: forward and dQ by 32 rows a workgroup on the fp32 pipe, which leaves delta and lse2 for dK/dV in parts."""
    w = W.custom_workload("pipe", lens, B, heads[0], heads[1], d, "f32", SPECS[mask], seed=99, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    g = H.GpuRun(w, tensors, table)
    assert set(P.dcp_plan_export_forms(g.plan, *heads, d, P.DCP_F32).values()) == {P.DCP_FORM_SHARED}
    groups = P.dcp_plan_export_part_groups(g.plan, *heads, d)
    assert groups[:2] == (0, 0) and groups[2] > 0
    got = dict(zip(NAMES, g.forward() + g.backward()))
    H.check(w, got, H.oracle_full(w, tensors, table), NAMES, f"D{d} {mask}")


LAYOUTS = [CASES[0], CASES[2], CASES[4], CASES[6]]   # D 32 and 64, one group of waves and several


def _in_parts(plan, case, dkv=True):
    d, _, _, heads, _ = case
    forms, groups = P.dcp_plan_export_forms(plan, *heads, d, P.DCP_F32), P.dcp_plan_export_part_groups(plan, *heads, d)
    return all(forms[n] == P.DCP_FORM_SHARED and g > 0 for n, g in zip(("fwd", "dq", "dkv") if dkv else ("fwd", "dq"), groups)) and forms["bwd"] == P.DCP_FORM_SHARED


@pytest.mark.parametrize("slots", [False, True], ids=["whole", "slots"])
@pytest.mark.parametrize("case", LAYOUTS, ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_block_buffers(case, slots):
    """Permuted blocks with free ones between them; with slots, each query block in up to three partial results and their merge."""
    from tests.test_gpu_parity import _buffer_case
    d, lens, B, heads, _ = case
    w = W.custom_workload("buffers", lens, B, *heads, d, "f32", SPECS["lambda"], seed=100, input_scale=0.5)
    table = H.oracle_table(w)
    slot, n_slots = W.deal_divisions(table[:, 0], 3, 5)[:2] if slots else (None, 0)
    assert _in_parts(P.dcp_plan_create(w.cu_seqlens, B, table, slot, n_slots), case)
    _buffer_case(w, table, 0, np.random.default_rng(11), out_slot=slot, n_slots=n_slots)


@pytest.mark.parametrize("case", LAYOUTS, ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_strides_and_gradients_over_the_inputs(case):
    """Inputs as views of one projection, outputs in padded rows; then dQ over O, dK over K and dV over V: the same bits."""
    import torch
    d, lens, B, (hq, hkv), _ = case
    w, tensors, table, g = _run(case, "causal")
    ref = H.oracle_full(w, tensors, table)
    fused = torch.cat([g.q, g.k, g.v], dim=1).contiguous()
    q, k, v = fused[:, :hq], fused[:, hq:hq + hkv], fused[:, hq + hkv:]
    pad = lambda h: torch.full((w.total_tokens, h + 1, d + 8), float("nan"), device="cuda")
    full = [pad(h) for h in (hq, hq, hq, hkv, hkv)]
    do, out, dq, dk, dv = (x[:, :-1, :d] for x in full)
    do.copy_(g.dout)
    lse = torch.empty((hq, w.total_tokens), device="cuda")
    ws = torch.empty(max(256, P.dcp_bwd_workspace_bytes(g.plan, hq, hkv, d, P.DCP_F32)), dtype=torch.uint8, device="cuda")
    P.dcp_block_attn_fwd(g.plan, q, k, v, out, lse, w.softmax_scale)
    P.dcp_block_attn_bwd(g.plan, q, k, v, out, lse, do, dq, dk, dv, w.softmax_scale, ws)
    torch.cuda.synchronize()
    got = dict(zip(NAMES, (H.from_torch(x.contiguous()) for x in (out, lse, dq, dk, dv))))
    H.check(w, got, ref, NAMES, "strided")
    for x in full[1:]:
        assert torch.isnan(x[:, -1]).all() and torch.isnan(x[:, :, d:]).all(), "a row's padding was written"
    want = [x.contiguous() for x in (dq, dk, dv)]
    P.dcp_block_attn_bwd(g.plan, q, k, v, out, lse, do, out, k, v, w.softmax_scale, ws)
    torch.cuda.synchronize()
    for a, b, n in zip((out, k, v), want, NAMES[2:]):
        assert torch.equal(a, b), n


@pytest.mark.parametrize("mask", list(SPECS))
@pytest.mark.parametrize("case", LAYOUTS, ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_rows_switched_off_by_their_lse(case, mask):
    """Query rows whose LSE is -inf or NaN contribute nothing: the gradients are those of dO = 0 in these rows, to the bit."""
    w, _, _, g = _run(case, mask)
    g.forward_only()
    off = [0, 31, 32, 160, 161, 500, 1285]
    lse, dout = g.lse, g.dout
    lse_off = lse.clone()
    lse_off[:, off[:-2]] = float("-inf")
    lse_off[1, off[-2:]] = float("nan")
    g.dout = dout.clone()
    g.dout[off[:-2]] = 0
    g.dout[off[-2:], 1] = 0
    want = g.backward(lse=lse)
    g.dout = dout
    for name, a, b in zip(NAMES[2:], g.backward(lse=lse_off), want):
        assert (a == b).all(), name


@pytest.mark.parametrize("mask", list(SPECS))
@pytest.mark.parametrize("case", LAYOUTS, ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_inf_and_nan_reach_visible_pairs_only(case, mask):
    """Forward and backward against the thread-per-row kernels, one tensor at a time, with what test_gpu_nonfinite.py plants."""
    import torch
    from tests.test_gpu_nonfinite import PLANT, _same
    w, tensors, table, _ = _run(case, mask)
    for name, plants in PLANT.items():
        fast, slow = H.GpuRun(w, tensors, table), H.GpuRun(w, tensors, table, impl=P.DCP_IMPL_SCALAR)

        def plant(x):
            for tok, head, col, value in plants:
                x[tok, head, slice(None) if col is None else col] = float(value)
        if name != "out":
            for g in (fast, slow):
                plant(getattr(g, name))
        for a, b, n in zip(fast.forward(), slow.forward(), ("out", "lse")):
            _same(a, b, w, f"{name} planted, {n}")
        out, lse = slow.out.clone(), slow.lse.clone()
        if name == "out":
            plant(out)
        lse[~torch.isfinite(lse)] = 1.0
        for a, b, n in zip(fast.backward(out, lse), slow.backward(out, lse), NAMES[2:]):
            _same(a, b, w, f"{name} planted, {n}")


@pytest.mark.parametrize("case", [CASES[0], CASES[4]], ids=lambda c: f"D{c[0]}-g{c[4]}")
def test_static_workspace(case):
    """dcp_block_attn_bwd_static: the same bits."""
    import torch
    w, _, _, g = _run(case, "lambda")
    P.dcp_plan_prepare(g.plan, w.hq, w.hkv, w.d, P.DCP_F32)
    g.forward_only()
    g.backward_only(g.out, g.lse)
    got = [torch.full_like(x, float("nan")) for x in (g.dq, g.dk, g.dv)]
    P.dcp_block_attn_bwd_static(g.plan, g.q, g.k, g.v, g.out, g.lse, g.dout, *got, w.softmax_scale, g.ranges)
    torch.cuda.synchronize()
    for a, b, n in zip(got, (g.dq, g.dk, g.dv), NAMES[2:]):
        assert torch.equal(a, b), n


@pytest.mark.parametrize("d", [32, 64])
def test_ranges_past_four_gigabytes(d):
    """The last sequence of a batch of more than 2^28 packed tokens, whose blocks are in block buffers, gives the bits of the same sequence by
    itself: byte offsets into the range array pass 2^32 there."""
    import torch
    B, far, n, (hq, hkv) = 2048, 1 << 28, 1500, (16, 4)
    case = (d, [n], B, (hq, hkv), 0)
    w = W.custom_workload("near", [n], B, hq, hkv, d, "f32", SPECS["lambda"], seed=101, input_scale=0.5)
    g = H.GpuRun(w, W.make_tensors(w), np.array([[0, 0, W.MASK_RANGES]], np.int32))
    assert _in_parts(g.plan, case)
    g.forward_only()
    g.backward_only(g.out, g.lse)
    nb = far // B + 1
    plan = P.dcp_plan_create(np.array([0, far, far + n], np.int32), B, np.array([[nb - 1, nb - 1, W.MASK_RANGES]], np.int32))
    slot = np.full(nb, -1, np.int32)
    slot[-1] = 0
    P.dcp_plan_set_block_buffers(plan, slot, 1, slot, 1)
    assert _in_parts(plan, case)
    ranges = torch.zeros((far + n, 4), dtype=torch.int32, device="cuda")
    near = torch.from_numpy(w.ranges).cuda()
    for c in (0, 2):
        near[near[:, c + 1] > near[:, c], c:c + 2] += far
    ranges[far:] = near
    rows = lambda x: torch.cat([x, torch.zeros((B - n,) + tuple(x.shape[1:]), device="cuda")])
    q, k, v, do = (rows(x) for x in (g.q, g.k, g.v, g.dout))
    out, dq, dk, dv = (torch.zeros_like(x) for x in (q, q, k, v))
    lse = torch.zeros((hq, B), device="cuda")
    P.dcp_block_attn_fwd(plan, q, k, v, out, lse, w.softmax_scale, ranges)
    ws = torch.empty(P.dcp_bwd_workspace_bytes(plan, hq, hkv, d, P.DCP_F32), dtype=torch.uint8, device="cuda")
    P.dcp_block_attn_bwd(plan, q, k, v, out, lse, do, dq, dk, dv, w.softmax_scale, ws, ranges)
    torch.cuda.synchronize()
    for name, a, b in zip(NAMES, (out[:n], lse[:, :n], dq[:n], dk[:n], dv[:n]), (g.out, g.lse, g.dq, g.dk, g.dv)):
        assert torch.equal(a, b), name
