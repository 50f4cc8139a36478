"""The bf16 kernels for heads of 32 and 64 at the sizes where they can go wrong, against the fp64 oracle: rows and blocks
around their 32-row sub-tiles, 64-row tiles and 128-row work items, every mask kind, slots and strided inputs.  Bounds:
those of bf16 I/O in helpers.TOL; and, for O, one bf16 rounding beside fp32 sums."""
import numpy as np
import pytest

from paper_2510_10620_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

LENS = [1, 31, 33, 63, 65, 127, 129, 257, 640]
ALL = ("out", "lse", "dq", "dk", "dv")


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("B,heads,spec", [
    (64, (2, 1), W.MaskSpec("causal")), (96, (3, 3), W.MaskSpec("lambda", window=70, sink=9)), (512, (8, 2), W.MaskSpec("shared_question")),
    (130, (4, 2), W.MaskSpec("window", window=40))], ids=lambda x: getattr(x, "kind", None))
def test_narrow_tiles(d, B, heads, spec):
    w = W.custom_workload("narrow", LENS, B, heads[0], heads[1], d, "bf16", spec, seed=63, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    ref = H.oracle_full(w, tensors, table)
    window = (spec.window, spec.sink) if spec.kind == "window" else None
    t = table.copy()
    if window:
        t[t[:, 2] == W.MASK_RANGES, 2] = W.MASK_WINDOW   # no range array: two numbers
    g = H.GpuRun(w, tensors, t, window=window)
    out, lse = g.forward()
    dq, dk, dv = g.backward()
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), ref, ALL, f"narrow D{d} B{B} {spec.kind}")
    # O = sum_j P_j v_j (and sum_j P_j = 1), rounded to bf16 once: half an ulp is at most 2^-8 |O|; the scores, weights and
    # fp32 sums add less than 2^-16 max |v|
    vmax = np.abs(W.to_f64(w, tensors["v"])).max()
    assert (np.abs(out - ref["out"]) <= 2.0 ** -8 * np.abs(ref["out"]) + 2.0 ** -16 * vmax).all()


def test_narrow_slots_strides_and_empty_rows():
    """Partial slots with their merge, a table that leaves rows without partners, q / k / v as views of one projection."""
    import torch
    w = W.custom_workload("narrow_s", [150, 260], 64, 4, 2, 64, "bf16", W.MaskSpec("causal"), seed=64, input_scale=0.5)
    tensors, table = W.make_tensors(w), H.oracle_table(w)[::2]
    slot, n_slots, _ = W.deal_divisions(table[:, 0], 2, 5)
    g = H.GpuRun(w, tensors, table, slot, n_slots)
    fused = torch.cat([g.q, g.k, g.v], dim=1).contiguous()
    g.q, g.k, g.v = fused[:, :4], fused[:, 4:6], fused[:, 6:8]
    out, lse = g.forward()
    dq, dk, dv = g.backward()
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), H.oracle_full(w, tensors, table), ALL, "narrow slots")


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("n_items,heads,form", [(64, (32, 16), 1), (65, (32, 16), 1), (65, (128, 128), 0)], ids=["split-64", "split-65", "shared"])
@pytest.mark.parametrize("spec,window_rows", [(W.MaskSpec("causal"), False), (W.MaskSpec("lambda", window=50, sink=9), False),
                                              (W.MaskSpec("lambda", window=50, sink=9), True)], ids=["causal", "ranges", "window"])
def test_narrow_dkv_on_both_sides_of_the_choice(d, n_items, heads, form, spec, window_rows):
    """dK/dV whose four waves split the other side, and the kernel that shares a tile among them (which takes launches of a great many items):
    sequences of 1 to 128 tokens beside one of 700."""
    import paper_2510_10620_amd as P
    lens = [700, 129, 128, 127, 65, 64, 33, 1] + [1 + 7 * i % 128 for i in range(n_items - 14)]
    w = W.custom_workload("narrow_rule", lens, 128, heads[0], heads[1], d, "bf16", spec, seed=72, input_scale=0.5)
    assert sum(-(-n // 128) for n in lens) == n_items
    tensors, table = W.make_tensors(w), H.oracle_table(w)
    ref = H.oracle_full(w, tensors, table)
    t = table.copy()
    if window_rows:
        t[t[:, 2] == W.MASK_RANGES, 2] = W.MASK_WINDOW
    g = H.GpuRun(w, tensors, t, window=(spec.window, spec.sink) if window_rows else None)
    forms = P.dcp_plan_export_forms(g.plan, *heads, d, P.DCP_BF16)
    assert forms["dkv"] == form and forms["bwd"] == P.DCP_FORM_SHARED
    out, lse = g.forward()
    dq, dk, dv = g.backward()
    H.check(w, dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv), ref, ALL, f"narrow D{d} {n_items} items {spec.kind}")


@pytest.mark.parametrize("d", [32, 64])
def test_narrow_weights_are_not_rounded(d):
    """P and dS enter the products over keys and queries with all their 24 bits.  Sequences of four tokens whose last two
    values (queries, keys, dO rows) are chosen so that the sums nearly cancel: what is left is 2^-18 of the terms, and
    its bf16 rounding as fine as 2^-26, so that an error of the weights shows.  Against the same sums in 64 bits."""
    import torch
    import paper_2510_10620_amd as P
    S, NH, n = 64, 2, 4
    rng = np.random.default_rng(66)
    bf = lambda x: W.bf16_bits_to_f64(W.f32_to_bf16_bits(np.asarray(x, np.float32)))
    rnd = lambda *s: bf(rng.standard_normal(s))
    scale = float(np.float32(1 / np.sqrt(d)))
    q, k, v, do = (np.zeros((S, n, NH, d)) for _ in range(4))
    A, B = slice(8, 8 + (d - 8) // 2), slice(8 + (d - 8) // 2, d)   # columns where q, where k is zero: free for the other
    q[..., :8], k[..., :8] = rnd(S, n, NH, 8), rnd(S, n, NH, 8)
    s = np.einsum("sihd,sjhd->shij", q, k) * scale
    s[:, :, ~np.tril(np.ones((n, n), bool))] = -np.inf
    lse = np.log(np.exp(s).sum(-1)).astype(np.float32)
    p = np.exp(s - lse[..., None])

    def cancel(x, w, cols):
        """x[:, 2:] so that sum_j w[.., j] x[:, j] is nearly zero; w [S, heads, n]."""
        x[:, :2, :, cols] = rnd(S, 2, NH, len(range(d)[cols]))
        for j in (2, 3):
            left = np.einsum("shj,sjhd->shd", w[..., :j], x[:, :j, :, cols])
            x[:, j, :, cols] = bf(np.clip(-left / w[..., j, None], -64, 64))
    cancel(v, p[:, :, 3], slice(0, d))
    cancel(do, p[:, :, :, 0], slice(0, 2))                           # dO in two columns: dP and delta are short sums
    o = np.einsum("shij,sjhd->sihd", p, v)
    ob = bf(o)
    dp, delta = np.einsum("sihd,sjhd->shij", do, v), np.einsum("sihd,sihd->shi", do, ob)
    mag = p * (np.einsum("sihd,sjhd->shij", abs(do), abs(v)) + np.einsum("sihd,sihd->shi", abs(do), abs(ob))[..., None])
    ds = p * (dp - delta[..., None])
    cancel(k, ds[:, :, 3], A)
    cancel(q, ds[:, :, :, 0], B)
    ref = dict(out=o[:, 3], dv=np.einsum("shi,sihd->shd", p[..., 0], do), dq=scale * np.einsum("shj,sjhd->shd", ds[:, :, 3], k),
               dk=scale * np.einsum("shi,sihd->shd", ds[..., 0], q))
    # fp32 arithmetic: a weight is good to 2^-21 (score, exponential, LSE), dP - delta to 2^-22 of its terms; twice that
    err = dict(out=2.0 ** -20 * np.einsum("shj,sjhd->shd", p[:, :, 3], abs(v)), dv=2.0 ** -20 * np.einsum("shi,sihd->shd", p[..., 0], abs(do)),
               dq=scale * np.einsum("shj,sjhd->shd", 2.0 ** -20 * abs(ds)[:, :, 3] + 2.0 ** -21 * mag[:, :, 3], abs(k)),
               dk=scale * np.einsum("shi,sihd->shd", 2.0 ** -20 * abs(ds)[..., 0] + 2.0 ** -21 * mag[..., 0], abs(q)))
    cu = (n * np.arange(S + 1)).astype(np.int32)
    table = np.array([[b, b, W.MASK_CAUSAL] for b in range(S)], np.int32)
    dev = lambda x: torch.from_numpy(x.reshape(S * n, NH, d)).to(torch.bfloat16).cuda()
    tq, tk, tv, tdo, to = (dev(x) for x in (q, k, v, do, ob))
    plan = P.dcp_plan_create(cu, 64, table)
    out, dq, dk, dv = (torch.empty_like(tq) for _ in range(4))
    lse_t = torch.empty((NH, S * n), device="cuda")
    P.dcp_block_attn_fwd(plan, tq, tk, tv, out, lse_t, scale, None)
    lse_t.copy_(torch.from_numpy(lse.transpose(1, 0, 2).reshape(NH, S * n).copy()))
    ws = torch.empty(max(256, P.dcp_bwd_workspace_bytes(plan, NH, NH, d, P.DCP_BF16)), dtype=torch.uint8, device="cuda")
    P.dcp_block_attn_bwd(plan, tq, tk, tv, to, lse_t, tdo, dq, dk, dv, scale, ws, None)
    torch.cuda.synchronize()
    host = lambda x, row: H.from_torch(x).reshape(S, n, NH, d)[:, row]
    got = dict(out=host(out, 3), dq=host(dq, 3), dk=host(dk, 0), dv=host(dv, 0))
    for name in ref:   # half an ulp of bf16 is at most 2^-8 of the value
        over = (np.abs(got[name] - ref[name]) - 2.0 ** -8 * (1 + 2.0 ** -8) * np.abs(ref[name])) / np.maximum(err[name], 1e-30)
        print(name, "error beyond the rounding of the result, of its bound:", over.max(), flush=True)
        assert over.max() <= 1, name
