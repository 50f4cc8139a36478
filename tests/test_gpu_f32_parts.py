"""The fp32 kernels that multiply in bf16 parts (D 32 and 64): one group of waves and several, odd head groups, ragged and one-token
sequences, against the fp64 oracle; values of every size, whose last bits are in the third part; an Inf in K, which leaves NaN in the parts
of a score that is -Inf."""
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
