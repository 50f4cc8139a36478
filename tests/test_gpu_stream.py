"""The streaming kernels where their splits end: heads and chunks that do not divide a workgroup's steps, a ragged last
workgroup, one to eight parts."""
import numpy as np
import pytest
import torch

import paper_2510_10620_amd as P
from paper_2510_10620_amd import workloads as W

pytestmark = pytest.mark.gpu


def _randn(shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, device="cuda", generator=g).to(dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("tokens,hq,d", [(1, 1, 8), (31, 3, 16), (33, 1, 32), (65, 6, 64), (100, 7, 128), (37, 33, 256), (64, 2, 8), (5, 40, 128)])
def test_delta_edges(tokens, hq, d, dtype):
    o, do = _randn((tokens, hq, d), dtype, 1), _randn((tokens, hq, d), dtype, 2)
    delta = torch.full((hq, tokens), float("nan"), device="cuda")
    P.dcp_bwd_delta(o, do, delta)
    ref = (o.double() * do.double()).sum(-1).T
    # d products summed in fp32: each of the d roundings is at most 2^-24 of the sum of the magnitudes
    bound = d * 2.0 ** -24 * (o.double() * do.double()).abs().sum(-1).T
    assert ((delta.double() - ref).abs() <= bound).all()


@pytest.mark.parametrize("src,dst", [(a, b) for a in (torch.bfloat16, torch.float32) for b in (torch.bfloat16, torch.float32)])
@pytest.mark.parametrize("n_parts", [1, 2, 3, 8])
@pytest.mark.parametrize("n", [8, 2040, 2056, 40008])
def test_sum_edges(n, n_parts, src, dst):
    parts = [_randn((n,), src, 10 + i) for i in range(n_parts)]
    out = torch.full((n,), float("nan"), device="cuda", dtype=dst)
    P.dcp_sum_partials(parts, out)
    ref = torch.zeros((n,), device="cuda")
    for p in parts:   # the documented order: first part to last, in fp32
        ref = ref + p.float()
    assert torch.equal(out, ref.to(dst))


@pytest.mark.parametrize("src,n,n_parts", [(torch.bfloat16, 1 << 26, 2), (torch.bfloat16, 1 << 26, 3), (torch.float32, (1 << 25) + 8, 3)])
def test_sum_on_both_sides_of_the_cache(src, n, n_parts):
    """268 MB of parts are read through the caches, 403 MB past them: the same sums."""
    parts = [_randn((n,), src, 10 + i) for i in range(n_parts)]
    out = torch.full((n,), float("nan"), device="cuda", dtype=torch.bfloat16)
    P.dcp_sum_partials(parts, out)
    ref = parts[0].float()
    for p in parts[1:]:
        ref = ref + p.float()
    assert torch.equal(out, ref.to(torch.bfloat16))


@pytest.mark.parametrize("d,hq", [(128, 1), (128, 3), (128, 8), (128, 16), (128, 24), (128, 40), (64, 5), (64, 32), (32, 7), (32, 64), (32, 100)])
def test_merge_of_none_to_six_partials(d, hq):
    """bf16 merge for head counts below, at and above the pairs of one step; blocks with 0 to 6 partials, short last blocks, a
    sequence shorter than its block.  Against fp64: half an ulp of the bf16 result is 2^-8 of it at most, the fp32 weights and
    sums of six terms add less than 2^-16 of the largest term."""
    B, lens = 16, [6 * 16 - 5, 3, 16]
    cu = W.cu_from_lengths(lens)
    table = [[i, j, 1 if i == j else 0] for i in range(6) for j in range(i + 1)] + [[6, 6, 1]]   # block 7 has no row: no partial
    table = np.array(table, dtype=np.int32)
    n_slots = len(table)
    plan = P.dcp_plan_create(cu, B, table, np.arange(n_slots, dtype=np.int32), n_slots)
    T = int(cu[-1])
    gen = torch.Generator(device="cuda").manual_seed(hq * 7 + d)
    o = torch.randn((n_slots, B, hq, d), device="cuda", generator=gen).to(torch.bfloat16)
    lse = torch.randn((n_slots, hq, B), device="cuda", generator=gen) * 3
    lse[torch.rand(lse.shape, device="cuda", generator=gen) < 0.2] = -float("inf")
    value = o.double()
    o = o.masked_fill((lse == -float("inf")).transpose(1, 2)[..., None], float("nan"))   # a dead partial's rows reach nothing
    out, l = torch.full((T, hq, d), float("nan"), device="cuda", dtype=torch.bfloat16), torch.full((hq, T), float("nan"), device="cuda")
    P.dcp_merge_partials(plan, o, lse, out, l)
    start, length = plan.export("BLK_START"), plan.export("BLK_LEN")
    for b in range(len(start)):
        s = np.nonzero(table[:, 0] == b)[0]
        n, a = int(length[b]), int(start[b])
        x = lse[s][:, :, :n].double()                                    # [parts, hq, n]
        ref_l = torch.logsumexp(x, 0) if len(s) else torch.full((hq, n), -float("inf"), device="cuda", dtype=torch.float64)
        wgt = torch.where(x > -float("inf"), torch.exp(x - ref_l), torch.zeros_like(x))
        terms = wgt.transpose(1, 2)[..., None] * value[s][:, :n]    # [parts, n, hq, d]
        ref = terms.sum(0) if len(s) else torch.zeros((n, hq, d), device="cuda", dtype=torch.float64)
        slack = 2.0 ** -16 * (terms.abs().amax() if len(s) else 0)
        assert ((out[a:a + n].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + slack).all(), (b, len(s))
        dead = ref_l == -float("inf")
        assert (l[:, a:a + n][dead] == -float("inf")).all()
        assert ((l[:, a:a + n].double() - ref_l)[~dead].abs() <= 1e-5).all(), (b, len(s))


@pytest.mark.parametrize("d,hq", [(128, 3), (128, 16), (64, 5), (32, 7)])
def test_merge_of_partials_whose_lse_is_not_finite(d, hq):
    """The bf16 merge gives NaN, zeros and -inf where the merge for any shape gives them (here on the same values in fp32), whichever of 1 to 6
    partials has LSE NaN, Inf or -inf; the other rows to a bf16 rounding."""
    B = 16
    table = np.array([[i, j, 1 if i == j else 0] for i in range(6) for j in range(i + 1)], dtype=np.int32)
    n_slots = len(table)
    plan = P.dcp_plan_create(np.array([0, 6 * B], np.int32), B, table, np.arange(n_slots, dtype=np.int32), n_slots)
    gen = torch.Generator(device="cuda").manual_seed(hq + d)
    o = torch.randn((n_slots, B, hq, d), device="cuda", generator=gen).to(torch.bfloat16)
    lse = torch.randn((n_slots, hq, B), device="cuda", generator=gen)
    kind = torch.rand(lse.shape, device="cuda", generator=gen)
    for at, value in ((0.5, "-inf"), (0.2, "nan"), (0.1, "inf")):
        lse[kind < at] = float(value)
    res = []
    for x in (o, o.float()):
        out, l = torch.full((6 * B, hq, d), 7.0, device="cuda", dtype=x.dtype), torch.full((hq, 6 * B), 7.0, device="cuda")
        P.dcp_merge_partials(plan, x, lse, out, l)
        res.append((out.double(), l.double()))
    (out, l), (ref, ref_l) = res
    assert torch.isnan(ref_l).any() and (ref_l == -float("inf")).any() and torch.isfinite(ref_l).any()
    for a, b, tol in ((out, ref, 2.0 ** -8), (l, ref_l, 2.0 ** -23)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
        fin = torch.isfinite(b)
        assert ((a - b).abs() <= tol * b.abs() + 2.0 ** -22)[fin].all()


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 8), (torch.float32, 64)])
@pytest.mark.parametrize("T", [1, 7, 8, 9, 32 * 1024 - 1, 32 * 1024])
def test_delta_tokens_per_workgroup(T, dtype, d):
    """Both sides of the rule for 8 or 32 tokens a workgroup, odd head counts.  fp32 sums of d terms in any order: d 2^-24 of
    the terms' magnitudes."""
    gen = torch.Generator(device="cuda").manual_seed(T)
    o, do = (torch.randn((T, 3, d), device="cuda", generator=gen).to(dtype) for _ in range(2))
    delta = torch.full((3, T), float("nan"), device="cuda")
    P.dcp_bwd_delta(o, do, delta)
    t = o.double() * do.double()
    assert ((delta.double() - t.sum(-1).T).abs() <= d * 2.0 ** -24 * t.abs().sum(-1).T).all()


@pytest.mark.parametrize("dtype,d,h,last", [(torch.bfloat16, 128, 17, 22 * 1024 - 1), (torch.bfloat16, 8, 3, 96 * 24), (torch.float32, 64, 3, 32 * 192),
                                            (torch.float32, 128, 5, 10 * 1024 - 1)])
def test_delta_tokens_per_workgroup_by_work(dtype, d, h, last):
    """The same where many heads, few chunks to a token or fp32 take 8 tokens a workgroup up to `last` tokens only."""
    for T in (last, last + 1):
        gen = torch.Generator(device="cuda").manual_seed(T)
        o, do = (torch.randn((T, h, d), device="cuda", generator=gen).to(dtype) for _ in range(2))
        delta = torch.full((h, T), float("nan"), device="cuda")
        P.dcp_bwd_delta(o, do, delta)
        t = o.double() * do.double()
        assert ((delta.double() - t.sum(-1).T).abs() <= d * 2.0 ** -24 * t.abs().sum(-1).T).all(), T
