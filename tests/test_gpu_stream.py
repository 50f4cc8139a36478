"""The streaming kernels where their splits end: heads and chunks that do not divide a workgroup's steps, a ragged last
workgroup, one to eight parts."""
import pytest
import torch

import paper_2510_10620_amd as P

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
