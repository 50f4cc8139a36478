"""A batch of more than 2^28 packed tokens of which a device's share is the last 200: byte offsets into the range array pass
2^32 there.  The blocks are in block buffers, so only the range array is long (4.3 GB)."""
import numpy as np
import pytest

from paper_2510_10620_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("bf16", 32), ("f32", 64)])
def test_ranges_past_four_gigabytes(dtype, d):
    """Forward and backward of the far sequence equal, to the bit, those of the same sequence in a batch of its own."""
    import torch
    import paper_2510_10620_amd as P
    B, far, n = 1 << 20, 1 << 28, 200
    w = W.custom_workload("near", [n], B, 2, 1, d, dtype, W.MaskSpec("lambda", window=70, sink=9), seed=70, input_scale=0.5)
    g = H.GpuRun(w, W.make_tensors(w), np.array([[0, 0, W.MASK_RANGES]], np.int32))
    g.forward_only()
    want = [g.out, g.lse] + [torch.from_numpy(x) for x in g.backward()]
    nb = far // B + 1
    plan = P.dcp_plan_create(np.array([0, far, far + n], np.int32), B, np.array([[nb - 1, nb - 1, W.MASK_RANGES]], np.int32))
    slot = np.full(nb, -1, np.int32)
    slot[-1] = 0
    P.dcp_plan_set_block_buffers(plan, slot, 1, slot, 1)
    ranges = torch.zeros((far + n, 4), dtype=torch.int32, device="cuda")
    ranges[far:] = torch.from_numpy(w.ranges).cuda()
    ranges[far:][ranges[far:, 1] > ranges[far:, 0], :2] += far
    ranges[far:][ranges[far:, 3] > ranges[far:, 2], 2:] += far
    rows = lambda x: torch.cat([x, torch.zeros((B - n,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda")])
    q, k, v, do = (rows(x) for x in (g.q, g.k, g.v, g.dout))
    out, dq, dk, dv = (torch.zeros_like(x) for x in (q, q, k, v))
    lse = torch.zeros((2, B), device="cuda")
    P.dcp_block_attn_fwd(plan, q, k, v, out, lse, w.softmax_scale, ranges)
    ws = torch.empty(P.dcp_bwd_workspace_bytes(plan, 2, 1, d, P.DCP_BF16 if dtype == "bf16" else P.DCP_F32), dtype=torch.uint8, device="cuda")
    P.dcp_block_attn_bwd(plan, q, k, v, out, lse, do, dq, dk, dv, w.softmax_scale, ws, ranges)
    torch.cuda.synchronize()
    for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), (out[:n], lse[:, :n], dq[:n], dk[:n], dv[:n]), want):
        assert (a.double().cpu() == b.double().cpu()).all(), name
