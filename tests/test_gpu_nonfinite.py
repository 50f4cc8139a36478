"""Values that are not finite, in the kernels for fp32 and for heads of 32 and 64: rows that the backward leaves out."""
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
