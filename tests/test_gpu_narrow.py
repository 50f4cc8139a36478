"""The bf16 kernels for heads of 32 and 64 at the sizes where they can go wrong, against the fp64 oracle: rows and blocks
around their 32-row sub-tiles, 64-row tiles and 128-row work items, every mask kind, slots and strided inputs.  Bounds:
those of bf16 I/O in helpers.TOL; and, for O, what 16 significant bits of P and one bf16 rounding allow."""
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
    # O = sum_j P_j v_j with P to 2^-17 (and sum_j P_j = 1), rounded to bf16 once: half an ulp is at most 2^-8 |O|; the
    # fp32 sums add less than 2^-17 max |v| again
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
