// The rows of a query-side workgroup whose four waves (or groups of four) share the other side's tiles, 32 rows a wave: narrow heads and
// fp32 in parts.
#pragma once
#include "mfma_common.h"
#include "nonfinite.h"

namespace dcp {
namespace {

// What the query-side kernels know about their workgroup's and their wave's rows.
struct NQTile {
  int head, hk, blk_start, row0, n_rows, q_lo, q_hi, qoff, wrow0, w_rows, wq_lo, wq_hi, qi, e0, e1, unit;
  bool qv;
  int4 qr;
  RangeBounds rb, wrb;   // of the workgroup's rows, of the wave's
};

// wave: of the RG that have different rows
template <bool RANGES, int RG = 4>
__device__ __forceinline__ bool nq_tile(const DevGroup& g, const KTensors& t, int lane, int wave, int (*wg_bounds)[8], NQTile* q) {
  int item, head_x;
  const int G = t.hq / t.hkv;
  if (!decode_wg(g, t.hkv, G * QSplitT<RG>::PARTS, &item, &head_x)) return false;
  const WorkItem w = plan_load(g.items, item);
  const QSplitT<RG> sp(uni(w.tile), uni(w.blk_len), head_x, G, wave);
  q->head = uni(sp.head);
  q->hk = head_x / (G * QSplitT<RG>::PARTS);
  q->unit = uni(w.unit); q->e0 = uni(w.e0); q->e1 = uni(w.e1);
  q->blk_start = uni(w.blk_start); q->qoff = uni(w.moff);
  q->row0 = sp.row0;
  q->n_rows = min(sp.rows, uni(w.blk_len) - q->row0);
  if (q->n_rows <= 0) return false;
  q->q_lo = q->blk_start + q->row0; q->q_hi = q->q_lo + q->n_rows - 1;
  q->wrow0 = uni(sp.wrow0);
  q->w_rows = max(0, min(32, q->n_rows - q->wrow0));
  q->wq_lo = q->q_lo + q->wrow0; q->wq_hi = q->wq_lo + q->w_rows - 1;
  const int r = q->wrow0 + (lane & 31);
  q->qv = r < q->n_rows;
  q->qi = q->q_lo + min(r, q->n_rows - 1);
  q->qr = make_int4(0, 0, 0, 0);
  q->wrb.init();
  q->rb.init();
  if (RANGES) {
    q->qr = unit_range_row(t, g, q->unit, q->qi);
    if (q->qv) q->wrb.add(q->qr);
    q->wrb.wave_reduce<32>();
    q->rb = q->wrb;
    if (sp.rows > 32) {   // the waves have different rows
      if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 2; k++) {
          wg_bounds[wave][4 * k] = q->wrb.lo_min[k]; wg_bounds[wave][4 * k + 1] = q->wrb.lo_max[k];
          wg_bounds[wave][4 * k + 2] = q->wrb.hi_min[k]; wg_bounds[wave][4 * k + 3] = q->wrb.hi_max[k];
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 2; k++) {
        for (int x = 0; x < RG; x++) {
          q->rb.lo_min[k] = min(q->rb.lo_min[k], wg_bounds[x][4 * k]); q->rb.lo_max[k] = max(q->rb.lo_max[k], wg_bounds[x][4 * k + 1]);
          q->rb.hi_min[k] = min(q->rb.hi_min[k], wg_bounds[x][4 * k + 2]); q->rb.hi_max[k] = max(q->rb.hi_max[k], wg_bounds[x][4 * k + 3]);
        }
        q->rb.lo_min[k] = uni(q->rb.lo_min[k]); q->rb.lo_max[k] = uni(q->rb.lo_max[k]);
        q->rb.hi_min[k] = uni(q->rb.hi_min[k]); q->rb.hi_max[k] = uni(q->rb.hi_max[k]);
      }
    }
  }
  return true;
}

// row r of the wave, for the functions of nonfinite.h
__device__ __forceinline__ FixRow fix_row(const NQTile& q, int r) {
  return {q.wq_lo + r, q.e0, q.e1,
          make_int4(__builtin_amdgcn_readlane(q.qr.x, r), __builtin_amdgcn_readlane(q.qr.y, r), __builtin_amdgcn_readlane(q.qr.z, r),
                    __builtin_amdgcn_readlane(q.qr.w, r))};
}

__device__ __forceinline__ void n_mask(f32x16& s, const NQTile& q, int kind, int ks32, int c0, int c1, int lane) {
  const RowRanges rr = row_ranges(kind, q.qi, c0, c1, q.qr);
  const int kb = ks32 + 4 * (lane >> 5);
#pragma unroll
  for (int r = 0; r < 16; r++)
    if (!rr.sees(kb + 8 * (r / 4) + (r % 4))) s[r] = -INFINITY;
}

}  // namespace
}  // namespace dcp
