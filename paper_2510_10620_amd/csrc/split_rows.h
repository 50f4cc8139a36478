// Workgroups that split the other side: their waves own the SAME 32 rows (queries in the forward and dQ, keys in dK/dV), take
// every eighth 32-row tile of the other side and meet once, in LDS, at the end (kernels_mfma_f32.hip, kernels_mfma_split.hip).
#pragma once
#include "device_utils.h"
#include "mfma_common.h"
#include "nonfinite.h"

namespace dcp {
namespace {

constexpr int kSplitWaves = kSplitThreads / 64;
constexpr int kSplitRows = 32;   // rows of a workgroup, and of a tile of the other side

// row of accumulator register r in a 32-row tile, without the lane's 4h
__device__ __forceinline__ constexpr int acc_row(int r) { return 8 * (r / 4) + r % 4; }

// The wave's tiles of a unit's table rows: 32-row tiles of the other side's blocks, numbered through the whole batch
// (t32), so that tile number mod NW deals them evenly to the NW waves whatever the block size.
template <int NW>
struct Walk {
  const int4* rec;
  int e, e_end, wave;
  int c0, c1, kind, moff, t32, lim, jt;
  __device__ Walk(const DevGroup& g, int e0, int e1, int wave_) : rec((const int4*)g.ent_rec) {
    e = e0 - 1; e_end = e1; wave = wave_; c0 = c1 = kind = moff = t32 = lim = 0; jt = 0;
  }
  __device__ __forceinline__ int ks() const { return c0 + kSplitRows * jt; }
  template <bool RANGES>
  __device__ __forceinline__ bool next(int q_hi, const RangeBounds& rb) {
    for (;;) {
      jt += NW;
      while (c0 + kSplitRows * jt >= lim) {
        if (++e >= e_end) return false;
        const int4 r = plan_load(rec, 2 * e);
        c0 = uni(r.x); c1 = c0 + uni(r.y); kind = uni(r.z); moff = uni(r.w);
        t32 = uni(plan_load(rec, 2 * e + 1).x);
        lim = kind == 1 ? min(c1, q_hi + 1) : c1;
        jt = (wave - t32) & (NW - 1);
      }
      if (!RANGES || kind != 2 || rb.may_see(ks(), min(ks() + kSplitRows, c1))) return true;
    }
  }
};

// What the query-side kernels know about their rows.
struct QTile {
  int head, hk, blk_start, row0, n_rows, q_lo, q_hi, qoff, qi, e0, e1, unit;
  int4 qr;
  RangeBounds rb;
};

template <bool RANGES>
__device__ __forceinline__ bool q_tile(const DevGroup& g, const KTensors& t, int lane, int bid, QTile* q) {
  int item, x;
  const int G = t.hq / t.hkv;
  if (!decode_wg(g, t.hkv, G * kSplitSub, &item, &x, bid)) return false;
  q->hk = x / (G * kSplitSub);
  q->head = q->hk * G + (x % (G * kSplitSub)) / kSplitSub;
  WorkItem w = plan_load(g.items, item);
  q->unit = uni(w.unit); q->e0 = uni(w.e0); q->e1 = uni(w.e1);
  q->blk_start = uni(w.blk_start); q->qoff = uni(w.moff);
  q->row0 = uni(w.tile) * (kSplitSub * kSplitRows) + (x % kSplitSub) * kSplitRows;
  q->n_rows = min(kSplitRows, uni(w.blk_len) - q->row0);
  if (q->n_rows <= 0) return false;
  q->q_lo = q->blk_start + q->row0;
  q->q_hi = q->q_lo + q->n_rows - 1;
  q->qi = q->q_lo + min(lane & 31, q->n_rows - 1);
  q->qr = make_int4(0, 0, 0, 0);
  q->rb.init();
  if (RANGES) {
    q->qr = range_row(t, q->qi, uni(plan_load(g.blk_s0, plan_load(g.unit_blk, q->unit))));
    q->rb.add(q->qr);
    q->rb.wave_reduce();
#pragma unroll
    for (int k = 0; k < 2; k++) {
      q->rb.lo_min[k] = uni(q->rb.lo_min[k]); q->rb.lo_max[k] = uni(q->rb.lo_max[k]);
      q->rb.hi_min[k] = uni(q->rb.hi_min[k]); q->rb.hi_max[k] = uni(q->rb.hi_max[k]);
    }
  }
  return true;
}

__device__ __forceinline__ void mask_keys(f32x16& s, const QTile& q, int kind, int ks, int c0, int c1, int lane) {
  const RowRanges rr = row_ranges(kind, q.qi, c0, c1, q.qr);
  const int kb = ks + 4 * (lane >> 5);
#pragma unroll
  for (int r = 0; r < 16; r++)
    if (!rr.sees(kb + acc_row(r))) s[r] = -INFINITY;
}

// row r of the workgroup, for the functions of nonfinite.h
__device__ __forceinline__ FixRow fix_row(const QTile& q, int r) {
  return {q.q_lo + r, q.e0, q.e1,
          make_int4(__builtin_amdgcn_readlane(q.qr.x, r), __builtin_amdgcn_readlane(q.qr.y, r), __builtin_amdgcn_readlane(q.qr.z, r),
                    __builtin_amdgcn_readlane(q.qr.w, r))};
}

}  // namespace
}  // namespace dcp
