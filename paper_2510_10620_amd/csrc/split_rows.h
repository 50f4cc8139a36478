// Workgroups that split the other side: their waves own the SAME 32 rows (queries in the forward and dQ, keys in dK/dV), take
// every NW-th 32-row tile of the other side (NW = 4 or 8 waves) and meet once, in LDS, at the end (kernels_mfma_f32.hip, eight waves and
// 32 or 16 rows; kernels_mfma_split.hip).
#pragma once
#include "device_utils.h"
#include "mfma_common.h"
#include "nonfinite.h"

namespace dcp {
namespace {

constexpr int kSplitWaves = kSplitThreads / 64;
constexpr int kSplitRows = 32;   // rows of a workgroup, and of a tile of the other side

// The lane number, opaque: what is derived from it is recomputed where it is used instead of being kept in registers.
__device__ __forceinline__ int fresh_lane() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}

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

// The wave's (query head, 32-query tile) pairs of a KV unit's table rows, dealt by tile number and head; 64 tiles of a block at a
// time, those that see none of the keys [k_lo, k_end) left out.  All state is wave-uniform.
template <int NW, bool RANGES>
struct QWalk {
  const int4* rec;
  const int4* qbounds;
  int e, e_end, wave, G, hh, base, n_t, q0, q1, kind, moff, t32, jt;
  uint64_t sees, all, todo;   // of the 64 tiles from `base` on: may see a key, every row sees every key; left of the current head
  __device__ QWalk(const DevGroup& g, int e0, int e1, int G_, int wave_, const int32_t* qb)
      : rec((const int4*)g.ent_rec), qbounds((const int4*)qb) {
    e = e0 - 1; e_end = e1; wave = wave_; G = G_; hh = G_ - 1; base = n_t = q0 = q1 = kind = moff = t32 = jt = 0; sees = all = todo = 0;
  }
  __device__ __forceinline__ int qs() const { return q0 + kSplitRows * jt; }
  __device__ __forceinline__ bool next(int k_lo, int k_end) {
    while (!todo) {
      if (++hh >= G) {
        hh = 0;
        base += 64;
        if (base >= n_t) {
          if (++e >= e_end) return false;
          const int4 r = plan_load(rec, 2 * e);
          q0 = uni(r.x); q1 = q0 + uni(r.y); kind = uni(r.z); moff = uni(r.w); t32 = uni(plan_load(rec, 2 * e + 1).x);
          n_t = (q1 - q0 + kSplitRows - 1) / kSplitRows;
          base = 0;
        }
        const int n = min(64, n_t - base);
        const uint64_t there = n >= 64 ? ~0ull : (1ull << n) - 1ull;
        if (RANGES && kind == 2) {
          const int lane = fresh_lane();
          bool see = false, every = false;
          if (lane < n) {
            const int4 a = qbounds[2 * (int64_t)(t32 + base + lane)], b = qbounds[2 * (int64_t)(t32 + base + lane) + 1];
            see = (k_lo < a.w && k_end > a.x) || (k_lo < b.w && k_end > b.x);           // RangeBounds::may_see
            every = (k_lo >= a.y && k_end <= a.z) || (k_lo >= b.y && k_end <= b.z);     // RangeBounds::all_see
          }
          sees = __ballot(see);
          all = __ballot(every);
        } else {
          const int first = kind == 1 ? max(0, (k_lo - q0) / kSplitRows - base) : 0;   // earlier tiles end before the first key
          sees = first >= 64 ? 0ull : there & (~0ull << first);
        }
      }
      todo = sees & ((NW == 8 ? 0x0101010101010101ull : 0x1111111111111111ull) << ((wave - t32 - hh) & (NW - 1)));
    }
    const int b = __builtin_ctzll(todo);
    todo &= todo - 1;
    jt = base + b;
    return true;
  }
  // every pair of the current tile and the keys [.., k_hi] (all kSplitRows of them there) is visible
  __device__ __forceinline__ bool full(int k_hi) const {
    return qs() + kSplitRows <= q1 && (kind == 0 || (kind == 1 && qs() >= k_hi) || (RANGES && kind == 2 && (all >> (jt & 63) & 1)));
  }
};

// What the query-side kernels know about their rows.
struct QTile {
  int head, hk, blk_start, row0, n_rows, q_lo, q_hi, qoff, qi, e0, e1, unit;
  int4 qr;
  RangeBounds rb;
};

// R: rows of the workgroup, which are the lanes' own rows modulo R
template <int R, bool RANGES>
__device__ __forceinline__ bool q_tile(const DevGroup& g, const KTensors& t, int lane, int bid, QTile* q) {
  constexpr int SUB = kItemRows / R;
  int item, x;
  const int G = t.hq / t.hkv;
  if (!decode_wg(g, t.hkv, G * SUB, &item, &x, bid)) return false;
  q->hk = x / (G * SUB);
  q->head = q->hk * G + (x % (G * SUB)) / SUB;
  WorkItem w = plan_load(g.items, item);
  q->unit = uni(w.unit); q->e0 = uni(w.e0); q->e1 = uni(w.e1);
  q->blk_start = uni(w.blk_start); q->qoff = uni(w.moff);
  q->row0 = uni(w.tile) * (kItemRows) + (x % SUB) * R;
  q->n_rows = min(R, uni(w.blk_len) - q->row0);
  if (q->n_rows <= 0) return false;
  q->q_lo = q->blk_start + q->row0;
  q->q_hi = q->q_lo + q->n_rows - 1;
  q->qi = q->q_lo + min(lane % R, q->n_rows - 1);
  q->qr = make_int4(0, 0, 0, 0);
  q->rb.init();
  if (RANGES) {
    q->qr = unit_range_row(t, g, q->unit, q->qi);
    q->rb.add(q->qr);
    q->rb.wave_reduce<R>();
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
