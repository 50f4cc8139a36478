// Blockwise attention forward on bf16 MFMA (Listing 1 line 5 + the in-kernel part of line 6).
//
// One workgroup (4 waves of 32 rows) owns 128 / HP query rows of HP = 1, 2 or 4 query heads of one KV head (QSplit)
// and walks the KV tiles (64 keys) of every table row of its output unit.  Scores are computed transposed,
// S^T = K Q^T, so that a lane owns one query column: the running max / sum are per-lane scalars,
// the only cross-lane step is one exchange between the two wave halves per 32 keys, and P^T in the
// MFMA accumulator layout is directly the B operand of O^T += V^T P^T.  K and V tiles are copied
// global -> LDS asynchronously one tile ahead into the other of two buffers; V^T fragments come
// from transposing LDS reads.  A 64-key tile that is fully visible to the wave takes a path with two
// independent score chains; tiles on a mask edge are handled per 32 keys with the per-element test.
#include "mfma_common.h"

namespace dcp {

static constexpr float kLazy = 8.f;  // rescale threshold, log2 units

static constexpr int kFwdWaves = 4;   // waves per workgroup; the step's inline tile copies and QSplit are written for four

// NQ: 32-query tiles per wave, which is 1 (QSplit).  It stays a parameter for the instruction schedule alone: with plain
// members in place of arrays of one, the variant for per-token ranges took 8.59 instead of 7.94 ms when this was measured
// (a 4 096-token window over 131 072 tokens; causal blockwise 2.66 and 2.75, the other variant the same).  Scalars that the two
// variants park in vector lanes: 14 with ranges, 24 without.
template <int NQ>
struct FwdState {
  bf16x8 qf[NQ][8];
  f32x16 o[NQ][4];
  float m[NQ], l[NQ];
  int qi[NQ];
  int4 qr[NQ];
  FragAddr fa;
  TileDmaT<16 / kFwdWaves> dmak, dmav;
};

// Scores of one 32-key sub-tile, S^T = K Q^T (one chain of 8 MFMAs), with the per-element mask test if MASK.
template <int NQ>
__device__ __forceinline__ void fwd_scores32(const FwdState<NQ>& st, const char* k_lds, int kt, int ks32, int kind, int c0,
                                             int c1, int lane, bool MASK, f32x16 (&s)[NQ]) {
  const int lh = lane >> 5;
#pragma unroll
  for (int nq = 0; nq < NQ; nq++)
#pragma unroll
    for (int r = 0; r < 16; r++) s[nq][r] = 0.f;
#pragma unroll
  for (int ksd = 0; ksd < 8; ksd++) {
    const bf16x8 a = frag_rm(k_lds, st.fa, 32 * kt, ksd);
#pragma unroll
    for (int nq = 0; nq < NQ; nq++) s[nq] = mfma(a, st.qf[nq][ksd], s[nq]);
  }
  if (MASK) {
#pragma unroll
    for (int nq = 0; nq < NQ; nq++) {
      const RowRanges rr = row_ranges(kind, st.qi[nq], c0, c1, st.qr[nq]);
      const int kb = ks32 + 4 * lh;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int key = kb + 8 * (r / 4) + (r % 4);
        if (!rr.sees(key)) s[nq][r] = -INFINITY;
      }
    }
  }
}

// Scores of a whole 64-key tile every pair of which is visible to the wave: the two 32-key score tiles are two
// independent MFMA chains, K fragments requested four k-steps ahead of the MFMAs that use them.
// DMA: the eight copy instructions of the next K and V tiles are issued here, one per k-step between the MFMAs
// (kb / vb: the tiles' first rows, lk / lv: the wave's part of the LDS stage they go to).
template <int NQ, bool DMA>
__device__ __forceinline__ void fwd_scores64(const FwdState<NQ>& st, const char* k_lds, f32x16 (&s)[2][NQ],
                                             const void* kb = nullptr, const void* vb = nullptr, unsigned lk = 0, unsigned lv = 0) {
#pragma unroll
  for (int kt = 0; kt < 2; kt++)
#pragma unroll
    for (int nq = 0; nq < NQ; nq++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[kt][nq][r] = 0.f;
  constexpr int PF = 4;
  bf16x8 ka[8][2];
#pragma unroll
  for (int ksd = 0; ksd < PF; ksd++)
#pragma unroll
    for (int kt = 0; kt < 2; kt++) ka[ksd][kt] = frag_rm(k_lds, st.fa, 32 * kt, ksd);
#pragma unroll
  for (int ksd = 0; ksd < 8; ksd++) {
    __builtin_amdgcn_sched_barrier(0);
    if (DMA) {
      if (ksd < 4) st.dmak.issue(ksd, kb, lk);
      else st.dmav.issue(ksd - 4, vb, lv);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (ksd + PF < 8) {
#pragma unroll
      for (int kt = 0; kt < 2; kt++) ka[ksd + PF][kt] = frag_rm(k_lds, st.fa, 32 * kt, ksd + PF);
    }
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
#pragma unroll
      for (int nq = 0; nq < NQ; nq++) s[kt][nq] = mfma(ka[ksd][kt], st.qf[nq][ksd], s[kt][nq]);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Online softmax over the 64 keys of a tile and O^T += V^T P^T.  This is the only code that touches the output
// accumulators: every kind of tile (fully visible, mask edge, half skipped) computes its scores on its own path and
// joins here, so the accumulators never meet at a control-flow merge with different register assignments (which
// costs a copy of all 64 of them, there and back, per tile).  For tables with per-token ranges this form
// replaced one with a section per kind of tile, 9 984 -> 9 814 us forward and backward in the case named at KvIter::next.
// One straight block, in which the P.V
// MFMAs of the first 32 keys are issued between the exponentials of the second 32 (the scheduling groups below say
// so; exponentials are their own instruction class there).  NQ = 1.  v0_lds, v1_lds: the V rows of the first and second 32 keys.
// two: the second 32 keys have weights other than 0.  A skipped half has scores -inf, so P = 0; without ranges (two = true) its MFMAs
// run all the same and add nothing, with ranges the seen half comes first and the other's are left out: 0 x V would make NaN of
// an Inf in rows that nothing sees, and blocks of 16 and 32 keys are half a tile each (6 174 tokens, 32/8 heads, blocks of 16, a window of
// 812: 1 409 -> 1 332 us, 1 243 with a section per kind of tile).
template <int NQ>
__device__ __forceinline__ void fwd_softmax_pv(FwdState<NQ>& st, f32x16 (&s)[2][NQ], const char* v0_lds, const char* v1_lds, float c_log2, bool two) {
  static_assert(NQ == 1, "one query per lane");
  bf16x8 va[4];
#pragma unroll
  for (int dt = 0; dt < 4; dt++) va[dt] = frag_tr(v0_lds, st.fa, 0, dt);
  __builtin_amdgcn_sched_barrier(0);
  float mx = fmaxf(fmaxf(s[0][0][0], s[0][0][1]), s[1][0][0]);
  mx = fmaxf(mx, s[1][0][1]);
#pragma unroll
  for (int r = 2; r < 16; r += 2) {
    mx = fmaxf(fmaxf(mx, s[0][0][r]), s[0][0][r + 1]);
    mx = fmaxf(fmaxf(mx, s[1][0][r]), s[1][0][r + 1]);
  }
  mx = xhalf_max(mx);
  // The reference max m is raised only when the tile's max exceeds it by more than 2^kLazy (in the exp2 domain): until then
  // P = exp2(c (s - m)) stays below 2^kLazy, exact in fp32 and bf16 range, and the accumulators need no rescaling.  O and l are
  // divided by the same sum at the end, so the result does not depend on which m was used.  A row that has seen no key yet keeps
  // m = -inf and uses 0.
  const bool raise = (mx - st.m[0]) * c_log2 > kLazy;
  const float m_new = raise ? mx : st.m[0];
  const float m_use = m_new == -INFINITY ? 0.f : m_new;
  const float mc = m_use * c_log2;
  if (__any(raise)) {
    const float alpha = raise ? __builtin_amdgcn_exp2f((st.m[0] - m_use) * c_log2) : 1.f;
    st.l[0] *= alpha;
#pragma unroll
    for (int dt = 0; dt < 4; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) st.o[0][dt][r] *= alpha;
  }
  st.m[0] = m_new;
  // first 32 keys
  float sum0 = 0.f;
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const float e = __builtin_amdgcn_exp2f(fmaf(s[0][0][r], c_log2, -mc));
    s[0][0][r] = e;
    sum0 += e;
  }
  const bf16x8 p00 = pack_frag(s[0][0], 0), p01 = pack_frag(s[0][0], 1);
  __builtin_amdgcn_sched_barrier(0);
  // region: 8 MFMAs of the first 32 keys + the exponentials of the second 32, interleaved by the group barriers below
  bf16x8 vb[4], vc[4];
#pragma unroll
  for (int dt = 0; dt < 4; dt++) vb[dt] = frag_tr(v0_lds, st.fa, 16, dt);
#pragma unroll
  for (int dt = 0; dt < 4; dt++) st.o[0][dt] = mfma(va[dt], p00, st.o[0][dt]);
#pragma unroll
  for (int dt = 0; dt < 4; dt++) vc[dt] = frag_tr(v1_lds, st.fa, 0, dt);
#pragma unroll
  for (int dt = 0; dt < 4; dt++) st.o[0][dt] = mfma(vb[dt], p01, st.o[0][dt]);
  float sum1 = 0.f;
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const float e = __builtin_amdgcn_exp2f(fmaf(s[1][0][r], c_log2, -mc));
    s[1][0][r] = e;
    sum1 += e;
  }
#pragma unroll
  for (int i = 0; i < 8; i++) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // two LDS reads for the MFMAs to come
    __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);   // two exponentials
    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);   // their multiply-adds and the running sum
  }
  __builtin_amdgcn_sched_barrier(0);
  st.l[0] += sum0 + sum1;
  if (!two) return;
  const bf16x8 p10 = pack_frag(s[1][0], 0), p11 = pack_frag(s[1][0], 1);
#pragma unroll
  for (int dt = 0; dt < 4; dt++) vb[dt] = frag_tr(v1_lds, st.fa, 16, dt);
#pragma unroll
  for (int dt = 0; dt < 4; dt++) st.o[0][dt] = mfma(vc[dt], p10, st.o[0][dt]);
#pragma unroll
  for (int dt = 0; dt < 4; dt++) st.o[0][dt] = mfma(vb[dt], p11, st.o[0][dt]);
}

// RANGES = false: the table has no row with per-token ranges (RANGES or WINDOW) and every use of them folds away.
template <int NQ, bool RANGES>
__global__ __launch_bounds__(64 * kFwdWaves, 2) void mfma_fwd_kernel(DevGroup g, KTensors t) {
  static_assert(NQ == 1, "a wave has 32 rows");
  if (!RANGES) t.masked = 0;
  // two stages, each [K tile | V tile]
  __shared__ __attribute__((aligned(1024))) char stage0[2 * kTileBytes];
  __shared__ __attribute__((aligned(1024))) char stage1[2 * kTileBytes];
  __shared__ int wg_bounds[kFwdWaves][8];

  int item, head_x;
  const int G = t.hq / t.hkv;
  if (!decode_wg(g, t.hkv, G, &item, &head_x)) return;
  const int hk = head_x / G;
  WorkItem w = plan_load(g.items, item);
  w.unit = uni(w.unit); w.tile = uni(w.tile); w.e0 = uni(w.e0); w.e1 = uni(w.e1);
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const int blk_start = uni(w.blk_start), blk_len = uni(w.blk_len);
  const int qoff = uni(w.moff);                       // rows of the Q-type buffers: packed index + qoff
  const QSplit sp(w.tile, blk_len, head_x, G, wave);
  const int head = uni(sp.head), row0 = sp.row0;      // first row of the workgroup inside the block
  const int n_rows = min(sp.rows, blk_len - row0);    // its valid rows
  if (n_rows <= 0) return;
  const int q_lo = blk_start + row0, q_hi = q_lo + n_rows - 1;
  const int wrow0 = uni(sp.wrow0);                    // wave's first row inside the tile
  const int w_rows = max(0, min(32, n_rows - wrow0)); // wave's valid rows
  const int wq_lo = q_lo + wrow0, wq_hi = wq_lo + w_rows - 1;

  FwdState<NQ> st;
  st.fa.init(lane);
  st.dmak.init(wave, lane, t.k_st);
  st.dmav.init(wave, lane, t.v_st);
  bool qv[NQ];
  RangeBounds wrb;
  wrb.init();
#pragma unroll
  for (int nq = 0; nq < NQ; nq++) {
    const int r = wrow0 + nq * 32 + li;
    qv[nq] = r < n_rows;
    st.qi[nq] = q_lo + min(r, n_rows - 1);
    st.qr[nq] = make_int4(0, 0, 0, 0);
    if (RANGES) st.qr[nq] = unit_range_row(t, g, w.unit, st.qi[nq]);
    // Q fragments (B operand: lane = query column li, d = 16 ks + 8 lh ..)
    const bf16_t* qp = (const bf16_t*)t.q + (int64_t)(st.qi[nq] + qoff) * t.q_st + (int64_t)head * t.q_sh + 8 * lh;
#pragma unroll
    for (int ks = 0; ks < 8; ks++) st.qf[nq][ks] = as_frag(*(const uint4*)(qp + 16 * ks));
    if (RANGES && qv[nq]) wrb.add(st.qr[nq]);
  }
  RangeBounds rb = wrb;  // workgroup bounds
  if (RANGES) {
    wrb.wave_reduce<32>();
    rb = wrb;
    if (sp.rows > 32) {   // the waves have different rows
      if (lane == 0) {
        wg_bounds[wave][0] = wrb.lo_min[0]; wg_bounds[wave][1] = wrb.lo_max[0]; wg_bounds[wave][2] = wrb.hi_min[0]; wg_bounds[wave][3] = wrb.hi_max[0];
        wg_bounds[wave][4] = wrb.lo_min[1]; wg_bounds[wave][5] = wrb.lo_max[1]; wg_bounds[wave][6] = wrb.hi_min[1]; wg_bounds[wave][7] = wrb.hi_max[1];
      }
      __syncthreads();
      rb.init();
      for (int x = 0; x < kFwdWaves; x++) {
        rb.lo_min[0] = min(rb.lo_min[0], wg_bounds[x][0]); rb.lo_max[0] = max(rb.lo_max[0], wg_bounds[x][1]);
        rb.hi_min[0] = min(rb.hi_min[0], wg_bounds[x][2]); rb.hi_max[0] = max(rb.hi_max[0], wg_bounds[x][3]);
        rb.lo_min[1] = min(rb.lo_min[1], wg_bounds[x][4]); rb.lo_max[1] = max(rb.lo_max[1], wg_bounds[x][5]);
        rb.hi_min[1] = min(rb.hi_min[1], wg_bounds[x][6]); rb.hi_max[1] = max(rb.hi_max[1], wg_bounds[x][7]);
      }
#pragma unroll
      for (int k = 0; k < 2; k++) {
        rb.lo_min[k] = uni(rb.lo_min[k]); rb.lo_max[k] = uni(rb.lo_max[k]); rb.hi_min[k] = uni(rb.hi_min[k]); rb.hi_max[k] = uni(rb.hi_max[k]);
      }
    }
  }

#pragma unroll
  for (int nq = 0; nq < NQ; nq++) {
    st.m[nq] = -INFINITY; st.l[nq] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) st.o[nq][dt][r] = 0.f;
  }
  const float c_log2 = t.scale * 1.44269504088896340736f;
  const bf16_t* kbase = (const bf16_t*)t.k + (int64_t)hk * t.k_sh;
  const bf16_t* vbase = (const bf16_t*)t.v + (int64_t)hk * t.v_sh;

  KvIter it(g, w.e0, w.e1);
  bool have = it.next<RANGES>(q_hi, rb);
  if (have) {
    st.dmak.load(stage0, kbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
    st.dmav.load(stage0 + kTileBytes, vbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
  }
  DCP_WAIT_VMCNT(0);
  __syncthreads();

  // one pipeline step: prefetch the next tile into `nxt`, compute the current one from `cur`
  auto step = [&](const char* cur, char* nxt) {
    const int ks = it.ks, c0 = it.c0, c1 = it.c1, kind = RANGES ? it.kind : (it.kind & 1);
    // the score paths join in one softmax + PV section (4 % faster: no copies of the accumulators at the merge)
    f32x16 s[2][NQ];
    bool pv;
    const char* v0 = cur + kTileBytes;   // V of the first and the second 32 keys
    const char* v1 = v0 + 32 * kRowBytes;
    bool two = true;
    const bool common = !RANGES || kind < 2 ? ks + 2 * kTN <= (kind ? min(c1, wq_lo + 1) : c1)
                                            : ks + 2 * kTN <= c1 && wrb.all_see(ks, ks + 2 * kTN);
    if (w_rows > 0 && common) {
      // The common step, found with a handful of scalar instructions: this tile and the next one of the same table
      // row are whole and visible to every row of the wave.  The iterator moves by one tile, nothing is classified,
      // and the copies of the next tile are issued between the score MFMAs: issued back to back at the top of the
      // step, the copy instructions of the four waves queue behind one another at the address unit and the waves
      // issue nothing else meanwhile; the general path's scalar bookkeeping costs some hundred issue slots more.
      it.jt++;
      it.ks += kTN;
      fwd_scores64<NQ, true>(st, cur, s, uni_ptr((const char*)kbase + (int64_t)(it.ks + it.moff) * st.dmak.sb),
                             uni_ptr((const char*)vbase + (int64_t)(it.ks + it.moff) * st.dmav.sb),
                             st.dmak.lds_of(nxt, wave), st.dmav.lds_of(nxt + kTileBytes, wave));
      pv = true;
    } else {
      have = it.next<RANGES>(q_hi, rb);
      if (have) {
        st.dmak.load(nxt, kbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
        st.dmav.load(nxt + kTileBytes, vbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
      }
      const int cls0 = w_rows > 0 ? classify32(kind, ks, c1, wq_lo, wq_hi, wrb) : kSkip;
      const int cls1 = w_rows > 0 ? classify32(kind, ks + 32, c1, wq_lo, wq_hi, wrb) : kSkip;
      pv = cls0 != kSkip || cls1 != kSkip;
      if (cls0 == kFull && cls1 == kFull) {
        fwd_scores64<NQ, false>(st, cur, s);
      } else if (pv) {
        if constexpr (RANGES) {   // the half that is seen comes first, and the other one's V rows meet nothing
          const int first = cls0 != kSkip ? 0 : 1;
          two = cls0 != kSkip && cls1 != kSkip;
          v0 += first * 32 * kRowBytes;
          fwd_scores32<NQ>(st, cur + first * 32 * kRowBytes, 0, ks + 32 * first, kind, c0, c1, lane, (first ? cls1 : cls0) == kPartial, s[0]);
          if (two) {
            fwd_scores32<NQ>(st, cur, 1, ks + 32, kind, c0, c1, lane, cls1 == kPartial, s[1]);
          } else {
#pragma unroll
            for (int r = 0; r < 16; r++) s[1][0][r] = -INFINITY;
          }
        } else {
#pragma unroll
          for (int kt = 0; kt < 2; kt++) {
            const int cls = kt ? cls1 : cls0;
            if (cls != kSkip) {
              fwd_scores32<NQ>(st, cur, kt, ks + 32 * kt, kind, c0, c1, lane, cls == kPartial, s[kt]);
            } else {
#pragma unroll
              for (int nq = 0; nq < NQ; nq++)
#pragma unroll
                for (int r = 0; r < 16; r++) s[kt][nq][r] = -INFINITY;
            }
          }
        }
      }
    }
    if (pv) fwd_softmax_pv<NQ>(st, s, v0, v1, c_log2, !RANGES || two);
    DCP_WAIT_VMCNT(0);
    __syncthreads();  // the copy into `nxt` has landed and `cur` may be overwritten
  };
  while (have) {
    step(stage0, stage1);
    if (!have) break;
    step(stage1, stage0);
  }

  // ---- epilogue: O = acc / l, LSE = ln2 * (m c + log2 l); the output tile goes out in whole rows (the tile stages
  // are free after the last step's barrier, two waves stage in each)
  static_assert(2 * 32 * kORow <= 2 * kTileBytes, "two waves stage their output tiles in one tile stage");
  char* ot = (wave < 2 ? stage0 : stage1) + (wave & 1) * (32 * kORow);
  const int slot = plan_load(g.unit_out, w.unit);
#pragma unroll
  for (int nq = 0; nq < NQ; nq++) {
    const float lt = xhalf_sum(st.l[nq]);
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const float lse = lt > 0.f ? (st.m[nq] * c_log2 + __builtin_amdgcn_logf(lt)) * 0.69314718055994530942f : -INFINITY;
    const int brow0 = row0 + wrow0 + nq * 32;   // the wave's first row inside the block
    if (qv[nq] && lh == 0) {
      if (slot < 0) t.lse[(int64_t)head * t.q_rows + blk_start + brow0 + li + qoff] = lse;
      else t.lse[((int64_t)slot * t.hq + head) * t.block_size + brow0 + li] = lse;
    }
    bf16_t* op = slot < 0 ? (bf16_t*)t.out + (int64_t)(blk_start + brow0 + qoff) * t.o_st + (int64_t)head * t.o_sh
                          : (bf16_t*)t.out + (((int64_t)slot * t.block_size + brow0) * t.hq + head) * kD;
    store_tile32(ot, st.o[nq], inv, lane, n_rows - wrow0 - nq * 32, op, slot < 0 ? t.o_st : (int64_t)t.hq * kD);
  }
}

bool mfma_supports(int32_t dtype, int32_t d) { return (dtype == DCP_BF16 || dtype == DCP_F32) && (d == 32 || d == 64 || d == 128); }

dcp_status_t mfma_fwd(const DevGroup& g, const KTensors& t, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  if (t.dtype == DCP_F32) return t.part_groups ? mfma_f32_parts_fwd(g, t, s) : mfma_f32_fwd(g, t, 32, s);
  if (t.d != kD) return mfma_narrow_fwd(g, t, s);
  const int grid = xcd_grid(g, t.hkv, t.hq / t.hkv);
  if (t.masked) hipLaunchKernelGGL((mfma_fwd_kernel<1, true>), dim3(grid), dim3(64 * kFwdWaves), 0, s, g, t);
  else hipLaunchKernelGGL((mfma_fwd_kernel<1, false>), dim3(grid), dim3(64 * kFwdWaves), 0, s, g, t);
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

}  // namespace dcp
