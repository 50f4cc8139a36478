// Blockwise attention, forward and backward, for bf16 tensors with narrow heads (D = 32, 64) on bf16 MFMA: the structure
// of the D = 128 kernels (transposed scores, 64-row LDS tiles copied one ahead, transposing reads, one workgroup of four
// waves x 32 rows per 128-row work item) with two differences.
//
//  * P and dS stay fp32 numbers: they go into the products over keys (queries) as three bf16 parts of 8 bits whose sum they
//    are, each part a product of its own with the same bf16 operand on the other side (8 x 8 bits, exact in fp32).  Two
//    rounded parts cost 17-19 % less time (16 384 causal tokens, 16/4 heads, D 64: forward 454 -> 545 us with the third, dQ
//    500 -> 600, dK/dV 1 047 -> 1 291) but leave 2^-18 of every weight, which the fp32 weights of the thread-per-row kernels
//    do not: their results were 1e-6 of the norm farther from a 64-bit reference, and far more where a sum cancels.
//  * Nothing is scheduled by hand: with D = 64 a workgroup needs a third of the registers and half the LDS of the D = 128
//    kernels, several are resident per CU, and their waves fill one another's waits.
//
// LDS tiles: tile_layout.h.
// Measured against one thread per row (16 384 causal tokens, 16/4 heads, D 64): forward 21.8 -> 0.54 ms, dQ 36.0 -> 0.60,
// dK/dV 76.8 -> 1.29 ms.  What bounds them on large batches is the MFMA rate that the chip holds on real data: counting
// the three parts of P and dS the three kernels execute 1 090, 1 128 and 950 TFLOP/s (65 536 causal tokens, log-normal).
#include "mfma_dkv_kernel.h"
#include "nonfinite.h"
#include "query_rows.h"
#include "tile_layout.h"

namespace dcp {

namespace {

constexpr float kLazyN = 8.f;   // the running maximum is raised when a tile exceeds it by more than 2^8

template <int D> using Narrow = TileLayout<D>;

// fragment addresses of a lane (see FragAddr): rows enter the swizzle through row % 16 only
template <int D>
struct NAddr {
  int rm[Narrow<D>::KS], tr[Narrow<D>::DT][2];
  __device__ __forceinline__ void init(int lane) {
    const int li = lane & 31, lh = lane >> 5, j = lane & 15, blk = lane >> 4, r0 = 4 * (blk >> 1) + (j >> 2);
#pragma unroll
    for (int ks = 0; ks < Narrow<D>::KS; ks++) rm[ks] = Narrow<D>::off(li, 2 * ks + lh);
#pragma unroll
    for (int dt = 0; dt < Narrow<D>::DT; dt++) {
      const int col = 32 * dt + 16 * (blk & 1) + 4 * (j & 3);
      tr[dt][0] = Narrow<D>::off(r0, col >> 3) + (col & 7) * 2;
      tr[dt][1] = Narrow<D>::off(r0 + 8, col >> 3) + (col & 7) * 2;
    }
  }
  __device__ __forceinline__ bf16x8 rows(const char* tile, int row0, int ks) const {
    return as_frag(*(const uint4*)(tile + row0 * Narrow<D>::kRow + rm[ks]));
  }
  __device__ __forceinline__ bf16x8 cols(const char* tile, int row0, int dt) const {
    typedef __attribute__((address_space(3))) s16x4* lds_p;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(tile + row0 * Narrow<D>::kRow + tr[dt][0]));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(tile + row0 * Narrow<D>::kRow + tr[dt][1]));
    s16x8 v;
    v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3]; v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
    return __builtin_bit_cast(bf16x8, v);
  }
};

// Asynchronous copy of a 64-row tile by NW waves (see TileDmaT): instruction u of wave w fills the lines
// 4 (w + NW u) .. + 3, whole multiples of 16 rows apart, so that they share the swizzle.
template <int D, int NW = 4>
struct NDma {
  static_assert(4 * NW * Narrow<D>::RPL % 16 == 0, "the rows of a wave's instructions share row % 16");
  static constexpr int PW = Narrow<D>::kBytes / 1024 / NW;
  unsigned off0;
  int sb, row, ch;
  __device__ __forceinline__ void init(int wave, int lane, int64_t stride_t) {
    sb = (int)stride_t * 2;
    const int line = 4 * wave + (lane >> 4), x = (lane & 15) ^ Narrow<D>::swz(line);
    row = line * Narrow<D>::RPL + x / Narrow<D>::CPR;
    ch = (x % Narrow<D>::CPR) * 16;
    off0 = (unsigned)(row * sb + ch);
  }
  __device__ __forceinline__ void load(char* tile, const bf16_t* base, int row_start, int row_last, int wave) const {
    const void* b = uni_ptr((const char*)base + (int64_t)row_start * sb);
    const unsigned l0 = lds_addr(tile) + wave * 1024;
    const int lim = row_last - row_start;
    constexpr int RU = 4 * NW * Narrow<D>::RPL;   // rows between a wave's instructions
#pragma unroll
    for (int u = 0; u < PW; u++) {
      if (lim >= kTN - 1) dma16(off0, (const char*)b + (int64_t)(RU * u) * sb, l0 + u * NW * 1024);
      else dma16((unsigned)(min(row + RU * u, lim) * sb + ch), b, l0 + u * NW * 1024);
    }
  }
};

// store_tile32 for D columns
template <int D>
__device__ __forceinline__ void store_rows32(char* ot, const f32x16 (&acc)[D / 32], float mul, int lane, int n_valid, bf16_t* row0_ptr,
                                             int64_t stride) {
  constexpr int OR = Narrow<D>::kORow, CPR = Narrow<D>::CPR;
  const int li = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      uint2 pk;
      pk.x = pack_bf16x2(acc[dt][4 * a] * mul, acc[dt][4 * a + 1] * mul);
      pk.y = pack_bf16x2(acc[dt][4 * a + 2] * mul, acc[dt][4 * a + 3] * mul);
      *(uint2*)(ot + li * OR + 2 * (32 * dt + 8 * a + 4 * lh)) = pk;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int i = 0; i < 32 * CPR / 64; i++) {
    const int r = i * (64 / CPR) + lane / CPR, c = lane % CPR;
    const uint4 piece = *(const uint4*)(ot + r * OR + 16 * c);
    if (r < n_valid) *(uint4*)(row0_ptr + (int64_t)r * stride + 8 * c) = piece;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Rows r < n_valid of a wave's D x 32 tile (lane = row) that hold a value which is not finite, as a bit mask.
template <int D>
__device__ __forceinline__ uint32_t rows_not_finite(const f32x16 (&acc)[D / 32], int n_valid) {
  float probe = 0.f;
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) probe = finite_probe(acc[dt][r], probe);
  const uint64_t bad = __ballot(probe != 0.f);
  return ((uint32_t)bad | (uint32_t)(bad >> 32)) & (n_valid < 32 ? (1u << n_valid) - 1u : 0xffffffffu);
}

template <int D>
__device__ __forceinline__ void load_own(bf16x8 (&f)[D / 16], const void* base, int64_t row, int64_t st, int64_t head_off, int lane) {
  const bf16_t* p = (const bf16_t*)base + row * st + head_off + 8 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) f[ks] = as_frag(*(const uint4*)(p + 16 * ks));
}

}  // namespace

template <int D, bool RANGES>
__global__ __launch_bounds__(kNarrowThreads, 4) void narrow_fwd_kernel(DevGroup g, KTensors t) {
  typedef Narrow<D> N;
  __shared__ __attribute__((aligned(1024))) char stages[4 * N::kBytes];   // two stages, each [K tile | V tile]
  __shared__ int wg_bounds[4][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), li = lane & 31, lh = lane >> 5;
  NQTile q;
  if (!nq_tile<RANGES>(g, t, lane, wave, wg_bounds, &q)) return;
  NAddr<D> fa;
  fa.init(lane);
  NDma<D> dmak, dmav;
  dmak.init(wave, lane, t.k_st);
  dmav.init(wave, lane, t.v_st);
  bf16x8 qf[N::KS];
  load_own<D>(qf, t.q, q.qi + q.qoff, t.q_st, (int64_t)q.head * t.q_sh, lane);
  f32x16 o[N::DT];
#pragma unroll
  for (int dt = 0; dt < N::DT; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[dt][r] = 0.f;
  float m = -INFINITY, l = 0.f;
  const float c_log2 = t.scale * kLog2e;
  const bf16_t* kbase = (const bf16_t*)t.k + (int64_t)q.hk * t.k_sh;
  const bf16_t* vbase = (const bf16_t*)t.v + (int64_t)q.hk * t.v_sh;
  KvIter it(g, q.e0, q.e1);
  bool have = it.next<RANGES>(q.q_hi, q.rb);
  auto issue = [&](char* stage) {
    dmak.load(stage, kbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
    dmav.load(stage + N::kBytes, vbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
  };
  if (have) issue(stages);
  DCP_WAIT_VMCNT(0);
  __syncthreads();
  int buf = 0;
  while (have) {
    const char* k_lds = stages + buf;
    const char* v_lds = k_lds + N::kBytes;
    const int ks = it.ks, c0 = it.c0, c1 = it.c1, kind = RANGES ? it.kind : (it.kind & 1);
    have = it.next<RANGES>(q.q_hi, q.rb);
    buf ^= 2 * N::kBytes;
    if (have) issue(stages + buf);
    int cls[2] = {kSkip, kSkip};
    if (q.w_rows > 0) {
      cls[0] = classify32(kind, ks, c1, q.wq_lo, q.wq_hi, q.wrb);
      cls[1] = classify32(kind, ks + 32, c1, q.wq_lo, q.wq_hi, q.wrb);
    }
    if (cls[0] != kSkip || cls[1] != kSkip) {
      f32x16 s[2];
#pragma unroll
      for (int kt = 0; kt < 2; kt++) {
#pragma unroll
        for (int r = 0; r < 16; r++) s[kt][r] = 0.f;
#pragma unroll
        for (int x = 0; x < N::KS; x++) s[kt] = mfma(fa.rows(k_lds, 32 * kt, x), qf[x], s[kt]);
      }
      if (cls[0] != kFull) n_mask(s[0], q, kind, ks, c0, c1, lane);        // a skipped half sees nothing under its mask
      if (cls[1] != kFull) n_mask(s[1], q, kind, ks + 32, c0, c1, lane);
      float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
      for (int r = 1; r < 16; r++) mx = fmaxf(fmaxf(mx, s[0][r]), s[1][r]);
      mx = xhalf_max(mx);
      const bool raise = (mx - m) * c_log2 > kLazyN;   // lazily, as in the D = 128 kernel
      const float m_new = raise ? mx : m;
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float mc = m_use * c_log2;
      if (__any(raise)) {
        const float alpha = raise ? __builtin_amdgcn_exp2f((m - m_use) * c_log2) : 1.f;
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < N::DT; dt++)
#pragma unroll
          for (int r = 0; r < 16; r++) o[dt][r] *= alpha;
      }
      m = m_new;
#pragma unroll
      for (int kt = 0; kt < 2; kt++) {
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          s[kt][r] = __builtin_amdgcn_exp2f(fmaf(s[kt][r], c_log2, -mc));
          sum += s[kt][r];
        }
        l += sum;
#pragma unroll
        for (int c = 0; c < 2; c++) {
          bf16x8 p[3];
          pack_split(s[kt], c, p);
#pragma unroll
          for (int dt = 0; dt < N::DT; dt++) {
            const bf16x8 v = fa.cols(v_lds, 32 * kt + 16 * c, dt);
#pragma unroll
            for (int k = 0; k < 3; k++) o[dt] = mfma(v, p[k], o[dt]);
          }
        }
      }
    }
    DCP_WAIT_VMCNT(0);
    __syncthreads();
  }
  char* ot = stages + wave * (32 * N::kORow);
  static_assert(4 * 32 * N::kORow <= 4 * N::kBytes, "the waves' output tiles fit in the stages");
  const int slot = plan_load(g.unit_out, q.unit);
  const float lt = xhalf_sum(l);
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  const float lse = lt > 0.f ? (m * c_log2 + __builtin_amdgcn_logf(lt)) * 0.69314718055994530942f : -INFINITY;
  const int brow0 = q.row0 + q.wrow0;
  if (q.qv && lh == 0) {
    if (slot < 0) t.lse[(int64_t)q.head * t.q_rows + q.blk_start + brow0 + li + q.qoff] = lse;
    else t.lse[((int64_t)slot * t.hq + q.head) * t.block_size + brow0 + li] = lse;
  }
  bf16_t* op = slot < 0 ? (bf16_t*)t.out + (int64_t)(q.blk_start + brow0 + q.qoff) * t.o_st + (int64_t)q.head * t.o_sh
                        : (bf16_t*)t.out + (((int64_t)slot * t.block_size + brow0) * t.hq + q.head) * D;
  const int64_t op_st = slot < 0 ? t.o_st : (int64_t)t.hq * D;
  uint32_t again = rows_not_finite<D>(o, q.w_rows);
  store_rows32<D>(ot, o, inv, lane, q.w_rows, op, op_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again);
      if (lane_of(lt, r) != lane_of(lt, r)) continue;   // a NaN score: all of the row is NaN already
      const FixRow f = fix_row(q, r);
      const float mr = lane_of(m, r);
      fix_out<bf16_t, D>(a.g, a.t, f, q.hk, (const bf16_t*)a.t.q + (int64_t)(f.qi + q.qoff) * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                         mr == -INFINITY ? 0.f : mr * c_log2, lane_of(inv, r), op + r * op_st);
    }
  }
}

template <int D, bool RANGES>
__global__ __launch_bounds__(kNarrowThreads, 3) void narrow_dq_kernel(DevGroup g, KTensors t) {
  typedef Narrow<D> N;
  __shared__ __attribute__((aligned(1024))) char stages[4 * N::kBytes];
  __shared__ int wg_bounds[4][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), lh = lane >> 5;
  NQTile q;
  if (!nq_tile<RANGES>(g, t, lane, wave, wg_bounds, &q)) return;
  NAddr<D> fa;
  fa.init(lane);
  NDma<D> dmak, dmav;
  dmak.init(wave, lane, t.k_st);
  dmav.init(wave, lane, t.v_st);
  bf16x8 qf[N::KS], dof[N::KS], of[N::KS];
  load_own<D>(qf, t.q, q.qi + q.qoff, t.q_st, (int64_t)q.head * t.q_sh, lane);
  load_own<D>(dof, t.dout, q.qi + q.qoff, t.do_st, (int64_t)q.head * t.do_sh, lane);
  load_own<D>(of, t.out_in, q.qi + q.qoff, t.o_st, (int64_t)q.head * t.o_sh, lane);
  // the backward preprocess, fused as in the D = 128 kernel
  float delta = 0.f;
#pragma unroll
  for (int x = 0; x < N::KS; x++)
#pragma unroll
    for (int e = 0; e < 8; e++) delta = fmaf((float)of[x][e], (float)dof[x][e], delta);
  delta = xhalf_sum(delta);
  const int64_t at = (int64_t)q.head * t.q_rows + q.qi + q.qoff;
  const float lse2 = row_lse2(t.lse[at], &delta);
  if (q.qv && lh == 0) { t.delta_w[at] = -delta; t.lse2_w[at] = lse2; }
  f32x16 dq[N::DT];
#pragma unroll
  for (int dt = 0; dt < N::DT; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) dq[dt][r] = 0.f;
  const float c_log2 = t.scale * kLog2e;
  const bf16_t* kbase = (const bf16_t*)t.k + (int64_t)q.hk * t.k_sh;
  const bf16_t* vbase = (const bf16_t*)t.v + (int64_t)q.hk * t.v_sh;
  KvIter it(g, q.e0, q.e1);
  bool have = it.next<RANGES>(q.q_hi, q.rb);
  auto issue = [&](char* stage) {
    dmak.load(stage, kbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
    dmav.load(stage + N::kBytes, vbase, it.ks + it.moff, it.c1 - 1 + it.moff, wave);
  };
  if (have) issue(stages);
  DCP_WAIT_VMCNT(0);
  __syncthreads();
  int buf = 0;
  while (have) {
    const char* k_lds = stages + buf;
    const char* v_lds = k_lds + N::kBytes;
    const int ks = it.ks, c0 = it.c0, c1 = it.c1, kind = RANGES ? it.kind : (it.kind & 1);
    have = it.next<RANGES>(q.q_hi, q.rb);
    buf ^= 2 * N::kBytes;
    if (have) issue(stages + buf);
#pragma unroll
    for (int kt = 0; kt < 2; kt++) {
      const int cls = q.w_rows > 0 ? classify32(kind, ks + 32 * kt, c1, q.wq_lo, q.wq_hi, q.wrb) : kSkip;
      if (cls == kSkip) continue;
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = -delta; }
#pragma unroll
      for (int x = 0; x < N::KS; x++) {
        s = mfma(fa.rows(k_lds, 32 * kt, x), qf[x], s);
        dp = mfma(fa.rows(v_lds, 32 * kt, x), dof[x], dp);
      }
      if (cls == kPartial) n_mask(s, q, kind, ks + 32 * kt, c0, c1, lane);
#pragma unroll
      for (int r = 0; r < 16; r++) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lse2)) * dp[r];
#pragma unroll
      for (int c = 0; c < 2; c++) {
        bf16x8 ds[3];
        pack_split(s, c, ds);
#pragma unroll
        for (int dt = 0; dt < N::DT; dt++) {
          const bf16x8 kc = fa.cols(k_lds, 32 * kt + 16 * c, dt);
#pragma unroll
          for (int k = 0; k < 3; k++) dq[dt] = mfma(kc, ds[k], dq[dt]);
        }
      }
    }
    DCP_WAIT_VMCNT(0);
    __syncthreads();
  }
  bf16_t* dqp = (bf16_t*)t.dq + (int64_t)(q.wq_lo + q.qoff) * t.dq_st + (int64_t)q.head * t.dq_sh;
  uint32_t again = rows_not_finite<D>(dq, q.w_rows);
  store_rows32<D>(stages + wave * (32 * N::kORow), dq, t.scale, lane, q.w_rows, dqp, t.dq_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again);
      const FixRow f = fix_row(q, r);
      const int64_t mem = f.qi + q.qoff;
      fix_dq<bf16_t, D>(a.g, a.t, f, q.hk, (const bf16_t*)a.t.q + mem * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                        (const bf16_t*)a.t.dout + mem * a.t.do_st + (int64_t)q.head * a.t.do_sh, lane_of(lse2, r), lane_of(delta, r), dqp + r * a.t.dq_st);
    }
  }
}

// A workgroup's eight waves are NG groups of KW waves: a wave has 32 keys, the groups own the same 128 keys and take the query
// tiles in turn, each with LDS stages of its own, and add their sums at the end.  It serves launches of many short items, whose
// start it shares among four waves' keys (1 000 sequences of 20 tokens, 8/2 heads, D 64: 73 us, 84 with 32 keys a workgroup); the
// others go to kernels_mfma_split.hip (65 536 tokens, 16/4 heads, D 64 / 32: 2.94 / 2.13 here and 2.87 / 1.79 ms there).
template <int D, bool RANGES>
__global__ __launch_bounds__(kNarrowDkvThreads, 2) void narrow_dkv_kernel(DevGroup g, KTensors t) {
  constexpr int KW = 4, NG = 2;
  typedef Narrow<D> N;
  // stage: Q tile, dO tile, then per query row lse2, -delta and ranges, and the range bounds of the tile's two halves
  constexpr int LSE = 2 * N::kBytes, DEL = LSE + 256, RNG = DEL + 256, BND = RNG + 1024, STAGE = BND + 1024;
  constexpr int kStage = RANGES ? STAGE : RNG;
  __shared__ __attribute__((aligned(1024))) char all_stages[2 * NG * kStage];
  int item, hk;
  if (!decode_wg(g, t.hkv, 1, &item, &hk)) return;
  const int G = t.hq / t.hkv;
  const WorkItem w = plan_load(g.items, item);
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6) % KW, group = uni(tid >> 6) / KW, li = lane & 31, lh = lane >> 5;
  char* stages = all_stages + group * (2 * kStage);
  const int koff = uni(w.moff), row0 = uni(w.tile) * 128, n_rows = min(128, uni(w.blk_len) - row0);
  const int seq0 = RANGES ? uni(plan_load(g.blk_s0, plan_load(g.unit_blk, uni(w.unit)))) : 0;
  const int k_lo = uni(w.blk_start) + row0, k_end = k_lo + n_rows, wrow0 = wave * 32;
  const int w_rows = max(0, min(32, n_rows - wrow0));
  const int wk_lo = k_lo + wrow0, wk_hi = wk_lo + w_rows - 1;
  bf16x8 kf[N::KS], vf[N::KS];
  const int kl = min(wk_lo + li, k_end - 1) + koff;
  load_own<D>(kf, t.k, kl, t.k_st, (int64_t)hk * t.k_sh, lane);
  load_own<D>(vf, t.v, kl, t.v_st, (int64_t)hk * t.v_sh, lane);
  f32x16 dk[N::DT], dv[N::DT];
#pragma unroll
  for (int dt = 0; dt < N::DT; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) { dk[dt][r] = 0.f; dv[dt][r] = 0.f; }
  const float c_log2 = t.scale * kLog2e;
  NAddr<D> fa;
  fa.init(lane);
  NDma<D, KW> dmaq, dmao;
  dmaq.init(wave, lane, t.q_st);
  dmao.init(wave, lane, t.do_st);
  QIter<RANGES> it(g, uni(w.e0), uni(w.e1), G, t.qbounds);
  auto issue = [&](char* stage) {
    const int head = hk * G + it.hh, last = it.q1 - 1;
    dmaq.load(stage, (const bf16_t*)t.q + (int64_t)head * t.q_sh, it.qs + it.moff, last + it.moff, wave);
    dmao.load(stage + N::kBytes, (const bf16_t*)t.dout + (int64_t)head * t.do_sh, it.qs + it.moff, last + it.moff, wave);
    const int ql = min(lane, last - it.qs);   // row of the tile: the lane's 32-bit offset runs from the tile's first row
    const int64_t at = (int64_t)head * t.q_rows + it.qs + it.moff;
    if (wave == 0) dma4((unsigned)ql * 4u, uni_ptr(t.lse2 + at), lds_addr(stage + LSE));
    if (wave == 1) dma4((unsigned)ql * 4u, uni_ptr(t.delta + at), lds_addr(stage + DEL));
    if (RANGES && wave == KW - 2 && it.kind == 2) {
      if (t.window > 0) *((int4*)(stage + RNG) + lane) = range_row(t, it.qs + ql, seq0);
      else dma16((unsigned)ql * 16u, uni_ptr(t.ranges + 4 * (int64_t)it.qs), lds_addr(stage + RNG));
    }
    if (RANGES && wave == KW - 1 && it.kind == 2)
      dma16((unsigned)(lane & 3) * 16u, uni_ptr(t.qbounds + (int64_t)(it.t32 + 2 * it.jt) * 8), lds_addr(stage + BND));
  };
  // group x takes tiles x, x + NG, ..; `alive`: group 0 has a tile in this step (every group finds out on its way)
  auto skip = [&](int n) {
    for (; n > 0; n--)
      if (!it.next(k_lo, k_end)) return false;
    return true;
  };
  bool alive = skip(1), have = alive && skip(group);
  if (have) issue(stages);
  DCP_WAIT_VMCNT(0);
  __syncthreads();
  int buf = 0;
  while (alive) {
    const char* cur = stages + buf;
    const char* q_lds = cur;
    const char* do_lds = cur + N::kBytes;
    const int qs = it.qs, q1 = it.q1, kind = it.kind;
    const bool now = have;
    alive = have && skip(NG - group);
    have = alive && skip(group);
    buf ^= kStage;
    if (have) issue(stages + buf);
    if (now && w_rows > 0) {
#pragma unroll 1
      for (int qt = 0; qt < 2; qt++) {
        const int qs32 = qs + 32 * qt;
        if (qs32 >= q1) break;
        const bool whole = qs32 + 32 <= q1 && w_rows == 32;
        int cls = kPartial;
        if (kind == 0) cls = whole ? kFull : kPartial;
        if (kind == 1) cls = min(qs32 + 31, q1 - 1) < wk_lo ? kSkip : ((whole && qs32 >= wk_hi) ? kFull : kPartial);
        if (RANGES && kind == 2) {
          const int4* bp = (const int4*)(cur + BND) + 2 * qt;
          const int4 a = bp[0], b = bp[1];
          RangeBounds qb;
          qb.lo_min[0] = uni(a.x); qb.lo_max[0] = uni(a.y); qb.hi_min[0] = uni(a.z); qb.hi_max[0] = uni(a.w);
          qb.lo_min[1] = uni(b.x); qb.lo_max[1] = uni(b.y); qb.hi_min[1] = uni(b.z); qb.hi_max[1] = uni(b.w);
          if (!qb.may_see(wk_lo, wk_hi + 1)) cls = kSkip;
          else if (whole && qb.all_see(wk_lo, wk_hi + 1)) cls = kFull;
        }
        if (cls == kSkip) continue;
        const float* lse_lds = (const float*)(cur + LSE) + 32 * qt + 4 * lh;
        const float* dl_lds = (const float*)(cur + DEL) + 32 * qt + 4 * lh;
        f32x16 s, dp;
#pragma unroll
        for (int a = 0; a < 4; a++) {
          const float4 d4 = *(const float4*)(dl_lds + 8 * a);
          dp[4 * a] = d4.x; dp[4 * a + 1] = d4.y; dp[4 * a + 2] = d4.z; dp[4 * a + 3] = d4.w;
        }
#pragma unroll
        for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
        for (int x = 0; x < N::KS; x++) {
          s = mfma(fa.rows(q_lds, 32 * qt, x), kf[x], s);
          dp = mfma(fa.rows(do_lds, 32 * qt, x), vf[x], dp);
        }
        if (cls == kPartial) {
          // which of the wave's 32 keys query row (l & 31) sees, as a bit mask of lane l (see the D = 128 kernel)
          const int row = lane & 31, qq = qs32 + row;
          int lo1 = 0, hi1 = kind == 1 ? qq + 1 : INT32_MAX, lo2 = 0, hi2 = 0;
          if (RANGES && kind == 2) {
            const int4 rg = ((const int4*)(cur + RNG))[32 * qt + row];
            lo1 = rg.x; hi1 = rg.y; lo2 = rg.z; hi2 = rg.w;
          }
          uint32_t vis = (keys_below(hi1, wk_lo) & ~keys_below(lo1, wk_lo)) | (keys_below(hi2, wk_lo) & ~keys_below(lo2, wk_lo));
          vis &= keys_below(k_end, wk_lo);
          vis = qq < q1 ? vis : 0u;
#pragma unroll
          for (int r = 0; r < 16; r++) {
            const int r0 = 8 * (r / 4) + (r % 4);
            const uint64_t cond = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)vis, r0) |
                                  ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)vis, r0 + 4) << 32);
            s[r] = __builtin_amdgcn_inverse_ballot_w64(cond) ? s[r] : -INFINITY;
          }
        }
#pragma unroll
        for (int a = 0; a < 4; a++) {
          const float4 l4 = *(const float4*)(lse_lds + 8 * a);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
          for (int b = 0; b < 4; b++) {
            const int r = 4 * a + b;
            s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lv[b]));
            dp[r] *= s[r];
          }
        }
#pragma unroll
        for (int c = 0; c < 2; c++) {
          bf16x8 p[3], ds[3];
          pack_split(s, c, p);
          pack_split(dp, c, ds);
#pragma unroll
          for (int dt = 0; dt < N::DT; dt++) {
            const bf16x8 a = fa.cols(do_lds, 32 * qt + 16 * c, dt), b = fa.cols(q_lds, 32 * qt + 16 * c, dt);
#pragma unroll
            for (int k = 0; k < 3; k++) {
              dv[dt] = mfma(a, p[k], dv[dt]);
              dk[dt] = mfma(b, ds[k], dk[dt]);
            }
          }
        }
      }
    }
    DCP_WAIT_VMCNT(0);
    __syncthreads();
  }
  // the other groups leave their sums in LDS (register by register), group 0 adds them to its own and stores
  constexpr int SUMS = 64 * 32 * N::DT;   // floats per wave
  static_assert((NG - 1) * KW * SUMS * 4 <= 2 * NG * kStage && KW * 32 * N::kORow <= 2 * NG * kStage, "the sums and the output tiles fit in the stages");
  float* sums = (float*)all_stages + lane;
  if (group > 0) {
    float* p = sums + ((group - 1) * KW + wave) * SUMS;
#pragma unroll
    for (int dt = 0; dt < N::DT; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) { p[64 * (32 * dt + r)] = dk[dt][r]; p[64 * (32 * dt + 16 + r)] = dv[dt][r]; }
  }
  __syncthreads();
  if (group == 0) {
    for (int y = 0; y < NG - 1; y++) {
      const float* p = sums + (y * KW + wave) * SUMS;
#pragma unroll
      for (int dt = 0; dt < N::DT; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) { dk[dt][r] += p[64 * (32 * dt + r)]; dv[dt][r] += p[64 * (32 * dt + 16 + r)]; }
    }
  }
  __syncthreads();
  if (group > 0) return;
  char* ot = all_stages + wave * (32 * N::kORow);
  bf16_t* dkp = (bf16_t*)t.dk + (int64_t)(wk_lo + koff) * t.dk_st + (int64_t)hk * t.dk_sh;
  bf16_t* dvp = (bf16_t*)t.dv + (int64_t)(wk_lo + koff) * t.dv_st + (int64_t)hk * t.dv_sh;
  uint32_t again = rows_not_finite<D>(dk, w_rows) | rows_not_finite<D>(dv, w_rows);
  store_rows32<D>(ot, dk, t.scale, lane, w_rows, dkp, t.dk_st);
  store_rows32<D>(ot, dv, 1.f, lane, w_rows, dvp, t.dv_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    const WorkItem w1 = plan_load(a.g.items, item);
    const int s0 = RANGES ? uni(plan_load(a.g.blk_s0, plan_load(a.g.unit_blk, uni(w1.unit)))) : 0;
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again), j = wk_lo + r;
      fix_dkv<bf16_t, D>(a.g, a.t, j, uni(w1.e0), uni(w1.e1), hk, s0, (const bf16_t*)a.t.k + (int64_t)(j + koff) * a.t.k_st + (int64_t)hk * a.t.k_sh,
                         (const bf16_t*)a.t.v + (int64_t)(j + koff) * a.t.v_st + (int64_t)hk * a.t.v_sh, dkp + r * a.t.dk_st, dvp + r * a.t.dv_st);
    }
  }
}

#define DCP_NARROW_LAUNCH(KERNEL)                                                              \
  const dim3 grid(xcd_grid(g, t.hkv, t.hq / t.hkv)), block(256);                               \
  if (t.masked) {                                                                              \
    if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, true>), grid, block, 0, s, g, t);            \
    else hipLaunchKernelGGL((KERNEL<64, true>), grid, block, 0, s, g, t);                      \
  } else {                                                                                     \
    if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, false>), grid, block, 0, s, g, t);           \
    else hipLaunchKernelGGL((KERNEL<64, false>), grid, block, 0, s, g, t);                     \
  }                                                                                            \
  DCP_HIP_TRY(hipGetLastError());                                                              \
  return DCP_OK;

dcp_status_t mfma_narrow_fwd(const DevGroup& g, const KTensors& t, hipStream_t s) { DCP_NARROW_LAUNCH(narrow_fwd_kernel) }
dcp_status_t mfma_narrow_dq(const DevGroup& g, const KTensors& t, hipStream_t s) { DCP_NARROW_LAUNCH(narrow_dq_kernel) }

dcp_status_t mfma_narrow_dkv(const DevGroup& g, const KTensors& t, hipStream_t s) {
  const dim3 grid(xcd_grid(g, t.hkv, 1)), block(kNarrowDkvThreads);
  if (t.masked) {
    if (t.d == 32) hipLaunchKernelGGL((narrow_dkv_kernel<32, true>), grid, block, 0, s, g, t);
    else hipLaunchKernelGGL((narrow_dkv_kernel<64, true>), grid, block, 0, s, g, t);
  } else {
    if (t.d == 32) hipLaunchKernelGGL((narrow_dkv_kernel<32, false>), grid, block, 0, s, g, t);
    else hipLaunchKernelGGL((narrow_dkv_kernel<64, false>), grid, block, 0, s, g, t);
  }
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

}  // namespace dcp
