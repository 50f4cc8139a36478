// Blockwise attention, forward and backward, for fp32 tensors (D = 32, 64, 128) on fp32 MFMA (v_mfma_f32_32x32x2_f32).
//
// What bounds it: the matrix pipe.  An fp32 MFMA takes 64 cycles for 64 x 4 bytes of operand A, a sixteenth of the
// bf16 rate, so a CU asks for 16 B/clk of streamed operands at most and the L1 / L2 serve them straight into registers:
// the other side's tiles are not staged in LDS, no barrier sits in the loops, and the waves of a workgroup run
// independently.  That freedom is used to split the contraction inside the workgroup: its eight waves own the SAME 32
// rows (kept in LDS, operand B) and take every eighth 32-row tile of the other side, and their partial results meet
// once, in LDS, at the end -- a small batch has eight times the parallel work it would have with a wave per 32 rows.
// Streamed operands come in chunks of at most 32 registers, the next one on its way under the 32 MFMAs of the current,
// so that two waves fit on a SIMD at every D.  Operand layouts (lane l, i = l % 32, h = l / 32):
//   "rows" fragment: floats 8j + 4h .. + 3 of row i (j = 0 .. D/8 - 1): A or B operand of a product over D (the
//     contraction index may be permuted as long as both operands agree);
//   "cols" fragment: entry r holds columns DT i .. DT i + DT - 1 (DT = D/32) of row 8 (r/4) + 4h + r%4: A operand of a
//     product over rows whose B operand is a score tile as the accumulator holds it (register r, lane (column, h)).
//     Column DT m + dt of the result is row m of accumulator tile dt.
// Measured, forward + backward, against the scalar family's thread per row: 8 192 causal tokens (log-normal, median
// 1 024), 8/2 heads, D 64: 55.2 -> 1.60 ms (forward 0.35, dQ 0.49, dK/dV 0.78 ms: 99 / 106 / 88 TFLOP/s executed; a
// large fp32 matrix product reaches 152 on this card); 512 tokens, one head: 1 067 -> 54 us.  Four waves with the own
// rows in registers took 2.36 ms (the dK/dV kernel spilled, and its 512 workgroups of one round waited for the longest).
#include "device_utils.h"
#include "split_rows.h"

namespace dcp {

namespace {

constexpr float kLog2eF = 1.44269504088896340736f;
constexpr float kLn2F = 0.69314718055994530942f;
constexpr int kThreads = kSplitThreads, kWaves = kSplitWaves, kRows = kSplitRows, kSub = kSplitSub;
constexpr float kRaise = 8.f;   // the running maximum is raised when a tile exceeds it by more than 2^8

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Chunks: NC per fragment, at most 32 registers each (D = 128: 16, its accumulators leave no more).
template <int D> struct Chunks { static constexpr int NC = D == 128 ? 4 : 1, NJ = D / 8 / NC, NR = 16 / NC; };
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
template <int D> struct RowChunk { f32x4 c[Chunks<D>::NJ]; };
template <int D> struct ColChunk { float v[Chunks<D>::NR][D / 32]; };

// The lane number, opaque: what the loads below derive from it is recomputed per tile instead of being kept in dozens of
// registers across the loop.
__device__ __forceinline__ int fresh_lane() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}

// Wave-uniform base + 32-bit lane offset, in the global address space (a pointer rebuilt from integers is a flat one to
// the compiler: flat loads take 64-bit lane addresses and the LDS counter too).
typedef const __attribute__((address_space(1))) char* gbase_t;
__device__ __forceinline__ gbase_t gbase(const void* p) { return (gbase_t)(uint64_t)uni_ptr(p); }
template <class T> __device__ __forceinline__ T gload(gbase_t b, unsigned off) { return *(const __attribute__((address_space(1))) T*)(b + off); }

// Chunk c of rows row0 .. row0 + 31 of a [rows, heads, D] tensor (head applied to base; stride in elements), rows past
// `last` repeat it.
template <int D>
__device__ __forceinline__ void load_rows(RowChunk<D>& f, const float* base, int64_t stride, int row0, int last, int c) {
  const int lane = fresh_lane(), i = lane & 31, h = lane >> 5;
  const gbase_t b = gbase(base + (int64_t)row0 * stride);
  const unsigned off = (unsigned)min(i, last - row0) * (unsigned)stride * 4u + 16u * h;
#pragma unroll
  for (int j = 0; j < Chunks<D>::NJ; j++) f.c[j] = gload<f32x4>(b, off + 32 * (c * Chunks<D>::NJ + j));
}

template <int D>
__device__ __forceinline__ void load_cols(ColChunk<D>& f, const float* base, int64_t stride, int row0, int last, int c) {
  constexpr int DT = D / 32, NR = Chunks<D>::NR;
  const int lane = fresh_lane(), i = lane & 31, h = lane >> 5;
  const gbase_t b = gbase(base + (int64_t)row0 * stride);
  const int lim = last - row0;
  auto get = [&](int r, unsigned off) {
    if constexpr (DT == 4) { const f32x4 x = gload<f32x4>(b, off); f.v[r][0] = x.x; f.v[r][1] = x.y; f.v[r][2] = x.z; f.v[r][3] = x.w; }
    else if constexpr (DT == 2) { const f32x2v x = gload<f32x2v>(b, off); f.v[r][0] = x.x; f.v[r][1] = x.y; }
    else f.v[r][0] = gload<float>(b, off);
  };
  if (lim >= kRows - 1) {
    const unsigned off = (unsigned)(4 * h) * (unsigned)stride * 4u + 4u * DT * i;
#pragma unroll
    for (int r = 0; r < NR; r++) get(r, off + (unsigned)acc_row(c * NR + r) * (unsigned)stride * 4u);
  } else {
#pragma unroll
    for (int r = 0; r < NR; r++) get(r, (unsigned)min(acc_row(c * NR + r) + 4 * h, lim) * (unsigned)stride * 4u + 4u * DT * i);
  }
}

// one value per row of the score tile: element r of the lane is row acc_row(r) + 4h
__device__ __forceinline__ f32x16 load_per_row(const float* p, int lim) {
  const int h = fresh_lane() >> 5;
  const gbase_t b = gbase(p);
  f32x16 v;
#pragma unroll
  for (int r = 0; r < 16; r++) v[r] = gload<float>(b, 4u * (unsigned)min(acc_row(r) + 4 * h, lim));
  return v;
}

// The workgroup's own 32 rows in LDS, rows of D + 4 floats (16-byte reads of 16 consecutive rows then fall into 64
// different banks), copied by all threads; rows past `last` repeat it.
template <int D>
__device__ __forceinline__ void own_rows(float* lds, const float* base, int64_t stride, int row0, int last) {
  for (int x = threadIdx.x; x < kRows * (D / 4); x += kThreads) {
    const int row = x / (D / 4), c = x % (D / 4);
    *(float4*)(lds + row * (D + 4) + 4 * c) = *(const float4*)(base + (int64_t)min(row0 + row, last) * stride + 4 * c);
  }
}

// s += A B over chunk c of D: A streamed rows, B the own rows in LDS
template <int D>
__device__ __forceinline__ f32x16 dot_rows(const RowChunk<D>& a, const float* lds, int lane, int c, f32x16 s) {
  const float* b = lds + (lane & 31) * (D + 4) + 4 * (lane >> 5) + 8 * Chunks<D>::NJ * c;
#pragma unroll
  for (int j = 0; j < Chunks<D>::NJ; j++) {
    const float4 x = *(const float4*)(b + 8 * j);
    s = mfma_f32(a.c[j].x, x.x, s);
    s = mfma_f32(a.c[j].y, x.y, s);
    s = mfma_f32(a.c[j].z, x.z, s);
    s = mfma_f32(a.c[j].w, x.w, s);
  }
  return s;
}

template <int D>
__device__ __forceinline__ void add_cols(const ColChunk<D>& a, const f32x16& p, int c, f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int r = 0; r < Chunks<D>::NR; r++)
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) acc[dt] = mfma_f32(a.v[r][dt], p[c * Chunks<D>::NR + r], acc[dt]);
}

__device__ __forceinline__ f32x16 splat(float x) {
  f32x16 v;
#pragma unroll
  for (int r = 0; r < 16; r++) v[r] = x;
  return v;
}

// A wave's D x 32 accumulator tile (lane = row of the result) into its LDS slab, rows of D + 4 floats.
template <int D>
__device__ __forceinline__ void stage_acc(float* slab, const f32x16 (&acc)[D / 32], int lane) {
  constexpr int DT = D / 32;
  float* row = slab + (lane & 31) * (D + 4) + 4 * DT * (lane >> 5);
#pragma unroll
  for (int a = 0; a < 4; a++)
#pragma unroll
    for (int x = 0; x < DT; x++) {   // four consecutive columns: 4 x .. 4 x + 3 of the 4 DT that rows m = 8a + 4h .. + 3 hold
      float4 v;
      v.x = acc[(4 * x) % DT][4 * a + (4 * x) / DT];
      v.y = acc[(4 * x + 1) % DT][4 * a + (4 * x + 1) / DT];
      v.z = acc[(4 * x + 2) % DT][4 * a + (4 * x + 2) / DT];
      v.w = acc[(4 * x + 3) % DT][4 * a + (4 * x + 3) / DT];
      *(float4*)(row + 8 * DT * a + 4 * x) = v;
    }
}

// Adds the waves' slabs up in wave order and stores rows r < n_rows.  wgt: factor of each (wave, row), or null (1).  Returns
// which of the wave's four rows (4 wave + bit) hold a value that is not finite.
template <int D>
__device__ __forceinline__ uint32_t store_sum(const float* slabs, const float* wgt, float mul, int n_rows, float* dst, int64_t stride) {
  const int row = threadIdx.x / 16, seg = threadIdx.x % 16;
  static_assert(kThreads == 16 * kRows, "16 threads per row");
  float probe = 0.f;
  if (row < n_rows)
    for (int col = 4 * seg; col < D; col += 64) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < kWaves; w++) {
        const float4 b = *(const float4*)(slabs + (w * kRows + row) * (D + 4) + col);
        const float f = wgt ? wgt[w * kRows + row] : mul;
        a.x = fmaf(b.x, f, a.x); a.y = fmaf(b.y, f, a.y); a.z = fmaf(b.z, f, a.z); a.w = fmaf(b.w, f, a.w);
      }
      *(float4*)(dst + (int64_t)row * stride + col) = a;
      probe = finite_probe(a.x, finite_probe(a.y, finite_probe(a.z, finite_probe(a.w, probe))));
    }
  const uint64_t bad = __ballot(probe != 0.f);
  return ((bad & 0xffffull) != 0) | ((bad & 0xffff0000ull) != 0) << 1 | ((bad & 0xffff00000000ull) != 0) << 2 | ((bad >> 48) != 0) << 3;
}

}  // namespace

// LDS of the three kernels: a slab per wave for its partial result; the first two hold the own rows during the loop.
#define DCP_FENCE() __builtin_amdgcn_sched_barrier(0)

template <int D, bool RANGES>
__global__ __launch_bounds__(kThreads, 2) void f32_fwd_kernel(DevGroup g, KTensors t) {
  constexpr int NC = Chunks<D>::NC, SLAB = kRows * (D + 4);
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * SLAB];
  __shared__ float sm[kWaves][kRows], sl[kWaves][kRows];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), li = lane & 31, lh = lane >> 5;
  QTile q;
  if (!q_tile<RANGES>(g, t, lane, blockIdx.x, &q)) return;
  own_rows<D>(slabs, (const float*)t.q + (int64_t)q.head * t.q_sh, t.q_st, q.q_lo + q.qoff, q.q_hi + q.qoff);
  const float* kb = (const float*)t.k + (int64_t)q.hk * t.k_sh;
  const float* vb = (const float*)t.v + (int64_t)q.hk * t.v_sh;
  const float c_log2 = t.scale * kLog2eF;
  float m = -INFINITY, l = 0.f;
  f32x16 o[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) o[dt] = splat(0.f);
  Walk<kWaves> it(g, q.e0, q.e1, wave);
  bool have = it.next<RANGES>(q.q_hi, q.rb);
  RowChunk<D> kc;
  if (have) load_rows<D>(kc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
  __syncthreads();
  while (have) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = it.kind, r0 = ks + it.moff, r1 = c1 - 1 + it.moff;
    f32x16 s = splat(0.f);
    ColChunk<D> vc, vn;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D> kn;
      if (c + 1 < NC) load_rows<D>(kn, kb, t.k_st, r0, r1, c + 1);
      else load_cols<D>(vc, vb, t.v_st, r0, r1, 0);
      DCP_FENCE();
      s = dot_rows<D>(kc, slabs, lane, c, s);
      DCP_FENCE();
      kc = kn;
    }
    if (classify32(kind, ks, c1, q.q_lo, q.q_hi, q.rb) != kFull) mask_keys(s, q, kind, ks, c0, c1, lane);
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; r++) mx = fmaxf(mx, s[r]);
    mx = xhalf_max(mx);
    const bool raise = (mx - m) * c_log2 > kRaise;
    const float m_new = raise ? mx : m;
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__any(raise)) {
      const float alpha = raise ? __builtin_amdgcn_exp2f((m - m_use) * c_log2) : 1.f;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[dt][r] *= alpha;
    }
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r++) {
      s[r] = __builtin_amdgcn_exp2f((s[r] - m_use) * c_log2);
      sum += s[r];
    }
    l += sum;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) {
        load_cols<D>(vn, vb, t.v_st, r0, r1, c + 1);
      } else {
        have = it.next<RANGES>(q.q_hi, q.rb);
        if (have) load_rows<D>(kc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
      }
      DCP_FENCE();
      add_cols<D>(vc, s, c, o);
      DCP_FENCE();
      vc = vn;
    }
  }
  l = xhalf_sum(l);
  if (lh == 0) { sm[wave][li] = m; sl[wave][li] = l; }
  __syncthreads();   // the own rows' slab is free
  stage_acc<D>(slabs + wave * SLAB, o, lane);
  // every wave's weight for its rows, the row's LSE
  float mt = -INFINITY, lt = 0.f, f[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; w++) mt = fmaxf(mt, sm[w][li]);
#pragma unroll
  for (int w = 0; w < kWaves; w++) {
    f[w] = sm[w][li] > -INFINITY ? __builtin_amdgcn_exp2f((sm[w][li] - mt) * c_log2) : 0.f;
    lt = fmaf(f[w], sl[w][li], lt);
  }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  __syncthreads();
  if (wave == 0 && lh == 0) {
#pragma unroll
    for (int w = 0; w < kWaves; w++) sl[w][li] = f[w] * inv;
  }
  __syncthreads();
  const int slot = plan_load(g.unit_out, q.unit);
  if (wave == 0 && lh == 0 && li < q.n_rows) {
    const float lse = lt > 0.f ? (mt * c_log2 + __builtin_amdgcn_logf(lt)) * kLn2F : -INFINITY;
    if (slot < 0) t.lse[(int64_t)q.head * t.q_rows + q.q_lo + q.qoff + li] = lse;
    else t.lse[((int64_t)slot * t.hq + q.head) * t.block_size + q.row0 + li] = lse;
  }
  float* op = slot < 0 ? (float*)t.out + (int64_t)(q.q_lo + q.qoff) * t.o_st + (int64_t)q.head * t.o_sh
                       : (float*)t.out + (((int64_t)slot * t.block_size + q.row0) * t.hq + q.head) * D;
  const int64_t op_st = slot < 0 ? t.o_st : (int64_t)t.hq * D;
  uint32_t again = store_sum<D>(slabs, &sl[0][0], 1.f, q.n_rows, op, op_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = 4 * wave + __builtin_ctz(again);
      if (lane_of(lt, r) != lane_of(lt, r)) continue;   // a NaN score: all of the row is NaN already
      const FixRow f = fix_row(q, r);
      const float mr = lane_of(mt, r);
      fix_out<float, D>(a.g, a.t, f, q.hk, (const float*)a.t.q + (int64_t)(f.qi + q.qoff) * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                        mr == -INFINITY ? 0.f : mr * c_log2, lane_of(inv, r), op + r * op_st);
    }
  }
}

template <int D, bool RANGES>
__global__ __launch_bounds__(kThreads, 2) void f32_dq_kernel(DevGroup g, KTensors t) {
  constexpr int NC = Chunks<D>::NC, SLAB = kRows * (D + 4);
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * SLAB];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), li = lane & 31, lh = lane >> 5;
  QTile q;
  if (!q_tile<RANGES>(g, t, lane, blockIdx.x, &q)) return;
  const float* q_lds = slabs;
  const float* do_lds = slabs + SLAB;
  own_rows<D>(slabs, (const float*)t.q + (int64_t)q.head * t.q_sh, t.q_st, q.q_lo + q.qoff, q.q_hi + q.qoff);
  own_rows<D>(slabs + SLAB, (const float*)t.dout + (int64_t)q.head * t.do_sh, t.do_st, q.q_lo + q.qoff, q.q_hi + q.qoff);
  __syncthreads();
  // the backward preprocess, fused: delta = sum_d dO * O of the lane's row, left (negated) with the rescaled LSE in
  // the workspace for the dK/dV kernel
  float delta = 0.f;
#pragma unroll
  for (int c = 0; c < NC; c++) {
    RowChunk<D> oc;
    load_rows<D>(oc, (const float*)t.out_in + (int64_t)q.head * t.o_sh, t.o_st, q.q_lo + q.qoff, q.q_hi + q.qoff, c);
#pragma unroll
    for (int j = 0; j < Chunks<D>::NJ; j++) {
      const float4 x = *(const float4*)(do_lds + li * (D + 4) + 4 * lh + 8 * (Chunks<D>::NJ * c + j));
      delta = fmaf(oc.c[j].x, x.x, delta); delta = fmaf(oc.c[j].y, x.y, delta);
      delta = fmaf(oc.c[j].z, x.z, delta); delta = fmaf(oc.c[j].w, x.w, delta);
    }
  }
  delta = xhalf_sum(delta);
  const int64_t at = (int64_t)q.head * t.q_rows + q.qi + q.qoff;
  const float lse2 = row_lse2(t.lse[at], &delta);
  if (wave == 0 && lh == 0 && li < q.n_rows) { t.delta_w[at] = -delta; t.lse2_w[at] = lse2; }
  const float* kb = (const float*)t.k + (int64_t)q.hk * t.k_sh;
  const float* vb = (const float*)t.v + (int64_t)q.hk * t.v_sh;
  const float c_log2 = t.scale * kLog2eF;
  f32x16 dq[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) dq[dt] = splat(0.f);
  Walk<kWaves> it(g, q.e0, q.e1, wave);
  bool have = it.next<RANGES>(q.q_hi, q.rb);
  RowChunk<D> rc;
  if (have) load_rows<D>(rc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
  while (have) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = it.kind, r0 = ks + it.moff, r1 = c1 - 1 + it.moff;
    f32x16 s = splat(0.f), dp = splat(-delta);
    ColChunk<D> cc, cn;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D> rn;
      if (c + 1 < NC) load_rows<D>(rn, kb, t.k_st, r0, r1, c + 1);
      else load_rows<D>(rn, vb, t.v_st, r0, r1, 0);
      DCP_FENCE();
      s = dot_rows<D>(rc, q_lds, lane, c, s);
      DCP_FENCE();
      rc = rn;
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D> rn;
      if (c + 1 < NC) load_rows<D>(rn, vb, t.v_st, r0, r1, c + 1);
      else load_cols<D>(cc, kb, t.k_st, r0, r1, 0);
      DCP_FENCE();
      dp = dot_rows<D>(rc, do_lds, lane, c, dp);
      DCP_FENCE();
      rc = rn;
    }
    if (classify32(kind, ks, c1, q.q_lo, q.q_hi, q.rb) != kFull) mask_keys(s, q, kind, ks, c0, c1, lane);
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lse2)) * dp[r];
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) {
        load_cols<D>(cn, kb, t.k_st, r0, r1, c + 1);
      } else {
        have = it.next<RANGES>(q.q_hi, q.rb);
        if (have) load_rows<D>(rc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
      }
      DCP_FENCE();
      add_cols<D>(cc, s, c, dq);
      DCP_FENCE();
      cc = cn;
    }
  }
  __syncthreads();   // the own rows' slabs are free
  stage_acc<D>(slabs + wave * SLAB, dq, lane);
  __syncthreads();
  float* dqp = (float*)t.dq + (int64_t)(q.q_lo + q.qoff) * t.dq_st + (int64_t)q.head * t.dq_sh;
  uint32_t again = store_sum<D>(slabs, nullptr, t.scale, q.n_rows, dqp, t.dq_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = 4 * wave + __builtin_ctz(again);
      const FixRow f = fix_row(q, r);
      const int64_t mem = f.qi + q.qoff;
      fix_dq<float, D>(a.g, a.t, f, q.hk, (const float*)a.t.q + mem * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                       (const float*)a.t.dout + mem * a.t.do_st + (int64_t)q.head * a.t.do_sh, lane_of(lse2, r), lane_of(delta, r), dqp + r * a.t.dq_st);
    }
  }
}

// dK / dV of 32 keys of one KV head: the waves take every eighth (query head, 32-query tile) of the listed q blocks.
template <int D, bool RANGES>
__global__ __launch_bounds__(kThreads, 2) void f32_dkv_kernel(DevGroup g, KTensors t) {
  constexpr int NC = Chunks<D>::NC, SLAB = kRows * (D + 4);
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * SLAB];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  int item, x;
  const int G = t.hq / t.hkv;
  if (!decode_wg(g, t.hkv, kSub, &item, &x)) return;
  const int hk = x / kSub;
  const WorkItem w = plan_load(g.items, item);
  const int e1 = uni(w.e1), koff = uni(w.moff);
  const int row0 = uni(w.tile) * (kSub * kRows) + (x % kSub) * kRows;
  const int n_rows = min(kRows, uni(w.blk_len) - row0);
  if (n_rows <= 0) return;
  const int k_lo = uni(w.blk_start) + row0, k_hi = k_lo + n_rows - 1;
  const int seq0 = RANGES ? uni(plan_load(g.blk_s0, plan_load(g.unit_blk, uni(w.unit)))) : 0;
  const float* k_lds = slabs;
  const float* v_lds = slabs + SLAB;
  own_rows<D>(slabs, (const float*)t.k + (int64_t)hk * t.k_sh, t.k_st, k_lo + koff, k_hi + koff);
  own_rows<D>(slabs + SLAB, (const float*)t.v + (int64_t)hk * t.v_sh, t.v_st, k_lo + koff, k_hi + koff);
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) { dk[dt] = splat(0.f); dv[dt] = splat(0.f); }
  const float c_log2 = t.scale * kLog2eF;

  const int4* rec = (const int4*)g.ent_rec;
  const int4* qbounds = (const int4*)t.qbounds;
  int e = uni(w.e0) - 1, hh = G - 1, q0 = 0, q1 = 0, kind = 0, moff = 0, t32 = 0, n_t = 0, jt0 = 0, jt = 0;
  RangeBounds qb;   // of the current tile's rows (RANGES rows of the table)
  auto next = [&]() {
    for (;;) {
      jt += kWaves;
      while (jt >= n_t) {
        if (++hh >= G) {
          if (++e >= e1) return false;
          hh = 0;
          const int4 r = plan_load(rec, 2 * e);
          q0 = uni(r.x); q1 = q0 + uni(r.y); kind = uni(r.z); moff = uni(r.w); t32 = uni(plan_load(rec, 2 * e + 1).x);
          n_t = (q1 - q0 + kRows - 1) / kRows;
          jt0 = kind == 1 ? max(0, (k_lo - q0) / kRows) : 0;
        }
        jt = jt0 + ((wave - t32 - jt0 - hh) & (kWaves - 1));
      }
      if (!RANGES || kind != 2) return true;
      const int4 a = qbounds[2 * (t32 + jt)], b = qbounds[2 * (t32 + jt) + 1];
      qb.lo_min[0] = uni(a.x); qb.lo_max[0] = uni(a.y); qb.hi_min[0] = uni(a.z); qb.hi_max[0] = uni(a.w);
      qb.lo_min[1] = uni(b.x); qb.lo_max[1] = uni(b.y); qb.hi_min[1] = uni(b.z); qb.hi_max[1] = uni(b.w);
      if (qb.may_see(k_lo, k_hi + 1)) return true;
    }
  };
  auto q_base = [&](int head) { return (const float*)t.q + (int64_t)head * t.q_sh; };
  bool have = next();
  RowChunk<D> rc;
  if (have) load_rows<D>(rc, q_base(hk * G + hh), t.q_st, q0 + kRows * jt + moff, q1 - 1 + moff, 0);
  __syncthreads();
  while (have) {
    const int qs = q0 + kRows * jt, q_end = q1, r0 = qs + moff, r1 = q1 - 1 + moff, kd = kind, head = hk * G + hh;
    const bool whole = qs + kRows <= q_end && n_rows == kRows;
    const bool full = whole && (kd == 0 || (kd == 1 && qs >= k_hi) || (RANGES && kd == 2 && qb.all_see(k_lo, k_hi + 1)));
    const float* qp = q_base(head);
    const float* dop = (const float*)t.dout + (int64_t)head * t.do_sh;
    const int lim = min(kRows, q_end - qs) - 1;
    f32x16 s = splat(0.f), dp;
    ColChunk<D> cc, cn;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D> rn;
      if (c + 1 < NC) {
        load_rows<D>(rn, qp, t.q_st, r0, r1, c + 1);
      } else {
        load_rows<D>(rn, dop, t.do_st, r0, r1, 0);
        dp = load_per_row(t.delta + (int64_t)head * t.q_rows + r0, lim);   // -delta: dP starts from it
      }
      DCP_FENCE();
      s = dot_rows<D>(rc, k_lds, lane, c, s);
      DCP_FENCE();
      rc = rn;
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D> rn;
      if (c + 1 < NC) load_rows<D>(rn, dop, t.do_st, r0, r1, c + 1);
      else load_cols<D>(cc, dop, t.do_st, r0, r1, 0);
      DCP_FENCE();
      dp = dot_rows<D>(rc, v_lds, lane, c, dp);
      DCP_FENCE();
      rc = rn;
    }
    const f32x16 lse2 = load_per_row(t.lse2 + (int64_t)head * t.q_rows + r0, lim);
    if (!full) {
      const int ln = fresh_lane(), kj = k_lo + (ln & 31);
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int i = qs + acc_row(r) + 4 * (ln >> 5);
        bool vis = i < q_end && kj <= k_hi;
        if (kd == 1) vis = vis && kj <= i;
        if (RANGES && kd == 2) {
          const int4 rg = range_row(t, min(i, q_end - 1), seq0);
          vis = vis && ((kj >= rg.x && kj < rg.y) || (kj >= rg.z && kj < rg.w));
        }
        if (!vis) s[r] = -INFINITY;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lse2[r]));
      dp[r] *= s[r];
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) load_cols<D>(cn, dop, t.do_st, r0, r1, c + 1);
      else load_cols<D>(cn, qp, t.q_st, r0, r1, 0);
      DCP_FENCE();
      add_cols<D>(cc, s, c, dv);
      DCP_FENCE();
      cc = cn;
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) {
        load_cols<D>(cn, qp, t.q_st, r0, r1, c + 1);
      } else {
        have = next();
        if (have) load_rows<D>(rc, q_base(hk * G + hh), t.q_st, q0 + kRows * jt + moff, q1 - 1 + moff, 0);
      }
      DCP_FENCE();
      add_cols<D>(cc, dp, c, dk);
      DCP_FENCE();
      cc = cn;
    }
  }
  float* slab = slabs + wave * SLAB;
  __syncthreads();   // the own rows' slabs are free
  stage_acc<D>(slab, dk, lane);
  __syncthreads();
  float* dkp = (float*)t.dk + (int64_t)(k_lo + koff) * t.dk_st + (int64_t)hk * t.dk_sh;
  float* dvp = (float*)t.dv + (int64_t)(k_lo + koff) * t.dv_st + (int64_t)hk * t.dv_sh;
  uint32_t again = store_sum<D>(slabs, nullptr, t.scale, n_rows, dkp, t.dk_st);
  __syncthreads();
  stage_acc<D>(slab, dv, lane);
  __syncthreads();
  again |= store_sum<D>(slabs, nullptr, 1.f, n_rows, dvp, t.dv_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    const WorkItem w1 = plan_load(a.g.items, item);
    const int s0 = RANGES ? uni(plan_load(a.g.blk_s0, plan_load(a.g.unit_blk, uni(w1.unit)))) : 0;
    for (; again; again &= again - 1) {
      const int r = 4 * wave + __builtin_ctz(again), j = k_lo + r;
      fix_dkv<float, D>(a.g, a.t, j, uni(w1.e0), uni(w1.e1), hk, s0, (const float*)a.t.k + (int64_t)(j + koff) * a.t.k_st + (int64_t)hk * a.t.k_sh,
                        (const float*)a.t.v + (int64_t)(j + koff) * a.t.v_st + (int64_t)hk * a.t.v_sh, dkp + r * a.t.dk_st, dvp + r * a.t.dv_st);
    }
  }
}

#define DCP_F32_LAUNCH(KERNEL, INNER)                                                                                     \
  const dim3 grid(xcd_grid(g, t.hkv, INNER)), block(kThreads);                                                         \
  if (t.masked) {                                                                                                         \
    if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, true>), grid, block, 0, s, g, t);                                       \
    else if (t.d == 64) hipLaunchKernelGGL((KERNEL<64, true>), grid, block, 0, s, g, t);                                  \
    else hipLaunchKernelGGL((KERNEL<128, true>), grid, block, 0, s, g, t);                                                \
  } else {                                                                                                                \
    if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, false>), grid, block, 0, s, g, t);                                      \
    else if (t.d == 64) hipLaunchKernelGGL((KERNEL<64, false>), grid, block, 0, s, g, t);                                 \
    else hipLaunchKernelGGL((KERNEL<128, false>), grid, block, 0, s, g, t);                                               \
  }                                                                                                                       \
  DCP_HIP_TRY(hipGetLastError());                                                                                         \
  return DCP_OK;

dcp_status_t mfma_f32_fwd(const DevGroup& g, const KTensors& t, hipStream_t s) { DCP_F32_LAUNCH(f32_fwd_kernel, t.hq / t.hkv * kSub) }
dcp_status_t mfma_f32_dq(const DevGroup& g, const KTensors& t, hipStream_t s) { DCP_F32_LAUNCH(f32_dq_kernel, t.hq / t.hkv * kSub) }
dcp_status_t mfma_f32_dkv(const DevGroup& g, const KTensors& t, hipStream_t s) { DCP_F32_LAUNCH(f32_dkv_kernel, kSub) }

}  // namespace dcp
