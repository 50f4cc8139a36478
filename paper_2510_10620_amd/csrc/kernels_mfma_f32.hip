// Blockwise attention, forward and backward, for fp32 tensors (D = 32, 64, 128) on fp32 MFMA (v_mfma_f32_32x32x2_f32, 16x16x4).
//
// What bounds it: the matrix pipe.  An fp32 MFMA takes 64 cycles for 64 x 4 bytes of operand A, a sixteenth of the
// bf16 rate, so a CU asks for 16 B/clk of streamed operands at most and the L1 / L2 serve them straight into registers:
// the other side's tiles are not staged in LDS, no barrier sits in the loops, and the waves of a workgroup run
// independently.  That freedom is used to split the contraction inside the workgroup: its eight waves own the SAME 32 or 16
// rows (kept in LDS, operand B) and take every eighth 32-row tile of the other side, and their partial results meet
// once, in LDS, at the end -- a small batch has eight times the parallel work it would have with a wave per 32 rows.
// With D = 32 and 64 full launches go to kernels_mfma_f32_parts.hip; 32 rows here are for D = 128, and for the forward and dQ of few long walks
// (3 950 tokens in one sequence, 4/2 heads, D 64: 95 and 131 us, in parts 167 and 233, 16 rows 100 and 154).
// 16 rows (16 x 16 x 4 MFMAs, the same rate) serve launches that leave most of the chip idle or wait for their longest item: a
// small batch is a few dozen workgroups whose CUs' matrix pipes are what its time is made of, and half the rows are twice the
// workgroups (512 tokens, one head, D 64: forward / dQ / dK/dV 12.7 / 16.5 / 21.9 -> 8.9 / 11.6 / 14.5 us; 8 192, 8/2 heads, where the parts are
// faster than both, 358 / 503 / 804 -> 377 / 608 / 748: twice the streamed bytes a product), and their backward is one launch where both halves fit the chip (26.1 ->
// 16.9; the dK/dV workgroups work delta out for themselves, from O).
// Streamed operands come in chunks of at most 32 registers (16 with 16 rows: four waves on a SIMD then), the next one on its way
// under the MFMAs of the current, so that two waves fit on a SIMD at every D.  Operand layouts: Fp below;
//   "rows" fragment: floats 4 H j + 4h .. + 3 of row i: A or B operand of a product over D (the contraction index may be permuted
//     as long as both operands agree);
//   "cols" fragment: columns DT i .. DT i + DT - 1 (DT = D / R) of a score value's row: A operand of a product over rows whose
//     B operand is a score tile as the accumulator holds it.  Column DT m + dt of the result is row m of accumulator tile dt.
// Measured, forward + backward, against the scalar family's thread per row: 8 192 causal tokens (log-normal, median
// 1 024), 8/2 heads, D 64: 55.2 -> 1.54 ms (a large fp32 matrix product reaches 152 TFLOP/s on this card, these 90 to 106); 512
// tokens, one head: 1 067 -> 26 us.  Four waves with the own
// rows in registers took 2.36 ms (the dK/dV kernel spilled, and its 512 workgroups of one round waited for the longest).
#include "device_utils.h"
#include "split_rows.h"

namespace dcp {

namespace {

constexpr float kLog2eF = 1.44269504088896340736f;
constexpr float kLn2F = 0.69314718055994530942f;
constexpr int kThreads = kSplitThreads, kWaves = kSplitWaves;
constexpr int kOther = kSplitRows;   // rows of a tile of the other side
constexpr float kRaise = 8.f;   // the running maximum is raised when a tile exceeds it by more than 2^8

// A workgroup owns R rows, 32 or 16: the columns of 32 x 32 x 2 or 16 x 16 x 4 MFMAs, of which NT cover the 32 rows of a tile of the
// other side.  Lane l: own row l % R, h = l / R of H = 64 / R; the H lanes of an own row hold NV = 32 / H values of a score tile,
// value v that of row H * 4 * (v / 4) + 4 h + v % 4.
template <int R> struct Fp;
template <> struct Fp<32> {
  typedef f32x16 Acc;
  static constexpr int H = 2, NT = 1, NV = 16, AR = 16;   // AR: registers of an accumulator tile
  static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <> struct Fp<16> {
  typedef float Acc __attribute__((ext_vector_type(4)));
  static constexpr int H = 4, NT = 2, NV = 8, AR = 4;
  static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};
// a score tile as its accumulators hold it
template <int R> struct Score {
  typename Fp<R>::Acc t[Fp<R>::NT];
  __device__ __forceinline__ float get(int v) const { return t[v / Fp<R>::AR][v % Fp<R>::AR]; }
  __device__ __forceinline__ void set(int v, float x) { t[v / Fp<R>::AR][v % Fp<R>::AR] = x; }
  __device__ __forceinline__ void fill(float x) {
#pragma unroll
    for (int v = 0; v < Fp<R>::NV; v++) set(v, x);
  }
};
template <int R> __device__ __forceinline__ constexpr int val_row(int v) { return 4 * Fp<R>::H * (v / 4) + v % 4; }   // without the lane's 4 h

// combined over the H lanes of an own row, in every one of them
template <int R> __device__ __forceinline__ float own_max(float x) {
  if (R == 16) x = fmaxf(x, __shfl_xor(x, 16));
  return xhalf_max(x);
}
template <int R> __device__ __forceinline__ float own_sum(float x) {
  if (R == 16) x += __shfl_xor(x, 16);
  return xhalf_sum(x);
}

// Chunks: NC per fragment, at most 32 registers each (D = 128: 16, its accumulators leave no more).
template <int D, int R> struct Chunks { static constexpr int NC = D == 128 ? 4 : R == 16 ? D / 32 : 1, NJ = D / 8 / NC; };
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
// "rows": NT x NJ / NT pieces, piece (a, j) floats 4 H j + 4 h .. + 3 of row 32 / NT a + l % R
template <int D, int R> struct RowChunk { f32x4 c[Chunks<D, R>::NJ]; };
// "cols": NV / NC values' rows, D H / 64 columns each
template <int D, int R> struct ColChunk { float v[Fp<R>::NV / Chunks<D, R>::NC][D * Fp<R>::H / 64]; };

// Wave-uniform base + 32-bit lane offset, in the global address space (a pointer rebuilt from integers is a flat one to
// the compiler: flat loads take 64-bit lane addresses and the LDS counter too).
typedef const __attribute__((address_space(1))) char* gbase_t;
__device__ __forceinline__ gbase_t gbase(const void* p) { return (gbase_t)(uint64_t)uni_ptr(p); }
template <class T> __device__ __forceinline__ T gload(gbase_t b, unsigned off) { return *(const __attribute__((address_space(1))) T*)(b + off); }

// Chunk c of rows row0 .. row0 + 31 of a [rows, heads, D] tensor (head applied to base; stride in elements), rows past
// `last` repeat it.
template <int D, int R>
__device__ __forceinline__ void load_rows(RowChunk<D, R>& f, const float* base, int64_t stride, int row0, int last, int c) {
  constexpr int NT = Fp<R>::NT, J = Chunks<D, R>::NJ / NT, W = 4 * Fp<R>::H;   // J pieces of W floats across the lanes of a row
  const int lane = fresh_lane(), i = lane % R, h = lane / R;
  const gbase_t b = gbase(base + (int64_t)row0 * stride);
#pragma unroll
  for (int a = 0; a < NT; a++) {
    const unsigned off = (unsigned)min(i + R * a, last - row0) * (unsigned)stride * 4u + 16u * h;
#pragma unroll
    for (int j = 0; j < J; j++) f.c[a * J + j] = gload<f32x4>(b, off + 4 * W * (c * J + j));
  }
}

template <int D, int R>
__device__ __forceinline__ void load_cols(ColChunk<D, R>& f, const float* base, int64_t stride, int row0, int last, int c) {
  constexpr int DT = D * Fp<R>::H / 64, N = Fp<R>::NV / Chunks<D, R>::NC;
  const int lane = fresh_lane(), i = lane % R, h = lane / R;
  const gbase_t b = gbase(base + (int64_t)row0 * stride);
  const int lim = last - row0;
  auto get = [&](int r, unsigned off) {
    if constexpr (DT >= 4) {
#pragma unroll
      for (int x = 0; x < DT; x += 4) {
        const f32x4 y = gload<f32x4>(b, off + 4 * x);
        f.v[r][x] = y.x; f.v[r][x + 1] = y.y; f.v[r][x + 2] = y.z; f.v[r][x + 3] = y.w;
      }
    } else if constexpr (DT == 2) { const f32x2v x = gload<f32x2v>(b, off); f.v[r][0] = x.x; f.v[r][1] = x.y; }
    else f.v[r][0] = gload<float>(b, off);
  };
  if (lim >= kOther - 1) {
    const unsigned off = (unsigned)(4 * h) * (unsigned)stride * 4u + 4u * DT * i;
#pragma unroll
    for (int r = 0; r < N; r++) get(r, off + (unsigned)val_row<R>(c * N + r) * (unsigned)stride * 4u);
  } else {
#pragma unroll
    for (int r = 0; r < N; r++) get(r, (unsigned)min(val_row<R>(c * N + r) + 4 * h, lim) * (unsigned)stride * 4u + 4u * DT * i);
  }
}

// one value per row of the score tile
template <int R>
__device__ __forceinline__ Score<R> load_per_row(const float* p, int lim) {
  const int h = fresh_lane() / R;
  const gbase_t b = gbase(p);
  Score<R> s;
#pragma unroll
  for (int v = 0; v < Fp<R>::NV; v++) s.set(v, gload<float>(b, 4u * (unsigned)min(val_row<R>(v) + 4 * h, lim)));
  return s;
}

// The workgroup's own R rows in LDS, rows of D + 4 floats (16-byte reads of 16 consecutive rows then fall into 64
// different banks), copied by all threads; rows past `last` repeat it.
template <int D, int R>
__device__ __forceinline__ void own_rows(float* lds, const float* base, int64_t stride, int row0, int last) {
  for (int x = threadIdx.x; x < R * (D / 4); x += kThreads) {
    const int row = x / (D / 4), c = x % (D / 4);
    *(float4*)(lds + row * (D + 4) + 4 * c) = *(const float4*)(base + (int64_t)min(row0 + row, last) * stride + 4 * c);
  }
}

// s += A B over chunk c of D: A streamed rows, B the own rows in LDS
template <int D, int R>
__device__ __forceinline__ void dot_rows(const RowChunk<D, R>& a, const float* lds, int lane, int c, Score<R>& s) {
  constexpr int NT = Fp<R>::NT, J = Chunks<D, R>::NJ / NT, W = 4 * Fp<R>::H;
  const float* b = lds + (lane % R) * (D + 4) + 4 * (lane / R) + W * J * c;
#pragma unroll
  for (int j = 0; j < J; j++) {
    const float4 x = *(const float4*)(b + W * j);
    const float xe[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int t = 0; t < NT; t++) s.t[t] = Fp<R>::mfma(a.c[t * J + j][e], xe[e], s.t[t]);
  }
}

template <int D, int R> struct Out { typename Fp<R>::Acc t[D / R]; };   // a D x R result: tile dt, row m is column D / R m + dt
template <int D, int R>
__device__ __forceinline__ void zero(Out<D, R>& o) {
#pragma unroll
  for (int dt = 0; dt < D / R; dt++)
#pragma unroll
    for (int r = 0; r < Fp<R>::AR; r++) o.t[dt][r] = 0.f;
}

template <int D, int R>
__device__ __forceinline__ void add_cols(const ColChunk<D, R>& a, const Score<R>& p, int c, Out<D, R>& acc) {
  constexpr int N = Fp<R>::NV / Chunks<D, R>::NC;
#pragma unroll
  for (int r = 0; r < N; r++)
#pragma unroll
    for (int dt = 0; dt < D / R; dt++) acc.t[dt] = Fp<R>::mfma(a.v[r][dt], p.get(c * N + r), acc.t[dt]);
}

template <int R>
__device__ __forceinline__ void mask_vals(Score<R>& s, const QTile& q, int kind, int ks, int c0, int c1, int lane) {
  const RowRanges rr = row_ranges(kind, q.qi, c0, c1, q.qr);
  const int kb = ks + 4 * (lane / R);
#pragma unroll
  for (int v = 0; v < Fp<R>::NV; v++)
    if (!rr.sees(kb + val_row<R>(v))) s.set(v, -INFINITY);
}

// A wave's D x R accumulators (lane = row of the result) into its LDS slab, rows of D + 4 floats.
template <int D, int R>
__device__ __forceinline__ void stage_acc(float* slab, const Out<D, R>& acc, int lane) {
  constexpr int DT = D / R, H = Fp<R>::H;
  float* row = slab + (lane % R) * (D + 4) + 4 * DT * (lane / R);
#pragma unroll
  for (int a = 0; a < Fp<R>::AR / 4; a++)
#pragma unroll
    for (int x = 0; x < DT; x++) {   // four consecutive columns: 4 x .. 4 x + 3 of the 4 DT that rows m = 4 H a + 4 h .. + 3 hold
      float4 v;
      v.x = acc.t[(4 * x) % DT][4 * a + (4 * x) / DT];
      v.y = acc.t[(4 * x + 1) % DT][4 * a + (4 * x + 1) / DT];
      v.z = acc.t[(4 * x + 2) % DT][4 * a + (4 * x + 2) / DT];
      v.w = acc.t[(4 * x + 3) % DT][4 * a + (4 * x + 3) / DT];
      *(float4*)(row + 4 * H * DT * a + 4 * x) = v;
    }
}

// Adds the waves' slabs up in wave order and stores rows r < n_rows.  wgt: factor of each (wave, row), or null (1).  Returns which
// rows (bit r = row r of the workgroup) hold a value that is not finite, each in the wave that stored it.
template <int D, int R>
__device__ __forceinline__ uint32_t store_sum(const float* slabs, const float* wgt, float mul, int n_rows, float* dst, int64_t stride) {
  constexpr int TPR = kThreads / R, RPW = R / kWaves;   // threads per row, rows per wave
  const int row = threadIdx.x / TPR, seg = threadIdx.x % TPR;
  float probe = 0.f;
  if (row < n_rows)
    for (int col = 4 * seg; col < D; col += 4 * TPR) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < kWaves; w++) {
        const float4 b = *(const float4*)(slabs + (w * R + row) * (D + 4) + col);
        const float f = wgt ? wgt[w * R + row] : mul;
        a.x = fmaf(b.x, f, a.x); a.y = fmaf(b.y, f, a.y); a.z = fmaf(b.z, f, a.z); a.w = fmaf(b.w, f, a.w);
      }
      *(float4*)(dst + (int64_t)row * stride + col) = a;
      probe = finite_probe(a.x, finite_probe(a.y, finite_probe(a.z, finite_probe(a.w, probe))));
    }
  const uint64_t bad = __ballot(probe != 0.f);
  uint32_t rows = 0;
#pragma unroll
  for (int r = 0; r < RPW; r++)
    if ((bad >> (r * TPR)) & ((1ull << TPR) - 1)) rows |= 1u << (RPW * uni(threadIdx.x >> 6) + r);
  return rows;
}

}  // namespace

// LDS of the three kernels: a slab per wave for its partial result; the first two hold the own rows during the loop.
#define DCP_FENCE() __builtin_amdgcn_sched_barrier(0)

template <int D, int R, bool RANGES>
__global__ __launch_bounds__(kThreads, R == 16 ? 4 : 2) void f32_fwd_kernel(DevGroup g, KTensors t) {
  constexpr int NC = Chunks<D, R>::NC, SLAB = R * (D + 4);
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * SLAB];
  __shared__ float sm[kWaves][R], sl[kWaves][R];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), li = lane % R, lh = lane / R;
  QTile q;
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  if (!q_tile<R, RANGES>(g, t, lane, blockIdx.x, &q)) return;
  own_rows<D, R>(slabs, (const float*)t.q + (int64_t)q.head * t.q_sh, t.q_st, q.q_lo + q.qoff, q.q_hi + q.qoff);
  const float* kb = (const float*)t.k + (int64_t)q.hk * t.k_sh;
  const float* vb = (const float*)t.v + (int64_t)q.hk * t.v_sh;
  const float c_log2 = t.scale * kLog2eF;
  float m = -INFINITY, l = 0.f;
  Out<D, R> o;
  zero(o);
  Walk<kWaves> it(g, q.e0, q.e1, wave);
  bool have = it.template next<RANGES>(q.q_hi, q.rb);
  RowChunk<D, R> kc;
  if (have) load_rows<D, R>(kc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
  __syncthreads();
  while (have) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = it.kind, r0 = ks + it.moff, r1 = c1 - 1 + it.moff;
    Score<R> s;
    s.fill(0.f);
    ColChunk<D, R> vc, vn;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D, R> kn;
      if (c + 1 < NC) load_rows<D, R>(kn, kb, t.k_st, r0, r1, c + 1);
      else load_cols<D, R>(vc, vb, t.v_st, r0, r1, 0);
      DCP_FENCE();
      dot_rows<D, R>(kc, slabs, lane, c, s);
      DCP_FENCE();
      kc = kn;
    }
    if (classify32(kind, ks, c1, q.q_lo, q.q_hi, q.rb) != kFull) mask_vals<R>(s, q, kind, ks, c0, c1, lane);
    float mx = s.get(0);
#pragma unroll
    for (int v = 1; v < Fp<R>::NV; v++) mx = fmaxf(mx, s.get(v));
    mx = own_max<R>(mx);
    const bool raise = (mx - m) * c_log2 > kRaise;
    const float m_new = raise ? mx : m;
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__any(raise)) {
      const float alpha = raise ? __builtin_amdgcn_exp2f((m - m_use) * c_log2) : 1.f;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / R; dt++)
#pragma unroll
        for (int r = 0; r < Fp<R>::AR; r++) o.t[dt][r] *= alpha;
    }
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < Fp<R>::NV; v++) {
      s.set(v, __builtin_amdgcn_exp2f((s.get(v) - m_use) * c_log2));
      sum += s.get(v);
    }
    l += sum;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) {
        load_cols<D, R>(vn, vb, t.v_st, r0, r1, c + 1);
      } else {
        have = it.template next<RANGES>(q.q_hi, q.rb);
        if (have) load_rows<D, R>(kc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
      }
      DCP_FENCE();
      add_cols<D, R>(vc, s, c, o);
      DCP_FENCE();
      vc = vn;
    }
  }
  l = own_sum<R>(l);
  if (lh == 0) { sm[wave][li] = m; sl[wave][li] = l; }
  __syncthreads();   // the own rows' slab is free
  stage_acc<D, R>(slabs + wave * SLAB, o, lane);
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
  uint32_t again = store_sum<D, R>(slabs, &sl[0][0], 1.f, q.n_rows, op, op_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again);
      if (lane_of(lt, r) != lane_of(lt, r)) continue;   // a NaN score: all of the row is NaN already
      const FixRow f = fix_row(q, r);
      const float mr = lane_of(mt, r);
      fix_out<float, D>(a.g, a.t, f, q.hk, (const float*)a.t.q + (int64_t)(f.qi + q.qoff) * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                        mr == -INFINITY ? 0.f : mr * c_log2, lane_of(inv, r), op + r * op_st);
    }
  }
}

// BOTH: the launch holds the dK/dV workgroups as well, which then work out delta and the rescaled LSE for themselves.
template <int D, int R, bool RANGES, bool BOTH>
__device__ __forceinline__ void f32_dq(const DevGroup& g, const KTensors& t, float* slabs, int bid) {
  constexpr int NC = Chunks<D, R>::NC, SLAB = R * (D + 4), W = 4 * Fp<R>::H;
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), li = lane % R, lh = lane / R;
  QTile q;
  if (!q_tile<R, RANGES>(g, t, lane, bid, &q)) return;
  const float* q_lds = slabs;
  const float* do_lds = slabs + SLAB;
  own_rows<D, R>(slabs, (const float*)t.q + (int64_t)q.head * t.q_sh, t.q_st, q.q_lo + q.qoff, q.q_hi + q.qoff);
  own_rows<D, R>(slabs + SLAB, (const float*)t.dout + (int64_t)q.head * t.do_sh, t.do_st, q.q_lo + q.qoff, q.q_hi + q.qoff);
  const int64_t at = (int64_t)q.head * t.q_rows + q.qi + q.qoff;
  const float lse = t.lse[at];
  const float* kb = (const float*)t.k + (int64_t)q.hk * t.k_sh;
  const float* vb = (const float*)t.v + (int64_t)q.hk * t.v_sh;
  Walk<kWaves> it(g, q.e0, q.e1, wave);
  bool have = it.template next<RANGES>(q.q_hi, q.rb);
  // the backward preprocess, fused: delta = sum_d dO * O of the lane's row, left (negated) with the rescaled LSE in
  // the workspace for the dK/dV kernel
  const float* op = (const float*)t.out_in + (int64_t)(q.qi + q.qoff) * t.o_st + (int64_t)q.head * t.o_sh + 4 * lh;
  float4 o[D / W];
#pragma unroll
  for (int j = 0; j < D / W; j++) o[j] = *(const float4*)(op + W * j);
  __syncthreads();
  float delta = 0.f;
#pragma unroll
  for (int j = 0; j < D / W; j++) {
    const float4 x = *(const float4*)(do_lds + li * (D + 4) + 4 * lh + W * j);
    delta = fmaf(o[j].x, x.x, delta); delta = fmaf(o[j].y, x.y, delta);
    delta = fmaf(o[j].z, x.z, delta); delta = fmaf(o[j].w, x.w, delta);
  }
  delta = own_sum<R>(delta);
  const float lse2 = row_lse2(lse, &delta);
  if (!BOTH && wave == 0 && lh == 0 && li < q.n_rows) { t.delta_w[at] = -delta; t.lse2_w[at] = lse2; }
  const float c_log2 = t.scale * kLog2eF;
  Out<D, R> dq;
  zero(dq);
  RowChunk<D, R> rc;
  if (have) load_rows<D, R>(rc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
  while (have) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = it.kind, r0 = ks + it.moff, r1 = c1 - 1 + it.moff;
    Score<R> s, dp;
    s.fill(0.f);
    dp.fill(-delta);
    ColChunk<D, R> cc, cn;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D, R> rn;
      if (c + 1 < NC) load_rows<D, R>(rn, kb, t.k_st, r0, r1, c + 1);
      else load_rows<D, R>(rn, vb, t.v_st, r0, r1, 0);
      DCP_FENCE();
      dot_rows<D, R>(rc, q_lds, lane, c, s);
      DCP_FENCE();
      rc = rn;
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D, R> rn;
      if (c + 1 < NC) load_rows<D, R>(rn, vb, t.v_st, r0, r1, c + 1);
      else load_cols<D, R>(cc, kb, t.k_st, r0, r1, 0);
      DCP_FENCE();
      dot_rows<D, R>(rc, do_lds, lane, c, dp);
      DCP_FENCE();
      rc = rn;
    }
    if (classify32(kind, ks, c1, q.q_lo, q.q_hi, q.rb) != kFull) mask_vals<R>(s, q, kind, ks, c0, c1, lane);
#pragma unroll
    for (int v = 0; v < Fp<R>::NV; v++) s.set(v, __builtin_amdgcn_exp2f(fmaf(s.get(v), c_log2, -lse2)) * dp.get(v));
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) {
        load_cols<D, R>(cn, kb, t.k_st, r0, r1, c + 1);
      } else {
        have = it.template next<RANGES>(q.q_hi, q.rb);
        if (have) load_rows<D, R>(rc, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff, 0);
      }
      DCP_FENCE();
      add_cols<D, R>(cc, s, c, dq);
      DCP_FENCE();
      cc = cn;
    }
  }
  __syncthreads();   // the own rows' slabs are free
  stage_acc<D, R>(slabs + wave * SLAB, dq, lane);
  __syncthreads();
  float* dqp = (float*)t.dq + (int64_t)(q.q_lo + q.qoff) * t.dq_st + (int64_t)q.head * t.dq_sh;
  uint32_t again = store_sum<D, R>(slabs, nullptr, t.scale, q.n_rows, dqp, t.dq_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args(0, BOTH ? 2 * sizeof(DevGroup) : sizeof(DevGroup));
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again);
      const FixRow f = fix_row(q, r);
      const int64_t mem = f.qi + q.qoff;
      fix_dq<float, D>(a.g, a.t, f, q.hk, (const float*)a.t.q + mem * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                       (const float*)a.t.dout + mem * a.t.do_st + (int64_t)q.head * a.t.do_sh, lane_of(lse2, r), lane_of(delta, r), dqp + r * a.t.dq_st);
    }
  }
}

// dK / dV of R keys of one KV head: the waves take the (query head, 32-query tile) pairs of the listed q blocks in turn.
template <int D, int R, bool RANGES, bool BOTH>
__device__ __forceinline__ void f32_dkv(const DevGroup& g, const KTensors& t, float* slabs, int bid) {
  constexpr int NC = Chunks<D, R>::NC, SLAB = R * (D + 4), SUB = kItemRows / R, NV = Fp<R>::NV, NT = Fp<R>::NT;
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  int item, x;
  const int G = t.hq / t.hkv;
  if (!decode_wg(g, t.hkv, SUB, &item, &x, bid)) return;
  const int hk = x / SUB;
  const WorkItem w = plan_load(g.items, item);
  const int koff = uni(w.moff);
  const int row0 = uni(w.tile) * kItemRows + (x % SUB) * R;
  const int n_rows = min(R, uni(w.blk_len) - row0);
  if (n_rows <= 0) return;
  const int k_lo = uni(w.blk_start) + row0, k_hi = k_lo + n_rows - 1;
  const int seq0 = RANGES ? uni(plan_load(g.blk_s0, plan_load(g.unit_blk, uni(w.unit)))) : 0;
  const float* k_lds = slabs;
  const float* v_lds = slabs + SLAB;
  own_rows<D, R>(slabs, (const float*)t.k + (int64_t)hk * t.k_sh, t.k_st, k_lo + koff, k_hi + koff);
  own_rows<D, R>(slabs + SLAB, (const float*)t.v + (int64_t)hk * t.v_sh, t.v_st, k_lo + koff, k_hi + koff);
  Out<D, R> dk, dv;
  zero(dk);
  zero(dv);
  const float c_log2 = t.scale * kLog2eF;
  QWalk<kWaves, RANGES> it(g, uni(w.e0), uni(w.e1), G, wave, t.qbounds);
  auto q_base = [&](int head) { return (const float*)t.q + (int64_t)head * t.q_sh; };
  bool have = it.next(k_lo, k_hi + 1);
  RowChunk<D, R> rc;
  if (have) load_rows<D, R>(rc, q_base(hk * G + it.hh), t.q_st, it.qs() + it.moff, it.q1 - 1 + it.moff, 0);
  __syncthreads();
  while (have) {
    const int qs = it.qs(), q_end = it.q1, r0 = qs + it.moff, r1 = it.q1 - 1 + it.moff, kd = it.kind, head = hk * G + it.hh;
    const bool full = n_rows == R && it.full(k_hi);
    const float* qp = q_base(head);
    const float* dop = (const float*)t.dout + (int64_t)head * t.do_sh;
    const float* op = (const float*)t.out_in + (int64_t)head * t.o_sh;
    const int lim = min(kOther, q_end - qs) - 1;
    Score<R> s, dp, lse2;
    s.fill(0.f);
    dp.fill(0.f);
    ColChunk<D, R> cc, cn;
    RowChunk<D, R> oc;
    float dl[NT], ll[NT];   // BOTH: delta and LSE of rows l % R + R a
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D, R> rn;
      if (c + 1 < NC) {
        load_rows<D, R>(rn, qp, t.q_st, r0, r1, c + 1);
      } else {
        load_rows<D, R>(rn, dop, t.do_st, r0, r1, 0);
        if (!BOTH) dp = load_per_row<R>(t.delta + (int64_t)head * t.q_rows + r0, lim);   // -delta: dP starts from it
        if (BOTH) load_rows<D, R>(oc, op, t.o_st, r0, r1, 0);
      }
      DCP_FENCE();
      dot_rows<D, R>(rc, k_lds, lane, c, s);
      DCP_FENCE();
      rc = rn;
    }
    if (BOTH) {
#pragma unroll
      for (int a = 0; a < NT; a++) {
        dl[a] = 0.f;
        ll[a] = t.lse[(int64_t)head * t.q_rows + r0 + min(lane % R + R * a, lim)];
      }
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      RowChunk<D, R> rn;
      if (c + 1 < NC) load_rows<D, R>(rn, dop, t.do_st, r0, r1, c + 1);
      else load_cols<D, R>(cc, dop, t.do_st, r0, r1, 0);
      DCP_FENCE();
      dot_rows<D, R>(rc, v_lds, lane, c, dp);
      if (BOTH) {
#pragma unroll
        for (int j = 0; j < Chunks<D, R>::NJ; j++)
#pragma unroll
          for (int e = 0; e < 4; e++) dl[j / (Chunks<D, R>::NJ / NT)] = fmaf(oc.c[j][e], rc.c[j][e], dl[j / (Chunks<D, R>::NJ / NT)]);
        if (c + 1 < NC) load_rows<D, R>(oc, op, t.o_st, r0, r1, c + 1);
      }
      DCP_FENCE();
      rc = rn;
    }
    if (BOTH) {
#pragma unroll
      for (int a = 0; a < NT; a++) {
        dl[a] = own_sum<R>(dl[a]);
        ll[a] = row_lse2(ll[a], &dl[a]);
      }
#pragma unroll
      for (int v = 0; v < NV; v++) {
        const int a = v / (NV / NT), src = val_row<R>(v) % R + 4 * (lane / R);
        dp.set(v, dp.get(v) - __shfl(dl[a], src));
        lse2.set(v, __shfl(ll[a], src));
      }
    } else {
      lse2 = load_per_row<R>(t.lse2 + (int64_t)head * t.q_rows + r0, lim);
    }
    if (!full) {
      const int ln = fresh_lane(), kj = k_lo + ln % R;
#pragma unroll
      for (int v = 0; v < NV; v++) {
        const int i = qs + val_row<R>(v) + 4 * (ln / R);
        bool vis = i < q_end && kj <= k_hi;
        if (kd == 1) vis = vis && kj <= i;
        if (RANGES && kd == 2) {
          const int4 rg = range_row(t, min(i, q_end - 1), seq0);
          vis = vis && ((kj >= rg.x && kj < rg.y) || (kj >= rg.z && kj < rg.w));
        }
        if (!vis) s.set(v, -INFINITY);
      }
    }
#pragma unroll
    for (int v = 0; v < NV; v++) {
      s.set(v, __builtin_amdgcn_exp2f(fmaf(s.get(v), c_log2, -lse2.get(v))));
      dp.set(v, dp.get(v) * s.get(v));
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) load_cols<D, R>(cn, dop, t.do_st, r0, r1, c + 1);
      else load_cols<D, R>(cn, qp, t.q_st, r0, r1, 0);
      DCP_FENCE();
      add_cols<D, R>(cc, s, c, dv);
      DCP_FENCE();
      cc = cn;
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c + 1 < NC) {
        load_cols<D, R>(cn, qp, t.q_st, r0, r1, c + 1);
      } else {
        have = it.next(k_lo, k_hi + 1);
        if (have) load_rows<D, R>(rc, q_base(hk * G + it.hh), t.q_st, it.qs() + it.moff, it.q1 - 1 + it.moff, 0);
      }
      DCP_FENCE();
      add_cols<D, R>(cc, dp, c, dk);
      DCP_FENCE();
      cc = cn;
    }
  }
  float* slab = slabs + wave * SLAB;
  __syncthreads();   // the own rows' slabs are free
  stage_acc<D, R>(slab, dk, lane);
  __syncthreads();
  float* dkp = (float*)t.dk + (int64_t)(k_lo + koff) * t.dk_st + (int64_t)hk * t.dk_sh;
  float* dvp = (float*)t.dv + (int64_t)(k_lo + koff) * t.dv_st + (int64_t)hk * t.dv_sh;
  uint32_t again = store_sum<D, R>(slabs, nullptr, t.scale, n_rows, dkp, t.dk_st);
  __syncthreads();
  stage_acc<D, R>(slab, dv, lane);
  __syncthreads();
  again |= store_sum<D, R>(slabs, nullptr, 1.f, n_rows, dvp, t.dv_st);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args(BOTH ? sizeof(DevGroup) : 0, BOTH ? 2 * sizeof(DevGroup) : sizeof(DevGroup));
    const WorkItem w1 = plan_load(a.g.items, item);
    const int s0 = RANGES ? uni(plan_load(a.g.blk_s0, plan_load(a.g.unit_blk, uni(w1.unit)))) : 0;
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again), j = k_lo + r;
      fix_dkv<float, D, BOTH>(a.g, a.t, j, uni(w1.e0), uni(w1.e1), hk, s0, (const float*)a.t.k + (int64_t)(j + koff) * a.t.k_st + (int64_t)hk * a.t.k_sh,
                              (const float*)a.t.v + (int64_t)(j + koff) * a.t.v_st + (int64_t)hk * a.t.v_sh, dkp + r * a.t.dk_st, dvp + r * a.t.dv_st);
    }
  }
}

template <int D, int R, bool RANGES>
__global__ __launch_bounds__(kThreads, R == 16 ? 4 : 2) void f32_dq_kernel(DevGroup g, KTensors t) {
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * R * (D + 4)];
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  f32_dq<D, R, RANGES, false>(g, t, slabs, blockIdx.x);
}

template <int D, int R, bool RANGES>
__global__ __launch_bounds__(kThreads, R == 16 && D < 128 ? 4 : 2) void f32_dkv_kernel(DevGroup g, KTensors t) {
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * R * (D + 4)];
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  f32_dkv<D, R, RANGES, false>(g, t, slabs, blockIdx.x);
}

// The whole backward in one launch: the first n_dkv workgroups (a multiple of 8) are dK/dV's, the others dQ's.
template <int D, int R, bool RANGES>
__global__ __launch_bounds__(kThreads, 2) void f32_bwd_kernel(DevGroup gq, DevGroup gkv, KTensors t, int n_dkv) {
  __shared__ __attribute__((aligned(16))) float slabs[kWaves * R * (D + 4)];
  touch_args<2 * sizeof(DevGroup) + sizeof(KTensors)>();
  if ((int)blockIdx.x < n_dkv) f32_dkv<D, R, RANGES, true>(gkv, t, slabs, blockIdx.x);
  else f32_dq<D, R, RANGES, true>(gq, t, slabs, blockIdx.x - n_dkv);
}

#define DCP_F32_LAUNCH(KERNEL, R, GRID, ...)                                                                               \
  {                                                                                                                       \
    const dim3 grid(GRID), block(kThreads);                                                                               \
    if (t.masked) {                                                                                                       \
      if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, R, true>), grid, block, 0, s, __VA_ARGS__);                           \
      else if (t.d == 64) hipLaunchKernelGGL((KERNEL<64, R, true>), grid, block, 0, s, __VA_ARGS__);                      \
      else hipLaunchKernelGGL((KERNEL<128, R, true>), grid, block, 0, s, __VA_ARGS__);                                    \
    } else {                                                                                                              \
      if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, R, false>), grid, block, 0, s, __VA_ARGS__);                          \
      else if (t.d == 64) hipLaunchKernelGGL((KERNEL<64, R, false>), grid, block, 0, s, __VA_ARGS__);                     \
      else hipLaunchKernelGGL((KERNEL<128, R, false>), grid, block, 0, s, __VA_ARGS__);                                   \
    }                                                                                                                     \
  }

dcp_status_t mfma_f32_fwd(const DevGroup& g, const KTensors& t, int rows, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const int64_t n = xcd_grid(g, t.hkv, t.hq / t.hkv * (kItemRows / rows));
  if (rows == 16) DCP_F32_LAUNCH(f32_fwd_kernel, 16, n, g, t)
  else DCP_F32_LAUNCH(f32_fwd_kernel, 32, n, g, t)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}
dcp_status_t mfma_f32_dq(const DevGroup& g, const KTensors& t, int rows, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const int64_t n = xcd_grid(g, t.hkv, t.hq / t.hkv * (kItemRows / rows));
  if (rows == 16) DCP_F32_LAUNCH(f32_dq_kernel, 16, n, g, t)
  else DCP_F32_LAUNCH(f32_dq_kernel, 32, n, g, t)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}
dcp_status_t mfma_f32_dkv(const DevGroup& g, const KTensors& t, int rows, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const int64_t n = xcd_grid(g, t.hkv, kItemRows / rows);
  if (rows == 16) DCP_F32_LAUNCH(f32_dkv_kernel, 16, n, g, t)
  else if (t.masked) hipLaunchKernelGGL((f32_dkv_kernel<128, 32, true>), dim3(n), dim3(kThreads), 0, s, g, t);   // D = 128 alone
  else hipLaunchKernelGGL((f32_dkv_kernel<128, 32, false>), dim3(n), dim3(kThreads), 0, s, g, t);
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}
// 16 rows a workgroup
dcp_status_t mfma_f32_bwd(const DevGroup& gq, const DevGroup& gkv, const KTensors& t, hipStream_t s) {
  if (gq.n_items + gkv.n_items == 0) return DCP_OK;
  const int64_t n_dkv = xcd_grid(gkv, t.hkv, kItemRows / 16), n = n_dkv + xcd_grid(gq, t.hkv, t.hq / t.hkv * (kItemRows / 16));
  DCP_F32_LAUNCH(f32_bwd_kernel, 16, n, gq, gkv, t, (int)n_dkv)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

}  // namespace dcp
