// Blockwise attention, forward and backward, for bf16 tensors (D = 32, 64, 128) in launches that are too small, or too uneven,
// for the chip: a workgroup's four or eight waves own the same 32 rows and split the other side's tiles (split_rows.h).
//
// What bounds such a launch where a workgroup shares its tiles among 128 rows: one workgroup's chain.  1 000 tokens are 16 key
// tiles in series, ~1.1 us each, on 80 to 104 workgroups; dK/dV items whose blocks are long cannot be cut along their table rows
// and walk all query heads of their group (5 196 tokens, 16/4 heads, blocks of 4 096: 168 tiles, 374 us).  Here the chain is
// 1/8 (1/4) of that and a launch has four times the workgroups.  The price is traffic: a tile is read for 32 rows, not for 128, so
// that a full chip runs at 57 % (forward, dQ with D = 128) to 96 % (dK/dV) of the shared kernels' rate; which launch goes where is
// estimated in api.hip.  Four waves where workgroups are many (two fit on a CU with D = 128), eight where they are few.
// A wave copies its own tiles into its own LDS and waits for nobody, so the loops have no barrier.  One stage per operand is what
// eight waves have room for with D = 128: an operand's next tile is requested as soon as its last product has read the current one
// (K before the softmax, V before the next scores, ..); dK/dV with D < 128 has two stages (16 384 tokens, 16/4 heads, D 64:
// 1 180 -> 1 110 us).  The partial results meet once, in fp32, in LDS.
// Measured, shared kernels -> these: 1 508 tokens, 4/2 heads, D 128, forward / dQ / dK/dV 26 / 30 / 27 us -> 12 / 15 / 18 (here
// dK/dV stays with the first, see api.hip); 4 528 tokens, 4/1 heads, 31 / 39 / 83 -> 20 / 26 / 28; 7 866 tokens, 8/1 heads, D 64,
// 159 / 164 / 783 -> 94 / 110 / 377.
// dQ and dK/dV are one launch where both fit the chip at once, which spares a launch and its start (the dK/dV workgroups work
// delta out for themselves, from O): 620 tokens, 4/2 heads, forward and backward 51 -> 28 us with two launches, 23 with one.
#include "mfma_dkv_kernel.h"
#include "split_rows.h"
#include "tile_layout.h"

namespace dcp {

namespace {

constexpr float kLog2eS = 1.44269504088896340736f;
constexpr float kLn2S = 0.69314718055994530942f;
constexpr int kRows = kSplitRows, kSub = kSplitSub;
constexpr float kRaiseS = 8.f;   // the running maximum is raised when a tile exceeds it by more than 2^8

// P and dS enter their products as one bf16 operand (D = 128) or as three parts that add up to the fp32 values (D < 128), as in
// the kernels that share one tile among their waves.
template <int D> constexpr int kParts = D == 128 ? 1 : 3;
template <int D>
__device__ __forceinline__ void to_parts(const f32x16& s, int c, bf16x8 (&p)[kParts<D>]) {
  if constexpr (D == 128) p[0] = pack_frag(s, c);
  else pack_split(s, c, p);
}

template <int D> constexpr int kTile = kRows * 2 * D;             // bytes of a 32-row tile
template <int D> constexpr int kCopies = kTile<D> / 1024;         // copy instructions per tile
template <int D> constexpr int kSlab = kRows * (D + 4) * 4;       // bytes of a wave's fp32 partial result, rows of D + 4 floats
// a wave's LDS: two tiles, later its slab; in dK/dV, where D < 128 leaves room, two stages of two tiles
template <int D> constexpr int kRegion = kSlab<D> > 2 * kTile<D> ? kSlab<D> : 2 * kTile<D>;
template <int D> constexpr int kStages = D < 128 ? 2 : 1;
template <int D> constexpr int kRegionKv = D < 128 ? 4 * kTile<D> : kRegion<D>;

// Asynchronous copy of rows row0 .. row0 + 31 (past `last`: that row again) into the wave's own tile; stride in elements.
// Instruction u fills the lines 4u .. 4u + 3; its rows differ from instruction 0's in the swizzle by a constant.
template <int D>
__device__ __forceinline__ void copy_tile(char* tile, const bf16_t* base, int64_t stride, int row0, int last) {
  typedef TileLayout<D> L;
  const int lane = fresh_lane(), sb = (int)stride * 2;
  const int x = (lane & 15) ^ L::swz(lane >> 4), row = (lane >> 4) * L::RPL + x / L::CPR, ch = x % L::CPR;
  const char* b = (const char*)uni_ptr((const char*)base + (int64_t)row0 * sb);
  const unsigned lds = lds_addr(tile);
  const int lim = last - row0;
  if (lim >= kRows - 1) {
#pragma unroll
    for (int u = 0; u < kCopies<D>; u++) dma16((unsigned)(row * sb + ((ch ^ L::swz(4 * u)) << 4)), b + (int64_t)(4 * L::RPL * u) * sb, lds + 1024 * u);
  } else {
#pragma unroll
    for (int u = 0; u < kCopies<D>; u++) dma16((unsigned)(min(row + 4 * L::RPL * u, lim) * sb + ((ch ^ L::swz(4 * u)) << 4)), b, lds + 1024 * u);
  }
}

// A tile is read after the wait for its copy, and copied into again after the wait for the reads: no other wave touches it, so
// no barrier is needed.  The copies complete in order: with N newer instructions under way vmcnt(N) waits for the older ones.
template <int N> __device__ __forceinline__ void copies_landed() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void reads_done() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

template <int D>
__device__ __forceinline__ void own_frags(bf16x8 (&f)[D / 16], const void* base, int64_t row, int64_t st, int64_t head_off, int lane) {
  const bf16_t* p = (const bf16_t*)base + row * st + head_off + 8 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) f[ks] = as_frag(*(const uint4*)(p + 16 * ks));
}

// s += A B over D: A the rows of a tile, B the own rows; D = 128 reads one step ahead, more than that it has no registers for
template <int D>
__device__ __forceinline__ f32x16 chain(const Frags<D>& fa, const char* tile, const bf16x8 (&b)[D / 16], f32x16 s) {
  bf16x8 a = fa.rows(tile, 0);
#pragma unroll
  for (int x = 0; x < D / 16; x++) {
    bf16x8 n = a;
    if (x + 1 < D / 16) n = fa.rows(tile, x + 1);
    if (D == 128) __builtin_amdgcn_sched_barrier(0);
    s = mfma(a, b[x], s);
    a = n;
    if (D == 128) __builtin_amdgcn_sched_barrier(0);
  }
  return s;
}

// acc += (columns of the tile) x p, p a score tile as the accumulator holds it
template <int D>
__device__ __forceinline__ void add_cols(const Frags<D>& fa, const char* tile, const f32x16& s, f32x16 (&acc)[D / 32]) {
  if constexpr (D == 128) {
    bf16x8 p[2];
#pragma unroll
    for (int c = 0; c < 2; c++) p[c] = pack_frag(s, c);
    bf16x8 a = fa.cols(tile, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; i++) {
      bf16x8 n = a;
      if (i < 7) n = fa.cols(tile, (i + 1) >> 2, (i + 1) & 3);
      __builtin_amdgcn_sched_barrier(0);
      acc[i & 3] = mfma(a, p[i >> 2], acc[i & 3]);
      a = n;
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int c = 0; c < 2; c++) {
      bf16x8 p[kParts<D>];
      to_parts<D>(s, c, p);
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const bf16x8 a = fa.cols(tile, c, dt);
#pragma unroll
        for (int k = 0; k < kParts<D>; k++) acc[dt] = mfma(a, p[k], acc[dt]);
      }
    }
  }
}

template <int N>
__device__ __forceinline__ void zero(f32x16 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; i++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[i][r] = 0.f;
}

// A wave's D x 32 accumulator tile (lane = row of the result) into its slab.
template <int D>
__device__ __forceinline__ void stage_acc(char* slab, const f32x16 (&acc)[D / 32], int lane) {
  float* row = (float*)slab + (lane & 31) * (D + 4) + 4 * (lane >> 5);
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int a = 0; a < 4; a++)
      *(float4*)(row + 32 * dt + 8 * a) = make_float4(acc[dt][4 * a], acc[dt][4 * a + 1], acc[dt][4 * a + 2], acc[dt][4 * a + 3]);
}

// Columns col .. col + 7 of a row: the waves' slabs added up in wave order, wgt the factor of each (wave, row), or null for `mul`.
template <int D, int NW, int REGION>
__device__ __forceinline__ void slab_sum(const char* lds, int row, int col, const float* wgt, float mul, float (&a)[8]) {
#pragma unroll
  for (int i = 0; i < 8; i++) a[i] = 0.f;
#pragma unroll
  for (int w = 0; w < NW; w++) {
    const float* p = (const float*)(lds + w * REGION) + row * (D + 4) + col;
    const float4 x = *(const float4*)p, y = *(const float4*)(p + 4);
    const float f = wgt ? wgt[w * kRows + row] : mul;
    a[0] = fmaf(x.x, f, a[0]); a[1] = fmaf(x.y, f, a[1]); a[2] = fmaf(x.z, f, a[2]); a[3] = fmaf(x.w, f, a[3]);
    a[4] = fmaf(y.x, f, a[4]); a[5] = fmaf(y.y, f, a[5]); a[6] = fmaf(y.z, f, a[6]); a[7] = fmaf(y.w, f, a[7]);
  }
}

// Stores the sum of the slabs, rows r < n_rows, eight columns a thread.  Returns which rows (bit r = row r of the workgroup) hold
// a value that is not finite, each in the wave that stored it; D = 128 does not ask (see nonfinite.h).
template <int D, int NW, int REGION>
__device__ __forceinline__ uint32_t store_sum(const char* lds, const float* wgt, float mul, int n_rows, bf16_t* dst, int64_t stride) {
  constexpr int CPR = D / 8, N = kRows * CPR, T = 64 * NW;
  uint32_t rows = 0;
#pragma unroll
  for (int x0 = 0; x0 < N; x0 += T) {
    const int x = x0 + threadIdx.x, row = x / CPR, col = 8 * (x % CPR);
    float probe = 0.f;
    if (x < N && row < n_rows) {
      float a[8];
      slab_sum<D, NW, REGION>(lds, row, col, wgt, mul, a);
      uint4 o;
      o.x = pack_bf16x2(a[0], a[1]); o.y = pack_bf16x2(a[2], a[3]); o.z = pack_bf16x2(a[4], a[5]); o.w = pack_bf16x2(a[6], a[7]);
      *(uint4*)(dst + (int64_t)row * stride + col) = o;
      if constexpr (D < 128) {
#pragma unroll
        for (int i = 0; i < 8; i++) probe = finite_probe(a[i], probe);
      }
    }
    if constexpr (D < 128) {
      const uint64_t bad = __ballot(probe != 0.f);
      const int first = (x0 + 64 * uni(threadIdx.x >> 6)) / CPR;
#pragma unroll
      for (int r = 0; r < 64 / CPR; r++)
        if ((bad >> (r * CPR)) & ((1ull << CPR) - 1)) rows |= 1u << ((first + r) & 31);
    }
  }
  return rows;
}

}  // namespace

template <int D, int NW, bool RANGES>
__global__ __launch_bounds__(64 * NW, 2) void split_fwd_kernel(DevGroup g, KTensors t) {
  typedef TileLayout<D> L;
  __shared__ __attribute__((aligned(1024))) char lds[NW * kRegion<D>];
  __shared__ float sm[NW][kRows], sl[NW][kRows];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), li = lane & 31, lh = lane >> 5;
  QTile q;
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  if (!q_tile<kRows, RANGES>(g, t, lane, blockIdx.x, &q)) return;
  const int slot = plan_load(g.unit_out, q.unit);
  char* k_lds = lds + wave * kRegion<D>;
  char* v_lds = k_lds + kTile<D>;
  const bf16_t* kb = (const bf16_t*)t.k + (int64_t)q.hk * t.k_sh;
  const bf16_t* vb = (const bf16_t*)t.v + (int64_t)q.hk * t.v_sh;
  Walk<NW> it(g, q.e0, q.e1, wave);
  bool have = it.template next<RANGES>(q.q_hi, q.rb);
  bf16x8 qf[L::KS];
  own_frags<D>(qf, t.q, q.qi + q.qoff, t.q_st, (int64_t)q.head * t.q_sh, lane);
  if (have) {
    copy_tile<D>(k_lds, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
    copy_tile<D>(v_lds, vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
  }
  Frags<D> fa;
  fa.init(lane);
  const float c_log2 = t.scale * kLog2eS;
  float m = -INFINITY, l = 0.f;
  f32x16 o[L::DT];
  zero(o);
  while (have) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = it.kind;
    copies_landed<kCopies<D>>();   // K (V is newer)
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
    for (int x = 0; x < L::KS; x++) s = mfma(fa.rows(k_lds, x), qf[x], s);
    have = it.template next<RANGES>(q.q_hi, q.rb);
    reads_done();
    if (have) copy_tile<D>(k_lds, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
    if (classify32(kind, ks, c1, q.q_lo, q.q_hi, q.rb) != kFull) mask_keys(s, q, kind, ks, c0, c1, lane);
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; r++) mx = fmaxf(mx, s[r]);
    mx = xhalf_max(mx);
    const bool raise = (mx - m) * c_log2 > kRaiseS;   // lazily, as in the kernel that shares its tiles
    const float m_new = raise ? mx : m;
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float mc = m_use * c_log2;
    if (__any(raise)) {
      const float alpha = raise ? __builtin_amdgcn_exp2f((m - m_use) * c_log2) : 1.f;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < L::DT; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[dt][r] *= alpha;
    }
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r++) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -mc));
      sum += s[r];
    }
    l += sum;
    if (have) copies_landed<kCopies<D>>();   // V (the next K is newer)
    else copies_landed<0>();
#pragma unroll
    for (int c = 0; c < 2; c++) {
      bf16x8 p[kParts<D>];
      to_parts<D>(s, c, p);
#pragma unroll
      for (int dt = 0; dt < L::DT; dt++) {
        const bf16x8 v = fa.cols(v_lds, c, dt);
#pragma unroll
        for (int k = 0; k < kParts<D>; k++) o[dt] = mfma(v, p[k], o[dt]);
      }
    }
    reads_done();
    if (have) copy_tile<D>(v_lds, vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
  }
  l = xhalf_sum(l);
  if (lh == 0) { sm[wave][li] = m; sl[wave][li] = l; }
  stage_acc<D>(k_lds, o, lane);
  __syncthreads();
  // every wave's weight for its rows, the row's LSE
  float mt = -INFINITY, lt = 0.f, f[NW];
#pragma unroll
  for (int w = 0; w < NW; w++) mt = fmaxf(mt, sm[w][li]);
#pragma unroll
  for (int w = 0; w < NW; w++) {
    f[w] = sm[w][li] > -INFINITY ? __builtin_amdgcn_exp2f((sm[w][li] - mt) * c_log2) : 0.f;
    lt = fmaf(f[w], sl[w][li], lt);
  }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  __syncthreads();
  if (wave == 0 && lh == 0) {
#pragma unroll
    for (int w = 0; w < NW; w++) sl[w][li] = f[w] * inv;
    if (li < q.n_rows) {
      const float lse = lt > 0.f ? (mt * c_log2 + __builtin_amdgcn_logf(lt)) * kLn2S : -INFINITY;
      if (slot < 0) t.lse[(int64_t)q.head * t.q_rows + q.q_lo + q.qoff + li] = lse;
      else t.lse[((int64_t)slot * t.hq + q.head) * t.block_size + q.row0 + li] = lse;
    }
  }
  __syncthreads();
  bf16_t* op = slot < 0 ? (bf16_t*)t.out + (int64_t)(q.q_lo + q.qoff) * t.o_st + (int64_t)q.head * t.o_sh
                        : (bf16_t*)t.out + (((int64_t)slot * t.block_size + q.row0) * t.hq + q.head) * D;
  const int64_t op_st = slot < 0 ? t.o_st : (int64_t)t.hq * D;
  uint32_t again = store_sum<D, NW, kRegion<D>>(lds, &sl[0][0], 1.f, q.n_rows, op, op_st);
  if constexpr (D < 128)
    if (again) {
      DCP_WAIT_VMCNT(0);   // the stores above come first
      const KernelArgs a = kernel_args();
      for (; again; again &= again - 1) {
        const int r = __builtin_ctz(again);
        if (lane_of(lt, r) != lane_of(lt, r)) continue;   // a NaN score: all of the row is NaN already
        const FixRow fr = fix_row(q, r);
        const float mr = lane_of(mt, r);
        fix_out<bf16_t, D>(a.g, a.t, fr, q.hk, (const bf16_t*)a.t.q + (int64_t)(fr.qi + q.qoff) * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                           mr == -INFINITY ? 0.f : mr * c_log2, lane_of(inv, r), op + r * op_st);
      }
    }
}

// BOTH: the launch holds the dK/dV workgroups as well, which then work out delta and the rescaled LSE for themselves.
template <int D, int NW, bool RANGES, bool BOTH>
__device__ __forceinline__ void split_dq(const DevGroup& g, const KTensors& t, char* lds, int bid) {
  typedef TileLayout<D> L;
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), lh = lane >> 5;
  QTile q;
  if (!q_tile<kRows, RANGES>(g, t, lane, bid, &q)) return;
  char* k_lds = lds + wave * kRegion<D>;
  char* v_lds = k_lds + kTile<D>;
  const bf16_t* kb = (const bf16_t*)t.k + (int64_t)q.hk * t.k_sh;
  const bf16_t* vb = (const bf16_t*)t.v + (int64_t)q.hk * t.v_sh;
  const int64_t at = (int64_t)q.head * t.q_rows + q.qi + q.qoff;
  const float lse = t.lse[at];
  bf16x8 qf[L::KS], dof[L::KS];
  own_frags<D>(dof, t.dout, q.qi + q.qoff, t.do_st, (int64_t)q.head * t.do_sh, lane);
  float delta = 0.f;
  {
    // the backward preprocess, fused: delta = sum_d dO * O of the lane's row, left (negated) with the rescaled LSE in the
    // workspace for the dK/dV kernel
    bf16x8 of[L::KS];
    own_frags<D>(of, t.out_in, q.qi + q.qoff, t.o_st, (int64_t)q.head * t.o_sh, lane);
    own_frags<D>(qf, t.q, q.qi + q.qoff, t.q_st, (int64_t)q.head * t.q_sh, lane);
#pragma unroll
    for (int x = 0; x < L::KS; x++)
#pragma unroll
      for (int e = 0; e < 8; e++) delta = fmaf((float)of[x][e], (float)dof[x][e], delta);
  }
  Walk<NW> it(g, q.e0, q.e1, wave);
  bool have = it.template next<RANGES>(q.q_hi, q.rb);
  if (have) {
    copy_tile<D>(v_lds, vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
    copy_tile<D>(k_lds, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
  }
  delta = xhalf_sum(delta);
  float lse2;
  if constexpr (D == 128) lse2 = fmaxf(lse * kLog2eS, -3.402823466e38f);
  else lse2 = row_lse2(lse, &delta);
  if (!BOTH && wave == 0 && lh == 0 && (lane & 31) < q.n_rows) { t.delta_w[at] = -delta; t.lse2_w[at] = lse2; }
  Frags<D> fa;
  fa.init(lane);
  const float c_log2 = t.scale * kLog2eS;
  f32x16 dq[L::DT];
  zero(dq);
  while (have) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = it.kind;
    copies_landed<kCopies<D>>();   // V (K is newer)
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = -delta; }
    dp = chain<D>(fa, v_lds, dof, dp);
    have = it.template next<RANGES>(q.q_hi, q.rb);
    reads_done();
    if (have) {
      copy_tile<D>(v_lds, vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
      copies_landed<kCopies<D>>();   // K (the next V is newer)
    } else {
      copies_landed<0>();
    }
    s = chain<D>(fa, k_lds, qf, s);
    if (classify32(kind, ks, c1, q.q_lo, q.q_hi, q.rb) != kFull) mask_keys(s, q, kind, ks, c0, c1, lane);
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lse2)) * dp[r];
    add_cols<D>(fa, k_lds, s, dq);
    reads_done();
    if (have) copy_tile<D>(k_lds, kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
  }
  stage_acc<D>(k_lds, dq, lane);
  __syncthreads();
  bf16_t* dqp = (bf16_t*)t.dq + (int64_t)(q.q_lo + q.qoff) * t.dq_st + (int64_t)q.head * t.dq_sh;
  uint32_t again = store_sum<D, NW, kRegion<D>>(lds, nullptr, t.scale, q.n_rows, dqp, t.dq_st);
  if constexpr (D < 128)
    if (again) {
      DCP_WAIT_VMCNT(0);   // the stores above come first
      const KernelArgs a = kernel_args(0, BOTH ? 2 * sizeof(DevGroup) : sizeof(DevGroup));
      for (; again; again &= again - 1) {
        const int r = __builtin_ctz(again);
        const FixRow f = fix_row(q, r);
        const int64_t mem = f.qi + q.qoff;
        fix_dq<bf16_t, D>(a.g, a.t, f, q.hk, (const bf16_t*)a.t.q + mem * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                          (const bf16_t*)a.t.dout + mem * a.t.do_st + (int64_t)q.head * a.t.do_sh, lane_of(lse2, r), lane_of(delta, r), dqp + r * a.t.dq_st);
      }
    }
}

// per wave, for the query rows of a tile: lse2 [64], -delta [64], ranges [64] (32 rows, and what the other lanes of a copy repeat)
template <bool RANGES> constexpr int kRowBytesLds = RANGES ? 1536 : 512;

// dK / dV of 32 keys of one KV head: the waves take the (query head, 32-query tile) pairs of the listed q blocks in turn.
template <int D, int NW, bool RANGES, bool BOTH>
__device__ __forceinline__ void split_dkv(const DevGroup& g, const KTensors& t, char* lds, char* row_lds, int bid) {
  typedef TileLayout<D> L;
  int item, x;
  if (!decode_wg(g, t.hkv, kSub, &item, &x, bid)) return;
  const int hk = x / kSub, G = t.hq / t.hkv;
  const WorkItem w = plan_load(g.items, item);
  const int wave = uni(threadIdx.x >> 6);
  const int koff = uni(w.moff), trow = (x % kSub) * kRows;   // trow: first row inside the 128-key item
  const int row0 = uni(w.tile) * (kSub * kRows) + trow;
  const int n_rows = min(kRows, uni(w.blk_len) - row0);
  if (n_rows <= 0) return;
  const int k_lo = uni(w.blk_start) + row0, k_end = k_lo + n_rows;
  const int seq0 = RANGES ? uni(plan_load(g.blk_s0, plan_load(g.unit_blk, uni(w.unit)))) : 0;
  char* region = lds + wave * kRegionKv<D>;
  char* do_lds = region;
  char* q_lds = do_lds + kTile<D>;
  char* lse_lds = row_lds + wave * (kStages<D> * kRowBytesLds<RANGES>);
  char* dl_lds = lse_lds + 256;
  char* rg_lds = lse_lds + 512;
  int stage = 0;
  auto other_stage = [&]() {
    const int x = stage ? -1 : 1;
    stage ^= 1;
    do_lds += x * 2 * kTile<D>; q_lds += x * 2 * kTile<D>;
    lse_lds += x * kRowBytesLds<RANGES>; dl_lds += x * kRowBytesLds<RANGES>; rg_lds += x * kRowBytesLds<RANGES>;
  };
  QWalk<NW, RANGES> it(g, uni(w.e0), uni(w.e1), G, wave, t.qbounds);
  // what a tile needs first (dO and the row values), and Q, which is free last.  With one stage (D = 128) the next dO is under way
  // during the product that still reads Q; with two both are during the whole of the current tile.
  auto copy_do = [&]() {
    const int head = hk * G + it.hh, r0 = it.qs() + it.moff, last = it.q1 - 1 + it.moff;
    const unsigned ql = (unsigned)min(fresh_lane(), last - r0);
    dma4(ql * 4u, uni_ptr((BOTH ? t.lse : t.lse2) + (int64_t)head * t.q_rows + r0), lds_addr(lse_lds));
    if (!BOTH) dma4(ql * 4u, uni_ptr(t.delta + (int64_t)head * t.q_rows + r0), lds_addr(dl_lds));
    if (RANGES && it.kind == 2 && t.window <= 0) dma16(ql * 16u, uni_ptr(t.ranges + 4 * (int64_t)it.qs()), lds_addr(rg_lds));
    copy_tile<D>(do_lds, (const bf16_t*)t.dout + (int64_t)head * t.do_sh, t.do_st, r0, last);
  };
  auto copy_q = [&]() {
    copy_tile<D>(q_lds, (const bf16_t*)t.q + (int64_t)(hk * G + it.hh) * t.q_sh, t.q_st, it.qs() + it.moff, it.q1 - 1 + it.moff);
  };
  // BOTH: the tile's rows of O, for delta; requested with its dO, or (D = 128, no registers to keep them in) with the wait for it
  bf16x8 of[BOTH ? L::KS : 1];
  auto load_o = [&]() {
    if constexpr (BOTH) {
      const int lane = fresh_lane(), row = min(it.qs() + (lane & 31), it.q1 - 1) + it.moff;
      own_frags<D>(of, t.out_in, row, t.o_st, (int64_t)(hk * G + it.hh) * t.o_sh, lane);
    }
  };
  bool have = it.next(k_lo, k_end);
  bf16x8 kf[L::KS], vf[L::KS];
  {
    const int lane = threadIdx.x & 63;
    const int kl = min(k_lo + (lane & 31), k_end - 1) + koff;
    own_frags<D>(kf, t.k, kl, t.k_st, (int64_t)hk * t.k_sh, lane);
    own_frags<D>(vf, t.v, kl, t.v_st, (int64_t)hk * t.v_sh, lane);
  }
  if (have) {
    if (D < 128) load_o();
    copy_do();
    copy_q();
  }
  f32x16 dk[L::DT], dv[L::DT];
  zero(dk);
  zero(dv);
  const float c_log2 = t.scale * kLog2eS;
  while (have) {
    const int lane = fresh_lane(), lh = lane >> 5;
    Frags<D> fa;
    fa.init(lane);
    const int qs = it.qs(), q1 = it.q1, kind = it.kind;
    const bool full = n_rows == kRows && it.full(k_end - 1);
    if (D == 128) {
      load_o();
      copies_landed<kCopies<D>>();   // dO and the row values (Q is newer)
    } else {
      copies_landed<0>();
    }
    uint32_t vis = 0xffffffffu;
    if (!full) {
      // which of the 32 keys query row (l & 31) sees, as a bit mask of lane l (see mfma_dkv_kernel.h)
      const int row = lane & 31, i = qs + row;
      int lo1 = 0, hi1 = kind == 1 ? i + 1 : INT32_MAX, lo2 = 0, hi2 = 0;
      if (RANGES && kind == 2) {
        int4 rg;
        if (t.window > 0) rg = range_row(t, i, seq0);
        else rg = ((const int4*)rg_lds)[row];
        lo1 = rg.x; hi1 = rg.y; lo2 = rg.z; hi2 = rg.w;
      }
      vis = (keys_below(hi1, k_lo) & ~keys_below(lo1, k_lo)) | (keys_below(hi2, k_lo) & ~keys_below(lo2, k_lo));
      vis &= keys_below(k_end, k_lo);
      vis = i < q1 ? vis : 0u;
    }
    if constexpr (BOTH) {
      float delta = 0.f;
#pragma unroll
      for (int ks = 0; ks < L::KS; ks++) {
        const bf16x8 d = fa.rows(do_lds, ks);
#pragma unroll
        for (int e = 0; e < 8; e++) delta = fmaf((float)of[ks][e], (float)d[e], delta);
      }
      delta = xhalf_sum(delta);
      const float lse = ((const float*)lse_lds)[lane & 31];
      const float lse2 = D == 128 ? fmaxf(lse * kLog2eS, -3.402823466e38f) : row_lse2(lse, &delta);
      ((float*)lse_lds)[lane & 31] = lse2;
      ((float*)dl_lds)[lane & 31] = -delta;
    }
    const char* do_cur = do_lds;
    const char* q_cur = q_lds;
    const char* lse_cur = lse_lds;
    const char* dl_cur = dl_lds;
    if constexpr (D < 128) {
      have = it.next(k_lo, k_end);
      other_stage();
      reads_done();
      if (have) { load_o(); copy_do(); copy_q(); }
    }
    f32x16 s, dp;
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const float4 d4 = *(const float4*)(dl_cur + 4 * (8 * a + 4 * lh));
      dp[4 * a] = d4.x; dp[4 * a + 1] = d4.y; dp[4 * a + 2] = d4.z; dp[4 * a + 3] = d4.w;
    }
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = 0.f;
    dp = chain<D>(fa, do_cur, vf, dp);
    if (D == 128) copies_landed<0>();   // Q
    s = chain<D>(fa, q_cur, kf, s);
    if (!full) {
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int r0 = acc_row(r);
        const uint64_t cond = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)vis, r0) |
                              ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)vis, r0 + 4) << 32);
        s[r] = __builtin_amdgcn_inverse_ballot_w64(cond) ? s[r] : -INFINITY;
      }
    }
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const float4 l4 = *(const float4*)(lse_cur + 4 * (8 * a + 4 * lh));
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
      for (int b = 0; b < 4; b++) {
        const int r = 4 * a + b;
        s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lv[b]));
        dp[r] *= s[r];
      }
    }
    // Eight waves, two on a SIMD: the one that multiplies goes before the other.  D 64, 16 384 tokens of which 10 829 in one sequence, 16/4
    // heads: 1 111 -> 1 075 us, 4 000 tokens, 8/2 heads: 52.7 -> 49.6; D 32: 673 -> 672.  Four waves: 1 057 -> 1 076.  Around the scores'
    // products: nothing.
    constexpr bool kFirst = D < 128 && NW == 8 && !BOTH;
    if constexpr (kFirst) __builtin_amdgcn_s_setprio(1);
    add_cols<D>(fa, do_cur, s, dv);
    if constexpr (D == 128) {
      have = it.next(k_lo, k_end);
      reads_done();
      if (have) copy_do();
    }
    add_cols<D>(fa, q_cur, dp, dk);
    if constexpr (kFirst) __builtin_amdgcn_s_setprio(0);
    if constexpr (D == 128) {
      reads_done();
      if (have) copy_q();
    }
  }
  const int lane = fresh_lane();
  bf16_t* dkp = (bf16_t*)t.dk + (int64_t)(k_lo + koff) * t.dk_st + (int64_t)hk * t.dk_sh;
  bf16_t* dvp = (bf16_t*)t.dv + (int64_t)(k_lo + koff) * t.dv_st + (int64_t)hk * t.dv_sh;
  stage_acc<D>(region, dk, lane);
  __syncthreads();
  uint32_t again = store_sum<D, NW, kRegionKv<D>>(lds, nullptr, t.scale, n_rows, dkp, t.dk_st);
  __syncthreads();
  stage_acc<D>(region, dv, lane);
  __syncthreads();
  again |= store_sum<D, NW, kRegionKv<D>>(lds, nullptr, 1.f, n_rows, dvp, t.dv_st);
  if constexpr (D < 128)
    if (again) {
      DCP_WAIT_VMCNT(0);   // the stores above come first
      const KernelArgs a = kernel_args(BOTH ? sizeof(DevGroup) : 0, BOTH ? 2 * sizeof(DevGroup) : sizeof(DevGroup));
      const WorkItem w1 = plan_load(a.g.items, item);
      const int s0 = RANGES ? uni(plan_load(a.g.blk_s0, plan_load(a.g.unit_blk, uni(w1.unit)))) : 0;
      for (; again; again &= again - 1) {
        const int r = __builtin_ctz(again), j = k_lo + r;
        fix_dkv<bf16_t, D, BOTH>(a.g, a.t, j, uni(w1.e0), uni(w1.e1), hk, s0, (const bf16_t*)a.t.k + (int64_t)(j + koff) * a.t.k_st + (int64_t)hk * a.t.k_sh,
                           (const bf16_t*)a.t.v + (int64_t)(j + koff) * a.t.v_st + (int64_t)hk * a.t.v_sh, dkp + r * a.t.dk_st, dvp + r * a.t.dv_st);
      }
    }
}

template <int D, int NW, bool RANGES>
__global__ __launch_bounds__(64 * NW, 2) void split_dq_kernel(DevGroup g, KTensors t) {
  __shared__ __attribute__((aligned(1024))) char lds[NW * kRegion<D>];
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  split_dq<D, NW, RANGES, false>(g, t, lds, blockIdx.x);
}

template <int D, int NW, bool RANGES>
__global__ __launch_bounds__(64 * NW, 2) void split_dkv_kernel(DevGroup g, KTensors t) {
  __shared__ __attribute__((aligned(1024))) char lds[NW * kRegionKv<D>];
  __shared__ __attribute__((aligned(1024))) char row_lds[NW * kStages<D> * kRowBytesLds<RANGES>];
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  split_dkv<D, NW, RANGES, false>(g, t, lds, row_lds, blockIdx.x);
}

// The whole backward in one launch: the first n_dkv workgroups (a multiple of 8) are dK/dV's, the others dQ's.
template <int D, int NW, bool RANGES>
__global__ __launch_bounds__(64 * NW, 2) void split_bwd_kernel(DevGroup gq, DevGroup gkv, KTensors t, int n_dkv) {
  __shared__ __attribute__((aligned(1024))) char lds[NW * kRegionKv<D>];
  __shared__ __attribute__((aligned(1024))) char row_lds[NW * kStages<D> * kRowBytesLds<RANGES>];
  touch_args<2 * sizeof(DevGroup) + sizeof(KTensors)>();
  if ((int)blockIdx.x < n_dkv) split_dkv<D, NW, RANGES, true>(gkv, t, lds, row_lds, blockIdx.x);
  else split_dq<D, NW, RANGES, true>(gq, t, lds, blockIdx.x - n_dkv);
}

#define DCP_SPLIT_LAUNCH(KERNEL, NW, GRID, ...)                                                                           \
  {                                                                                                                       \
    const dim3 grid(GRID), block(64 * NW);                                                                                \
    if (t.masked) {                                                                                                       \
      if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, NW, true>), grid, block, 0, s, __VA_ARGS__);                          \
      else if (t.d == 64) hipLaunchKernelGGL((KERNEL<64, NW, true>), grid, block, 0, s, __VA_ARGS__);                     \
      else hipLaunchKernelGGL((KERNEL<128, NW, true>), grid, block, 0, s, __VA_ARGS__);                                   \
    } else {                                                                                                              \
      if (t.d == 32) hipLaunchKernelGGL((KERNEL<32, NW, false>), grid, block, 0, s, __VA_ARGS__);                         \
      else if (t.d == 64) hipLaunchKernelGGL((KERNEL<64, NW, false>), grid, block, 0, s, __VA_ARGS__);                    \
      else hipLaunchKernelGGL((KERNEL<128, NW, false>), grid, block, 0, s, __VA_ARGS__);                                  \
    }                                                                                                                     \
  }

// waves: 4 or 8 per workgroup
dcp_status_t mfma_split_fwd(const DevGroup& g, const KTensors& t, int waves, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const int64_t n = xcd_grid(g, t.hkv, t.hq / t.hkv * kSub);
  if (waves == 4) DCP_SPLIT_LAUNCH(split_fwd_kernel, 4, n, g, t)
  else DCP_SPLIT_LAUNCH(split_fwd_kernel, 8, n, g, t)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}
dcp_status_t mfma_split_dq(const DevGroup& g, const KTensors& t, int waves, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const int64_t n = xcd_grid(g, t.hkv, t.hq / t.hkv * kSub);
  if (waves == 4) DCP_SPLIT_LAUNCH(split_dq_kernel, 4, n, g, t)
  else DCP_SPLIT_LAUNCH(split_dq_kernel, 8, n, g, t)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}
dcp_status_t mfma_split_dkv(const DevGroup& g, const KTensors& t, int waves, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const int64_t n = xcd_grid(g, t.hkv, kSub);
  if (waves == 4) DCP_SPLIT_LAUNCH(split_dkv_kernel, 4, n, g, t)
  else DCP_SPLIT_LAUNCH(split_dkv_kernel, 8, n, g, t)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}
dcp_status_t mfma_split_bwd(const DevGroup& gq, const DevGroup& gkv, const KTensors& t, int waves, hipStream_t s) {
  if (gq.n_items + gkv.n_items == 0) return DCP_OK;
  const int64_t n_dkv = xcd_grid(gkv, t.hkv, kSub), n = n_dkv + xcd_grid(gq, t.hkv, t.hq / t.hkv * kSub);
  if (waves == 4) DCP_SPLIT_LAUNCH(split_bwd_kernel, 4, n, gq, gkv, t, (int)n_dkv)
  else DCP_SPLIT_LAUNCH(split_bwd_kernel, 8, n, gq, gkv, t, (int)n_dkv)
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

}  // namespace dcp
