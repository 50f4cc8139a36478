// Blockwise attention, forward and backward, for fp32 tensors (D = 32, 64) on bf16 MFMA: every fp32 operand is the sum of three bf16
// parts.
//
// Why: an fp32 MFMA has a sixteenth of the bf16 rate, so fp32 numbers in parts are the faster operands as long as a product takes fewer
// than sixteen.  Rounded to nearest, three parts of 8 bits hold all 24 bits of a number (x = h + m + l, |m| <= 2^-8 |x|, |l| <= 2^-17 |x|),
// and of the nine products of two such sums the six largest are kept: h h, h m, m h, m m, h l, l h.  What is left out is below 2^-24 of
// the product, and the sums over a tile start at zero and are added to the running ones by one rounded addition, where a chain of fp32
// MFMAs rounds the running sum once per two products.  Relative errors against 64 bits (norms; 8 192 tokens, 8/2 heads, D 64), fp32 MFMA ->
// these: out 1.23e-7 -> 0.82e-7, LSE 6.08e-8 -> 6.08e-8, dQ 3.78e-7 -> 3.52e-7, dK 8.30e-7 -> 3.87e-7, dV 8.04e-7 -> 3.24e-7.
//
// What bounds it: matrix and vector pipe together.  Cutting a value takes 5.5 vector instructions, a 32 x 32 tile 48 MFMAs (forward, D 64)
// to 96 (dK/dV), so a wave that cuts its own tiles works as long on that as on the products; the chip runs the full launches at 1.0 to
// 1.25 PFLOP/s of bf16 products, the rate that it holds on real data in the kernels for bf16 tensors too.
//
// Forward and dQ: tiles of 32 rows of K and V are fetched to registers, cut once for all waves of a group and put into LDS as three
// planes, from which rows and transposed columns are read as in bf16.  A step has two barriers, and what one half of it reads is written
// in the other, so that one buffer per operand is enough:
//   forward  scores from K, V written | P V, next K written
//   dQ       dP from V, K written     | scores and dQ from K, next V written
// Where the chip is full of equal work a workgroup is one group of four waves that share their tiles (two or three workgroups on a CU, whose
// halves of a step fall beside one another); elsewhere it is two groups of four waves (D 64) or four of two (D 32) that take the tiles in
// turn, half a step apart, and meet at the end.  16 384 tokens in 8 sequences, 16/4 heads, D 64, one group / two: forward 362 / 401 us, dQ 490 /
// 587; 8 192 tokens of which 5 582 in one sequence, 8/2 heads: 303 / 227, 380 / 324.
// Against fp32 MFMA with 32 rows a workgroup, the last batch: forward / dQ / dK/dV 357 / 500 / 723 (16 rows) -> 227 / 324 / 466 us, and 1 to 3 %
// more with the factors of kUp below.
#include "mfma_dkv_kernel.h"
#include "query_rows.h"
#include "split_rows.h"
#include "tile_layout.h"

namespace dcp {

namespace {

// A bf16 ends at 2^-133, an fp32 number at 2^-149: times 2^16 every one has three parts that add up to it.  So the operands that a result is
// linear in are cut times 2^16 (V in the forward; K, V and dO in dQ; Q, dO and V in dK/dV, and dS is 2^32 times itself through dP), and the
// sums are put right before they are stored.  What overflows for it, operands of 2^112 and gradients of 2^80, is not finite in the parts and
// worked out again.  64 more multiplications a tile in dK/dV (96 values are cut), 8 and 16 in the others: 8 192 tokens, 8/2 heads, forward / dQ /
// dK/dV 237 / 336 / 484 -> 240 / 337 / 496 us.  Not so P, and Q and K in the forward's scores: their last bits, at 2^-134, count in a weight
// below 2^-117 (which has lost as many to the rounding of its exponent, and is 0 below 2^-126) and in a score against a factor beyond 2^108.
constexpr float kUp = 0x1p16f, kDown = 0x1p-16f;
constexpr float kLn2P = 0.69314718055994530942f;
constexpr float kRaiseP = 8.f;   // the running maximum is raised when a tile exceeds it by more than 2^8
constexpr int kTR = 32;          // rows of a tile of the other side

template <int D> constexpr int kPlane = kTR * 2 * D;             // bytes of one part of a tile
template <int D> constexpr int kOperand = 3 * kPlane<D>;
template <int D> constexpr int kSlabP = kTR * (D + 4);           // floats of a wave's result, rows of D + 4

typedef float pf32x4 __attribute__((ext_vector_type(4)));

// Two values as two bf16 of each part, rounded to nearest: the remainders are exact, and the last one fits.
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = pack_bf16x2(a, b);
  a -= __uint_as_float(h << 16); b -= __uint_as_float(h & 0xffff0000u);
  m = pack_bf16x2(a, b);
  a -= __uint_as_float(m << 16); b -= __uint_as_float(m & 0xffff0000u);
  l = pack_bf16x2(a, b);
}
struct Parts { bf16x8 p[3]; };
__device__ __forceinline__ Parts split8(const float (&x)[8], float mul = 1.f) {
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; e++) split2(x[2 * e] * mul, x[2 * e + 1] * mul, w[0][e], w[1][e], w[2][e]);
  Parts r;
#pragma unroll
  for (int k = 0; k < 3; k++) r.p[k] = as_frag(make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]));
  return r;
}
// registers 8c .. 8c + 7 of a score tile
__device__ __forceinline__ Parts split_acc(const f32x16& s, int c) {
  const float x[8] = {s[8 * c], s[8 * c + 1], s[8 * c + 2], s[8 * c + 3], s[8 * c + 4], s[8 * c + 5], s[8 * c + 6], s[8 * c + 7]};
  return split8(x);
}

// c += a b, the small products first
__device__ __forceinline__ f32x16 mul6(const Parts& a, const Parts& b, f32x16 c) {
  c = mfma(a.p[2], b.p[0], c);
  c = mfma(a.p[0], b.p[2], c);
  c = mfma(a.p[1], b.p[1], c);
  c = mfma(a.p[1], b.p[0], c);
  c = mfma(a.p[0], b.p[1], c);
  return mfma(a.p[0], b.p[0], c);
}

template <int D> struct OwnParts { Parts s[D / 16]; };   // the lane's row: floats 16 ks + 8 h .. + 7 of each step ks
template <int D>
__device__ __forceinline__ void read_own(float (&x)[D / 16][8], const void* base, int64_t row, int64_t st, int64_t head_off, int lane) {
  const float* p = (const float*)base + row * st + head_off + 8 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) load8<float>(p + 16 * ks, x[ks]);
}
template <int D>
__device__ __forceinline__ void cut_own(OwnParts<D>& o, const float (&x)[D / 16][8], float mul = 1.f) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) o.s[ks] = split8(x[ks], mul);
}

// Own rows that meet a tile times kUp in the scores are cut times kDown, so that the products are the scores and overflow no sooner; small
// ones, whose last bits that would take, times 2^32, and the scores' factor makes up for it.
template <int D>
__device__ __forceinline__ bool are_small(const float (&x)[D / 16][8]) {
  float m = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++)
#pragma unroll
    for (int e = 0; e < 8; e++) m = fmaxf(m, fabsf(x[ks][e]));
  return !__any(m >= 0x1p-40f);
}
__device__ __forceinline__ float own_mul(bool small) { return small ? 0x1p32f : kDown; }
__device__ __forceinline__ float score_factor(float scale, bool small) { return scale * kLog2e * (small ? 0x1p-48f : 1.f); }

// ... and into LDS, as a tile of 32 rows
template <int D>
__device__ __forceinline__ void put_own(char* lds, const Frags<D>& fa, const OwnParts<D>& o) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++)
#pragma unroll
    for (int k = 0; k < 3; k++) *(uint4*)(lds + k * kPlane<D> + (fa.rm ^ (ks << 5))) = __builtin_bit_cast(uint4, o.s[ks].p[k]);
}

template <int D>
__device__ __forceinline__ Parts get_own(const char* lds, const Frags<D>& fa, int ks) {
  Parts a;
#pragma unroll
  for (int k = 0; k < 3; k++) a.p[k] = fa.rows(lds + k * kPlane<D>, ks);
  return a;
}

// A tile of the other side on its way: memory -> registers -> three planes in LDS, by the 64 RG threads of a group, eight floats at a
// time.
template <int D, int RG>
struct Fetch {
  static constexpr int CPR = D / 8, N = kTR * CPR, T = 64 * RG, PER = N < T ? 1 : N / T;
  pf32x4 v[PER][2];
  static __device__ __forceinline__ int tid() { return (int)(fresh_lane() + (uni(threadIdx.x >> 6) % RG) * 64); }
  static __device__ __forceinline__ bool idle() { return N < T && uni(threadIdx.x >> 6) % RG >= N / 64; }
  // rows row0 .. row0 + 31, past `last` that row again; head applied to base, stride in elements
  __device__ __forceinline__ void load(const float* base, int64_t stride, int row0, int last) {
    if (idle()) return;
    typedef const __attribute__((address_space(1))) char* gp;
    const gp b = (gp)(uint64_t)uni_ptr(base + (int64_t)row0 * stride);
    const int x = tid(), lim = last - row0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const unsigned off = (unsigned)min((x + T * i) / CPR, lim) * (unsigned)stride * 4u + 32u * ((x + T * i) % CPR);
      v[i][0] = *(const __attribute__((address_space(1))) pf32x4*)(b + off);
      v[i][1] = *(const __attribute__((address_space(1))) pf32x4*)(b + off + 16);
    }
  }
  __device__ __forceinline__ void put(char* lds, float mul = 1.f) const {
    if (idle()) return;
    const int x = tid();
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const float f[8] = {v[i][0][0], v[i][0][1], v[i][0][2], v[i][0][3], v[i][1][0], v[i][1][1], v[i][1][2], v[i][1][3]};
      const Parts q = split8(f, mul);
      char* at = lds + TileLayout<D>::off((x + T * i) / CPR, (x + T * i) % CPR);
#pragma unroll
      for (int k = 0; k < 3; k++) *(uint4*)(at + k * kPlane<D>) = __builtin_bit_cast(uint4, q.p[k]);
    }
  }
};

// s += A B over D: A the rows of a tile, B the own rows
template <int D>
__device__ __forceinline__ f32x16 dot_parts(const Frags<D>& fa, const char* tile, const OwnParts<D>& b, f32x16 s) {
#pragma unroll
  for (int x = 0; x < D / 16; x++) s = mul6(get_own<D>(tile, fa, x), b.s[x], s);
  return s;
}
// (columns 32 dt .. of the tile) x p, p the parts of a score tile as the accumulator holds it
template <int D>
__device__ __forceinline__ f32x16 cols_parts(const Frags<D>& fa, const char* tile, const Parts (&p)[2], int dt) {
  f32x16 x;
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = 0.f;
#pragma unroll
  for (int c = 0; c < 2; c++) {
    Parts a;
#pragma unroll
    for (int k = 0; k < 3; k++) a.p[k] = fa.cols(tile + k * kPlane<D>, c, dt);
    x = mul6(a, p[c], x);
  }
  return x;
}

template <int N>
__device__ __forceinline__ void clear(f32x16 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; i++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[i][r] = 0.f;
}

// A wave's D x 32 accumulator tile (lane = row of the result), times mul, into its slab, rows of D + 4 floats.
template <int D>
__device__ __forceinline__ void stage_slab(float* slab, const f32x16 (&acc)[D / 32], float mul, int lane) {
  float* row = slab + (lane & 31) * (D + 4) + 4 * (lane >> 5);
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int a = 0; a < 4; a++)
      *(float4*)(row + 32 * dt + 8 * a) = make_float4(acc[dt][4 * a] * mul, acc[dt][4 * a + 1] * mul, acc[dt][4 * a + 2] * mul, acc[dt][4 * a + 3] * mul);
}

// Rows r0 .. r0 + ROWS - 1 of NG slabs (`pitch` floats apart) added up in order, each times its factor (one for all, or lane r of an
// array of one per slab for row r), rows r < n_valid stored.  Returns which rows hold a value that is not finite, as a bit mask.
template <int NG> __device__ __forceinline__ float slab_factor(const float (&f)[NG], int w, int r) { return __shfl(f[w], r); }
__device__ __forceinline__ float slab_factor(float f, int, int) { return f; }
template <int D, int NG, int ROWS, class F>
__device__ __forceinline__ uint32_t store_slabs(const float* slab, int pitch, int r0, const F& mul, int n_valid, float* dst, int64_t stride, int lane) {
  constexpr int LPR = D / 4, RPI = 64 / LPR;   // lanes per row, rows per instruction
  uint32_t rows = 0;
#pragma unroll
  for (int i = 0; i < ROWS; i += RPI) {
    const int r = r0 + i + lane / LPR, col = 4 * (lane % LPR);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < NG; w++) {
      const float4 b = *(const float4*)(slab + w * pitch + r * (D + 4) + col);
      const float f = slab_factor(mul, w, r);
      a.x = fmaf(b.x, f, a.x); a.y = fmaf(b.y, f, a.y); a.z = fmaf(b.z, f, a.z); a.w = fmaf(b.w, f, a.w);
    }
    float probe = 0.f;
    if (r < n_valid) {
      *(float4*)(dst + (int64_t)r * stride + col) = a;
      probe = finite_probe(a.x, finite_probe(a.y, finite_probe(a.z, finite_probe(a.w, probe))));
    }
    const uint64_t bad = __ballot(probe != 0.f);
#pragma unroll
    for (int x = 0; x < RPI; x++)
      if ((bad >> (x * LPR)) & ((1ull << LPR) - 1)) rows |= 1u << ((r0 + i + x) & 31);
  }
  return rows;
}

// LDS of a query-side workgroup: K and V of every group, later the waves' results
template <int D, int RG, int NG> constexpr int kQueryLds = NG * 2 * kOperand<D> > NG * RG * 4 * kSlabP<D> ? NG * 2 * kOperand<D> : NG * RG * 4 * kSlabP<D>;

// Whether any of NG groups has another tile, for odd and even steps: all of them go on until none has.
template <int NG>
struct More {
  int (*flag)[NG];
  __device__ __forceinline__ void put(int p, int group, bool first_wave, bool have) const {
    if (NG > 1 && first_wave && (threadIdx.x & 63) == 0) flag[p][group] = have;
  }
  __device__ __forceinline__ bool any(int p, bool have) const {
    if (NG == 1) return have;
    int y = 0;
#pragma unroll
    for (int z = 0; z < NG; z++) y |= flag[p][z];
    return uni(y) != 0;
  }
};

}  // namespace

template <int D, int RG, int NG, bool RANGES>
__global__ __launch_bounds__(64 * RG * NG, 2) void f32p_fwd_kernel(DevGroup g, KTensors t) {
  __shared__ __attribute__((aligned(1024))) char lds[kQueryLds<D, RG, NG>];
  __shared__ int wg_bounds[RG][8], flags[2][NG];
  __shared__ float sm[NG][RG][32], sl[NG][RG][32];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), rg = wave % RG, group = wave / RG, li = lane & 31, lh = lane >> 5;
  NQTile q;
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  if (!nq_tile<RANGES, RG>(g, t, lane, rg, wg_bounds, &q)) return;
  const More<NG> more{flags};
  char* k_lds = lds + group * 2 * kOperand<D>;
  char* v_lds = k_lds + kOperand<D>;
  const float* kb = (const float*)t.k + (int64_t)q.hk * t.k_sh;
  const float* vb = (const float*)t.v + (int64_t)q.hk * t.v_sh;
  Walk<NG> it(g, q.e0, q.e1, group);
  bool have = it.template next<RANGES>(q.q_hi, q.rb);
  Fetch<D, RG> fk, fv;
  if (have) {
    fk.load(kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
    fv.load(vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
  }
  OwnParts<D> qf;
  {
    float x[D / 16][8];
    read_own<D>(x, t.q, q.qi + q.qoff, t.q_st, (int64_t)q.head * t.q_sh, lane);
    cut_own<D>(qf, x);
  }
  Frags<D> fa;
  fa.init(lane);
  const float c_log2 = t.scale * kLog2e;
  float m = -INFINITY, l = 0.f;
  f32x16 o[D / 32];
  clear(o);
  if (have) fk.put(k_lds);
  more.put(1, group, rg == 0, have);
  __syncthreads();
  bool alive = more.any(1, have);
  const bool late = NG > 1 && group >= NG / 2;   // half a step behind
  int par = 0;
  if (late) __syncthreads();
  while (alive) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = RANGES ? it.kind : (it.kind & 1);
    const bool now = NG == 1 || have;
    f32x16 s;
    if (now) {
      have = it.template next<RANGES>(q.q_hi, q.rb);
      if (have) fk.load(kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
#pragma unroll
      for (int r = 0; r < 16; r++) s[r] = 0.f;
      s = dot_parts<D>(fa, k_lds, qf, s);
      fv.put(v_lds, kUp);
    }
    more.put(par, group, rg == 0, have);
    __syncthreads();
    if (now) {
      if (have) fv.load(vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
      if (classify32(kind, ks, c1, q.wq_lo, q.wq_hi, q.wrb) != kFull) n_mask(s, q, kind, ks, c0, c1, lane);
      float mx = s[0];
#pragma unroll
      for (int r = 1; r < 16; r++) mx = fmaxf(mx, s[r]);
      mx = xhalf_max(mx);
      const bool raise = (mx - m) * c_log2 > kRaiseP;
      const float m_new = raise ? mx : m;
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = raise ? __builtin_amdgcn_exp2f((m - m_use) * c_log2) : 1.f;
      m = m_new;
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        s[r] = __builtin_amdgcn_exp2f((s[r] - m_use) * c_log2);
        sum += s[r];
      }
      l = fmaf(l, alpha, sum);
      const Parts p[2] = {split_acc(s, 0), split_acc(s, 1)};
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const f32x16 x = cols_parts<D>(fa, v_lds, p, dt);
#pragma unroll
        for (int r = 0; r < 16; r++) o[dt][r] = fmaf(o[dt][r], alpha, x[r]);
      }
      fk.put(k_lds);   // nothing reads it if there is no next tile
    }
    __syncthreads();
    alive = more.any(par, have);
    par ^= 1;
  }
  if (NG > 1 && !late) __syncthreads();
  // the groups' results meet: a wave stores its share of its rows
  float mt = m, lt = xhalf_sum(l), f[NG];
  f[0] = 1.f;
  if (NG > 1 && lh == 0) { sm[group][rg][li] = m; sl[group][rg][li] = lt; }
  float* slabs = (float*)lds;
  stage_slab<D>(slabs + wave * kSlabP<D>, o, kDown, lane);
  __syncthreads();
  if (NG > 1) {
    mt = -INFINITY;
    lt = 0.f;
#pragma unroll
    for (int w = 0; w < NG; w++) mt = fmaxf(mt, sm[w][rg][li]);
#pragma unroll
    for (int w = 0; w < NG; w++) {
      f[w] = sm[w][rg][li] > -INFINITY ? __builtin_amdgcn_exp2f((sm[w][rg][li] - mt) * c_log2) : 0.f;
      lt = fmaf(f[w], sl[w][rg][li], lt);
    }
  }
  const int slot = plan_load(g.unit_out, q.unit);
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
#pragma unroll
  for (int w = 0; w < NG; w++) f[w] *= inv;
  const int brow0 = q.row0 + q.wrow0;
  float* lp = slot < 0 ? t.lse + (int64_t)q.head * t.q_rows + q.wq_lo + q.qoff : t.lse + ((int64_t)slot * t.hq + q.head) * t.block_size + brow0;
  constexpr int MINE = 32 / NG;   // rows of a wave here: it stores and repairs both O and LSE of them, in this order
  if (li / MINE == group && q.qv && lh == 0) lp[li] = lt > 0.f ? (mt * c_log2 + __builtin_amdgcn_logf(lt)) * kLn2P : -INFINITY;
  float* op = slot < 0 ? (float*)t.out + (int64_t)(q.wq_lo + q.qoff) * t.o_st + (int64_t)q.head * t.o_sh
                       : (float*)t.out + (((int64_t)slot * t.block_size + brow0) * t.hq + q.head) * D;
  const int64_t op_st = slot < 0 ? t.o_st : (int64_t)t.hq * D;
  uint32_t again = store_slabs<D, NG, MINE>(slabs + rg * kSlabP<D>, RG * kSlabP<D>, MINE * group, f, q.w_rows, op, op_st, lane);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again);
      const FixRow fr = fix_row(q, r);
      const float* qp = (const float*)a.t.q + (int64_t)(fr.qi + q.qoff) * a.t.q_st + (int64_t)q.head * a.t.q_sh;
      const float mr = lane_of(mt, r), lr = lane_of(lt, r);
      // an operand that is not finite has no parts: where it met the scores they are worked out again too
      if (lr != lr) fix_scores_and_out<float, D>(a.g, a.t, fr, q.hk, qp, op + r * op_st, lp + r);
      else fix_out<float, D>(a.g, a.t, fr, q.hk, qp, mr == -INFINITY ? 0.f : mr * c_log2, lane_of(inv, r), op + r * op_st);
    }
  }
}

template <int D, int RG, int NG, bool RANGES>
__global__ __launch_bounds__(64 * RG * NG, 2) void f32p_dq_kernel(DevGroup g, KTensors t) {
  __shared__ __attribute__((aligned(1024))) char lds[kQueryLds<D, RG, NG>];
  __shared__ int wg_bounds[RG][8], flags[2][NG];
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), rg = wave % RG, group = wave / RG, lh = lane >> 5;
  NQTile q;
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  if (!nq_tile<RANGES, RG>(g, t, lane, rg, wg_bounds, &q)) return;
  const More<NG> more{flags};
  char* k_lds = lds + group * 2 * kOperand<D>;
  char* v_lds = k_lds + kOperand<D>;
  const float* kb = (const float*)t.k + (int64_t)q.hk * t.k_sh;
  const float* vb = (const float*)t.v + (int64_t)q.hk * t.v_sh;
  Walk<NG> it(g, q.e0, q.e1, group);
  bool have = it.template next<RANGES>(q.q_hi, q.rb);
  Fetch<D, RG> fk, fv;
  if (have) {
    fv.load(vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
    fk.load(kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
  }
  const int64_t mem = q.qi + q.qoff, at = (int64_t)q.head * t.q_rows + mem;
  const float lse = t.lse[at];
  OwnParts<D> qf, dof;
  float delta = 0.f;
  bool small;
  {
    // the backward preprocess, fused: delta = sum_d dO * O of the lane's row, left (negated) with the rescaled LSE in the
    // workspace for the dK/dV kernel
    float x[D / 16][8], y[D / 16][8];
    read_own<D>(x, t.dout, mem, t.do_st, (int64_t)q.head * t.do_sh, lane);
    read_own<D>(y, t.out_in, mem, t.o_st, (int64_t)q.head * t.o_sh, lane);
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++)
#pragma unroll
      for (int e = 0; e < 8; e++) delta = fmaf(y[ks][e], x[ks][e], delta);
    cut_own<D>(dof, x, kUp);
    read_own<D>(x, t.q, mem, t.q_st, (int64_t)q.head * t.q_sh, lane);
    small = are_small<D>(x);
    cut_own<D>(qf, x, own_mul(small));
  }
  delta = xhalf_sum(delta);
  const float lse2 = row_lse2(lse, &delta), delta_up = delta * (kUp * kUp);
  if (group == 0 && q.qv && lh == 0) { t.delta_w[at] = -delta; t.lse2_w[at] = lse2; }
  Frags<D> fa;
  fa.init(lane);
  const float c_log2 = score_factor(t.scale, small);
  f32x16 dq[D / 32];
  clear(dq);
  if (have) fv.put(v_lds, kUp);
  more.put(1, group, rg == 0, have);
  __syncthreads();
  bool alive = more.any(1, have);
  const bool late = NG > 1 && group >= NG / 2;   // half a step behind
  int par = 0;
  if (late) __syncthreads();
  while (alive) {
    const int ks = it.ks(), c0 = it.c0, c1 = it.c1, kind = RANGES ? it.kind : (it.kind & 1);
    const bool now = NG == 1 || have;
    f32x16 dp;
    if (now) {
      have = it.template next<RANGES>(q.q_hi, q.rb);
      if (have) fv.load(vb, t.v_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
#pragma unroll
      for (int r = 0; r < 16; r++) dp[r] = -delta_up;
      dp = dot_parts<D>(fa, v_lds, dof, dp);
      fk.put(k_lds, kUp);
    }
    more.put(par, group, rg == 0, have);
    __syncthreads();
    if (now) {
      if (have) fk.load(kb, t.k_st, it.ks() + it.moff, it.c1 - 1 + it.moff);
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; r++) s[r] = 0.f;
      s = dot_parts<D>(fa, k_lds, qf, s);
      if (classify32(kind, ks, c1, q.wq_lo, q.wq_hi, q.wrb) != kFull) n_mask(s, q, kind, ks, c0, c1, lane);
#pragma unroll
      for (int r = 0; r < 16; r++) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lse2)) * dp[r];
      const Parts p[2] = {split_acc(s, 0), split_acc(s, 1)};
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const f32x16 x = cols_parts<D>(fa, k_lds, p, dt);
#pragma unroll
        for (int r = 0; r < 16; r++) dq[dt][r] += x[r];
      }
      fv.put(v_lds, kUp);   // nothing reads it if there is no next tile
    }
    __syncthreads();
    alive = more.any(par, have);
    par ^= 1;
  }
  if (NG > 1 && !late) __syncthreads();
  float* slabs = (float*)lds;
  stage_slab<D>(slabs + wave * kSlabP<D>, dq, kDown * kDown * kDown, lane);
  __syncthreads();
  float* dqp = (float*)t.dq + (int64_t)(q.wq_lo + q.qoff) * t.dq_st + (int64_t)q.head * t.dq_sh;
  constexpr int MINE = 32 / NG;
  uint32_t again = store_slabs<D, NG, MINE>(slabs + rg * kSlabP<D>, RG * kSlabP<D>, MINE * group, t.scale, q.w_rows, dqp, t.dq_st, lane);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again);
      const FixRow f = fix_row(q, r);
      const int64_t row = f.qi + q.qoff;
      fix_dq<float, D>(a.g, a.t, f, q.hk, (const float*)a.t.q + row * a.t.q_st + (int64_t)q.head * a.t.q_sh,
                       (const float*)a.t.dout + row * a.t.do_st + (int64_t)q.head * a.t.do_sh, lane_of(lse2, r), lane_of(delta, r), dqp + r * a.t.dq_st);
    }
  }
}

// dK / dV of 32 keys of one KV head: NG waves take the (query head, 32-query tile) pairs in turn, two on a SIMD: eight, or where the chip
// is full of equal work four, whose start and end fall beside another workgroup's loop (see part_groups in api.hip).  The rows of a tile
// are an A operand as they come from memory: a wave cuts them in registers, multiplies them from there, and puts them into LDS of its own
// for the transposed reads alone, dO first and Q after it into the same place, so that the loop has no barrier.  The keys' parts are in
// LDS for all waves.  What is live then fits 256 registers: the sums (64), the parts of one operand (48), the next tile's rows as they come
// (32, 64 during the last products) and one score tile or its parts; the two fences keep the compiler from holding more (with D 64 one
// register is spilled, three under ranges).  A wave that
// multiplies goes before one that cuts, or both would cut and then both multiply.  8 192 tokens of which 5 582 in one sequence, 8/2 heads,
// D 64 (the longest chain decides) and 16 384 in 8 equal ones, 16/4 heads: four waves that hold their keys' parts, one on a SIMD, 543 and
// 914 us; four that read them from LDS, two on a SIMD, 659 and 816; eight 507 and 862, with priorities 483 and 844, with two fences of
// four 466 and 815; four with both 647 and 782.
template <int D, int NG, bool RANGES>
__global__ __launch_bounds__(64 * NG, 2) void f32p_dkv_kernel(DevGroup g, KTensors t) {
  constexpr int KS = D / 16, SUB = kItemRows / 32;
  constexpr int kSums = NG * 2 * kSlabP<D> * 4;
  __shared__ __attribute__((aligned(1024))) char lds[(NG + 2) * kOperand<D> > kSums ? (NG + 2) * kOperand<D> : kSums];   // a tile of every wave, K, V
  __shared__ float row_vals[NG][64];   // lse2 and -delta of the tile's rows
  __shared__ int k_small;
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), li = lane & 31, lh = lane >> 5;
  touch_args<sizeof(DevGroup) + sizeof(KTensors)>();
  int item, x;
  if (!decode_wg(g, t.hkv, SUB, &item, &x)) return;
  const int hk = x / SUB, G = t.hq / t.hkv;
  const WorkItem w = plan_load(g.items, item);
  const int koff = uni(w.moff), row0 = uni(w.tile) * kItemRows + (x % SUB) * 32, n_rows = min(32, uni(w.blk_len) - row0);
  if (n_rows <= 0) return;
  const int seq0 = RANGES ? uni(plan_load(g.blk_s0, plan_load(g.unit_blk, uni(w.unit)))) : 0;
  const int k_lo = uni(w.blk_start) + row0, k_end = k_lo + n_rows;
  char* mine = lds + wave * kOperand<D>;
  char* k_lds = lds + NG * kOperand<D>;
  char* v_lds = k_lds + kOperand<D>;
  float* vals = row_vals[wave];
  QWalk<NG, RANGES> it(g, uni(w.e0), uni(w.e1), G, wave, t.qbounds);
  float rq[KS][8], rd[KS][8], rv = 0.f;   // the next tile as it comes
  int head = 0, r0 = 0, lim = 0;          // its head, first row in memory and last row of it
  auto fetch = [&](float (&r)[KS][8], const void* base, int64_t st, int64_t sh) {
    const int ln = fresh_lane();
    typedef const __attribute__((address_space(1))) char* gp;
    const gp b = (gp)(uint64_t)uni_ptr((const float*)base + (int64_t)r0 * st + (int64_t)head * sh);
    const unsigned off = (unsigned)min(ln & 31, lim) * (unsigned)st * 4u + 32u * (ln >> 5);
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int y = 0; y < 2; y++) {
        const pf32x4 a = *(const __attribute__((address_space(1))) pf32x4*)(b + off + 64 * ks + 16 * y);
#pragma unroll
        for (int e = 0; e < 4; e++) r[ks][4 * y + e] = a[e];
      }
  };
  auto load_do = [&]() {
    fetch(rd, t.dout, t.do_st, t.do_sh);
    const int ln = fresh_lane();
    rv = ((ln < 32 ? t.lse2 : t.delta) + (int64_t)head * t.q_rows)[r0 + min(ln & 31, lim)];
  };
  auto load_q = [&]() { fetch(rq, t.q, t.q_st, t.q_sh); };
  auto at_next = [&]() { head = hk * G + it.hh; r0 = it.qs() + it.moff; lim = it.q1 - 1 - it.qs(); };
  bool have = it.next(k_lo, k_end);
  if (have) { at_next(); load_do(); load_q(); }
  Frags<D> fa;
  fa.init(lane);
  if (wave < 2) {
    float y[KS][8];
    const int kl = min(k_lo + li, k_end - 1) + koff;
    if (wave == 0) read_own<D>(y, t.k, kl, t.k_st, (int64_t)hk * t.k_sh, lane);
    else read_own<D>(y, t.v, kl, t.v_st, (int64_t)hk * t.v_sh, lane);
    OwnParts<D> o;
    const bool small = are_small<D>(y);
    cut_own<D>(o, y, wave ? kUp : own_mul(small));
    put_own<D>(wave ? v_lds : k_lds, fa, o);
    if (wave == 0 && lane == 0) k_small = small;
  }
  __syncthreads();
  f32x16 dk[D / 32], dv[D / 32];
  clear(dk);
  clear(dv);
  const float c_log2 = score_factor(t.scale, uni(k_small) != 0);
  OwnParts<D> rows;   // dO, then Q, then the next dO
  if (have) cut_own<D>(rows, rd, kUp);
  while (have) {
    const int qs = it.qs(), q1 = it.q1, kind = it.kind;
    const bool full = n_rows == 32 && it.full(k_end - 1);
    vals[fresh_lane()] = rv * (fresh_lane() < 32 ? 1.f : kUp * kUp);
    f32x16 s, dp;
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const float4 d4 = *(const float4*)(vals + 32 + 8 * a + 4 * lh);
      dp[4 * a] = d4.x; dp[4 * a + 1] = d4.y; dp[4 * a + 2] = d4.z; dp[4 * a + 3] = d4.w;
    }
    put_own<D>(mine, fa, rows);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) dp = mul6(rows.s[ks], get_own<D>(v_lds, fa, ks), dp);
    cut_own<D>(rows, rq, kUp);
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) s = mul6(rows.s[ks], get_own<D>(k_lds, fa, ks), s);
    __builtin_amdgcn_s_setprio(0);
    have = it.next(k_lo, k_end);
    if (have) at_next();   // past the last tile it is that one again, unused
    load_do();
    __builtin_amdgcn_sched_barrier(0);
    if (!full) {
      // which of the 32 keys query row (l & 31) sees, as a bit mask of lane l (see mfma_dkv_kernel.h)
      const int i = qs + li;
      int lo1 = 0, hi1 = kind == 1 ? i + 1 : INT32_MAX, lo2 = 0, hi2 = 0;
      if (RANGES && kind == 2) {
        const int4 r = range_row(t, min(i, q1 - 1), seq0);
        lo1 = r.x; hi1 = r.y; lo2 = r.z; hi2 = r.w;
      }
      uint32_t vis = (keys_below(hi1, k_lo) & ~keys_below(lo1, k_lo)) | (keys_below(hi2, k_lo) & ~keys_below(lo2, k_lo));
      vis &= keys_below(k_end, k_lo);
      vis = i < q1 ? vis : 0u;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int m0 = acc_row(r);
        const uint64_t cond = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)vis, m0) |
                              ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)vis, m0 + 4) << 32);
        s[r] = __builtin_amdgcn_inverse_ballot_w64(cond) ? s[r] : -INFINITY;
      }
    }
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const float4 l4 = *(const float4*)(vals + 8 * a + 4 * lh);
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
      for (int b = 0; b < 4; b++) {
        const int r = 4 * a + b;
        s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_log2, -lv[b]));
        dp[r] *= s[r];
      }
    }
    __builtin_amdgcn_s_setprio(1);
    {
      const Parts p[2] = {split_acc(s, 0), split_acc(s, 1)};
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const f32x16 a = cols_parts<D>(fa, mine, p, dt);
#pragma unroll
        for (int r = 0; r < 16; r++) dv[dt][r] += a[r];
      }
    }
    put_own<D>(mine, fa, rows);   // Q takes dO's place, behind the reads (one wave's LDS operations are done in order)
    load_q();
    {
      const Parts p[2] = {split_acc(dp, 0), split_acc(dp, 1)};
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const f32x16 b = cols_parts<D>(fa, mine, p, dt);
#pragma unroll
        for (int r = 0; r < 16; r++) dk[dt][r] += b[r];
      }
    }
    __builtin_amdgcn_s_setprio(0);
    cut_own<D>(rows, rd, kUp);   // nothing uses it if there is no next tile
    __builtin_amdgcn_sched_barrier(0);
  }
  // the waves' sums meet, and a wave stores some of the rows
  constexpr int kPitch = 2 * kSlabP<D>;
  float* slabs = (float*)lds;
  __syncthreads();   // K and V have been read
  stage_slab<D>(slabs + wave * kPitch, dk, kDown * kDown * kDown, lane);
  stage_slab<D>(slabs + wave * kPitch + kSlabP<D>, dv, kDown, lane);
  __syncthreads();
  float* dkp = (float*)t.dk + (int64_t)(k_lo + koff) * t.dk_st + (int64_t)hk * t.dk_sh;
  float* dvp = (float*)t.dv + (int64_t)(k_lo + koff) * t.dv_st + (int64_t)hk * t.dv_sh;
  constexpr int MINE = 32 / NG > 256 / D ? 32 / NG : 256 / D;   // no fewer than an instruction stores
  if (MINE * wave >= 32) return;
  uint32_t again = store_slabs<D, NG, MINE>(slabs, kPitch, MINE * wave, t.scale, n_rows, dkp, t.dk_st, lane) |
                   store_slabs<D, NG, MINE>(slabs + kSlabP<D>, kPitch, MINE * wave, 1.f, n_rows, dvp, t.dv_st, lane);
  if (again) {
    DCP_WAIT_VMCNT(0);   // the stores above come first
    const KernelArgs a = kernel_args();
    const WorkItem w1 = plan_load(a.g.items, item);
    const int s0 = RANGES ? uni(plan_load(a.g.blk_s0, plan_load(a.g.unit_blk, uni(w1.unit)))) : 0;
    for (; again; again &= again - 1) {
      const int r = __builtin_ctz(again), j = k_lo + r;
      fix_dkv<float, D>(a.g, a.t, j, uni(w1.e0), uni(w1.e1), hk, s0, (const float*)a.t.k + (int64_t)(j + koff) * a.t.k_st + (int64_t)hk * a.t.k_sh,
                        (const float*)a.t.v + (int64_t)(j + koff) * a.t.v_st + (int64_t)hk * a.t.v_sh, dkp + r * a.t.dk_st, dvp + r * a.t.dv_st);
    }
  }
}

#define DCP_F32P_ONE(KERNEL, THREADS, ...) hipLaunchKernelGGL((KERNEL<__VA_ARGS__>), grid, dim3(THREADS), 0, s, g, t)
// one group of four waves, or two of four (D = 64) or four of two (D = 32)
#define DCP_F32P_LAUNCH(KERNEL)                                                                              \
  {                                                                                                          \
    if (g.n_items == 0) return DCP_OK;                                                                       \
    const dim3 grid(xcd_grid(g, t.hkv, t.hq / t.hkv * (t.part_groups > 1 && t.d == 32 ? 2 : 1)));                   \
    if (t.part_groups == 1) {                                                                                  \
      if (t.d == 32 && t.masked) DCP_F32P_ONE(KERNEL, 256, 32, 4, 1, true);                                  \
      else if (t.d == 32) DCP_F32P_ONE(KERNEL, 256, 32, 4, 1, false);                                        \
      else if (t.masked) DCP_F32P_ONE(KERNEL, 256, 64, 4, 1, true);                                          \
      else DCP_F32P_ONE(KERNEL, 256, 64, 4, 1, false);                                                       \
    } else {                                                                                                 \
      if (t.d == 32 && t.masked) DCP_F32P_ONE(KERNEL, 512, 32, 2, 4, true);                                  \
      else if (t.d == 32) DCP_F32P_ONE(KERNEL, 512, 32, 2, 4, false);                                        \
      else if (t.masked) DCP_F32P_ONE(KERNEL, 512, 64, 4, 2, true);                                          \
      else DCP_F32P_ONE(KERNEL, 512, 64, 4, 2, false);                                                       \
    }                                                                                                        \
    DCP_HIP_TRY(hipGetLastError());                                                                          \
    return DCP_OK;                                                                                           \
  }

dcp_status_t mfma_f32_parts_fwd(const DevGroup& g, const KTensors& t, hipStream_t s) DCP_F32P_LAUNCH(f32p_fwd_kernel)
dcp_status_t mfma_f32_parts_dq(const DevGroup& g, const KTensors& t, hipStream_t s) DCP_F32P_LAUNCH(f32p_dq_kernel)
dcp_status_t mfma_f32_parts_dkv(const DevGroup& g, const KTensors& t, hipStream_t s) {
  if (g.n_items == 0) return DCP_OK;
  const dim3 grid(xcd_grid(g, t.hkv, kSplitSub));
  if (t.part_groups == 1) {
    if (t.d == 32 && t.masked) DCP_F32P_ONE(f32p_dkv_kernel, 256, 32, 4, true);
    else if (t.d == 32) DCP_F32P_ONE(f32p_dkv_kernel, 256, 32, 4, false);
    else if (t.masked) DCP_F32P_ONE(f32p_dkv_kernel, 256, 64, 4, true);
    else DCP_F32P_ONE(f32p_dkv_kernel, 256, 64, 4, false);
  } else {
    if (t.d == 32 && t.masked) DCP_F32P_ONE(f32p_dkv_kernel, 512, 32, 8, true);
    else if (t.d == 32) DCP_F32P_ONE(f32p_dkv_kernel, 512, 32, 8, false);
    else if (t.masked) DCP_F32P_ONE(f32p_dkv_kernel, 512, 64, 8, true);
    else DCP_F32P_ONE(f32p_dkv_kernel, 512, 64, 8, false);
  }
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

}  // namespace dcp
