// Rows whose result is not finite, again and exactly (the MFMA kernels for fp32 and for narrow heads).
//
// Those kernels multiply whole tiles: a key that a row does not see has weight 0 but is multiplied all the same, and
// 0 x Inf = NaN, so one Inf or NaN in K, V, Q, O or dO would reach every row of its tile; and an operand that enters as
// several parts (pack_split) turns a visible Inf into Inf x 0.  A finite result of a row is proof that neither happened.
// A row whose result is not finite is therefore worked out once more from the pairs it really sees, one wave per row
// (lane = key of a 64-key step for the scores, lane = column for the sums, in table order): Inf and NaN then stand where the
// pairs' own arithmetic puts them.  Finite inputs pay one fused multiply-add per accumulator register at the end (nothing
// measurable: bf16, 16 384 tokens, 16/4 heads of 64, 576 / 640 / 1 339 us before and 577 / 641 / 1 319 with it).  Bound by latency where it runs: that bf16 batch forward and
// backward takes 2.9 ms finite, 10 with q, k, v all NaN (a row that is NaN in every column ends at once), 48 with V_5 NaN,
// 210 with one query in the middle NaN in every head (its keys' gradients are all worked out again, and are finite); the
// thread-per-row kernels took 133 in each case but the second.  fp32 in parts (8 192 tokens, longest 5 582, 8/2 heads of 64; forward, then
// forward and backward, ms): finite 0.27, 1.13; q, k, v all NaN 0.44, 1.52; in the longest sequence one K element NaN at its start 0.34,
// 1.27, in its middle 3.3, 6.2, Inf there 11.3, 22.7; one query NaN in every head 0.27, 22.4; V_5 NaN 10.6, 34.5.  The fp32 MFMA kernels,
// which work with Inf and NaN as they come and give a row of these to more waves, took 0.36, 1.61 | 0.36, 1.68 | 0.36, 1.63 | 0.35, 2.4 |
// 0.35, 8.5 | 0.39, 14.6 | 7.5, 22.5.
#pragma once
#include "mfma_common.h"

namespace dcp {

// The kernel's arguments (DevGroup, KTensors) once more, as the kernarg segment holds them: read when a row has to be worked
// out again, through a pointer the compiler cannot see through, so that the main loop keeps none of it in scalar
// registers (kept, they cost the dK/dV loops of narrow heads 18 lane reads per tile, 3 % of their time).
struct KernelArgs {
  DevGroup g;
  KTensors t;
};
// g_at, t_at: where they lie in the arguments
__device__ __forceinline__ KernelArgs kernel_args(int g_at = 0, int t_at = sizeof(DevGroup)) {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  KernelArgs a;
  __builtin_memcpy(&a.g, (const void*)((const __attribute__((address_space(4))) char*)p + g_at), sizeof(a.g));
  __builtin_memcpy(&a.t, (const void*)((const __attribute__((address_space(4))) char*)p + t_at), sizeof(a.t));
  return a;
}

template <typename T> __device__ __forceinline__ void load8(const T* p, float* f);
template <> __device__ __forceinline__ void load8<float>(const float* p, float* f) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}
template <> __device__ __forceinline__ void load8<bf16_t>(const bf16_t* p, float* f) {
  const uint4 u = *(const uint4*)p;
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; i++) { f[2 * i] = __uint_as_float(w[i] << 16); f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
}

template <typename T, int D>
__device__ __forceinline__ float dot_row(const T* a, const T* b) {
  float s = 0.f;
#pragma unroll 4
  for (int d = 0; d < D; d += 8) {
    float x[8], y[8];
    load8<T>(a + d, x);
    load8<T>(b + d, y);
#pragma unroll
    for (int i = 0; i < 8; i++) s = fmaf(x[i], y[i], s);
  }
  return s;
}

// NaN once some x is not finite, else 0; a finite result of a row means every term of it was
__device__ __forceinline__ float finite_probe(float x, float probe) { return fmaf(x, 0.f, probe); }

__device__ __forceinline__ float lane_of(float x, int l) { return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(x), l)); }

// acc[k] += weight of lane b x column (lane + 64 k) of that lane's row, for the lanes of `on` in order.  Eight rows are
// requested at once (the place of one that is not on takes another of the eight, unused).
template <typename T, int D>
__device__ __forceinline__ void add_rows(float (&acc)[(D + 63) / 64], float weight, uint64_t on, const T* row0, int64_t stride, int lane) {
  constexpr int K = (D + 63) / 64, U = 8;
  const int col = D % 64 == 0 ? lane : min(lane, D - 1);
#pragma unroll 1
  for (int b0 = 0; b0 < 64; b0 += U) {
    const unsigned m = (unsigned)(on >> b0) & ((1u << U) - 1u);
    if (!m) continue;
    float x[U][K];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int k = 0; k < K; k++)
        x[u][k] = Elem<T>::load(row0 + (int64_t)(b0 + ((m >> u) & 1 ? u : __builtin_ctz(m))) * stride + col + 64 * k);
#pragma unroll
    for (int u = 0; u < U; u++)
      if ((m >> u) & 1) {
        const float w = lane_of(weight, b0 + u);
#pragma unroll
        for (int k = 0; k < K; k++) acc[k] = fmaf(w, x[u][k], acc[k]);
      }
  }
}

template <int N>
__device__ __forceinline__ bool all_nan(const float (&acc)[N], bool column) {
  bool nan = true;
#pragma unroll
  for (int k = 0; k < N; k++) nan = nan && acc[k] != acc[k];
  return __all(nan || !column);   // nothing that follows changes a sum that is NaN
}

template <typename T, int D>
__device__ __forceinline__ void put_row(T* dst, const float (&acc)[(D + 63) / 64], float mul, int lane) {
#pragma unroll
  for (int k = 0; k < (D + 63) / 64; k++)
    if (D % 64 == 0 || lane < D) Elem<T>::store(dst + lane + 64 * k, acc[k] * mul);
}

// One query row: its packed index, its ranges, the table rows [e0, e1) of its unit, its rows of Q and (backward) dO.
struct FixRow {
  int qi, e0, e1;
  int4 qr;
};

// O of the row: exponents are taken against max2 (the row's reference maximum times c_log2), inv is 1 / the row's sum, and
// the weights are normalised before they meet V: the reference is raised lazily, so that exponentials reach 2^8, and with
// V beyond 2^120 a sum that is finite when normalised would overflow (as it may have in the kernel's own pass).
template <typename T, int D>
__device__ void fix_out(const DevGroup& g, const KTensors& t, const FixRow& f, int hk, const T* q, float max2, float inv, T* dst) {
  const int lane = threadIdx.x & 63;
  const float c_log2 = t.scale * 1.44269504088896340736f;
  const T* kb = (const T*)t.k + (int64_t)hk * t.k_sh;
  const T* vb = (const T*)t.v + (int64_t)hk * t.v_sh;
  float acc[(D + 63) / 64] = {};
  for (int e = f.e0; e < f.e1; e++) {
    const int c0 = uni(g.ent_start[e]), c1 = c0 + uni(g.ent_len[e]), kind = uni(g.ent_kind[e]), moff = uni(g.ent_moff[e]);
    for (int j0 = c0; j0 < c1; j0 += 64) {
      const int j = j0 + lane;
      const bool vis = j < c1 && key_visible(kind, f.qi, j, f.qr);
      const uint64_t on = __ballot(vis);
      if (!on) continue;
      float p = 0.f;
      if (vis) p = __builtin_amdgcn_exp2f(fmaf(dot_row<T, D>(q, kb + (int64_t)(j + moff) * t.k_st), c_log2, -max2)) * inv;
      add_rows<T, D>(acc, p, on, vb + (int64_t)(j0 + moff) * t.v_st, t.v_st, lane);
      if (all_nan(acc, lane < D)) { e = f.e1; break; }
    }
  }
  put_row<T, D>(dst, acc, 1.f, lane);
}

// The same for a row whose scores were not all worked out from what the inputs are (fp32 in parts: an Inf leaves NaN in the parts of its
// number): its maximum, its sum and its LSE too, in a walk before that of fix_out.  Exponents are differences of scores, as in the
// kernel, so that scores of any size do.  A score that is NaN or +Inf makes the whole row NaN, and ends the walk.
template <typename T, int D>
__device__ void fix_scores_and_out(const DevGroup& g, const KTensors& t, const FixRow& f, int hk, const T* q, T* dst, float* lse) {
  const int lane = threadIdx.x & 63;
  const float c_log2 = t.scale * 1.44269504088896340736f;
  const T* kb = (const T*)t.k + (int64_t)hk * t.k_sh;
  const T* vb = (const T*)t.v + (int64_t)hk * t.v_sh;
  float mx = -INFINITY, l = 0.f, acc[(D + 63) / 64] = {};   // the lane's maximum and its sum against that
  bool nan = false;
  for (int e = f.e0; e < f.e1 && !nan; e++) {
    const int c0 = uni(g.ent_start[e]), c1 = c0 + uni(g.ent_len[e]), kind = uni(g.ent_kind[e]), moff = uni(g.ent_moff[e]);
    for (int j0 = c0; j0 < c1 && !nan; j0 += 64) {
      const int j = j0 + lane;
      const bool vis = j < c1 && key_visible(kind, f.qi, j, f.qr);
      if (!__any(vis)) continue;
      const float s = vis ? dot_row<T, D>(q, kb + (int64_t)(j + moff) * t.k_st) : -INFINITY;
      nan = __any(!(s < INFINITY));
      const float m = fmaxf(mx, s);
      if (m > -INFINITY) l = fmaf(l, __builtin_amdgcn_exp2f((mx - m) * c_log2), __builtin_amdgcn_exp2f((s - m) * c_log2));
      mx = m;
    }
  }
  if (nan) {
    if (lane == 0) *lse = -INFINITY;
#pragma unroll
    for (int k = 0; k < (D + 63) / 64; k++) acc[k] = __builtin_nanf("");
    put_row<T, D>(dst, acc, 1.f, lane);
    return;
  }
  float m = mx;
#pragma unroll
  for (int x = 32; x > 0; x >>= 1) m = fmaxf(m, __shfl_xor(m, x));
  l = mx > -INFINITY ? l * __builtin_amdgcn_exp2f((mx - m) * c_log2) : 0.f;
#pragma unroll
  for (int x = 32; x > 0; x >>= 1) l += __shfl_xor(l, x);
  const float inv = l > 0.f ? 1.f / l : 0.f;
  if (lane == 0) *lse = l > 0.f ? (m * c_log2 + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f : -INFINITY;
  for (int e = l > 0.f ? f.e0 : f.e1; e < f.e1; e++) {
    const int c0 = uni(g.ent_start[e]), c1 = c0 + uni(g.ent_len[e]), kind = uni(g.ent_kind[e]), moff = uni(g.ent_moff[e]);
    for (int j0 = c0; j0 < c1; j0 += 64) {
      const int j = j0 + lane;
      const bool vis = j < c1 && key_visible(kind, f.qi, j, f.qr);
      const uint64_t on = __ballot(vis);
      if (!on) continue;
      const float p = vis ? __builtin_amdgcn_exp2f((dot_row<T, D>(q, kb + (int64_t)(j + moff) * t.k_st) - m) * c_log2) * inv : 0.f;
      add_rows<T, D>(acc, p, on, vb + (int64_t)(j0 + moff) * t.v_st, t.v_st, lane);
      if (all_nan(acc, lane < D)) { e = f.e1; break; }
    }
  }
  put_row<T, D>(dst, acc, 1.f, lane);
}

// dQ of the row, which is 0 for a row that is off (lse2 = +inf)
template <typename T, int D>
__device__ void fix_dq(const DevGroup& g, const KTensors& t, const FixRow& f, int hk, const T* q, const T* dout, float lse2, float delta, T* dst) {
  const int lane = threadIdx.x & 63;
  const float c_log2 = t.scale * 1.44269504088896340736f;
  const T* kb = (const T*)t.k + (int64_t)hk * t.k_sh;
  const T* vb = (const T*)t.v + (int64_t)hk * t.v_sh;
  float acc[(D + 63) / 64] = {};
  for (int e = lse2 < INFINITY ? f.e0 : f.e1; e < f.e1; e++) {
    const int c0 = uni(g.ent_start[e]), c1 = c0 + uni(g.ent_len[e]), kind = uni(g.ent_kind[e]), moff = uni(g.ent_moff[e]);
    for (int j0 = c0; j0 < c1; j0 += 64) {
      const int j = j0 + lane;
      const bool vis = j < c1 && key_visible(kind, f.qi, j, f.qr);
      const uint64_t on = __ballot(vis);
      if (!on) continue;
      float ds = 0.f;
      if (vis) {
        const float p = __builtin_amdgcn_exp2f(fmaf(dot_row<T, D>(q, kb + (int64_t)(j + moff) * t.k_st), c_log2, -lse2));
        ds = p * (dot_row<T, D>(dout, vb + (int64_t)(j + moff) * t.v_st) - delta);
      }
      add_rows<T, D>(acc, ds, on, kb + (int64_t)(j0 + moff) * t.k_st, t.k_st, lane);
      if (all_nan(acc, lane < D)) { e = f.e1; break; }
    }
  }
  put_row<T, D>(dst, acc, t.scale, lane);
}

// dK and dV of key j (packed index), table rows [e0, e1) of its block, over the query heads of KV head hk; t.lse2 and t.delta
// (negated) are the dQ kernel's, or (OWN) are worked out here, from the LSE and from O and dO
template <typename T, int D, bool OWN = false>
__device__ void fix_dkv(const DevGroup& g, const KTensors& t, int j, int e0, int e1, int hk, int seq0, const T* k, const T* v, T* dk_dst, T* dv_dst) {
  const int lane = threadIdx.x & 63, G = t.hq / t.hkv;
  const float c_log2 = t.scale * 1.44269504088896340736f;
  float dk[(D + 63) / 64] = {}, dv[(D + 63) / 64] = {};
  for (int e = e0; e < e1; e++) {
    const int q0 = uni(g.ent_start[e]), q1 = q0 + uni(g.ent_len[e]), kind = uni(g.ent_kind[e]), moff = uni(g.ent_moff[e]);
    for (int i0 = q0; i0 < q1; i0 += 64) {
      const int i = min(i0 + lane, q1 - 1);
      int4 r = make_int4(0, 0, 0, 0);
      if (kind == 2) r = range_row(t, i, seq0);
      const bool sees = i0 + lane < q1 && key_visible(kind, i, j, r);
      if (!__any(sees)) continue;
      for (int h = hk * G; h < (hk + 1) * G; h++) {
        const T* qb = (const T*)t.q + (int64_t)h * t.q_sh;
        const T* dob = (const T*)t.dout + (int64_t)h * t.do_sh;
        const int64_t at = (int64_t)h * t.q_rows + i + moff;
        float delta = 0.f;
        if (OWN) delta = dot_row<T, D>((const T*)t.out_in + (int64_t)(i + moff) * t.o_st + (int64_t)h * t.o_sh, dob + (int64_t)(i + moff) * t.do_st);
        else delta = -t.delta[at];
        const float lse2 = OWN ? row_lse2(t.lse[at], &delta) : t.lse2[at];
        const bool vis = sees && lse2 < INFINITY;
        const uint64_t on = __ballot(vis);
        if (!on) continue;
        float p = 0.f, ds = 0.f;
        if (vis) {
          p = __builtin_amdgcn_exp2f(fmaf(dot_row<T, D>(qb + (int64_t)(i + moff) * t.q_st, k), c_log2, -lse2));
          ds = p * (dot_row<T, D>(dob + (int64_t)(i + moff) * t.do_st, v) - delta);
        }
        add_rows<T, D>(dk, ds, on, qb + (int64_t)(i0 + moff) * t.q_st, t.q_st, lane);
        add_rows<T, D>(dv, p, on, dob + (int64_t)(i0 + moff) * t.do_st, t.do_st, lane);
      }
      if (all_nan(dk, lane < D) && all_nan(dv, lane < D)) { e = e1; break; }
    }
  }
  put_row<T, D>(dk_dst, dk, t.scale, lane);
  put_row<T, D>(dv_dst, dv, 1.f, lane);
}

}  // namespace dcp
