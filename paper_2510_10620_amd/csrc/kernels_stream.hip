// HBM-bound streaming kernels: the LSE-carrying merge of partial outputs ("RescaleAndSum",
// Listing 1 line 6; the paper's Blockwise Reduction instruction), the backward preprocess
// delta = rowsum(dO * O), and the plain gradient sum across blocks.  Each thread moves 16-byte
// vectors; all arithmetic is fp32.
#include "device_utils.h"
#include "kernels.h"
#include "mfma_common.h"

namespace dcp {

template <typename T> struct Vec8;  // 8 elements of D per thread
template <> struct Vec8<bf16_t> {
  typedef __bf16 hb8 __attribute__((ext_vector_type(8)));
  typedef float f8 __attribute__((ext_vector_type(8)));
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  typedef u4 Raw;   // 8 elements as memory holds them
  // NT: past the caches
  template <bool NT> static __device__ __forceinline__ Raw raw(const bf16_t* p) {
    if constexpr (NT) return __builtin_nontemporal_load((const u4*)p);
    else return *(const u4*)p;
  }
  static __device__ __forceinline__ void expand(const Raw& w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; i++) { f[2 * i] = __uint_as_float(w[i] << 16); f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
  }
  static __device__ __forceinline__ void load(const bf16_t* p, float* f) { expand(*(const u4*)p, f); }
  // round to nearest even with the hardware conversion (two values per instruction)
  static __device__ __forceinline__ u4 pack(const float* f) {
    const f8 v = {f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7]};
    return __builtin_bit_cast(u4, __builtin_convertvector(v, hb8));
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float* f) { *(u4*)p = pack(f); }
  // nontemporal: the line is not kept in the caches on its way out
  static __device__ __forceinline__ void store_nt(bf16_t* p, const float* f) { __builtin_nontemporal_store(pack(f), (u4*)p); }
};
template <> struct Vec8<float> {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  struct Raw { f32x4 a, b; };
  // a lane's 32 bytes are two loads, each of them half of every line that the wave touches
  template <bool NT> static __device__ __forceinline__ Raw raw(const float* p) {
    if constexpr (NT) return {__builtin_nontemporal_load((const f32x4*)p), __builtin_nontemporal_load((const f32x4*)(p + 4))};
    else return {*(const f32x4*)p, *(const f32x4*)(p + 4)};
  }
  static __device__ __forceinline__ void expand(const Raw& r, float* f) {
#pragma unroll
    for (int i = 0; i < 4; i++) { f[i] = r.a[i]; f[4 + i] = r.b[i]; }
  }
  static __device__ __forceinline__ void load(const float* p, float* f) {
    const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
  static __device__ __forceinline__ void store(float* p, const float* f) {
    *(float4*)p = make_float4(f[0], f[1], f[2], f[3]);
    *(float4*)(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
  }
  static __device__ __forceinline__ void store_nt(float* p, const float* f) {
    const f32x4 a = {f[0], f[1], f[2], f[3]}, b = {f[4], f[5], f[6], f[7]};
    __builtin_nontemporal_store(a, (f32x4*)p);
    __builtin_nontemporal_store(b, (f32x4*)(p + 4));
  }
};

// grid (8 * ceil(row groups / 8), n_blocks); a workgroup merges one group of ROWS rows of one q block for all heads.
// A thread item = (row, head, 8-wide chunk of D).
// Which row group a workgroup takes is chosen by XCD: the partial LSEs (and the merged LSE) of one head are
// contiguous along the rows, so 128 / (4 ROWS) neighbouring row groups share each of their cache lines; workgroup
// ids are dealt round-robin to the 8 XCDs, each with an L2 of its own, so with row group = blockIdx.x those
// neighbours sit on 8 different XCDs, every XCD fetches the whole line for 4 ROWS of its bytes, and the merged LSE
// goes out as partial lines (measured on the share benchmark: 48 % more bytes fetched than the partials hold).  With
// XCD x taking the x-th eighth of the row groups, the groups that share a line run on one XCD, close in time.
template <typename T, int ROWS>
__global__ __launch_bounds__(256) void merge_kernel(const int32_t* __restrict__ merge_ptr, const int32_t* __restrict__ merge_idx,
                                                    const int32_t* __restrict__ blk_mem0, const int32_t* __restrict__ blk_len,
                                                    int32_t block_size, const T* __restrict__ o_part,
                                                    const float* __restrict__ lse_part, T* __restrict__ out, int64_t o_st,
                                                    int64_t o_sh, float* __restrict__ lse, int64_t q_rows, int32_t hq,
                                                    int32_t d) {
  const int b = blockIdx.y;
  const int len = blk_len[b];
  const int mem0 = blk_mem0[b];   // the block's first row in out / lse; negative: the block is not in the buffer
  if (mem0 < 0) return;
  const int per_xcd = gridDim.x >> 3;
  const int row0 = ((blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3)) * ROWS;
  if (row0 >= len) return;
  const int p0 = merge_ptr[b], p1 = merge_ptr[b + 1];
  const int chunks = d / 8;
  const int n_items = min(ROWS, len - row0) * hq * chunks;
  for (int it = threadIdx.x; it < n_items; it += blockDim.x) {
    const int c = it % chunks, h = (it / chunks) % hq, row = row0 + it / (chunks * hq);
    float m = -INFINITY;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float tot = 0.f;
    for (int p = p0; p < p1; p++) m = fmaxf(m, lse_part[((int64_t)merge_idx[p] * hq + h) * block_size + row]);
    if (m > -INFINITY) {
      for (int p = p0; p < p1; p++) {
        const int slot = merge_idx[p];
        const float lp = lse_part[((int64_t)slot * hq + h) * block_size + row];
        if (lp == -INFINITY) continue;  // weight 0: never touch the partial's values
        const float wgt = expf(lp - m);
        tot += wgt;
        float f[8];
        Vec8<T>::load(o_part + (((int64_t)slot * block_size + row) * hq + h) * d + c * 8, f);
#pragma unroll
        for (int i = 0; i < 8; i++) acc[i] = fmaf(wgt, f[i], acc[i]);
      }
      const float inv = 1.f / tot;
#pragma unroll
      for (int i = 0; i < 8; i++) acc[i] *= inv;
    }
    const int64_t tok = (int64_t)mem0 + row;
    Vec8<T>::store_nt(out + tok * o_st + (int64_t)h * o_sh + c * 8, acc);
    if (c == 0) lse[(int64_t)h * q_rows + tok] = m > -INFINITY ? m + logf(tot) : -INFINITY;
  }
}

// The merge for bf16 with D = 8 CH.  The kernel above is bound by its own instructions, not by memory (index arithmetic with
// run-time divisors, and arithmetic it does not need when a q block has no partial or only one): here lane t keeps chunk t % CH
// and the (row, head) pairs of the workgroup's rows go round in steps of 256 / CH without a division, and there are three paths
// chosen per q block: no partial (the rows are zero-filled), one partial (weight 1: the row is copied, or zero-filled where its
// LSE is -inf), several (up to kMergePreload with every load issued before the arithmetic).  The results are the above kernel's for
// every LSE: one that is NaN makes the row NaN beside a partial with a weight and counts for nothing alone; +inf makes it NaN.
static constexpr int kMergePreload = 4;   // partial slots per q block up to which all of an item's loads are issued at once
typedef __bf16 hbf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int CH>
__global__ __launch_bounds__(256) void merge_rows_kernel(const int32_t* __restrict__ merge_ptr, const int32_t* __restrict__ merge_idx,
                                                         const int32_t* __restrict__ blk_mem0, const int32_t* __restrict__ blk_len,
                                                         int32_t block_size, int32_t rows, const bf16_t* __restrict__ o_part,
                                                         const float* __restrict__ lse_part, bf16_t* __restrict__ out, int64_t o_st,
                                                         int64_t o_sh, float* __restrict__ lse, int64_t q_rows, int32_t hq) {
  constexpr int STEP = 256 / CH;
  const int b = blockIdx.y;
  const int len = plan_load(blk_len, b), mem0 = plan_load(blk_mem0, b), p0 = plan_load(merge_ptr, b), n_p = plan_load(merge_ptr, b + 1) - p0;
  if (mem0 < 0) return;
  const int per_xcd = gridDim.x >> 3;
  const int row0 = ((blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3)) * rows;   // row groups by XCD, see merge_kernel
  if (row0 >= len) return;
  const int n_pairs = min(rows, len - row0) * hq;
  const int c = threadIdx.x % CH;
  int pair = threadIdx.x / CH, row = row0, h = pair, step_r = 0, step_h = STEP;
  if (hq < STEP) { row += pair / hq; h = pair % hq; step_r = STEP / hq; step_h = STEP % hq; }
  auto next = [&]() {
    pair += STEP; row += step_r; h += step_h;
    if (h >= hq) { h -= hq; row++; }
  };
  auto out_at = [&]() { return (u32x4*)(out + ((int64_t)mem0 + row) * o_st + (int64_t)h * o_sh + c * 8); };
  auto lse_of = [&](int slot) { return lse_part[((int64_t)slot * hq + h) * block_size + row]; };
  auto part_at = [&](int slot) { return (const u32x4*)(o_part + (((int64_t)slot * block_size + row) * hq + h) * (8 * CH) + c * 8); };
  const u32x4 zero = {0u, 0u, 0u, 0u};
  if (n_p == 0) {
    for (; pair < n_pairs; next()) {
      __builtin_nontemporal_store(zero, out_at());
      if (c == 0) lse[(int64_t)h * q_rows + mem0 + row] = -INFINITY;
    }
    return;
  }
  if (n_p == 1) {
    const int slot = plan_load(merge_idx, p0);
    const u32x4 nan = {0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u};
    for (; pair < n_pairs; next()) {
      const float lp = lse_of(slot);
      u32x4 v = __builtin_nontemporal_load(part_at(slot));
      v = lp < INFINITY ? v : nan;
      __builtin_nontemporal_store(lp > -INFINITY ? v : zero, out_at());
      if (c == 0) lse[(int64_t)h * q_rows + mem0 + row] = lp > -INFINITY ? lp + (lp - lp) : -INFINITY;
    }
    return;
  }
  for (; pair < n_pairs; next()) {
    float m = -INFINITY, tot = 0.f;
    f32x8 acc = {0, 0, 0, 0, 0, 0, 0, 0};
    if (n_p <= kMergePreload) {
      float lp[kMergePreload];
      u32x4 raw[kMergePreload];
#pragma unroll
      for (int k = 0; k < kMergePreload; k++)
        if (k < n_p) {
          const int slot = plan_load(merge_idx, p0 + k);
          lp[k] = lse_of(slot);
          raw[k] = __builtin_nontemporal_load(part_at(slot));
          m = fmaxf(m, lp[k]);   // of those that are not NaN
        }
#pragma unroll
      for (int k = 0; k < kMergePreload; k++)
        if (k < n_p) {
          const bool live = m > -INFINITY && lp[k] != -INFINITY;
          const float wgt = live ? expf(lp[k] - m) : 0.f;
          tot += wgt;
#pragma unroll
          for (int i = 0; i < 4; i++) {
            acc[2 * i] = fmaf(wgt, live ? __uint_as_float(raw[k][i] << 16) : 0.f, acc[2 * i]);
            acc[2 * i + 1] = fmaf(wgt, live ? __uint_as_float(raw[k][i] & 0xffff0000u) : 0.f, acc[2 * i + 1]);
          }
        }
    } else {
      for (int k = 0; k < n_p; k++) m = fmaxf(m, lse_of(merge_idx[p0 + k]));
      for (int k = 0; k < n_p; k++) {
        const int slot = merge_idx[p0 + k];
        const float lpk = lse_of(slot);
        if (lpk == -INFINITY || m == -INFINITY) continue;
        const float wgt = expf(lpk - m);
        tot += wgt;
        const u32x4 rw = *part_at(slot);
#pragma unroll
        for (int i = 0; i < 4; i++) {
          acc[2 * i] = fmaf(wgt, __uint_as_float(rw[i] << 16), acc[2 * i]);
          acc[2 * i + 1] = fmaf(wgt, __uint_as_float(rw[i] & 0xffff0000u), acc[2 * i + 1]);
        }
      }
    }
    acc *= m > -INFINITY ? 1.f / tot : 0.f;
    const hbf16x8 ob = __builtin_convertvector(acc, hbf16x8);   // round to nearest even in hardware
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4, ob), out_at());
    if (c == 0) lse[(int64_t)h * q_rows + mem0 + row] = m > -INFINITY ? m + logf(tot) : -INFINITY;
  }
}

dcp_status_t stream_merge(const int32_t* merge_ptr, const int32_t* merge_idx, const int32_t* blk_mem0,
                          const int32_t* blk_len, int32_t n_blocks, int32_t longest_block, int32_t block_size, const void* o_part,
                          const float* lse_part, void* out, int64_t o_st, int64_t o_sh, float* lse,
                          int64_t total_tokens, int32_t hq, int32_t d, int32_t dtype, hipStream_t s) {
  if (n_blocks == 0) return DCP_OK;
  if (dtype == DCP_BF16 && (d == 32 || d == 64 || d == 128)) {
    // One step of pairs per workgroup, at least one row: the most workgroups in flight measured fastest.  D 128, one, two, four
    // steps: 14 429 tokens, 4 heads, 51 MB 12.7 / 13.2 / 16.5 us; 65 536, 8 heads, 413 MB 78.5 / 80.6 / 86.7 (the kernel for any
    // shape 13.9 and 109.4); 24 heads 235.5 / 235.9 / 240.7 (315.5); 16 heads, 9 706 tokens in blocks of 4 096, 81 MB, 21.0 / 21.3 /
    // 22.5 (31.0 with a launch sized by the block size).
    const int rows = std::max(1, 256 / (d / 8) / hq);
    const int groups = (longest_block + rows - 1) / rows;
#define DCP_MERGE_ROWS(CH)                                                                                                 \
  hipLaunchKernelGGL(merge_rows_kernel<CH>, dim3(8 * ((groups + 7) / 8), n_blocks), dim3(256), 0, s, merge_ptr, merge_idx, \
                     blk_mem0, blk_len, block_size, rows, (const bf16_t*)o_part, lse_part, (bf16_t*)out, o_st, o_sh, lse, total_tokens, hq)
    if (d == 128) DCP_MERGE_ROWS(16);
    else if (d == 64) DCP_MERGE_ROWS(8);
    else DCP_MERGE_ROWS(4);
  } else {
#define DCP_MERGE(T)                                                                                                      \
  hipLaunchKernelGGL((merge_kernel<T, 4>), dim3(8 * (((longest_block + 3) / 4 + 7) / 8), n_blocks), dim3(256), 0, s, merge_ptr,     \
                     merge_idx, blk_mem0, blk_len, block_size, (const T*)o_part, lse_part, (T*)out, o_st, o_sh, lse, total_tokens, \
                     hq, d)
    if (dtype == DCP_BF16) DCP_MERGE(bf16_t);
    else DCP_MERGE(float);
  }
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

// delta[h, t] = sum_d dO[t,h,d] * O[t,h,d].  A workgroup covers TOK tokens x all heads; the
// d/8 lanes of one (token, head) reduce with shuffles; results pass through LDS so that each head
// row of delta is written in contiguous runs of TOK floats.

template <int CTRL> __device__ __forceinline__ float dpp_add(float x) {
  return x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
// Sum over aligned groups of `chunks` lanes (a power of two up to 32, uniform), in every lane of the group.
__device__ __forceinline__ float chunk_sum(float x, int chunks) {
  if (chunks > 1) x = dpp_add<0xb1>(x);     // quad_perm 1,0,3,2
  if (chunks > 2) x = dpp_add<0x4e>(x);     // quad_perm 2,3,0,1
  if (chunks > 4) x = dpp_add<0x141>(x);    // mirrored within 8 lanes: the other quad's sum
  if (chunks > 8) x = dpp_add<0x140>(x);    // mirrored within 16 lanes: the other half's sum
  if (chunks > 16) x += __shfl_xor(x, 16);
  return x;
}

template <typename T, int TOK>
__global__ __launch_bounds__(256) void delta_kernel(const T* __restrict__ o, int64_t o_st, int64_t o_sh,
                                                    const T* __restrict__ dout, int64_t do_st, int64_t do_sh,
                                                    float* __restrict__ delta, const float* __restrict__ lse,
                                                    float* __restrict__ lse2, int64_t total_tokens, int32_t hq,
                                                    int32_t d) {
  extern __shared__ float sm[];  // [hq][TOK + 1]
  const int64_t t0 = (int64_t)blockIdx.x * TOK;
  const int ntok = (int)min((int64_t)TOK, total_tokens - t0);
  // HBM-bound.  Thread x keeps chunk x % chunks; the (token, head) pairs of the workgroup go round in steps of
  // 256 / chunks without a division, and four steps' loads are requested before the first is reduced (in DPP steps, not
  // LDS ones): 65 536 tokens, 32 heads of 128 in bf16 207 -> 168-175 us, 6.0-6.4 TB/s.
  const int chunks = d / 8;  // power of two <= 32
  const int step = 256 / chunks, n_pairs = ntok * hq;
  const int c = threadIdx.x & (chunks - 1);
  const int step_t = step / hq, step_h = step % hq;
  int pair = threadIdx.x / chunks, tl = pair / hq, h = pair % hq;
  // bf16 past the caches; fp32, two loads a line, through them (16 MB of it 47 -> 40 us)
  constexpr bool NT = sizeof(T) == 2;
  constexpr int U = 4;
  for (int k = 0; k < n_pairs; k += U * step) {   // the same trip count for every thread: the reduction uses all lanes
    typename Vec8<T>::Raw a[U], b[U];
    int at[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      at[u] = pair < n_pairs ? h * (TOK + 1) + tl : -1;
      if (at[u] >= 0) {
        a[u] = Vec8<T>::template raw<NT>(o + (t0 + tl) * o_st + (int64_t)h * o_sh + c * 8);
        b[u] = Vec8<T>::template raw<NT>(dout + (t0 + tl) * do_st + (int64_t)h * do_sh + c * 8);
      }
      pair += step; tl += step_t; h += step_h;
      if (h >= hq) { h -= hq; tl++; }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      float sum = 0.f;
      if (at[u] >= 0) {
        float x[8], y[8];
        Vec8<T>::expand(a[u], x);
        Vec8<T>::expand(b[u], y);
#pragma unroll
        for (int i = 0; i < 8; i++) sum = fmaf(x[i], y[i], sum);
      }
      sum = chunk_sum(sum, chunks);
      if (at[u] >= 0 && c == 0) sm[at[u]] = sum;
    }
  }
  __syncthreads();
  for (int it = threadIdx.x; it < hq * ntok; it += blockDim.x) {
    const int h = it / ntok, tl = it % ntok;
    delta[(int64_t)h * total_tokens + t0 + tl] = sm[h * (TOK + 1) + tl];
    // log-sum-exp in the exp2 domain for the backward kernels; -inf (a row that saw nothing) becomes
    // the lowest finite float so that (masked score = -inf) - lse2 stays -inf and P = 0
    if (lse2) lse2[(int64_t)h * total_tokens + t0 + tl] = fmaxf(lse[(int64_t)h * total_tokens + t0 + tl] * 1.44269504088896340736f, -3.402823466e38f);
  }
}

dcp_status_t stream_delta(const void* o, int64_t o_st, int64_t o_sh, const void* dout, int64_t do_st, int64_t do_sh,
                          float* delta, const float* lse, float* lse2, int64_t total_tokens, int32_t hq, int32_t d,
                          int32_t dtype, hipStream_t s) {
  if (total_tokens == 0) return DCP_OK;
  // 32 tokens a workgroup make less than four workgroups a CU of a short batch, each with a chain of loads; 8 make four times the
  // starts, and with few chunks to a token threads without a load.  8 and 32 tokens, bf16, D 128: 16 384 tokens, 4 / 16 / 128 heads
  // 7.2 / 23.1 / 181 and 10.3 / 32.0 / 226 us; 24 576 tokens 9.4 / 33.7 / 281 and 11.1 / 35.5 / 255; 32 768 tokens 11.7 / 45.0 / 379
  // and 12.6 / 44.3 / 334; one head of 64, 4 096 / 16 384 tokens 3.8 / 5.0 and 3.6 / 3.8.  fp32, whose chunk is two loads: 32 heads of
  // 64, 8 192 / 12 288 tokens 21.7 / 31.9 and 23.1 / 30.2; one head 4.0 and 3.5 at 8 192.
  const int64_t chunks8 = 8 * (int64_t)hq * (d / 8);   // of 8 tokens
  const bool few = dtype == DCP_BF16 ? total_tokens < (hq <= 16 ? 32 * 1024 : 22 * 1024) && total_tokens <= 96 * chunks8
                                     : total_tokens < 10 * 1024 && total_tokens <= 32 * chunks8;
  const int tok = few ? 8 : 32;
  dim3 grid((unsigned)((total_tokens + tok - 1) / tok)), block(256);
  const size_t sm = (size_t)hq * (tok + 1) * sizeof(float);
#define DCP_DELTA(T, TOK)                                                                                                  \
  hipLaunchKernelGGL((delta_kernel<T, TOK>), grid, block, sm, s, (const T*)o, o_st, o_sh, (const T*)dout, do_st, do_sh, delta, lse, \
                     lse2, total_tokens, hq, d)
  if (dtype == DCP_BF16) {
    if (tok == 32) DCP_DELTA(bf16_t, 32);
    else DCP_DELTA(bf16_t, 8);
  } else {
    if (tok == 32) DCP_DELTA(float, 32);
    else DCP_DELTA(float, 8);
  }
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

struct PartPtrs {
  const void* p[8];
};

// HBM-bound.  One 16- or 32-byte piece per part and thread, all parts requested before the first is added: two bf16 parts of
// 512 MiB 293 -> 248-258 us (6.2-6.5 TB/s) against 4 096 workgroups that walked the arrays with one load at a time.
// What goes past the caches: bf16 results (16 bytes a lane, whole lines); fp32 results do not, their two stores a lane are
// half lines (one bf16 part of 2^28 elements to fp32: 403 us past, 272 through).  NT: the parts too, see stream_sum.
template <typename TI, typename TO, bool NT>
__global__ __launch_bounds__(256) void sum_kernel(PartPtrs parts, int32_t n_parts, TO* __restrict__ dst, int64_t n8) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (int64_t)gridDim.x * 256) {
    typename Vec8<TI>::Raw raw[8];
#pragma unroll
    for (int p = 0; p < 8; p++)
      if (p < n_parts) raw[p] = Vec8<TI>::template raw<NT>((const TI*)parts.p[p] + i * 8);
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < 8; p++)
      if (p < n_parts) {
        float f[8];
        Vec8<TI>::expand(raw[p], f);
#pragma unroll
        for (int k = 0; k < 8; k++) acc[k] += f[k];
      }
    if constexpr (sizeof(TO) == 2) Vec8<TO>::store_nt(dst + i * 8, acc);
    else Vec8<TO>::store(dst + i * 8, acc);
  }
}

dcp_status_t stream_sum(const void* const* parts, int32_t n_parts, int32_t parts_dtype, void* dst, int32_t dst_dtype,
                        int64_t n, hipStream_t s) {
  if (n == 0) return DCP_OK;
  PartPtrs pp{};
  for (int i = 0; i < n_parts; i++) pp.p[i] = parts[i];
  const int64_t n8 = n / 8;
  dim3 grid((unsigned)std::min<int64_t>((n8 + 255) / 256, 1 << 22)), block(256);   // one pass up to 2^33 elements
  // Parts that the 256 MB behind the L2s can hold are read through it (a kernel before may have left them there), larger
  // ones past it.  To bf16, past and through: four bf16 parts of 2^25 elements (268 MB) 56 and 47 us, two of 2^27 (537 MB) 124
  // and 133; two fp32 parts of 2^25 (268 MB) 53 and 46, of 2^26 (537 MB) 107 and 114.
  const bool nt = n * n_parts * (parts_dtype == DCP_F32 ? 4 : 2) > 300000000;
  if (parts_dtype == DCP_F32 && dst_dtype == DCP_BF16) {
    if (nt) hipLaunchKernelGGL((sum_kernel<float, bf16_t, true>), grid, block, 0, s, pp, n_parts, (bf16_t*)dst, n8);
    else hipLaunchKernelGGL((sum_kernel<float, bf16_t, false>), grid, block, 0, s, pp, n_parts, (bf16_t*)dst, n8);
  } else if (parts_dtype == DCP_F32 && dst_dtype == DCP_F32) {
    hipLaunchKernelGGL((sum_kernel<float, float, false>), grid, block, 0, s, pp, n_parts, (float*)dst, n8);
  } else if (parts_dtype == DCP_BF16 && dst_dtype == DCP_BF16) {
    if (nt) hipLaunchKernelGGL((sum_kernel<bf16_t, bf16_t, true>), grid, block, 0, s, pp, n_parts, (bf16_t*)dst, n8);
    else hipLaunchKernelGGL((sum_kernel<bf16_t, bf16_t, false>), grid, block, 0, s, pp, n_parts, (bf16_t*)dst, n8);
  } else {
    hipLaunchKernelGGL((sum_kernel<bf16_t, float, false>), grid, block, 0, s, pp, n_parts, (float*)dst, n8);
  }
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

// ------------------------------------------------------------------------------------ copy
// Blockwise Copy: one workgroup per chunk of at most kCopyChunkRows rows, 16 bytes per lane and
// load, four loads in flight per lane.  HBM-bound: 2 * row_bytes algorithmic bytes per row.
__global__ __launch_bounds__(256) void copy_kernel(const int32_t* __restrict__ chunks, int64_t n_chunks,
                                                   const char* __restrict__ src, int64_t src_stride,
                                                   char* __restrict__ dst, int64_t dst_stride, int32_t vec_per_row) {
  // every byte is touched once: nontemporal loads and stores keep the copy from displacing what the attention kernels
  // that run beside it hold in the caches (5.33 -> 5.77 TB/s on the 512 MiB Q-block copy)
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  auto ld = [](const char* p, int32_t i) -> u32x4 { return __builtin_nontemporal_load((const u32x4*)p + i); };
  auto st = [](char* p, int32_t i, u32x4 v) { __builtin_nontemporal_store(v, (u32x4*)p + i); };
  for (int64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
    const int32_t sr = chunks[3 * c], dr = chunks[3 * c + 1], nr = chunks[3 * c + 2];
    const char* sp = src + (int64_t)sr * src_stride;
    char* dp = dst + (int64_t)dr * dst_stride;
    const int32_t total = nr * vec_per_row;
    if (src_stride == (int64_t)vec_per_row * 16 && dst_stride == src_stride) {
      // rows are back to back in both buffers: one linear span
      int32_t i = threadIdx.x;
      for (; i + 768 < total; i += 1024) {
        const u32x4 a = ld(sp, i), b = ld(sp, i + 256), e = ld(sp, i + 512), f = ld(sp, i + 768);
        st(dp, i, a); st(dp, i + 256, b); st(dp, i + 512, e); st(dp, i + 768, f);
      }
      for (; i < total; i += 256) st(dp, i, ld(sp, i));
    } else {
      for (int32_t i = threadIdx.x; i < total; i += 256) {
        const int32_t r = i / vec_per_row, v = i - r * vec_per_row;
        st(dp + (int64_t)r * dst_stride, v, ld(sp + (int64_t)r * src_stride, v));
      }
    }
  }
}

dcp_status_t stream_copy(const int32_t* chunks, int64_t n_chunks, const void* src, int64_t src_stride, void* dst,
                         int64_t dst_stride, int64_t row_bytes, hipStream_t s) {
  if (n_chunks == 0) return DCP_OK;
  dim3 grid((unsigned)std::min<int64_t>(n_chunks, 256 * 64)), block(256);
  hipLaunchKernelGGL(copy_kernel, grid, block, 0, s, chunks, n_chunks, (const char*)src, src_stride, (char*)dst, dst_stride,
                     (int32_t)(row_bytes / 16));
  DCP_HIP_TRY(hipGetLastError());
  return DCP_OK;
}

}  // namespace dcp
