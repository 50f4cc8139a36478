// Launcher declarations: one function per kernel family, defined in the .hip files.
#pragma once
#include "dcp_internal.h"

namespace dcp {

// Plain-old-data copy of the caller's tensor descriptor plus derived fields, passed by value.
struct KTensors {
  const void *q, *k, *v, *dout, *out_in;
  void *out, *dq, *dk, *dv;
  float* lse;              // forward: output; backward: input
  float* delta_w;          // backward, MFMA family: where the dQ kernel leaves -delta and lse2 (the same arrays as below) for
  float* lse2_w;           //   the dK/dV kernel; null in the scalar family, where a preprocess kernel has filled them
  const float* delta;      // backward input [Hq,T]: delta (scalar family), -delta (MFMA family dK/dV, from the dQ kernel)
  const float* lse2;       // backward input [Hq,T]: max(lse * log2(e), -FLT_MAX); fp32 and D < 128: +inf where lse is -inf or NaN
  const int32_t* ranges;   // [T,4] or null (tables without RANGES rows)
  int32_t window, sink;    // window > 0: the table has WINDOW rows; their per-token ranges are worked out, not read
  int32_t masked;          // the table has RANGES or WINDOW rows (rows with per-token ranges)
  float* part;             // backward, or null: fp32 partial sums of split dK/dV items, [slot][KV head][dK, dV][128 keys][D]
  const int32_t* qbounds;  // backward, or null: [32-row tiles of all blocks + 1][8] bounds of the rows' ranges (RangeBounds order)
  int64_t q_st, q_sh, k_st, k_sh, v_st, v_sh, o_st, o_sh, do_st, do_sh, dq_st, dq_sh, dk_st, dk_sh, dv_st, dv_sh;
  int64_t q_rows;   // rows of the Q-type buffers (= packed tokens without block buffers): row pitch of lse / delta / lse2
  int32_t hq, hkv, d, block_size;
  int32_t dtype;           // dcp_dtype_t
  float scale;
  int32_t use_slots;
  int32_t by_head;         // dK/dV, bf16 with D = 128, masked: the query heads are the outer loop (dcp_plan::kv_by_head)
  int32_t part_groups;     // fp32, not 16 rows: 0 (32 rows a workgroup, fp32 pipe) or, with D < 128, in parts: 1 (four waves a workgroup) or 2 (eight)
};

#ifdef __HIPCC__
// The range-array entry of packed token i (s0 = first token of its sequence): read from the array, or, for a
// sliding window with sink, the window [lo, i + 1) with lo = max(i - window + 1, s0) and the sink tokens before it,
// [s0, min(s0 + sink, lo)) (two ranges that do not overlap).
__device__ __forceinline__ int4 range_row(const KTensors& t, int i, int s0) {
  if (t.window > 0) {
    const int lo = max(i - t.window + 1, s0);
    return make_int4(s0, min(s0 + t.sink, lo), lo, i + 1);
  }
  return ((const int4*)t.ranges)[i];
}
#endif

// Grid of a launch whose workgroups find their work with decode_wg: 8 times the largest number of workgroups any XCD
// needs for its (KV head, segment) units.
inline int64_t xcd_grid(const DevGroup& g, int heads_outer, int heads_inner) {
  const int upx = (heads_outer * g.n_seg) / 8;
  int64_t most = 0;
  for (int x = 0; x < 8; x++) {
    int64_t n = 0;
    for (int u = x * upx; u < (x + 1) * upx; u++) n += (int64_t)(g.seg[u % g.n_seg + 1] - g.seg[u % g.n_seg]) * heads_inner;
    most = n > most ? n : most;
  }
  return 8 * most;
}

// Workgroups that the kernels launch per work item and KV head, and their threads.  kSplit*: the kernels whose waves share 32
// rows (split_rows.h).
constexpr int kSplitSub = kItemRows / 32, kSplitThreads = 512, kNarrowThreads = 256, kNarrowDkvThreads = 512;

// A launch counts its threads in 32 bits.  Whether that of a query-side group (or the dK/dV group) of these kernels fits;
// the D = 128 kernels' tensors would outgrow the memory first.
inline bool mfma_launch_fits(const DevGroup& g, bool dkv, int32_t dtype, int32_t d, int hq, int hkv) {
  if (dtype == DCP_BF16 && d == 128) return true;
  if ((int64_t)g.n_items * hq < (UINT32_MAX >> 3) / (kSplitSub * kSplitThreads)) return true;   // whatever the XCDs' shares are
  const bool f32 = dtype == DCP_F32;
  const int per_item = (dkv ? 1 : hq / hkv) * (f32 ? kSplitSub : 1);
  return xcd_grid(g, hkv, per_item) * (f32 ? kSplitThreads : dkv ? kNarrowDkvThreads : kNarrowThreads) <= (int64_t)UINT32_MAX;
}

// Optional per-kernel event timing (see dcp_profile_enable).
struct ProfScope {
  int id;
  hipStream_t s;
  hipEvent_t stop = nullptr;
  ProfScope(int id, hipStream_t s, bool enabled = true);
  ~ProfScope();
};

// the backward behind dcp_block_attn_bwd (api.hip); may_alloc = false: fail rather than create device copies or events
dcp_status_t bwd_launch(dcp_plan_t* plan, const dcp_tensors_t* t, void* workspace, size_t workspace_bytes, hipStream_t s,
                        bool may_alloc);

// device address, on the current device, of the fixed workspace of dcp_block_attn_bwd_static (bwd_static.hip); the first
// call on a device looks it up
dcp_status_t static_scratch(void** ptr);

// scalar fp32-ALU family (any dtype; D in {32, 64, 128})
bool scalar_supports(int32_t d);
dcp_status_t scalar_fwd(const DevGroup& g, const KTensors& t, int32_t dtype, hipStream_t s);
dcp_status_t scalar_bwd_dq(const DevGroup& g, const KTensors& t, int32_t dtype, hipStream_t s);
dcp_status_t scalar_bwd_dkv(const DevGroup& g, const KTensors& t, int32_t dtype, hipStream_t s);

// MFMA family: bf16 with D = 128 (kernels_mfma_fwd / dq / dkv) and D in {32, 64} (kernels_mfma_narrow), fp32 with D in
// {32, 64, 128} (kernels_mfma_f32, kernels_mfma_f32_parts)
bool mfma_supports(int32_t dtype, int32_t d);
// the dK/dV kernel takes cut work items (KTensors::part)
inline bool mfma_splits_dkv(int32_t dtype, int32_t d) { return dtype == DCP_BF16 && d == 128; }
size_t mfma_dkv_part_bytes(int32_t n_pslots, int32_t hkv);   // size of KTensors::part for that many slots
dcp_status_t mfma_fwd(const DevGroup& g, const KTensors& t, hipStream_t s);
dcp_status_t mfma_bwd_dq(const DevGroup& g, const KTensors& t, hipStream_t s);
dcp_status_t mfma_bwd_dkv(const DevGroup& g, const KTensors& t, hipStream_t s);
// fp32 on the fp32 pipe, 32 or 16 rows per workgroup; f32_bwd is dQ and dK/dV in one launch (16 rows)
dcp_status_t mfma_f32_fwd(const DevGroup& g, const KTensors& t, int rows, hipStream_t s);
dcp_status_t mfma_f32_dq(const DevGroup& g, const KTensors& t, int rows, hipStream_t s);
dcp_status_t mfma_f32_dkv(const DevGroup& g, const KTensors& t, int rows, hipStream_t s);
dcp_status_t mfma_f32_bwd(const DevGroup& gq, const DevGroup& gkv, const KTensors& t, hipStream_t s);
// the part of mfma_fwd, mfma_bwd_dq and mfma_bwd_dkv for fp32 with D < 128 in bf16 parts
dcp_status_t mfma_f32_parts_fwd(const DevGroup& g, const KTensors& t, hipStream_t s);
dcp_status_t mfma_f32_parts_dq(const DevGroup& g, const KTensors& t, hipStream_t s);
dcp_status_t mfma_f32_parts_dkv(const DevGroup& g, const KTensors& t, hipStream_t s);
// the part of mfma_fwd, mfma_bwd_dq and mfma_bwd_dkv for bf16 with D < 128
dcp_status_t mfma_narrow_fwd(const DevGroup& g, const KTensors& t, hipStream_t s);
dcp_status_t mfma_narrow_dq(const DevGroup& g, const KTensors& t, hipStream_t s);
dcp_status_t mfma_narrow_dkv(const DevGroup& g, const KTensors& t, hipStream_t s);
// bf16 (any of these D), for launches that the others leave uneven or the chip half empty (kernels_mfma_split.hip): 4 or 8 waves
// per workgroup, work lists of whole items; split_bwd is dQ and dK/dV in one launch
dcp_status_t mfma_split_fwd(const DevGroup& g, const KTensors& t, int waves, hipStream_t s);
dcp_status_t mfma_split_dq(const DevGroup& g, const KTensors& t, int waves, hipStream_t s);
dcp_status_t mfma_split_dkv(const DevGroup& g, const KTensors& t, int waves, hipStream_t s);
dcp_status_t mfma_split_bwd(const DevGroup& gq, const DevGroup& gkv, const KTensors& t, int waves, hipStream_t s);
// per 32-row tile of every block: bounds of its rows' range arrays -> qbounds [n_t32 + 1][8]
dcp_status_t mfma_range_bounds(const DevGroup& g, const KTensors& t, const int32_t* blk_t32, int32_t n_blocks, int32_t longest_block,
                               int32_t* qbounds, hipStream_t s);

// streaming (HBM-bound) kernels
dcp_status_t stream_merge(const int32_t* merge_ptr, const int32_t* merge_idx, const int32_t* blk_mem0,
                          const int32_t* blk_len, int32_t n_blocks, int32_t longest_block, int32_t block_size, const void* o_part,
                          const float* lse_part, void* out, int64_t o_st, int64_t o_sh, float* lse,
                          int64_t total_tokens, int32_t hq, int32_t d, int32_t dtype, hipStream_t s);
dcp_status_t stream_delta(const void* o, int64_t o_st, int64_t o_sh, const void* dout, int64_t do_st, int64_t do_sh,
                          float* delta, const float* lse, float* lse2, int64_t total_tokens, int32_t hq, int32_t d,
                          int32_t dtype, hipStream_t s);
dcp_status_t stream_sum(const void* const* parts, int32_t n_parts, int32_t parts_dtype, void* dst, int32_t dst_dtype,
                        int64_t n, hipStream_t s);

// chunks: device int32 [n_chunks, 3] (src_row, dst_row, n_rows)
dcp_status_t stream_copy(const int32_t* chunks, int64_t n_chunks, const void* src, int64_t src_stride, void* dst,
                         int64_t dst_stride, int64_t row_bytes, hipStream_t s);

}  // namespace dcp
