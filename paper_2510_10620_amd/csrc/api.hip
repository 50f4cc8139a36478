// Launching entry points of the C ABI: argument validation (host side, complete before any
// launch), kernel-family selection, and the enqueue of the kernels on the caller's stream.
#include <algorithm>
#include <cmath>
#include <memory>
#include <string>
#include <vector>

#include "kernels.h"

using namespace dcp;

namespace dcp {
struct ProfRec { hipEvent_t a, b; };
static bool g_prof_on = false;
static std::vector<ProfRec> g_prof[7];
ProfScope::ProfScope(int id_, hipStream_t s_, bool enabled) : id(id_), s(s_) {
  if (!g_prof_on || !enabled) return;
  hipEvent_t a = nullptr;
  if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&stop) != hipSuccess) { stop = nullptr; return; }
  (void)hipEventRecord(a, s);
  g_prof[id].push_back({a, stop});
}
ProfScope::~ProfScope() {
  if (stop) (void)hipEventRecord(stop, s);
}
}  // namespace dcp

extern "C" dcp_status_t dcp_profile_enable(int32_t enable) {
  if (enable) {
    for (auto& v : g_prof) {
      for (auto& r : v) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
      v.clear();
    }
  }
  g_prof_on = enable != 0;
  return DCP_OK;
}

extern "C" dcp_status_t dcp_profile_read(int32_t kernel_id, double* total_ms, int64_t* launches) {
  if (kernel_id < 0 || kernel_id > 6 || !total_ms || !launches) return fail(DCP_ERR_INVALID_ARG, "bad kernel id or NULL output");
  double tot = 0;
  for (auto& r : g_prof[kernel_id]) {
    DCP_HIP_TRY(hipEventSynchronize(r.b));
    float ms = 0;
    DCP_HIP_TRY(hipEventElapsedTime(&ms, r.a, r.b));
    tot += ms;
  }
  *total_ms = tot;
  *launches = (int64_t)g_prof[kernel_id].size();
  return DCP_OK;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static dcp_status_t check_shape(const dcp_tensors_t* t) {
  if (!t) return fail(DCP_ERR_INVALID_ARG, "tensor descriptor is NULL");
  if (t->hq <= 0 || t->hkv <= 0 || t->d <= 0) return fail(DCP_ERR_INVALID_ARG, "hq, hkv, d must be positive");
  if (t->hq % t->hkv != 0) return fail(DCP_ERR_UNSUPPORTED, "hq must be a multiple of hkv");
  if (t->dtype != DCP_BF16 && t->dtype != DCP_F32) return fail(DCP_ERR_UNSUPPORTED, "dtype must be DCP_BF16 or DCP_F32");
  if (t->impl < DCP_IMPL_AUTO || t->impl > DCP_IMPL_MFMA) return fail(DCP_ERR_INVALID_ARG, "bad impl selector");
  if (!(t->softmax_scale > 0.f) || !std::isfinite(t->softmax_scale)) return fail(DCP_ERR_INVALID_ARG, "softmax_scale must be positive and finite");
  return DCP_OK;
}

static dcp_status_t check_tensor(const char* name, const void* p, int64_t st, int64_t sh, int32_t d) {
  if (!p) return fail(DCP_ERR_INVALID_ARG, std::string(name) + " is NULL");
  if (!aligned16(p)) return fail(DCP_ERR_INVALID_ARG, std::string(name) + " must be 16-byte aligned");
  if (sh < d || st < d || sh % 8 || st % 8) return fail(DCP_ERR_INVALID_ARG, std::string(name) + ": strides must be >= d and multiples of 8 elements");
  return DCP_OK;
}

// The fp32 and narrow-head MFMA kernels reach the rows of a tile through 32-bit byte offsets from its first row: 64 rows
// of 2 bytes or 32 rows of 4 bytes, so token strides of up to 2^24 elements stay below 2^31.  A tensor the call does not
// use has stride 0.
static bool short_strides(const dcp_tensors_t* t) {
  constexpr int64_t kMax = int64_t(1) << 24;
  return t->q_stride_t <= kMax && t->k_stride_t <= kMax && t->v_stride_t <= kMax && t->o_stride_t <= kMax && t->do_stride_t <= kMax &&
         t->dq_stride_t <= kMax && t->dk_stride_t <= kMax && t->dv_stride_t <= kMax;
}

// Chooses the kernel family.  AUTO: MFMA where it is covered and, outside bf16 with D = 128, the strides are short (and, as
// the callers check, the launch fits); else the thread-per-row kernels.  A caller that asks for MFMA by name gets the bf16, D = 128 kernels or a refusal.
static dcp_status_t pick_impl(const dcp_tensors_t* t, bool* use_mfma) {
  const bool wide = t->dtype == DCP_BF16 && t->d == 128;
  const bool m_ok = mfma_supports(t->dtype, t->d) && (wide || short_strides(t)), s_ok = scalar_supports(t->d);
  if (t->impl == DCP_IMPL_MFMA) {
    if (!wide) return fail(DCP_ERR_UNSUPPORTED, "DCP_IMPL_MFMA covers bf16 with head_dim 128 only");
    *use_mfma = true;
  } else if (t->impl == DCP_IMPL_SCALAR) {
    if (!s_ok) return fail(DCP_ERR_UNSUPPORTED, "scalar kernels cover head_dim 32, 64, 128");
    *use_mfma = false;
  } else {
    if (!m_ok && !s_ok) return fail(DCP_ERR_UNSUPPORTED, "no kernel covers this dtype / head_dim");
    *use_mfma = m_ok;
  }
  return DCP_OK;
}

// Whether the thread-per-row kernels are the faster ones: a walk over many short blocks costs the MFMA kernels a round trip to
// memory per table row and a mostly empty tile, the others a few instructions a key.  Times of a launch are estimated as
// walk x the rounds that its workgroups (waves) take on the chip, with constants fitted to both families' times for
// sequences of 1 to 64 tokens and blocks of 1 to 32.  Where the two are 2.5 times apart it is on the right side: fp32, D 64,
// 4/2 heads, forward + backward, thread per row against MFMA: 4 000 sequences of 8 tokens 1 148 and 4 060 us, 1 000 of 32
// 1 041 and 1 162, 500 of 64 1 079 and 677; one of 2 048 under a 64-token window in blocks of 4 996 and 2 258, of 16 458 and
// 273.  bf16 with D 64 has no such range (at most a tenth), and D 128 never had the choice.
static bool rows_are_faster(const dcp_plan_t* plan, const dcp_tensors_t* t, bool backward) {
  struct Fit { int32_t dtype, d; double row_us, start_rows, wgs, key_us, waves; };   // wgs, waves: as many run at once
  static const Fit fits[] = {{DCP_F32, 32, 2.4, 6.5, 280, 1.0, 1470}, {DCP_F32, 64, 4.0, 5, 256, 1.9, 700},
                             {DCP_F32, 128, 6.7, 5, 256, 5.3, 530}, {DCP_BF16, 32, 4.0, 3, 2048, 1.5, 1500}};
  for (const Fit& f : fits) {
    if (f.dtype != t->dtype || f.d != t->d) continue;
    const int group = t->hq / t->hkv;
    double mfma = 0, rows = 0;
    auto add = [&](const GroupSize& z, int heads, int g) {   // g: query heads walked by a workgroup or a thread
      if (z.tiles == 0) return;
      const double n_wgs = (double)z.tiles * heads, n_waves = (double)z.waves * heads;
      mfma += f.row_us * (f.start_rows + (z.tile_ents + z.tile_tiles * g / 8.0) / z.tiles) * std::max(1.0, n_wgs / f.wgs);
      rows += 12 + f.key_us * (2 + z.wave_keys * (double)g / z.waves) * std::max(1.0, n_waves / f.waves);
    };
    if (!backward) add(plan->size[0], t->hq, 1);
    else { add(plan->size[1], t->hq, 1); add(plan->size[2], t->hkv, group); }
    return rows < mfma;
  }
  return false;
}

// Which of the MFMA kernels a launch takes.  bf16: those that share a tile among the waves of a workgroup, or those whose four or
// eight waves split the other side (kernels_mfma_split.hip); fp32: 32 rows a workgroup or 16
// on the fp32 pipe (D < 128: and 32 rows a wave in bf16 parts, see kWalkFits).  The first kind streams least from the
// L2 and wins where the chip is full of equal work; the second finishes a long walk several times sooner and wins where a launch
// has few items or waits for its longest: bf16, 5 196 tokens, 16/4 heads, blocks of 4 096, dK/dV 374 and 130 us; 4 528 tokens, 4/1
// heads, forward 31 and 20; 65 536 tokens, 32/8 heads, forward 2.6 and 5.3 ms; fp32, 1 723 tokens, one head of 64, dK/dV 70 and 44 us,
// 8 192 tokens, 8/2 heads, dQ 504 and 608.  The time of a launch is estimated as
//     start + sqrt((chain x pairs of the longest item)^2 + (share x all pairs / 512)^2) + item x items / 512
// (a pair per query head for `share`; for dK/dV an item walks its KV head's whole group; 512 workgroups are resident) with
// constants (us; chain and share per million pairs) fitted to the times of 230 batches in bf16, 121 / 69 / 40 of them with D 128 /
// 64 / 32, and 32 in fp32 with D 128 (D 64 and 32 without parts, kPipeFits: 47 / 26): 1 to 1 000 sequences of 1 to 65 536 tokens, 1 to 16 KV heads, groups of 1 to 8, blocks of 64
// to 4 096.  The estimates are 12 to 27 % off, so the second kind is taken only where it is estimated at 0.9 (fp32: 0.85, D 32 and 64 0.9) of
// the first or less: over those batches no call was slower than with the first kind alone by more than 2 %, on average it took 0.87 /
// 0.64 / 0.71 of the time in the forward and 0.79 / 0.52 / 0.47 in the backward (fp32 without parts 0.78 / 0.88 / 0.92 and 0.66 / 0.71 / 0.66).
// bf16 with D 128 where no block has more than 64 rows: the pairs are those that are walked (LaunchSize), since a split workgroup has 32
// rows and walks such an item as long as one of 128 rows.  Counted as visible pairs, its dK/dV was estimated at 0.6 of its time: 5 765
// tokens, 8/2 heads, blocks of 64, backward 177 us with shared tiles and 329 in the form that was taken.  Shared tiles take 0.85 of
// their estimate there (the waves without rows leave their issue slots to the CU's other workgroup), hence
// kSureShort.  149 batches with blocks of 16 to 64: 34 were slower than with shared tiles alone by more than 3 %, up to 1.81 times; now
// 8 are, up to 1.13 (blocks of 64: 1.07).
// Per-token ranges, whose pairs are a guess (windows of 32 to 4 096, sinks, mask blocks, shared questions; blocks of 64 to 4 096), measured over
// 251 batches of all types: forward 0.63 to 0.96, backward 0.58 to 0.75 of the time of the first kind alone, single calls up to 1.05 of it.
// fp32 with D 32 and 64 (the kernels in parts beside 16 rows): 587 batches of 100 to 16 384 tokens, and what the second choice below makes of it.
struct LaunchFit { double start, chain, share, item; };
// bf16: shared tiles, four waves, eight waves; fp32: 32 rows and 16, with D < 128 in parts with several groups (dK/dV: eight waves), 16 rows, and
// in parts with one (kFull); kRows: the thread-per-row kernels
enum { kRows = DCP_FORM_ROWS, kShared = DCP_FORM_SHARED, kSplit = DCP_FORM_SPLIT, kSplit8 = DCP_FORM_SPLIT8, kForms, kFull = kSplit8 };
struct LaunchFits { int32_t dtype, d; double sure; LaunchFit fwd[kForms], dq[kForms], dkv[kForms], bwd[kForms]; };   // bwd: dQ and dK/dV in one launch
static const LaunchFits kFits[] = {
    {DCP_BF16, 128, 0.9, {{7.0, 128, 253, 5.7}, {5.0, 53.5, 373, 18.9}, {5.3, 30.1, 380, 41.1}}, {{7.3, 167, 335, 7.5}, {6.6, 50.4, 428, 29.6}, {7.8, 28.9, 433, 62.8}},
     {{9.4, 283, 500, 16.8}, {6.9, 77.3, 519, 29.0}, {8.2, 47.4, 531, 63.0}}, {{}, {8.6, 118, 1230, 31.5}, {9.6, 68.1, 1230, 66.7}}},
    {DCP_BF16, 64, 0.9, {{6.4, 198, 249, 2.8}, {4.7, 53.7, 282, 7.7}, {4.7, 23.9, 275, 17.3}}, {{6.4, 196, 294, 4.5}, {5.2, 54.0, 323, 14.9}, {5.6, 14.5, 378, 39.7}},
     {{7.3, 232, 509, 19.0}, {5.1, 84.6, 492, 21.9}, {5.1, 55.1, 510, 45.7}}, {{}, {5.3, 101, 940, 20.6}, {4.9, 60.5, 1010, 44.6}}},
    {DCP_BF16, 32, 0.9, {{5.0, 134, 181, 5.1}, {3.7, 42.6, 193, 9.0}, {3.3, 28.6, 209, 18.0}}, {{5.3, 137, 204, 5.1}, {4.1, 44.1, 207, 10.2}, {4.1, 29.4, 221, 18.9}},
     {{10.7, 180, 394, 11.3}, {6.1, 70.2, 341, 10.9}, {6.2, 43.3, 358, 19.8}}, {{}, {6.1, 80.7, 655, 11.7}, {4.5, 42.0, 779, 33.2}}},
    {DCP_F32, 128, 0.85, {{9.6, 223, 2220, 82.9}, {7.6, 151, 2810, 32.9}}, {{13.9, 314, 3240, 120}, {9.9, 248, 4860, 40.2}},
     {{15.9, 448, 3710, 183}, {10.8, 274, 4960, 89.9}}, {{}, {11.4, 364, 11050, 76.4}}},
    {DCP_F32, 64, 0.9, {{11.3, 271, 609, 17.7}, {7.25, 125, 1800, 25.6}, {12.2, 386, 394, 9.45}}, {{16.0, 399, 1130, 8.43}, {6.22, 225, 2860, 29.9}, {12.1, 519, 820, 6.74}},
     {{14.2, 159, 1350, 56.9}, {10.2, 142, 1880, 25.3}, {12.8, 207, 1360, 25.7}}, {{}, {9.09, 131, 6610, 44.6}}},
    {DCP_F32, 32, 0.9, {{8.31, 129, 554, 12.8}, {6.41, 64.8, 973, 22.4}, {9.42, 326, 420, 4.15}}, {{10.4, 159, 696, 21.4}, {7.08, 97.6, 1340, 22.9}, {10.4, 471, 462, 6.75}},
     {{10.1, 89.3, 1010, 16.8}, {6.24, 85.9, 2830, 23.2}, {9.24, 126, 913, 15.2}}, {{}, {8.83, 110, 2470, 38.4}}}};
static constexpr double kLaunchGap = 1.0;   // between two launches
static constexpr double kSureShort = 0.8, kSureShort8 = 0.7;   // `sure` of dK/dV over short blocks with four and eight waves
static bool short_blocks(const dcp_tensors_t* t, const LaunchSize& z) { return t->dtype == DCP_BF16 && t->d == 128 && z.walk > 0; }

static double launch_us(const LaunchFit& f, double longest, double total, double items) {
  return f.start + std::hypot(f.chain * longest * 1e-6, f.share * total / 512e6) + f.item * items / 512;
}

// The row of the table, or null where there is no choice: launches that may have more threads than 32 bits count.
static const LaunchFits* fits_of(const dcp_tensors_t* t, const LaunchSize& z) {
  if (z.items * t->hq >= (int64_t)((UINT32_MAX >> 3) / (kItemRows / 16 * kSplitThreads))) return nullptr;
  for (const LaunchFits& f : kFits)
    if (f.dtype == t->dtype && f.d == t->d) return &f;
  return nullptr;
}
static int last_form(const dcp_tensors_t* t) { return t->dtype == DCP_BF16 ? kSplit8 : kSplit; }

// The form of a launch whose estimates are us[kShared ..], and its estimate.  sure, sure8: for kSplit and kSplit8.
static int least_form(double sure, double sure8, const dcp_tensors_t* t, const double* us, double* out) {
  int best = kShared;
  double least = HUGE_VAL;
  for (int v = kSplit; v <= last_form(t); v++)
    if (us[v] < least && us[v] < (v == kSplit ? sure : sure8) * us[kShared]) { best = v; least = us[v]; }
  *out = us[best];
  return best;
}

// fp32 with D < 128 has four kernels for the forward and for dQ: on the fp32 pipe with 32 rows a workgroup or 16, in bf16 parts
// with one group of waves or several; dK/dV has 16 rows, and parts with four waves or eight (with 32 rows it was never the best).
// By pairs two of them come into question: the faster of those in parts and 16 rows (kFits: kFull, kShared, kSplit), or what the choice between 32 and 16 rows would be without parts (kPipeFits).  Where the
// second is estimated at 0.9 of the first or less by what the workgroups walk (WalkSize, kWalkFits), it is taken.  Pairs alone
// misjudge few long walks and short blocks, where workgroups of 128 rows in parts walk far longer than the pairs say: 4 407 tokens, 2/1
// heads of 64, blocks of 64, forward / dQ 191 / 253 us in parts, 107 / 145 and 81 / 130 on the fp32 pipe; 9 839 tokens under mask blocks of
// 256, 4/4 heads, 444 / 575 and 181 / 251, 136 / 216.  What is walked alone misjudges ranges, of which neither knows the widths.
// 1 294 batches each of D 32 and 64 (100 to 16 384 tokens, 1 to 40 sequences, blocks of 64 to 2 048, a third with ranges; the constants of
// kWalkFits fitted to the times of 905 of them, then moved within what those allow until the choices cost least): against kPipeFits
// alone 0.90 of the time on average, 20 (D 32) and 17 batches more than 3 % slower, 3 and 4 more than 10 %, up to 1.38 and 1.37 (with kFits
// alone 87 and 68, 39 and 37, up to 1.42 and 1.79); against kFits alone 0.99, 16 and 19 more than 3 % slower, none and 4 more than 10 %,
// up to 1.08 and 1.21.  The best kernel each time would take 0.97 of it.
static bool in_parts(const dcp_tensors_t* t) { return t->dtype == DCP_F32 && t->d < 128; }
struct PipeFits { int32_t d; double sure; LaunchFit f[3][2], bwd; };   // forward, dQ, dK/dV: 32 rows, 16 rows
static const PipeFits kPipeFits[] = {
    {64, 0.87, {{{6.9, 125, 1180, 41.4}, {5.4, 88.9, 1300, 31.5}}, {{8.7, 174, 1640, 54.4}, {6.3, 144, 2160, 38.8}}, {{12.5, 252, 1990, 61.7}, {8.1, 164, 2310, 31.5}}},
     {8.6, 170, 5574, 51.4}},
    {32, 0.86, {{{5.1, 70.8, 573, 21.1}, {4.8, 42.8, 748, 23.3}}, {{5.8, 97.3, 789, 24.6}, {4.8, 71.1, 1130, 27.4}}, {{6.6, 152, 1120, 52.6}, {5.9, 94.8, 1390, 26.6}}},
     {4.5, 109, 2975, 41.0}}};
enum { kPipe32, kPipe16, kParts1, kParts2, kF32Kernels };
struct WalkFits { int32_t d; LaunchFit f[3][kF32Kernels], bwd; };   // of WalkSize in place of pairs
static const WalkFits kWalkFits[] = {
    {64, {{{6.09, 115, 1420, 58.8}, {8.11, 90.4, 1450, 17.7}, {8.19, 437, 573, 3.12}, {10.5, 374, 506, 4.41}},
          {{5.24, 255, 1730, 42.1}, {7.15, 142, 1710, 26.6}, {14, 402, 869, 1.54}, {12.8, 396, 1570, 6.21}},
          {{}, {10.4, 208, 2210, 24.9}, {11.7, 195, 1280, 16.3}, {13.4, 159, 1340, 42.8}}}, {9.35, 190, 6200, 47.1}},
    {32, {{{5.13, 54.3, 725, 19.9}, {5.21, 38.9, 806, 33}, {5.52, 212, 351, 1.85}, {7.3, 101, 823, 8.82}},
          {{4.65, 71.1, 1350, 19.9}, {4.15, 69, 1020, 28.1}, {8.27, 374, 497, 1.38}, {10.7, 133, 706, 19.9}},
          {{}, {12.3, 152, 1380, 17}, {9.31, 119, 816, 12.6}, {12, 135, 656, 33.5}}}, {8.63, 85.3, 4180, 37.1}}};
static constexpr double kSecond = 0.9;   // the other choice is taken where it is estimated at this much of the first or less

struct F32Launch { double longest, total, items; };   // as launch_us takes them
// Of forward (gid 0), dQ (1), dK/dV (2), by pairs: the kernel with those in parts to choose from, that without, their estimates; the faster in parts.
struct F32Pick { int first, second, parts; double first_us, second_us; };
static F32Launch f32_pairs(dcp_plan_t* plan, const dcp_tensors_t* t, int gid) {
  const int group = t->hq / t->hkv;
  const LaunchSize& z = plan->host_items(gid, gid < 2 ? group : 0, xcd_segments(t->hkv)).size;
  return {(double)z.longest * (gid == 2 ? group : 1), (double)z.total * t->hq, (double)z.items * (gid == 2 ? t->hkv : t->hq)};
}
template <class F> static const F& f32_row(const F (&rows)[2], int32_t d) { return rows[rows[0].d == d ? 0 : 1]; }
static double launch_us(const LaunchFit& f, const F32Launch& x) { return launch_us(f, x.longest, x.total, x.items); }
static F32Pick f32_pick(const LaunchFits& fits, const dcp_tensors_t* t, int gid, const F32Launch& x) {
  const LaunchFit* f = gid == 0 ? fits.fwd : gid == 1 ? fits.dq : fits.dkv;
  const PipeFits& pf = f32_row(kPipeFits, t->d);
  const double p1 = launch_us(f[kFull], x), p2 = launch_us(f[kShared], x), r16 = launch_us(f[kSplit], x), parts = std::min(p1, p2);
  const double a = launch_us(pf.f[gid][0], x), b = launch_us(pf.f[gid][1], x);
  F32Pick c;
  const bool rows16 = r16 < fits.sure * parts, pipe16 = b < pf.sure * a;
  c.parts = p1 < p2 ? kParts1 : kParts2;
  c.first = rows16 ? kPipe16 : c.parts;
  c.first_us = rows16 ? r16 : parts;
  c.second = pipe16 ? kPipe16 : kPipe32;
  c.second_us = pipe16 ? b : a;
  return c;
}
// by what is walked
static F32Launch f32_walked(dcp_plan_t* plan, const dcp_tensors_t* t, int gid, int kernel, double items) {
  const WalkSize& w = plan->walk_size(gid);
  const int rows = kernel == kPipe16 ? 0 : kernel == kPipe32 || gid == 2 ? 1 : t->d == 32 && kernel == kParts2 ? 2 : 3;
  return {(double)w.longest * (gid == 2 ? t->hq / t->hkv : 1), (double)w.total[rows] * t->hq, items};
}
// The kernel of a launch, and its estimate by what is walked.
static int f32_kernel(dcp_plan_t* plan, const dcp_tensors_t* t, int gid, const F32Launch& x, const F32Pick& c, double* us) {
  const LaunchFit* f = f32_row(kWalkFits, t->d).f[gid];
  const double first = launch_us(f[c.first], f32_walked(plan, t, gid, c.first, x.items)), second = launch_us(f[c.second], f32_walked(plan, t, gid, c.second, x.items));
  const bool other = (gid < 2 || c.second == kPipe16) && second < kSecond * first;
  *us = other ? second : first;
  return other ? c.second : c.first;
}
static F32Choice f32_choose(dcp_plan_t* plan, const dcp_tensors_t* t) {
  F32Choice c{{kParts1, kParts1, kParts1}, {kParts1, kParts1, kParts1}, false};
  const int group = t->hq / t->hkv, n_seg = xcd_segments(t->hkv);
  F32Launch x[3];
  F32Pick p[3];
  double us[3];
  for (int gid = 0; gid < 3; gid++) {
    const LaunchFits* f = fits_of(t, plan->host_items(gid, gid < 2 ? group : 0, n_seg).size);
    if (!f) return c;
    x[gid] = f32_pairs(plan, t, gid);
    p[gid] = f32_pick(*f, t, gid, x[gid]);
    c.kernel[gid] = f32_kernel(plan, t, gid, x[gid], p[gid], &us[gid]);
    c.parts[gid] = p[gid].parts;
  }
  // one launch for dQ and dK/dV or two: the same way, each choice with its own two launches by pairs
  const LaunchFits* f = fits_of(t, plan->host_items(1, group, n_seg).size);
  const PipeFits& pf = f32_row(kPipeFits, t->d);
  const F32Launch xb{x[2].longest, x[2].total, x[2].items + x[1].items};
  const bool first = launch_us(f->bwd[kSplit], xb) < f->sure * (p[1].first_us + p[2].first_us + kLaunchGap);
  const bool second = launch_us(pf.bwd, xb) < pf.sure * (p[1].second_us + p[2].second_us + kLaunchGap);
  const double one = launch_us(f32_row(kWalkFits, t->d).bwd, f32_walked(plan, t, 2, kPipe16, xb.items)), two = us[1] + us[2] + kLaunchGap;
  c.one_launch = first == second ? first : first ? !(two < kSecond * one) : one < kSecond * two;
  return c;
}
// ... once for a plan and shape
static F32Choice f32_choice(dcp_plan_t* plan, const dcp_tensors_t* t) {
  const std::tuple<int, int, int> key(t->hq, t->hkv, t->d);
  {
    std::lock_guard<std::mutex> lock(plan->mu);
    const auto hit = plan->f32_choices.find(key);
    if (hit != plan->f32_choices.end()) return hit->second;
  }
  const F32Choice c = f32_choose(plan, t);
  std::lock_guard<std::mutex> lock(plan->mu);
  return plan->f32_choices.emplace(key, c).first->second;
}
static int f32_form(int kernel) { return kernel == kPipe16 ? kSplit : kShared; }
static int f32_groups(int kernel) { return kernel == kParts1 ? 1 : kernel == kParts2 ? 2 : 0; }

static int pick_q(const LaunchFits& fits, const LaunchFit* f, const dcp_tensors_t* t, const LaunchSize& z, double* us) {
  double x[kForms];
  const bool walked = short_blocks(t, z);
  const double longest = (double)(walked ? z.walk : z.longest), total = (double)(walked ? z.walk_total : z.total) * t->hq;
  for (int v = kShared; v <= last_form(t); v++) x[v] = launch_us(f[v], longest, total, (double)z.items * t->hq);
  return least_form(fits.sure, fits.sure, t, x, us);
}

struct BwdChoice { int dq, dkv, both; };   // both: the form of the one launch, or kShared (two launches)
static BwdChoice pick_bwd(const dcp_tensors_t* t, const LaunchSize& zq, const LaunchSize& zk, bool one_launch) {
  BwdChoice c{kShared, kShared, kShared};
  const LaunchFits* f = fits_of(t, zq);
  if (!f || !fits_of(t, zk)) return c;
  const bool walked = short_blocks(t, zk);
  const double group = t->hq / t->hkv, longest = (double)(walked ? zk.walk : zk.longest) * group,
               total = (double)(walked ? zk.walk_total : zk.total) * t->hq, items = (double)zk.items * t->hkv;
  double us_q = 0, us_k = 0, x[kForms];
  c.dq = pick_q(*f, f->dq, t, zq, &us_q);
  for (int v = kShared; v <= last_form(t); v++) x[v] = launch_us(f->dkv[v], longest, total, items);
  if (mfma_splits_dkv(t->dtype, t->d))   // shared tiles go over a list of cut items
    x[kShared] = launch_us(f->dkv[kShared], (double)(walked ? zk.walk_part : zk.longest_part) * group, total, (double)zk.parts * t->hkv);
  c.dkv = least_form(walked ? kSureShort : f->sure, walked ? kSureShort8 : f->sure, t, x, &us_k);
  double least = f->sure * (us_q + us_k + kLaunchGap);
  for (int v = kSplit; one_launch && v <= last_form(t); v++) {
    const double us = launch_us(f->bwd[v], longest, total, items + (double)zq.items * t->hq);
    if (us < least) { c.both = v; least = us; }
  }
  return c;
}

// Whether dQ and dK/dV may run side by side: each reads Q, K, V, O, dO and the LSE to its end, so no gradient may share memory with
// them.  Two launches allow dQ over O, dK over K and dV over V: a workgroup loads its own rows of these before it stores them,
// and dK/dV, which starts when dQ has ended, does not read O.  Tensors that only interleave count as sharing.
static bool one_launch_is_safe(const dcp_plan_t* plan, const dcp_tensors_t* t) {
  struct Span { uintptr_t lo, hi; };
  const int64_t es = t->dtype == DCP_BF16 ? 2 : 4;
  auto span = [&](const void* p, int64_t rows, int heads, int64_t st, int64_t sh) {
    const uintptr_t lo = (uintptr_t)p;
    return Span{lo, rows > 0 ? lo + (uintptr_t)(((rows - 1) * st + (heads - 1) * sh + t->d) * es) : lo};
  };
  const int64_t nq = plan->q_rows, nk = plan->kv_rows;
  const Span in[] = {span(t->q, nq, t->hq, t->q_stride_t, t->q_stride_h), span(t->k, nk, t->hkv, t->k_stride_t, t->k_stride_h),
                     span(t->v, nk, t->hkv, t->v_stride_t, t->v_stride_h), span(t->out, nq, t->hq, t->o_stride_t, t->o_stride_h),
                     span(t->dout, nq, t->hq, t->do_stride_t, t->do_stride_h),
                     {(uintptr_t)t->lse, (uintptr_t)t->lse + (uintptr_t)(t->hq * nq) * sizeof(float)}};
  const Span out[] = {span(t->dq, nq, t->hq, t->dq_stride_t, t->dq_stride_h), span(t->dk, nk, t->hkv, t->dk_stride_t, t->dk_stride_h),
                      span(t->dv, nk, t->hkv, t->dv_stride_t, t->dv_stride_h)};
  for (const Span& o : out)
    for (const Span& i : in)
      if (o.lo < i.hi && i.lo < o.hi) return false;
  return true;
}
static int waves_of(int form) { return form == kSplit ? 4 : 8; }

// The form of a forward over the list g.
static int fwd_form(dcp_plan_t* plan, const dcp_tensors_t* t, bool use_mfma, const DevGroup& g) {
  if (!use_mfma || !mfma_launch_fits(g, false, t->dtype, t->d, t->hq, t->hkv) || rows_are_faster(plan, t, false)) return kRows;
  if (in_parts(t)) return f32_form(f32_choice(plan, t).kernel[0]);
  const LaunchSize& z = plan->host_items(0, t->hq / t->hkv, xcd_segments(t->hkv)).size;
  const LaunchFits* f = fits_of(t, z);
  double us = 0;
  return f ? pick_q(*f, f->fwd, t, z, &us) : kShared;
}

// The forms of a backward over the lists gq and gkv, the latter of items cut for `heads` KV heads (0: whole items).
static BwdChoice bwd_forms(dcp_plan_t* plan, const dcp_tensors_t* t, bool use_mfma, const DevGroup& gq, const DevGroup& gkv, int cut, int heads,
                           bool one_launch) {
  if (!use_mfma || !mfma_launch_fits(gq, false, t->dtype, t->d, t->hq, t->hkv) ||
      !mfma_launch_fits(gkv, true, t->dtype, t->d, t->hq, t->hkv) || rows_are_faster(plan, t, true))
    return {kRows, kRows, kShared};
  if (in_parts(t)) {
    const F32Choice f = f32_choice(plan, t);
    return {f32_form(f.kernel[1]), f32_form(f.kernel[2]), one_launch && f.one_launch ? kSplit : kShared};
  }
  const int n_seg = xcd_segments(t->hkv);
  BwdChoice c = pick_bwd(t, plan->host_items(1, t->hq / t->hkv, n_seg).size, plan->host_items(2, cut, n_seg).size, one_launch);
  if (heads != 0) c.dkv = c.both = kShared;
  return c;
}

// KV heads the dK/dV list is cut for (0: whole items).  All other lists are the same for every kernel family, so a plan
// made ready for a shape serves it whichever family a call's strides or its `impl` choose.
static int cut_heads(bool use_mfma, int32_t dtype, int32_t d, int32_t hkv) { return use_mfma && mfma_splits_dkv(dtype, d) ? hkv : 0; }

// The list that the dK/dV launch of a call wants, as host_items names it: the split kernels take whole items.
static int dkv_heads(dcp_plan_t* plan, const dcp_tensors_t* t, bool use_mfma, int n_seg, bool one_launch) {
  const int cut = cut_heads(use_mfma, t->dtype, t->d, t->hkv);
  if (cut == 0) return 0;
  const BwdChoice c = pick_bwd(t, plan->host_items(1, t->hq / t->hkv, n_seg).size, plan->host_items(2, cut, n_seg).size, one_launch);
  return c.dkv != kShared || c.both != kShared ? 0 : cut;
}

static KTensors pack(const dcp_plan_t* plan, const dcp_tensors_t* t) {
  KTensors k{};
  k.q = t->q; k.k = t->k; k.v = t->v; k.dout = t->dout; k.out_in = t->out;
  k.out = t->out; k.dq = t->dq; k.dk = t->dk; k.dv = t->dv;
  k.lse = t->lse; k.delta = nullptr;
  k.ranges = plan->has_ranges ? t->attn_ranges : nullptr;   // kernels skip all range work when no row has per-token ranges
  k.window = plan->has_window ? plan->window : 0;
  k.sink = plan->has_window ? plan->sink : 0;
  k.masked = (plan->has_ranges || plan->has_window) ? 1 : 0;
  k.qbounds = nullptr;
  k.q_st = t->q_stride_t; k.q_sh = t->q_stride_h; k.k_st = t->k_stride_t; k.k_sh = t->k_stride_h;
  k.v_st = t->v_stride_t; k.v_sh = t->v_stride_h; k.o_st = t->o_stride_t; k.o_sh = t->o_stride_h;
  k.do_st = t->do_stride_t; k.do_sh = t->do_stride_h; k.dq_st = t->dq_stride_t; k.dq_sh = t->dq_stride_h;
  k.dk_st = t->dk_stride_t; k.dk_sh = t->dk_stride_h; k.dv_st = t->dv_stride_t; k.dv_sh = t->dv_stride_h;
  k.q_rows = plan->q_rows;
  k.hq = t->hq; k.hkv = t->hkv; k.d = t->d; k.dtype = t->dtype; k.block_size = plan->block_size;
  k.scale = t->softmax_scale;
  k.use_slots = plan->use_slots ? 1 : 0;
  k.by_head = plan->kv_by_head ? 1 : 0;
  return k;
}

extern "C" dcp_status_t dcp_plan_prepare(dcp_plan_t* plan, int32_t hq, int32_t hkv, int32_t d, int32_t dtype, int32_t impl,
                                         void* stream) {
  if (!plan) return fail(DCP_ERR_INVALID_ARG, "plan is NULL");
  dcp_tensors_t t{};
  t.hq = hq; t.hkv = hkv; t.d = d; t.dtype = dtype; t.impl = impl; t.softmax_scale = 1.f;
  dcp_status_t st = check_shape(&t);
  if (st != DCP_OK) return st;
  bool use_mfma = false;
  if ((st = pick_impl(&t, &use_mfma)) != DCP_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if ((st = plan->ensure_device(s)) != DCP_OK) return st;
  void* scratch_addr = nullptr;   // looked up here so that dcp_block_attn_bwd_static finds it ready
  if ((st = static_scratch(&scratch_addr)) != DCP_OK) return st;
  if (plan->total_tokens == 0) return DCP_OK;
  DevGroup g;
  const int n_seg = xcd_segments(hkv);
  if ((st = plan->group_for(0, s, &g, hq / hkv, n_seg)) != DCP_OK) return st;
  if ((st = plan->group_for(1, s, &g, hq / hkv, n_seg)) != DCP_OK) return st;
  if (use_mfma && in_parts(&t)) (void)f32_choice(plan, &t);
  return plan->group_for(2, s, &g, dkv_heads(plan, &t, use_mfma, n_seg, true), n_seg);
}

extern "C" dcp_status_t dcp_block_attn_fwd(dcp_plan_t* plan, const dcp_tensors_t* t, void* stream) {
  if (!plan) return fail(DCP_ERR_INVALID_ARG, "plan is NULL");
  dcp_status_t st = check_shape(t);
  if (st != DCP_OK) return st;
  bool use_mfma = false;
  if ((st = pick_impl(t, &use_mfma)) != DCP_OK) return st;
  if (plan->total_tokens == 0) return DCP_OK;
  if ((st = check_tensor("q", t->q, t->q_stride_t, t->q_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("k", t->k, t->k_stride_t, t->k_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("v", t->v, t->v_stride_t, t->v_stride_h, t->d)) != DCP_OK) return st;
  if (!t->out || !aligned16(t->out)) return fail(DCP_ERR_INVALID_ARG, "out is NULL or not 16-byte aligned");
  if (!t->lse) return fail(DCP_ERR_INVALID_ARG, "lse is NULL");
  if (!plan->use_slots && (st = check_tensor("out", t->out, t->o_stride_t, t->o_stride_h, t->d)) != DCP_OK) return st;
  if (plan->has_ranges && !t->attn_ranges) return fail(DCP_ERR_INVALID_ARG, "table has RANGES rows but attn_ranges is NULL");
  if (plan->has_window && plan->window <= 0) return fail(DCP_ERR_INVALID_ARG, "table has WINDOW rows but dcp_plan_set_window was not called");
  hipStream_t s = (hipStream_t)stream;
  DevGroup g;
  if ((st = plan->group_for(0, s, &g, t->hq / t->hkv, xcd_segments(t->hkv))) != DCP_OK) return st;
  const int form = fwd_form(plan, t, use_mfma, g);
  KTensors k = pack(plan, t);
  ProfScope ps(DCP_K_FWD, s);
  if (form == kRows) return scalar_fwd(g, k, t->dtype, s);
  if (form == kShared) {
    if (in_parts(t)) k.part_groups = f32_groups(f32_choice(plan, t).kernel[0]);
    return mfma_fwd(g, k, s);
  }
  return t->dtype == DCP_F32 ? mfma_f32_fwd(g, k, 16, s) : mfma_split_fwd(g, k, waves_of(form), s);
}

extern "C" dcp_status_t dcp_merge_partials(dcp_plan_t* plan, const void* o_part, const float* lse_part, void* out,
                                           int64_t o_stride_t, int64_t o_stride_h, float* lse, int32_t hq, int32_t d,
                                           int32_t dtype, void* stream) {
  if (!plan) return fail(DCP_ERR_INVALID_ARG, "plan is NULL");
  if (!plan->use_slots) return fail(DCP_ERR_INVALID_ARG, "plan was created without output slots");
  if (hq <= 0 || d <= 0 || d % 8) return fail(DCP_ERR_UNSUPPORTED, "merge needs hq > 0 and d a positive multiple of 8");
  if (dtype != DCP_BF16 && dtype != DCP_F32) return fail(DCP_ERR_UNSUPPORTED, "dtype must be DCP_BF16 or DCP_F32");
  if (plan->total_tokens == 0) return DCP_OK;
  if (plan->n_slots > 0 && (!o_part || !lse_part || !aligned16(o_part))) return fail(DCP_ERR_INVALID_ARG, "o_part / lse_part NULL or misaligned");
  dcp_status_t st = check_tensor("out", out, o_stride_t, o_stride_h, d);
  if (st != DCP_OK) return st;
  if (!lse) return fail(DCP_ERR_INVALID_ARG, "lse is NULL");
  hipStream_t s = (hipStream_t)stream;
  if ((st = plan->ensure_device(s)) != DCP_OK) return st;
  ProfScope ps(DCP_K_MERGE, s);
  return stream_merge(plan->d_merge_ptr, plan->d_merge_idx, plan->d_q_mem0, plan->d_fwd.blk_len, plan->n_blocks,
                      plan->longest_block, plan->block_size, o_part, lse_part, out, o_stride_t, o_stride_h, lse, plan->q_rows, hq, d,
                      dtype, s);
}

extern "C" dcp_status_t dcp_bwd_delta(const dcp_tensors_t* t, int64_t total_tokens, float* delta, void* stream) {
  if (!t) return fail(DCP_ERR_INVALID_ARG, "tensor descriptor is NULL");
  if (t->hq <= 0 || t->d <= 0 || t->d % 8 || t->d > 256 || (t->d & (t->d - 1))) return fail(DCP_ERR_UNSUPPORTED, "delta needs d a power of two in 8..256");
  if (t->dtype != DCP_BF16 && t->dtype != DCP_F32) return fail(DCP_ERR_UNSUPPORTED, "dtype must be DCP_BF16 or DCP_F32");
  if (total_tokens < 0) return fail(DCP_ERR_INVALID_ARG, "total_tokens < 0");
  if (total_tokens == 0) return DCP_OK;
  dcp_status_t st;
  if ((st = check_tensor("out", t->out, t->o_stride_t, t->o_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("dout", t->dout, t->do_stride_t, t->do_stride_h, t->d)) != DCP_OK) return st;
  if (!delta) return fail(DCP_ERR_INVALID_ARG, "delta is NULL");
  ProfScope ps(DCP_K_DELTA, (hipStream_t)stream);
  return stream_delta(t->out, t->o_stride_t, t->o_stride_h, t->dout, t->do_stride_t, t->do_stride_h, delta, nullptr,
                      nullptr, total_tokens, t->hq, t->d, t->dtype, (hipStream_t)stream);
}

// Workspace layout: delta [Hq, rows] | lse2 [Hq, rows] | range-bound summaries | partial dK / dV sums of split items.
struct BwdWorkspace {
  size_t n_hT, n_bounds, n_part;
  size_t total() const { return 2 * n_hT + n_bounds + n_part; }
};

static BwdWorkspace bwd_workspace(dcp_plan_t* plan, int32_t hq, int32_t hkv, int32_t d, int32_t dtype) {
  BwdWorkspace w{};
  w.n_hT = (size_t)hq * (size_t)plan->q_rows * sizeof(float);
  w.n_hT = (w.n_hT + 255) & ~(size_t)255;
  // range-bound summaries of every 32-row tile (+1 spare entry), only for tables with RANGES or WINDOW rows
  w.n_bounds = (plan->has_ranges || plan->has_window) ? ((size_t)plan->blk_t32.back() + 1) * 8 * sizeof(int32_t) : 0;
  w.n_bounds = (w.n_bounds + 255) & ~(size_t)255;
  if (hkv > 0 && mfma_splits_dkv(dtype, d)) w.n_part = mfma_dkv_part_bytes(plan->host_items(2, hkv, xcd_segments(hkv)).n_pslots, hkv);
  return w;
}

extern "C" dcp_status_t dcp_plan_export_dkv_items(dcp_plan_t* plan, int32_t hkv, int32_t* dst, int64_t capacity_rows,
                                                  int64_t* n_items_out) {
  if (!plan || !n_items_out) return fail(DCP_ERR_INVALID_ARG, "plan or n_items_out is NULL");
  if (hkv <= 0) return fail(DCP_ERR_INVALID_ARG, "hkv must be positive");
  const HostItems& hi = plan->host_items(2, hkv, xcd_segments(hkv));
  *n_items_out = (int64_t)hi.items.size();
  if (dst) {
    if (capacity_rows < (int64_t)hi.items.size()) return fail(DCP_ERR_INVALID_ARG, "export capacity too small");
    for (size_t i = 0; i < hi.items.size(); i++) {
      const WorkItem& w = hi.items[i];
      dst[5 * i] = w.unit; dst[5 * i + 1] = w.tile; dst[5 * i + 2] = w.e0; dst[5 * i + 3] = w.e1; dst[5 * i + 4] = w.pslot;
    }
  }
  return DCP_OK;
}

extern "C" dcp_status_t dcp_plan_export_dkv_segments(dcp_plan_t* plan, int32_t hkv, int32_t* n_seg_out, int32_t* seg_out) {
  if (!plan || !n_seg_out || !seg_out) return fail(DCP_ERR_INVALID_ARG, "plan, n_seg_out or seg_out is NULL");
  if (hkv <= 0) return fail(DCP_ERR_INVALID_ARG, "hkv must be positive");
  const HostItems& hi = plan->host_items(2, hkv, xcd_segments(hkv));
  *n_seg_out = hi.n_seg;
  for (int k = 0; k <= 8; k++) seg_out[k] = hi.seg[k];
  return DCP_OK;
}

extern "C" dcp_status_t dcp_plan_export_forms(dcp_plan_t* plan, int32_t hq, int32_t hkv, int32_t d, int32_t dtype, int32_t* forms) {
  if (!plan || !forms) return fail(DCP_ERR_INVALID_ARG, "plan or forms is NULL");
  dcp_tensors_t t{};
  t.hq = hq; t.hkv = hkv; t.d = d; t.dtype = dtype; t.softmax_scale = 1.f;
  dcp_status_t st = check_shape(&t);
  bool use_mfma = false;
  if (st == DCP_OK) st = pick_impl(&t, &use_mfma);
  if (st != DCP_OK) return st;
  const int n_seg = xcd_segments(hkv), cut = cut_heads(use_mfma, dtype, d, hkv), heads = dkv_heads(plan, &t, use_mfma, n_seg, true);
  auto list = [&](int gid, int h) {
    const HostItems& hi = plan->host_items(gid, h, n_seg);
    DevGroup g{};
    g.n_items = (int32_t)hi.items.size();
    g.n_seg = hi.n_seg;
    for (int k = 0; k <= 8; k++) g.seg[k] = hi.seg[k];
    return g;
  };
  forms[0] = fwd_form(plan, &t, use_mfma, list(0, hq / hkv));
  const BwdChoice c = bwd_forms(plan, &t, use_mfma, list(1, hq / hkv), list(2, heads), cut, heads, true);
  forms[1] = c.dq; forms[2] = c.dkv; forms[3] = c.both;
  return DCP_OK;
}

extern "C" dcp_status_t dcp_plan_export_part_groups(dcp_plan_t* plan, int32_t hq, int32_t hkv, int32_t d, int32_t* groups) {
  if (!plan || !groups) return fail(DCP_ERR_INVALID_ARG, "plan or groups is NULL");
  dcp_tensors_t t{};
  t.hq = hq; t.hkv = hkv; t.d = d; t.dtype = DCP_F32; t.softmax_scale = 1.f;
  const dcp_status_t st = check_shape(&t);
  if (st != DCP_OK) return st;
  const F32Choice c = in_parts(&t) ? f32_choice(plan, &t) : F32Choice{};
  for (int gid = 0; gid < 3; gid++) groups[gid] = in_parts(&t) ? f32_groups(c.kernel[gid] == kPipe16 ? c.parts[gid] : c.kernel[gid]) : 0;
  return DCP_OK;
}

extern "C" size_t dcp_bwd_workspace_bytes(const dcp_plan_t* plan, int32_t hq, int32_t hkv, int32_t d, int32_t dtype) {
  if (!plan || hq <= 0) return 0;
  // the work lists are cached in the plan the first time a size or a launch asks for them
  return bwd_workspace(const_cast<dcp_plan_t*>(plan), hq, hkv, d, dtype).total();
}

// The backward behind both of its entry points.  may_alloc = false: the plan's device copies must exist already
// (dcp_plan_prepare) and no per-kernel timing events are created, so the call neither allocates nor synchronises.
dcp_status_t dcp::bwd_launch(dcp_plan_t* plan, const dcp_tensors_t* t, void* workspace, size_t workspace_bytes, hipStream_t s,
                             bool may_alloc) {
  if (!plan) return fail(DCP_ERR_INVALID_ARG, "plan is NULL");
  dcp_status_t st = check_shape(t);
  if (st != DCP_OK) return st;
  bool use_mfma = false;
  if ((st = pick_impl(t, &use_mfma)) != DCP_OK) return st;
  if (plan->total_tokens == 0) return DCP_OK;
  if ((st = check_tensor("q", t->q, t->q_stride_t, t->q_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("k", t->k, t->k_stride_t, t->k_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("v", t->v, t->v_stride_t, t->v_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("out", t->out, t->o_stride_t, t->o_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("dout", t->dout, t->do_stride_t, t->do_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("dq", t->dq, t->dq_stride_t, t->dq_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("dk", t->dk, t->dk_stride_t, t->dk_stride_h, t->d)) != DCP_OK) return st;
  if ((st = check_tensor("dv", t->dv, t->dv_stride_t, t->dv_stride_h, t->d)) != DCP_OK) return st;
  if (!t->lse) return fail(DCP_ERR_INVALID_ARG, "lse is NULL");
  if (plan->has_ranges && !t->attn_ranges) return fail(DCP_ERR_INVALID_ARG, "table has RANGES rows but attn_ranges is NULL");
  if (plan->has_window && plan->window <= 0) return fail(DCP_ERR_INVALID_ARG, "table has WINDOW rows but dcp_plan_set_window was not called");
  const BwdWorkspace wsz = bwd_workspace(plan, t->hq, t->hkv, t->d, t->dtype);
  const size_t need = wsz.total();
  if (!workspace || workspace_bytes < need) return fail(DCP_ERR_WORKSPACE, "workspace is NULL or smaller than dcp_bwd_workspace_bytes");
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(DCP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  DevGroup gq, gkv;
  const int n_seg = xcd_segments(t->hkv);
  if ((st = plan->group_for(1, s, &gq, t->hq / t->hkv, n_seg, may_alloc)) != DCP_OK) return st;
  // Whole or cut dK/dV items: what the choice of kernels wants.  Where that list cannot be created now and the plan holds the
  // other one, the other one: whole items serve every kernel, cut ones only the one that shares its tiles.
  const int cut = cut_heads(use_mfma, t->dtype, t->d, t->hkv);
  const bool one_launch = one_launch_is_safe(plan, t);
  int heads = dkv_heads(plan, t, use_mfma, n_seg, one_launch);
  if (cut && !plan->has_items(2, heads, n_seg) && plan->has_items(2, cut - heads, n_seg) && (!may_alloc || is_capturing(s))) heads = cut - heads;
  if ((st = plan->group_for(2, s, &gkv, heads, n_seg, may_alloc)) != DCP_OK) return st;
  const BwdChoice form = bwd_forms(plan, t, use_mfma, gq, gkv, cut, heads, one_launch);
  use_mfma = form.dq != kRows;
  KTensors k = pack(plan, t);
  const size_t n_hT = wsz.n_hT;
  k.part = (float*)((char*)workspace + 2 * wsz.n_hT + wsz.n_bounds);
  float* delta = (float*)workspace;
  float* lse2 = (float*)((char*)workspace + n_hT);
  k.delta = delta;
  k.lse2 = lse2;
  if (k.masked && use_mfma) {
    int32_t* qb = (int32_t*)((char*)workspace + 2 * n_hT);
    k.qbounds = qb;
    if ((st = mfma_range_bounds(gkv, k, plan->d_blk_t32, plan->n_blocks, plan->longest_block, qb, s)) != DCP_OK) return st;
  }
  if (form.both != kShared) {
    ProfScope ps(DCP_K_DKV, s, may_alloc);
    return t->dtype == DCP_F32 ? mfma_f32_bwd(gq, gkv, k, s) : mfma_split_bwd(gq, gkv, k, waves_of(form.both), s);
  }
  if (use_mfma) {
    // the MFMA dQ kernel computes delta and the rescaled LSE of its own rows and leaves them for the dK/dV kernel
    k.delta_w = delta;
    k.lse2_w = lse2;
  } else {
    ProfScope ps(DCP_K_DELTA, s, may_alloc);
    if ((st = stream_delta(t->out, t->o_stride_t, t->o_stride_h, t->dout, t->do_stride_t, t->do_stride_h, delta,
                           t->lse, lse2, plan->q_rows, t->hq, t->d, t->dtype, s)) != DCP_OK) return st;
  }
  {
    ProfScope ps(DCP_K_DQ, s, may_alloc);
    if (form.dq == kRows) st = scalar_bwd_dq(gq, k, t->dtype, s);
    else if (form.dq == kShared) {
      if (in_parts(t)) k.part_groups = f32_groups(f32_choice(plan, t).kernel[1]);
      st = mfma_bwd_dq(gq, k, s);
    }
    else st = t->dtype == DCP_F32 ? mfma_f32_dq(gq, k, 16, s) : mfma_split_dq(gq, k, waves_of(form.dq), s);
    if (st != DCP_OK) return st;
  }
  ProfScope ps(DCP_K_DKV, s, may_alloc);
  if (form.dkv == kRows) return scalar_bwd_dkv(gkv, k, t->dtype, s);
  if (form.dkv == kShared) {
    if (in_parts(t)) k.part_groups = f32_groups(f32_choice(plan, t).kernel[2]);
    return mfma_bwd_dkv(gkv, k, s);
  }
  return t->dtype == DCP_F32 ? mfma_f32_dkv(gkv, k, 16, s) : mfma_split_dkv(gkv, k, waves_of(form.dkv), s);
}

extern "C" dcp_status_t dcp_block_attn_bwd(dcp_plan_t* plan, const dcp_tensors_t* t, void* workspace,
                                           size_t workspace_bytes, void* stream) {
  return bwd_launch(plan, t, workspace, workspace_bytes, (hipStream_t)stream, true);
}

extern "C" dcp_status_t dcp_sum_partials(const void* const* parts, int32_t n_parts, int32_t parts_dtype, void* dst,
                                         int32_t dst_dtype, int64_t n_elems, void* stream) {
  if (n_parts < 1 || n_parts > 8 || !parts) return fail(DCP_ERR_INVALID_ARG, "n_parts must be 1..8 and parts non-NULL");
  if (n_elems < 0 || n_elems % 8) return fail(DCP_ERR_INVALID_ARG, "n_elems must be a non-negative multiple of 8");
  if ((parts_dtype != DCP_BF16 && parts_dtype != DCP_F32) || (dst_dtype != DCP_BF16 && dst_dtype != DCP_F32))
    return fail(DCP_ERR_UNSUPPORTED, "dtype must be DCP_BF16 or DCP_F32");
  if (n_elems == 0) return DCP_OK;
  if (!dst || !aligned16(dst)) return fail(DCP_ERR_INVALID_ARG, "dst is NULL or misaligned");
  for (int i = 0; i < n_parts; i++)
    if (!parts[i] || !aligned16(parts[i])) return fail(DCP_ERR_INVALID_ARG, "a partial pointer is NULL or misaligned");
  ProfScope ps(DCP_K_SUM, (hipStream_t)stream);
  return stream_sum(parts, n_parts, parts_dtype, dst, dst_dtype, n_elems, (hipStream_t)stream);
}

extern "C" dcp_status_t dcp_copy_list_create(dcp_copy_list_t** list, const int32_t* entries, int64_t n, int64_t src_rows,
                                             int64_t dst_rows) {
  if (!list) return fail(DCP_ERR_INVALID_ARG, "list is NULL");
  *list = nullptr;
  if (n < 0 || (n > 0 && !entries)) return fail(DCP_ERR_INVALID_ARG, "entries is NULL or n < 0");
  if (src_rows < 0 || dst_rows < 0 || src_rows > INT32_MAX || dst_rows > INT32_MAX)
    return fail(DCP_ERR_INVALID_ARG, "src_rows / dst_rows must lie in [0, 2^31)");
  std::unique_ptr<dcp_copy_list> cl(new dcp_copy_list);
  cl->src_rows = src_rows; cl->dst_rows = dst_rows;
  std::vector<std::pair<int64_t, int64_t>> dsts, srcs;   // [begin, end)
  for (int64_t i = 0; i < n; i++) {
    const int64_t sr = entries[3 * i], dr = entries[3 * i + 1], nr = entries[3 * i + 2];
    if (sr < 0 || dr < 0 || nr < 0) return fail(DCP_ERR_BAD_TABLE, "copy entry " + std::to_string(i) + " has a negative field");
    if (sr + nr > src_rows) return fail(DCP_ERR_BAD_TABLE, "copy entry " + std::to_string(i) + " reads past the source buffer");
    if (dr + nr > dst_rows) return fail(DCP_ERR_BAD_TABLE, "copy entry " + std::to_string(i) + " writes past the destination buffer");
    if (nr == 0) continue;
    dsts.push_back({dr, dr + nr});
    srcs.push_back({sr, sr + nr});
    for (int64_t r = 0; r < nr; r += kCopyChunkRows) {
      cl->chunks.push_back((int32_t)(sr + r));
      cl->chunks.push_back((int32_t)(dr + r));
      cl->chunks.push_back((int32_t)std::min<int64_t>(kCopyChunkRows, nr - r));
    }
  }
  std::sort(dsts.begin(), dsts.end());
  for (size_t i = 1; i < dsts.size(); i++)
    if (dsts[i].first < dsts[i - 1].second) return fail(DCP_ERR_BAD_TABLE, "two copy entries write overlapping destination rows");
  // would a destination range overlap a source range if both buffers were the same allocation?
  std::sort(srcs.begin(), srcs.end());
  size_t j = 0;
  for (size_t i = 0; i < dsts.size() && cl->alias_safe; i++) {
    while (j < srcs.size() && srcs[j].second <= dsts[i].first) j++;
    for (size_t k = j; k < srcs.size() && srcs[k].first < dsts[i].second; k++)
      if (srcs[k].second > dsts[i].first) { cl->alias_safe = false; break; }
  }
  *list = cl.release();
  return DCP_OK;
}

extern "C" dcp_status_t dcp_copy_list_destroy(dcp_copy_list_t* list) {
  if (!list) return DCP_OK;
  if (list->d_chunks) (void)hipFree(list->d_chunks);
  delete list;
  return DCP_OK;
}

extern "C" dcp_status_t dcp_blockwise_copy(dcp_copy_list_t* list, const void* src, int64_t src_stride, void* dst,
                                           int64_t dst_stride, int64_t row_bytes, void* stream) {
  if (!list) return fail(DCP_ERR_INVALID_ARG, "list is NULL");
  if (row_bytes <= 0 || row_bytes % 16 || row_bytes / 16 > (1 << 24)) return fail(DCP_ERR_INVALID_ARG, "row_bytes must be a positive multiple of 16 (at most 2^28)");
  if (src_stride < row_bytes || dst_stride < row_bytes || src_stride % 16 || dst_stride % 16)
    return fail(DCP_ERR_INVALID_ARG, "row strides must be multiples of 16 and at least row_bytes");
  if (list->chunks.empty()) return DCP_OK;
  if (!src || !dst || !aligned16(src) || !aligned16(dst)) return fail(DCP_ERR_INVALID_ARG, "src or dst is NULL or misaligned");
  {
    // extents the list can touch
    const char* s0 = (const char*)src; const char* s1 = s0 + (list->src_rows - 1) * src_stride + row_bytes;
    const char* d0 = (const char*)dst; const char* d1 = d0 + (list->dst_rows - 1) * dst_stride + row_bytes;
    const bool overlap = list->src_rows > 0 && list->dst_rows > 0 && s0 < d1 && d0 < s1;
    if (overlap && !(src == dst && src_stride == dst_stride && list->alias_safe))
      return fail(DCP_ERR_INVALID_ARG, "source and destination buffers overlap (allowed only as the same buffer with a list whose destination ranges avoid its source ranges)");
  }
  hipStream_t s = (hipStream_t)stream;
  {
    std::lock_guard<std::mutex> lock(list->mu);
    int dev = -1;
    DCP_HIP_TRY(hipGetDevice(&dev));
    if (list->d_chunks && list->device != dev) return fail(DCP_ERR_INVALID_ARG, "copy list was first used on another device");
    if (!list->d_chunks) {
      const size_t bytes = list->chunks.size() * sizeof(int32_t);
      DCP_HIP_TRY(hipMalloc((void**)&list->d_chunks, bytes));
      hipError_t e = hipMemcpyAsync(list->d_chunks, list->chunks.data(), bytes, hipMemcpyHostToDevice, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (e != hipSuccess) {
        (void)hipFree(list->d_chunks);
        list->d_chunks = nullptr;
        return fail(DCP_ERR_HIP, std::string("copy list upload: ") + hipGetErrorString(e));
      }
      list->device = dev;
    }
  }
  ProfScope ps(DCP_K_COPY, s);
  return stream_copy(list->d_chunks, (int64_t)(list->chunks.size() / 3), src, src_stride, dst, dst_stride, row_bytes, s);
}

extern "C" const char* dcp_version(void) { return "dcp_attn 0.1 (gfx950)"; }
