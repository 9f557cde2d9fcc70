// Internal declarations shared by the kernels and the C-ABI layer of the FiCoCo library.
// gfx950 only (64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/ficoco.h"

namespace ficoco {

constexpr int kWave = 64;
constexpr int kCandPad = 2048;     // floats of padding behind the approximate correlation block (one pass of its reader)
constexpr int kGramStage = 32;     // features per K stage of the matrix-core kernel (its K ranges are counted in stages)
constexpr int kVec = 8;            // elements per lane per load in the streaming kernels
constexpr int kSelMax = 8;         // order statistics kept in registers by the fast threshold path
constexpr int kReduceThreads = 256;
constexpr int kSelectThreads = 1024;
constexpr int kMaxSelectN = 12288; // visual tokens / grid cells the per-image select kernel holds in LDS

// Workspace layout: byte offsets from a 256-byte aligned base, 0 = absent.
struct Plan {
  int n_disc;            // N^S
  int n_out;             // n_tot - N^S
  // attention reduction
  int col_strips;        // column strips of the visual keys
  int strip_groups;      // 8-column groups per strip
  int row_lanes;         // rows processed concurrently by one workgroup
  int rows_per_wg;       // visual-block rows per workgroup
  int n_chunks;          // row chunks of the A block (partials of the received attention)
  int a_row0, a_rows;    // rows of A that carry a role (first, count)
  int a_shift;           // rows by which the first chunk is shortened so that visual row 0 starts a chunk
  int map_pitch;         // floats per row of the head-mean map (N rounded up to 64: read in whole 64-entry steps)
  // threshold selection
  int sel_m;             // order statistics needed: n_keep - floor(eps (n_keep-1))
  int sel_f;             // floor(p)
  double sel_g;          // fractional part of p
  bool dense_rows;       // sel_m > kSelMax: rows are materialised and selected bit by bit
  bool need_features;    // unit rows / norms
  size_t abar;           // float  [B][N][map_pitch]  head-mean visual x visual map, TRANSPOSED: [key token][query token]
  size_t recv_part;      // double [B][n_chunks][N]
  size_t cls;            // double [B][N]
  size_t ttext;          // double [B][N][M]      head-mean text->visual map, transposed
  size_t inv_norm;       // double [B][N]         1/|F_i| (0 for a zero row)
  size_t xhat;           // bf16   [B][N][Df]     unit rows rounded to bfloat16
  size_t colsum_part;    // double [2][B][f_chunks][Df] column sums of unit rows and of rows (unit_rows_summed: [B][f_chunks][Df], of unit rows)
  size_t colmean;        // double [2][B][Df] (mean unit row, mean raw row), then the parts of |mean raw row|^2
  size_t fterm;          // double [B][N]         feature-derived score term
  size_t fterm2;         // double [B][N]
  size_t slot_of;        // int32  [B][N]         keep slot of a preserved token, -1 if discarded
  size_t tgt_ptr;        // int32  [B][n_keep+1]
  size_t tgt_src;        // int32  [B][N^S*k_max] discarded token index per edge, by target
  size_t tgt_alpha;      // double [B][N^S*k_max]
  size_t hub_list, hub_cnt;   // int32 [B][n_keep], [B]: preserved tokens with long buckets (inverted lists only)
  int bkt_cap;           // fused step: edges kept per target while the lists are written (0: none)
  int cnt_stride;        // counters are this many int32 apart
  size_t bkt_cnt;        // int32  [B][n_keep][cnt_stride] edges per target
  size_t bkt_src;        // int32  [B][n_keep][bkt_cap]   their sources (bucket_entry), in order of arrival
  size_t bkt_w;          // double [B][n_keep][bkt_cap]   their weights
  size_t beyond;         // bytes of the regions that the limit of the static scratch does not count (qk_norm, bkt_*)
  size_t rowbuf;         // double [B][N^S][n_keep] (dense_rows only)
  size_t ct;             // float  [splits][B][N^S][n_keep]  approximate cosines (matrix-core path)
  size_t cmax;           // double [B][M]
  // exact re-evaluation of the cosine-derived score terms (select stage), present with those terms only
  size_t ex_nrm;         // double [B][N]
  size_t ex_mu;          // double [B][Df + 1]
  size_t ex_u;           // double [B][8][Df]
  size_t ex_g;           // double [B][8][N]
  size_t ex_list;        // int32  [B][N]
  int fixed_k;           // >= 0: targets per discarded token fixed by the caller (0: no edges), -1: adaptive
  bool extra_token;      // the additional token of the convergent form is written
  bool qk;               // the maps are formed from queries and keys on the fly (attn_qk.hip)
  int qk_nq, qk_visq;    // query rows that form needs, and how many of them are visual (all or none)
  int qk_images;         // images whose row normalisers the workspace holds at a time
  size_t qk_norm;        // float2 [qk_images][H][qk_nq] row normalisers
  bool use_gram;         // cosine correlation proposed by the MFMA tile kernel
  int gram_splits, gram_st_per_split;   // K ranges of that kernel and their length in 32-feature stages
  int f_chunks, f_rows_per_wg, Df;
  size_t total;
};

// scratch: bytes the whole workspace may have at most, as far as the lists of the targets can be cut down to it
int make_plan(const ficoco_problem& p, Plan& plan, const char** why, size_t scratch = SIZE_MAX);

// ---- launchers (all asynchronous on `s`) -----------------------------------------------
// text_elsewhere: the text-profile kernel is not launched here (text_with_features: it rides in the
// feature stage's launch)
void launch_attn_reduce(const ficoco_problem& p, const Plan& pl, char* ws, hipStream_t s, bool text_elsewhere = false);
void launch_attn_qk(const ficoco_problem& p, const Plan& pl, char* ws, hipStream_t s);
constexpr int kQkTile = 64;        // query rows of a column partial of the query/key form
// The row normalisers are kept for as many images at a time as fit in this many bytes (at least one).
constexpr size_t kQkNormBytes = (size_t)8 << 20;
// With more keys than kQkMaxKeys, and for FiCoCo-L, at most kQkLongMaxHeads heads are taken: one image of FiCoCo-V then
// stays within those bytes whatever its length is, as the static scratch requires (640 keys would need 1600 heads
// for as much), and FiCoCo-L, which has no static form, has the same limit.
constexpr int kQkMaxKeys = 640, kQkLongMaxHeads = 64;
static_assert((size_t)kQkLongMaxHeads * (kMaxSelectN + 1) * sizeof(float2) <= kQkNormBytes, "one image");
// with_text: the launch of the row-norm kernel also forms the text profiles and the launch of the
// column-sum kernel their statistics (with_cmax: the column maxima too), see text_with_features
void launch_features(const ficoco_problem& p, const Plan& pl, char* ws, hipStream_t s, bool with_text = false,
                     bool with_cmax = false);
// The feature stage is norms and unit rows only (no score term reads the features; the cosine
// correlation does): the score stage's launch of the filter kernel takes them along on workgroups
// of its own, and launch_features does nothing.
inline bool rows_with_filter(const ficoco_problem& p, const Plan& pl) {
  return pl.need_features && p.red_src != FICOCO_R_SIM_MEAN && p.sem_src != FICOCO_G_EQ_TOKEN;
}
// FiCoCo-L with 32 or more text queries: the fused step forms the column maxima of the text
// profiles in the score stage's launch (select.hip), and its correlate stage does not.
inline bool text_stats_in_score(const ficoco_problem& p) {
  return p.variant == FICOCO_VARIANT_L && p.sem_src == FICOCO_G_TEXT_ATTN && p.M >= 32;
}
// FiCoCo-L whose score reads both the features (column sums: four dependent launches) and the text
// profiles (two dependent launches): the two chains do not depend on each other, so where score
// and reduction are issued by the same call the text kernels ride in the launches of the feature
// kernels instead of standing in line before and after them.
inline bool text_with_features(const ficoco_problem& p, const Plan& pl) {
  return text_stats_in_score(p) && p.A_text != nullptr && pl.need_features && !rows_with_filter(p, pl);
}
// FiCoCo-L whose redundancy term is the mean cosine, in bfloat16: norms, unit rows and their column sums in one pass over the
// tokens (features.hip), where a row fills four to sixteen wavefronts with 16 bytes a lane: 2048 to 8192 features (narrower
// rows leave a workgroup too few wavefronts; FiCoCo-V keeps its workspace, which the static scratch bounds).
// Not where its workgroups fill the chip badly and the separate passes are faster.  Step in us, one pass / separate: nine or ten wavefronts, of which one
// workgroup has a compute unit of sixteen to itself, above 8192 rows (5120 features, 64 text tokens: 8 x 690 145.8 / 151.8, 12 x 690 184.5 / 183.9, 8 x 1152
// 221.2 / 214.6, with 200 252.3 / 241.1; 4096 features 170.8 / 179.7); thirteen and more with over four workgroups of text profiles a compute unit in
// the launch (8192 features, 200 text tokens: 32 x 200 253.3 / 263.6, 24 x 576 455.7 / 486.7, 64 x 64 263.6 / 251.2, 128 x 33 414.4 / 393.4); and where no
// unit rows are wanted (correlation by attention), above 4096 features and one workgroup a compute unit (7 x 585 tokens, 8192 features, 259 workgroups 142.8 /
// 130.3, 12 x 364, 6144, 276 124.7 / 119.0; 16 x 195, 6144, 208 86.6 / 93.7): relative to the separate passes 0.95 to 0.99
// at 200 to 256 workgroups, 1.03 to 1.08 at 257 to 300, beyond 1.00 (5120, 6144 features) and 1.04 (7168, 8192); 4096 features 0.97, 1.00 and 0.98.
inline bool unit_rows_summed(const ficoco_problem& p, int Df) {
  if (p.variant != FICOCO_VARIANT_L || p.dtype != FICOCO_BF16 || p.red_src != FICOCO_R_SIM_MEAN || Df % kVec != 0 || Df < 2048 || Df > 8192) return false;
  if (Df > 4096 && Df <= 5120 && (int64_t)p.B * p.N > 8192) return false;
  if (p.corr_src != FICOCO_C_COSINE && Df > 4096 && (int64_t)p.B * ((p.N + 15) / 16) > 256) return false;
  return !(Df > 6144 && p.A_text != nullptr && (int64_t)p.B * ((p.M + 7) / 8) > 1024);
}
// Rows of a workgroup there: 16, or 8 where those would be fewer than half as many workgroups as there are compute units.  us per step with
// 16, with 8 and in the separate passes before: one sequence of 576 tokens, 5120 features 73.2 / 66.0 / 71.6, four of 200 82.2 / 74.2 /
// 79.1; four of 576 91.9 / 97.3 / 97.8, eight of 690 172 / 183 / 187.
inline int unit_rows_per_wg(const ficoco_problem& p) { return (int64_t)p.B * ((p.N + 15) / 16) >= 128 ? 16 : 8; }
// The column partials of the reduction are added by a launch of their own (combine_partials_kernel) instead of by the one workgroup of
// an image's filter: from 48 partials a thread of that workgroup (chunks x columns a thread) on.  us behind the reduction, added by the filter and
// so: 33 partials of 1024 columns 25.0 / 23.9 and, four images, 27.7 / 26.7; 66 of 1025 columns 28.1 / 27.4, 82 (1296) 31.4 / 28.4, 108 (1728)
// 36.5 / 30.2, 126 (2000) 41.5 / 30.6; without a map 58 (576) 30.8 / 29.9; from queries and keys 46 (1440) 27.9 / 27.9, 54 (1728) 31.6 / 28.8, 108 (2304) 47.6 / 40.5.
inline bool partials_combined(const ficoco_problem& p, const Plan& pl) {
  return p.red_src == FICOCO_R_ATTN_RECV && (int64_t)pl.n_chunks * ((p.N + kSelectThreads - 1) / kSelectThreads) > 48;
}
// text_stats_done: the text statistics were formed by the feature stage's launches
void launch_score(const ficoco_problem& p, const Plan& pl, char* ws, double* scores, hipStream_t s,
                  bool text_stats_done = false);
void launch_filter(const ficoco_problem& p, const Plan& pl, char* ws, const double* scores,
                   int32_t* discard_idx, int32_t* keep_idx, hipStream_t s);
// pos_out: the filter also writes the position ids of the preserved tokens (a fused step: the
// compress stage is then called without them), or null
void launch_select(const ficoco_problem& p, const Plan& pl, char* ws, double* scores, bool do_score,
                   bool do_filter, int32_t* discard_idx, int32_t* keep_idx, int32_t* overflow,
                   hipStream_t s, bool text_stats_done = false, int32_t* pos_out = nullptr);
void launch_correlate(const ficoco_problem& p, const Plan& pl, char* ws, const int32_t* discard_idx,
                      const int32_t* keep_idx, int32_t* edge_cnt, int32_t* edge_tgt,
                      double* edge_alpha, int32_t* overflow, bool fused,
                      hipEvent_t gram_start, hipEvent_t gram_stop, hipStream_t s, int gram_repeat = 1);
// The tiles that the block of approximate cosines is cut into (Plan::use_gram): 128 x 128, 192 x 192 or 256 x 192.
enum GramForm { kGramSquare, kGramWide, kGramTall };
GramForm gram_form(const ficoco_problem& p, const Plan& pl);
// Bound of their error.  Every step of an accumulation adds at most 2^-22 of the sum of its terms' magnitudes; the
// magnitudes of all K ranges together add up to at most |x||y|, so the length that counts is that of one range.
inline float gram_delta(const Plan& pl) {
  const int len = pl.gram_st_per_split * kGramStage;
  return (float)((len < pl.Df ? len : pl.Df) + 4 * pl.gram_splits) * 2.384185791015625e-07f;
}
void launch_gather(const ficoco_problem& p, const Plan& pl, const int32_t* keep_idx, const void* in,
                   int64_t sb, int64_t sn, int row_bytes, void* out, hipStream_t s);
void launch_corr_gap(const ficoco_problem& p, const Plan& pl, char* ws, const int32_t* discard_idx,
                     const int32_t* keep_idx, double* gap, hipStream_t s);
// targets_listed: the call follows the correlate stage of the same fused step, which filled the
// targets' lists; otherwise the compress stage works from the edge lists it is given alone
void launch_compress(const ficoco_problem& p, const Plan& pl, char* ws, const int32_t* discard_idx,
                     const int32_t* keep_idx, const int32_t* edge_cnt, const int32_t* edge_tgt,
                     const double* edge_alpha, void* X_out, int32_t* pos_out,
                     hipStream_t s, bool targets_listed = false);
// In a fused step the correlate stage drops every edge into the list of its target (bkt_*: a counter that
// the filter stage clears, and up to bkt_cap (source, weight) pairs in order of arrival), and the
// merge takes a row's sources from there.  Targets with more sources than a list holds work from the
// edge lists; above kMatchMaxRows those with more than kHubMin sources are listed as they appear (hub_list).
// A staged compress call has the edge lists alone: up to kMatchMaxRows discarded tokens
// every workgroup of the merge scans the image's lists in LDS, above that they are first bucketed by
// target (compress.hip), the discarded rows cut into invert_groups() shares of invert_share_rows()
// consecutive rows, one workgroup of the bucketing kernel per share.
constexpr int kMatchMaxRows = 1024;
constexpr int kInvertRows = 512;
constexpr int kHubMin = 32;        // targets with more sources than this are merged by a whole workgroup
// Entries per target up to kMatchMaxRows discarded tokens and above: as many as a wavefront, and a workgroup, puts in
// order.  (16 for the former: 37 us instead of 19 where two dozen of 144 targets have 17 to 29 sources.)
constexpr int kBucketCap = 32, kBucketCapLong = 256;
constexpr size_t kBucketBytes = (size_t)8 << 20;         // at most, for one image: more targets keep fewer
static_assert(kMaxSelectN <= (1 << 16), "row and token of an entry");
__host__ __device__ __forceinline__ int bucket_entry(int row, int token) { return row << 16 | token; }   // ascending like the rows
inline bool edges_inverted(const Plan& pl) { return pl.n_disc > kMatchMaxRows; }
inline int invert_groups(const Plan& pl) { return (pl.n_disc + kInvertRows - 1) / kInvertRows; }
inline int invert_share_rows(const Plan& pl) {
  const int g = invert_groups(pl);
  return g > 0 ? (pl.n_disc + g - 1) / g : 1;
}

// ---- device helpers ----------------------------------------------------------------------
typedef uint16_t bf16_t;

template <typename T> struct __attribute__((packed, aligned(2))) Pack8 { T v[kVec]; };

__device__ __forceinline__ double widen(bf16_t x) {
  return (double)__uint_as_float(((uint32_t)x) << 16);
}
__device__ __forceinline__ double widen(float x) { return (double)x; }

// Raw bits of 8 consecutive elements, loaded from an address that is only element aligned
// (kept unconverted so that many loads can be in flight before the first use).
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> { uint4 a; };
template <> struct Raw8<float> { float4 a, b; };

__device__ __forceinline__ void load_raw(const bf16_t* __restrict__ p, Raw8<bf16_t>& r) {
  __builtin_memcpy(&r.a, p, 16);
}
__device__ __forceinline__ void load_raw(const float* __restrict__ p, Raw8<float>& r) {
  __builtin_memcpy(&r.a, p, 16);
  __builtin_memcpy(&r.b, p + 4, 16);
}
__device__ __forceinline__ void add_raw(const Raw8<bf16_t>& r, double (&acc)[kVec]) {
  const uint32_t w[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc[2 * j] += (double)__uint_as_float(w[j] << 16);
    acc[2 * j + 1] += (double)__uint_as_float(w[j] & 0xffff0000u);
  }
}
__device__ __forceinline__ void add_raw(const Raw8<float>& r, double (&acc)[kVec]) {
  acc[0] += r.a.x; acc[1] += r.a.y; acc[2] += r.a.z; acc[3] += r.a.w;
  acc[4] += r.b.x; acc[5] += r.b.y; acc[6] += r.b.z; acc[7] += r.b.w;
}

// acc += w * (the 8 elements held raw): product and sum are rounded separately, as the plain
// statement of Eq. 2 does, so that the sums are the same doubles (a fused multiply-add differs in
// the last bit, which shows where a sum cancels)
__device__ __forceinline__ void fma_raw(const Raw8<bf16_t>& r, double w, double (&acc)[kVec]) {
#pragma clang fp contract(off)
  const uint32_t q[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc[2 * j] += w * (double)__uint_as_float(q[j] << 16);
    acc[2 * j + 1] += w * (double)__uint_as_float(q[j] & 0xffff0000u);
  }
}
__device__ __forceinline__ void fma_raw(const Raw8<float>& r, double w, double (&acc)[kVec]) {
#pragma clang fp contract(off)
  acc[0] += w * r.a.x; acc[1] += w * r.a.y; acc[2] += w * r.a.z; acc[3] += w * r.a.w;
  acc[4] += w * r.b.x; acc[5] += w * r.b.y; acc[6] += w * r.b.z; acc[7] += w * r.b.w;
}

// Between the loads of a batch and their first use: the instruction scheduler moves nothing
// across this point.  Left to itself it may pull a load down to its use to save registers,
// which turns a batch of loads in flight back into one memory round trip after the other.
__device__ __forceinline__ void issue_fence() { __builtin_amdgcn_sched_barrier(0); }

// ---- reductions over the 64 lanes of a wavefront ----------------------------------------------------
// Every lane must be active and every lane gets the result.  The first four steps pair lanes inside
// a row of 16 with data-parallel-primitive moves (lane ^ 1, lane ^ 2, then the mirror images inside
// 8 and inside 16 lanes, which reach the other half because the halves are uniform by then), the
// four row results are read out by lane and combined as (r0 op r1) op (r2 op r3): a fixed tree,
// and no trip through the LDS permute path (a butterfly of six of those costs several hundred
// cycles in kernels that are chains of dependent steps).  `op` must be commutative.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false); }
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) { return __int_as_float(dpp_move<CTRL>(__float_as_int(x))); }
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  return __hiloint2double(dpp_move<CTRL>(__double2hiint(x)), dpp_move<CTRL>(__double2loint(x)));
}
__device__ __forceinline__ int lane_value(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ float lane_value(float x, int l) { return __int_as_float(lane_value(__float_as_int(x), l)); }
__device__ __forceinline__ double lane_value(double x, int l) {
  return __hiloint2double(lane_value(__double2hiint(x), l), lane_value(__double2loint(x), l));
}
template <typename T, typename F>
__device__ __forceinline__ T wave_reduce(T v, F op) {
  v = op(v, dpp_move<0xB1>(v));      // quad_perm [1,0,3,2]: lane ^ 1
  v = op(v, dpp_move<0x4E>(v));      // quad_perm [2,3,0,1]: lane ^ 2
  v = op(v, dpp_move<0x141>(v));     // mirror inside 8 lanes
  v = op(v, dpp_move<0x140>(v));     // mirror inside 16 lanes
  return op(op(lane_value(v, 0), lane_value(v, 16)), op(lane_value(v, 32), lane_value(v, 48)));
}
// Inclusive prefix sum over the lanes of a wavefront (every lane active): four shifted adds inside
// each row of 16 (a lane whose source would lie before its row adds zero), then the totals of
// the rows before a lane's own, read out of lanes 15, 31 and 47.
template <int CTRL>
__device__ __forceinline__ int dpp_move_or_zero(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
__device__ __forceinline__ int wave_scan_inclusive(int v) {
  v += dpp_move_or_zero<0x111>(v);   // row_shr:1
  v += dpp_move_or_zero<0x112>(v);   // row_shr:2
  v += dpp_move_or_zero<0x114>(v);   // row_shr:4
  v += dpp_move_or_zero<0x118>(v);   // row_shr:8
  const int r0 = lane_value(v, 15), r1 = lane_value(v, 31), r2 = lane_value(v, 47);
  const int row = (int)(threadIdx.x % kWave) / 16;
  return v + (row >= 1 ? r0 : 0) + (row >= 2 ? r1 : 0) + (row >= 3 ? r2 : 0);
}

// The value of lane ^ 4: rows shifted by four lanes up for the first quad of a pair, down for the second.
__device__ __forceinline__ int lane_xor_4(int v) {
  const int up = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false);      // row_shl:4 into quads 0 and 2
  return __builtin_amdgcn_update_dpp(up, v, 0x114, 0xF, 0xA, false);             // row_shr:4 into quads 1 and 3
}
__device__ __forceinline__ double lane_xor_4(double v) {
  return __hiloint2double(lane_xor_4(__double2hiint(v)), lane_xor_4(__double2loint(v)));
}
// all bits cleared (eight zeros) unless `keep`: selects, no branch
__device__ __forceinline__ void keep_raw_if(Raw8<bf16_t>& r, bool keep) {
  r.a.x = keep ? r.a.x : 0u; r.a.y = keep ? r.a.y : 0u; r.a.z = keep ? r.a.z : 0u; r.a.w = keep ? r.a.w : 0u;
}
__device__ __forceinline__ void keep_raw_if(Raw8<float>& r, bool keep) {
  r.a.x = keep ? r.a.x : 0.0f; r.a.y = keep ? r.a.y : 0.0f; r.a.z = keep ? r.a.z : 0.0f; r.a.w = keep ? r.a.w : 0.0f;
  r.b.x = keep ? r.b.x : 0.0f; r.b.y = keep ? r.b.y : 0.0f; r.b.z = keep ? r.b.z : 0.0f; r.b.w = keep ? r.b.w : 0.0f;
}

// the 8 elements held raw, as doubles
__device__ __forceinline__ void widen_raw(const Raw8<bf16_t>& r, double (&out)[kVec]) {
  const uint32_t q[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    out[2 * j] = (double)__uint_as_float(q[j] << 16);
    out[2 * j + 1] = (double)__uint_as_float(q[j] & 0xffff0000u);
  }
}
__device__ __forceinline__ void widen_raw(const Raw8<float>& r, double (&out)[kVec]) {
  out[0] = r.a.x; out[1] = r.a.y; out[2] = r.a.z; out[3] = r.a.w;
  out[4] = r.b.x; out[5] = r.b.y; out[6] = r.b.z; out[7] = r.b.w;
}

// 8 consecutive elements from an address that is only element aligned.
template <typename T>
__device__ __forceinline__ void load8(const T* __restrict__ p, double (&out)[kVec]);

template <>
__device__ __forceinline__ void load8<bf16_t>(const bf16_t* __restrict__ p, double (&out)[kVec]) {
  uint4 r;
  __builtin_memcpy(&r, p, 16);
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    out[2 * j] = (double)__uint_as_float(w[j] << 16);
    out[2 * j + 1] = (double)__uint_as_float(w[j] & 0xffff0000u);
  }
}
template <>
__device__ __forceinline__ void load8<float>(const float* __restrict__ p, double (&out)[kVec]) {
  float4 a, b;
  __builtin_memcpy(&a, p, 16);
  __builtin_memcpy(&b, p + 4, 16);
  out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
  out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
}

// Workgroups are handed to the 8 XCDs round-robin by their linear id, and every XCD has its
// own L2.  This maps the linear id to a logical id such that consecutive logical ids (the
// tiles of one image) run on the same XCD and share its L2.  Logical ids >= total are idle.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_logical_id(int linear, int total) {
  const int per = (total + kXcds - 1) / kXcds;
  return (linear % kXcds) * per + linear / kXcds;
}
__host__ __device__ __forceinline__ int xcd_padded_total(int total) {
  return ((total + kXcds - 1) / kXcds) * kXcds;
}

// Inclusive scan of one int per thread over the workgroup (wavefront shuffles, then the
// wavefront totals through LDS); returns this thread's inclusive value, *total receives the
// sum.  scratch: at least blockDim.x / 64 ints.
__device__ __forceinline__ int block_scan_inclusive(int v, int* scratch, int* total) {
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave, nw = blockDim.x / kWave;
  const int incl = wave_scan_inclusive(v);
  __syncthreads();
  if (lane == kWave - 1) scratch[wv] = incl;
  __syncthreads();
  int before = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const int t = scratch[w];
    before += w < wv ? t : 0;
    tot += t;
  }
  *total = tot;
  __syncthreads();
  return incl + before;
}

// The nearest float of a double lies on the same side of every midpoint between two bfloat16 as the
// double itself, unless it IS such a midpoint (its low half reads 0x8000; denormals are kept, so the
// same holds there).
__device__ __forceinline__ bool bf16_midpoint(float f) { return (__float_as_uint(f) & 0xffffu) == 0x8000u; }
// `off`: any double with the sign of value - midpoint, zero for a tie: one step off the midpoint on that side
__device__ __forceinline__ float off_midpoint(float f, double off) {
  const uint32_t u = __float_as_uint(f);
  return off == 0.0 ? f : __uint_as_float((off > 0.0) == ((u >> 31) == 0u) ? u + 1u : u - 1u);
}
__device__ __forceinline__ uint32_t bf16_bits(float f) {  // nearest bfloat16 of a float, ties to even, in the high half
  const uint32_t u = __float_as_uint(f);
  return u + 0x7fffu + ((u >> 16) & 1u);
}

// Round a double to the nearest bfloat16, ties to even, straight from double (no
// intermediate float rounding).  The spacing at binary exponent e is 2^(max(e,-126)-7).
__device__ __forceinline__ bf16_t to_bf16(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  int e = (int)((u >> 52) & 0x7ff) - 1023;
  e = e < -126 ? -126 : e;
  const double r = ldexp(rint(ldexp(x, 7 - e)), e - 7);
  return (bf16_t)(__float_as_uint((float)r) >> 16);
}
__device__ __forceinline__ void store_token(bf16_t* p, double x) { *p = to_bf16(x); }
__device__ __forceinline__ void store_token(float* p, double x) { *p = (float)x; }

}  // namespace ficoco
