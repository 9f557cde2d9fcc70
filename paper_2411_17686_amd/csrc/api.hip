// C-ABI layer: argument checks, workspace plan and the stage / fused-step entry points
// declared in include/ficoco.h.  Host code only; every launch goes to the caller's stream.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>

#include "common.hpp"

// Scratch of the allocation-free entry point (ficoco_v_step_static): the workspace of a step
// lives in this file-scope device array instead of caller memory.  Every GPU the library runs
// on holds its own copy for the life of the process.  Host code never passes the array's name to
// a kernel (on the host it is a stand-in symbol, not a device address): ficoco_create asks the
// runtime for the array's address on the ctx's device and keeps it in g_static_ws.
// Behind FICOCO_STATIC_SCRATCH_BYTES there is room for the row normalisers of the query/key form and for
// the targets' lists, which that limit does not count (the lists are cut down to what is left).
constexpr size_t kStaticScratchBytes = FICOCO_STATIC_SCRATCH_BYTES + ficoco::kQkNormBytes + ficoco::kBucketBytes;
static_assert(kStaticScratchBytes == (size_t)48 << 20, "the size that ficoco.h states");
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static void* g_static_ws[kMaxDevices];    // per device, filled by ficoco_create (written once per device with the same value)

struct ficoco_ctx {
  int device;
  hipEvent_t probe_start, probe_stop;   // measurement hook, both null when off
  int probe_kernel;
  char err[512];
};

namespace ficoco {

// Row lanes, 8-column groups (at most) and rows of a reduction workgroup with the head-mean map to store, whose chunks are
// multiples of 8 rows (whole 32-byte sectors of the transposed map).
//
// The usual shape is 8 lanes x 24 groups (32 beyond 1024 columns) with rows for about 512 workgroups: its loads lie close together in
// memory, and few, long workgroups leave room for those of other streams.  Others take its place where they are faster, by the 16-byte loads that a
// row and a column group take (`loads`: heads, twice as many in float32).  Step in us, usual / taken:
//   16 x 16 lanes, 16 rows: short sequences, up to 512 workgroups (8 x 256 tokens, 16 heads 26.9 / 25.4); with more than sixteen loads where the usual
//     shape has 16 rows too (49 x 86, 40 heads of bfloat16 35.2 / 29.1, 12 x 219, 32 of float32, the worst of 84, 36.7 / 37.6), with 8 below 256 of them
//     (8 x 232, 40 heads of bfloat16 28.6 / 27.3; from there on 20 x 180, 24 heads 28.4 / 30.8).
//   32 x 8, 32 rows, a row a thread: up to sixteen loads in flight, and few partials for the one workgroup of the filter.  1 x 576 tokens, 8 heads
//     25.9 / 24.1, 3 x 576 28.7 / 27.1.  As far as 1300 workgroups (five a compute unit: 8 x 576, 12 heads 39.7 / 39.6; with sixteen loads 1187; few heads
//     700, from where two rows a thread are better).  Beyond sixteen loads a thread makes several trips with one row in hand: up to three workgroups a compute
//     unit, the [CLS] rows' among them (3 x 658, 20 heads of bfloat16, 726 of them 39.9 / 34.5, 9 x 378, 12 of float32, 702 35.6 / 34.4, 6 x 443, 40 of
//     bfloat16, 630 57.7 / 48.3, 3 x 660, 16 of float32, 726 44.2 / 39.0; worst 1 x 1004, 40 of bfloat16, 528 43.2 / 46.2), or 1100 of them where the usual shape
//     has 24 rows, three a thread (2 x 1017, 40 of bfloat16, 1056 80.4 / 67.1, 2 x 918, 16 of float32, 900 55.1 / 53.7; worst 15 x 315, 16 of float32, 825
//     48.3 / 50.4); with more than forty loads one, where the second is half a launch (2 x 488, 40 heads of float32, 272 of them: 40.0 / 43.6, 2 x 472 with 256 38.9 / 34.7), or two where
//     the usual shape has 16 rows or more, which is short of loads in flight (3 x 510, 40 of float32, 408 of them 59.1 / 51.3, 6 x 359, 64 of bfloat16, 468
//     60.1 / 49.5); for short sequences none (46 x 144, 40 heads of float32 56.4 / 63.1, 16 x 144 of a decoder in bfloat16 35.8 / 38.5).
//     In float32 such a row is a chain of batches of eight heads, two loads each, and the chip is better filled with shorter chunks where its workgroups are
//     few: from 50 on up to forty loads (304 tokens, 16 heads, one image with 50 22.8 / 23.5), from 100 on beyond (1 x 320, 40 heads 24.8 / 26.2, 1 x 448
//     with 98 28.3 / 27.3, 2 x 288 with 90 25.1 / 26.3, 2 x 376 with 144 28.6 / 28.4).
//   16 x 16, 32 rows, two a thread: few heads up to 2500 workgroups (8 x 576, 4 heads 31.1 / 30.2; beyond, several steps in flight lose by it: 48 x 576, one
//     head 54.6 / 59.2) and again from 9000 on (47 x 1145, one head 231 / 210, in flight 217 / 202), others from 6000 on (4 x 2880, 16 heads 314 / 311), and
//     beyond 1024 columns, where the usual shape has 32 rows, up to forty loads (3 x 1129, 40 heads of bfloat16 124 / 106, 4 x 1714, 20 150 / 147, worst
//     7 x 1092, 32 155 / 163; over 1600 such problems 1.016).
// Of 24500 problems (40 to 2900 tokens, 1 to 64 images, 1 to 64 heads) the step is 1.015 times as fast as with the usual shape alone, 117 are more than 3 %
// slower (26 more than 5 %), three steps in flight 1.006 times.  (With 8 x 24 lanes and 32 rows for all calls beyond 700 workgroups some were by up to
// 16 %: 11 x 348, 32 heads, launch 22.1 usual, 30.9.)
//
// What the static scratch may hold is a fixed size, so no shape has fewer rows (more partials) than the usual one, whose
// partials it has always had room for: the 16 rows end where that takes 24.
static int rows_for_512(int64_t strip_rows) { return (int)std::min<int64_t>(((strip_rows + 511) / 512 + 7) / 8 * 8, 32); }
struct MapShape { int lanes, groups, rows; };
static MapShape map_shape(const ficoco_problem& p, int rows) {
  const int groups = (p.N + kVec - 1) / kVec, wide = groups > 128 ? 32 : 24;
  auto wgs = [&](int g, int r) { return (int64_t)p.B * ((groups + g - 1) / g) * ((p.N + r - 1) / r); };
  const MapShape usual{8, wide, rows_for_512((int64_t)p.B * ((groups + wide - 1) / wide) * rows)};
  const int loads = p.dtype == FICOCO_BF16 ? p.H : 2 * p.H;
  const bool is_short = p.N <= 256;
  if (is_short && wgs(24, 8) <= 256) return usual;         // every workgroup has a compute unit of its own
  if (is_short && usual.rows <= 16 && wgs(16, 16) <= (loads <= 16 || usual.rows == 16 ? 512 : 255)) return {16, 16, 16};
  const int64_t most = wgs(8, 32), all = most + (int64_t)p.B * ((groups + 7) / 8) * ((std::max(rows - p.N, 0) + 31) / 32);    // (the [CLS] row has a chunk of its own)
  const int beyond = p.dtype == FICOCO_BF16 || loads <= 24 ? 0 : loads <= 40 ? 50 : 100;
  const bool fills = loads < 8    ? most <= 700
                     : loads <= 16 ? most <= std::min(1300, 19000 / loads)
                     : is_short    ? false
                     : loads <= 40 ? all <= (usual.rows == 24 ? 1100 : 768)
                                   : all <= (usual.rows >= 16 ? 512 : 256);
  if (most > beyond && fills) return {32, 8, 32};
  const bool two_rows = loads < 8 ? most <= 2500 || most > 9000 : most > 6000 || (groups > 128 && usual.rows == 32 && loads <= 40);
  return two_rows ? MapShape{16, 16, 32} : usual;
}
// Workgroups the reduction aims at where it has no such map to store.
constexpr int64_t kWgTarget = 1024;

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int make_plan(const ficoco_problem& p, Plan& pl, const char** why, size_t scratch) {
  static const char* kNone = "";
  *why = kNone;
  std::memset(&pl, 0, sizeof(pl));
#define REQUIRE(c, msg) do { if (!(c)) { *why = msg; return FICOCO_EINVAL; } } while (0)
  REQUIRE(p.variant == FICOCO_VARIANT_V || p.variant == FICOCO_VARIANT_L, "variant must be V or L");
  REQUIRE(p.dtype == FICOCO_F32 || p.dtype == FICOCO_BF16, "dtype must be F32 or BF16");
  REQUIRE(p.B >= 1 && p.D >= 1 && p.n_tot >= 1, "B, D, n_tot must be positive");
  REQUIRE(p.N >= 1 && p.vis_begin >= 0 && p.vis_begin + (int64_t)p.N <= p.n_tot,
          "visual span [vis_begin, vis_begin+N) must lie inside the sequence");
  REQUIRE(p.n_keep >= 0 && p.n_keep <= p.N, "n_keep must be in [0, N]");
  REQUIRE(p.n_keep >= 1 || p.N == 0, "n_keep must be >= 1 (nothing to recycle into)");
  REQUIRE(p.N <= kMaxSelectN, "N exceeds the per-image limit of the filter kernel (12288)");
  REQUIRE(p.X != nullptr, "X is NULL");
  REQUIRE(p.x_stride_n >= p.D && p.x_stride_b >= 0, "bad X strides");
  REQUIRE(p.eps >= 0.0f && p.eps <= 1.0f, "eps must be in [0, 1]");
  REQUIRE(p.k_max >= 1, "k_max must be >= 1");
  REQUIRE(p.k_max <= kMaxSelectN, "k_max exceeds 12288 (N^S * k_max is indexed with 32-bit integers)");
  REQUIRE(p.k_mode >= FICOCO_K_ADAPTIVE && p.k_mode <= FICOCO_K_CONVERGENT, "unknown k_mode");
  REQUIRE(p.compress_mode == FICOCO_COMPRESS_SELF || p.compress_mode == FICOCO_COMPRESS_AVERAGE,
          "unknown compress_mode");
  if (p.k_mode == FICOCO_K_FIXED)
    REQUIRE(p.fixed_k >= 0 && p.fixed_k <= p.k_max, "fixed_k must be in [0, k_max]");
  REQUIRE(p.red_src >= 0 && p.red_src <= 2 && p.sem_src >= 0 && p.sem_src <= 3 &&
              p.corr_src >= 0 && p.corr_src <= 1, "unknown source selector");
  const bool L = p.variant == FICOCO_VARIANT_L;
  const bool need_A = p.red_src == FICOCO_R_ATTN_RECV || p.sem_src == FICOCO_G_CLS_ATTN ||
                      p.corr_src == FICOCO_C_ATTN;
  // queries and keys in place of the maps: FiCoCo-V with an attention-derived term and no A;
  // FiCoCo-L with neither A nor A_text (the decoder's causal maps; the M text tokens follow the visual span)
  const bool qk = p.A == nullptr && p.Q != nullptr && p.K != nullptr && (L ? p.A_text == nullptr : need_A);
  if (qk) {
    REQUIRE(p.H >= 1 && p.qk_n >= 1 && p.qk_stride_n >= p.d_head && p.qk_stride_h >= 0 && p.qk_stride_b >= 0,
            "bad Q / K shape or strides");
    REQUIRE(p.qk_begin >= 0 && p.qk_begin <= p.vis_begin && p.vis_begin + p.N <= p.qk_begin + p.qk_n,
            "Q / K do not cover the visual tokens");
    if (L)
      REQUIRE(p.M >= 1 && p.vis_begin + p.N + (int64_t)p.M <= p.qk_begin + (int64_t)p.qk_n,
              "Q / K do not cover the M text tokens behind the visual span");
    if (p.sem_src == FICOCO_G_CLS_ATTN)
      REQUIRE(p.cls_index >= p.qk_begin && p.cls_index < p.qk_begin + p.qk_n &&
                  (p.cls_index < p.vis_begin || p.cls_index >= p.vis_begin + p.N),
              "cls_index must be a row of Q / K outside the visual span");
    REQUIRE(p.qk_scale > 0.0f && p.qk_scale < 1e30f, "qk_scale must be positive and finite");
    if (p.qk_dtype != FICOCO_BF16 || !(p.d_head == 32 || p.d_head == 64 || p.d_head == 128) ||
        ((L || p.qk_n > kQkMaxKeys) && p.H > kQkLongMaxHeads) || p.qk_stride_n % 8 != 0 || p.qk_stride_h % 8 != 0 ||
        p.qk_stride_b % 8 != 0 || ((uintptr_t)p.Q & 15) || ((uintptr_t)p.K & 15)) {
      *why = "queries / keys: bfloat16, 16-byte aligned rows and d_head in {32,64,128} are supported (beyond 640 rows and for FiCoCo-L: at most 64 heads)";
      return FICOCO_EUNSUPPORTED;
    }
  } else if (need_A) {
    REQUIRE(p.A != nullptr, "A is NULL but an attention-derived term is selected");
    REQUIRE(p.H >= 1, "H must be positive");
    REQUIRE(p.a_nq >= 1 && p.a_nk >= 1 && p.a_stride_q >= p.a_nk, "bad A shape / strides");
    REQUIRE(p.a_k_begin <= p.vis_begin && p.vis_begin + p.N <= p.a_k_begin + p.a_nk,
            "A does not cover the visual keys");
    if (p.red_src == FICOCO_R_ATTN_RECV || p.corr_src == FICOCO_C_ATTN)
      REQUIRE(p.a_q_begin <= p.vis_begin && p.vis_begin + p.N <= p.a_q_begin + p.a_nq,
              "A does not cover the visual queries");
    if (p.sem_src == FICOCO_G_CLS_ATTN)
      REQUIRE(p.cls_index >= p.a_q_begin && p.cls_index < p.a_q_begin + p.a_nq &&
                  (p.cls_index < p.vis_begin || p.cls_index >= p.vis_begin + p.N),
              "cls_index must be a query row of A outside the visual span");
  }
  if (L) {
    REQUIRE(p.sem_src == FICOCO_G_TEXT_ATTN, "FiCoCo-L uses the text-attention term (Eq. 3)");
    REQUIRE((qk || p.A_text != nullptr) && p.M >= 1 && p.H >= 1, "A_text / M missing for FiCoCo-L");
    REQUIRE(p.gamma >= 0.0f && p.gamma <= 1.0f, "gamma (Eq. 4) must be in [0, 1]");
    if (!qk)
      REQUIRE(p.at_stride_q >= p.at_nk && p.at_k_begin <= p.vis_begin &&
                  p.vis_begin + p.N <= p.at_k_begin + p.at_nk, "A_text does not cover the visual keys");
  } else {
    REQUIRE(p.sem_src != FICOCO_G_TEXT_ATTN, "the text-attention term belongs to FiCoCo-L");
  }
  if (p.red_src == FICOCO_R_VECTOR) REQUIRE(p.recv_vec != nullptr && p.H >= 1, "recv_vec is NULL");
  if (p.sem_src == FICOCO_G_VECTOR) REQUIRE(p.sem_vec != nullptr && p.H >= 1, "sem_vec is NULL");
  const bool penalty = !L && p.window > 0;
  if (penalty) {
    REQUIRE(p.grid_g >= 1 && p.grid_h >= 1 && p.grid_w >= 1, "grid dimensions must be positive");
    const int64_t cells = (int64_t)p.grid_g * p.grid_h * p.grid_w;
    REQUIRE(cells >= p.N && cells <= kMaxSelectN, "grid must have between N and 12288 cells");
    REQUIRE(p.pos != nullptr || cells == p.N, "pos is NULL but the grid has more cells than tokens");
  }
  pl.need_features = p.red_src == FICOCO_R_SIM_MEAN || p.sem_src == FICOCO_G_EQ_TOKEN ||
                     p.corr_src == FICOCO_C_COSINE;
  pl.Df = p.F ? p.Df : p.D;
  if (pl.need_features && p.F)
    REQUIRE(p.Df >= 1 && p.f_stride_n >= p.Df, "bad F shape / strides");
#undef REQUIRE

  pl.n_disc = p.N - p.n_keep;
  pl.extra_token = p.k_mode == FICOCO_K_CONVERGENT && pl.n_disc > 0;
  pl.n_out = p.n_tot - pl.n_disc + (pl.extra_token ? 1 : 0);
  // targets per discarded token fixed by the caller (ablation): 0 = no edges at all
  pl.fixed_k = p.k_mode == FICOCO_K_FIXED ? std::min(p.fixed_k, p.n_keep) : -1;
  if (p.k_mode == FICOCO_K_CONVERGENT) pl.fixed_k = 0;

  // attention reduction geometry
  // Column strips.  With the head-mean map to store they are narrow at any width: the workgroup turns its
  // tile of the map in LDS, strip columns x chunk rows (map_shape).  Without it, up to 1024 key columns, a strip has
  // at most 24 8-column groups: a workgroup is then (row lanes) x (groups of the strip) with several row lanes, covers many
  // query rows and leaves few per-chunk column partials behind (measured: 3 strips of 24 groups beat 1 strip
  // of 72 at 576 columns by 4 %).  Wider maps take wide strips (their partials are a small share of the traffic): the
  // fewest strips that keep at least 80 % of the threads busy, else the busiest of the next 8 choices.
  const int groups = (p.N + kVec - 1) / kVec;
  const bool map_tile = p.corr_src == FICOCO_C_ATTN;
  const bool vis_rows = p.red_src == FICOCO_R_ATTN_RECV || p.corr_src == FICOCO_C_ATTN;
  if (need_A && !qk) {
    int lo = p.vis_begin - p.a_q_begin, hi = lo + p.N;  // visual query rows
    if (!vis_rows) { lo = hi = p.cls_index - p.a_q_begin; ++hi; }
    if (p.sem_src == FICOCO_G_CLS_ATTN) {
      const int c = p.cls_index - p.a_q_begin;
      if (c < lo) lo = c;
      if (c + 1 > hi) hi = c + 1;
    }
    pl.a_row0 = lo;
    pl.a_rows = hi - lo;
  }
  const MapShape ms = map_shape(p, pl.a_rows);
  if (map_tile) {
    pl.col_strips = (groups + ms.groups - 1) / ms.groups;
    pl.strip_groups = (groups + pl.col_strips - 1) / pl.col_strips;
    pl.row_lanes = ms.lanes;
  } else {
    const int max_groups = groups <= 128 ? 24 : kReduceThreads;
    const int s_min = std::max((groups + kReduceThreads - 1) / kReduceThreads, (groups + max_groups - 1) / max_groups);
    int best_busy = -1;
    for (int sN = s_min; sN < s_min + 8; ++sN) {
      const int sg = (groups + sN - 1) / sN;
      const int rl = kReduceThreads / sg;
      if (rl * sg > best_busy) { best_busy = rl * sg; pl.col_strips = sN; pl.strip_groups = sg; pl.row_lanes = rl; }
      if (best_busy * 5 >= kReduceThreads * 4) break;
    }
  }
  auto rows_per_wg = [&](int rows) {
    if (map_tile) return ms.rows;
    // aim at ~kWgTarget workgroups
    const int64_t want = std::max<int64_t>(((int64_t)p.B * pl.col_strips * rows + kWgTarget - 1) / kWgTarget, 1);
    return (int)((want + pl.row_lanes - 1) / pl.row_lanes) * pl.row_lanes;
  };
  pl.qk = qk;
  if (qk) {
    // the visual queries where a visual-to-visual term is selected, then the [CLS] query or the text
    // queries; one column partial per tile of visual queries
    pl.qk_visq = p.red_src == FICOCO_R_ATTN_RECV || p.corr_src == FICOCO_C_ATTN ? p.N : 0;
    pl.qk_nq = pl.qk_visq + (L ? p.M : p.sem_src == FICOCO_G_CLS_ATTN ? 1 : 0);
    pl.n_chunks = (pl.qk_visq + kQkTile - 1) / kQkTile;
  } else if (need_A) {
    pl.rows_per_wg = rows_per_wg(pl.a_rows);
    pl.a_shift = 0;
    if (p.corr_src == FICOCO_C_ATTN && vis_rows) {
      // The head-mean map is stored transposed, a chunk's rows of one key column as one piece:
      // chunks of a multiple of 8 rows that start at multiples of it, counted from visual row 0,
      // make every piece whole 32-byte sectors.
      const int lead = (p.vis_begin - p.a_q_begin) - pl.a_row0;      // role rows before visual row 0 (the [CLS] query)
      pl.a_shift = (pl.rows_per_wg - lead % pl.rows_per_wg) % pl.rows_per_wg;
    }
    pl.n_chunks = (pl.a_rows + pl.a_shift + pl.rows_per_wg - 1) / pl.rows_per_wg;
  } else {
    pl.n_chunks = 0;
  }

  // threshold selection: p = eps (n-1) evaluated in double from the float eps
  if (p.n_keep >= 1) {
    const double q = (double)p.eps * (double)(p.n_keep - 1);
    const double f = std::floor(q);
    pl.sel_f = (int)f;
    pl.sel_g = q - f;
    pl.sel_m = p.n_keep - pl.sel_f;
    if (pl.fixed_k > 0) {      // fixed K: the threshold is the K-th largest value itself
      pl.sel_m = pl.fixed_k;
      pl.sel_f = p.n_keep - pl.fixed_k;
      pl.sel_g = 0.0;
    }
    pl.dense_rows = pl.sel_m > kSelMax;
  }

  // feature pass geometry (column sums over the tokens)
  if (pl.need_features) {
    // two batches of 8 rows per wavefront: half the workgroups (one round on the chip) and half the partials
    pl.f_rows_per_wg = unit_rows_summed(p, pl.Df) ? unit_rows_per_wg(p) : 64;
    pl.f_chunks = (p.N + pl.f_rows_per_wg - 1) / pl.f_rows_per_wg;
  }

  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes ? bytes : 1); return o; };
  const size_t B = p.B, N = p.N;
  pl.map_pitch = (p.N + 63) / 64 * 64;     // whole 64-entry steps: a wavefront reads a row without clamping
  pl.abar = take(p.corr_src == FICOCO_C_ATTN ? B * N * (size_t)pl.map_pitch * sizeof(float) : 0);
  pl.recv_part = take(B * (size_t)pl.n_chunks * N * sizeof(double));
  pl.cls = take(B * N * sizeof(double));
  pl.ttext = take(L ? B * N * (size_t)p.M * sizeof(double) : 0);
  pl.inv_norm = take(pl.need_features ? B * N * sizeof(double) : 0);
  pl.xhat = take(p.corr_src == FICOCO_C_COSINE ? B * N * (size_t)pl.Df * sizeof(bf16_t) : 0);
  pl.colsum_part = take(pl.need_features ? (unit_rows_summed(p, pl.Df) ? 1 : 2) * B * (size_t)pl.f_chunks * pl.Df * sizeof(double) : 0);
  pl.colmean = take(pl.need_features ? (2 * B * (size_t)pl.Df + B * (size_t)((pl.Df + 255) / 256)) * sizeof(double) : 0);   // two means, then |mu|^2 in parts
  pl.fterm = take(B * N * sizeof(double));
  pl.fterm2 = take(B * N * sizeof(double));
  pl.slot_of = take((B * N + 64) * sizeof(int32_t));    // + one 64-entry step: rows of it are read in whole steps
  pl.tgt_ptr = take(B * (size_t)(p.n_keep + 1) * sizeof(int32_t));
  pl.tgt_src = take(B * (size_t)pl.n_disc * p.k_max * sizeof(int32_t));
  pl.tgt_alpha = take(B * (size_t)pl.n_disc * p.k_max * sizeof(double));
  pl.hub_list = take(B * (size_t)p.n_keep * sizeof(int32_t));
  pl.hub_cnt = take(B * sizeof(int32_t));
  if (qk) {
    // equal rounds of as many images as have room
    const size_t per = (size_t)p.H * pl.qk_nq * sizeof(float2);
    const size_t most = std::max<size_t>(1, kQkNormBytes / std::max<size_t>(per, 1));
    const size_t rounds = (B + most - 1) / most;
    pl.qk_images = (int)((B + rounds - 1) / rounds);
    pl.qk_norm = take(per * pl.qk_images);
    pl.beyond += align_up(per * pl.qk_images);
  }
  pl.rowbuf = take(pl.dense_rows ? B * (size_t)pl.n_disc * p.n_keep * sizeof(double) : 0);
  pl.use_gram = p.corr_src == FICOCO_C_COSINE && !pl.dense_rows && pl.Df % 8 == 0 && p.k_max <= 64 &&
                pl.n_disc > 0;
  pl.gram_splits = 1;
  pl.gram_st_per_split = (pl.Df + kGramStage - 1) / kGramStage;
  if (pl.use_gram) {
    // Few output tiles: cut K so that the matrix-core kernel still fills the chip (about two
    // workgroups per compute unit), each range at least 256 features long; the partial blocks are
    // added, in a fixed order, where they are read.
    // At most 8 ranges, or 16 of a decoder's layer as long as they are one workgroup per compute unit: a tile's time is its
    // stages, but every range is also a block to write and to read.  Stage of 8 / 16 ranges, 4096 features: 1 image of 432 x 144
    // (8 tiles) 22.2 / 21.4 us, 8 of 256 x 128 (16) 27.7 / 26.8, 3 of 432 x 144 (24) 26.9 / 27.9; 5120: 24.6 / 22.5, 29.8 / 29.3,
    // 1 of 800 x 384 (21 tiles) 29.3 / 31.0.  (The other variant keeps to 8: what its scratch may hold is a fixed size.)
    const int64_t tiles = (int64_t)p.B * ((pl.n_disc + 127) / 128) * ((p.n_keep + 127) / 128);
    int splits = (int)((512 + tiles - 1) / tiles);
    splits = std::min(splits, std::min(L && tiles <= 16 ? 16 : 8, pl.Df / 256));
    if (splits < 1) splits = 1;
    const int st_all = (pl.Df + kGramStage - 1) / kGramStage;
    pl.gram_st_per_split = (st_all + splits - 1) / splits;
    pl.gram_splits = (st_all + pl.gram_st_per_split - 1) / pl.gram_st_per_split;
  }
  // + padding: the row kernel reads whole 2048-target passes
  pl.ct = take(pl.use_gram ? (pl.gram_splits * B * (size_t)pl.n_disc * p.n_keep + kCandPad) * sizeof(float) : 0);
  pl.cmax = take(L ? B * (size_t)p.M * sizeof(double) : 0);
  const bool exact_terms = p.red_src == FICOCO_R_SIM_MEAN || p.sem_src == FICOCO_G_EQ_TOKEN;
  pl.ex_nrm = take(exact_terms ? B * N * sizeof(double) : 0);
  pl.ex_mu = take(exact_terms ? B * (size_t)(pl.Df + 1) * sizeof(double) : 0);
  pl.ex_u = take(exact_terms ? B * 8 * (size_t)pl.Df * sizeof(double) : 0);
  pl.ex_g = take(exact_terms ? B * 8 * N * sizeof(double) : 0);
  pl.ex_list = take(exact_terms ? B * N * sizeof(int32_t) : 0);
  if (pl.n_disc > 0) {
    // The targets' lists.  A caller's workspace has room for them whatever the batch is (at 384 of 576 tokens
    // they are a tenth of the head-mean map): bounded by what all images together may take, they ended at
    // B = 219 there, and what they gain with them (256 images of one head 302 us without, 280 with them; 32 x
    // 2881 tokens 740 and 658).  Up to kMatchMaxRows discarded tokens half as many entries do where a target has no more
    // than two sources on average by attention (64 images of one head, 0.5 sources: 84.0 us with 32 entries, 78.5 with
    // 16; 256 images, 2 sources: 288 and 282; 16 images, 19 sources: 212 and 365); the counts of like tokens spread
    // more (cosine, 0.5 sources: the merge 12.4 and 15.1 us).  In a scratch of given size the lists take what the rest
    // leaves; below a quarter / an eighth of the full length nothing is gained.
    const size_t targets = (size_t)p.n_keep, entry = sizeof(int32_t) + sizeof(double);
    const bool is_long = edges_inverted(pl);
    const int per_row = pl.fixed_k >= 0 ? pl.fixed_k : std::max(pl.sel_m - 1, 1);      // targets of a row
    const int64_t edges = (int64_t)pl.n_disc * per_row;
    // The adds to counters of one cache line queue, about 11 ns each (16 images with one preserved token of 576,
    // whose counters share a line: 109 us for the correlate stage, 9 without the adds).  Where the targets
    // have four sources or more on average, and above kMatchMaxRows, each counter has 64 bytes of its own: step with
    // the counters packed and apart 217.8 and 131.7 us there, 94.0 and 79.8 at 16 preserved, 46.7 and 40.9 at
    // 32, 39.3 and 39.0 at 96 (5 sources); 8064 rows with 1152 targets 34 and 28 us for the stage.  Below, the filter
    // and the merge, which write and read the lines, lose what the adds gain (40.0 and 40.3 at 144, 3 sources).
    pl.cnt_stride = is_long || edges >= 4 * (int64_t)p.n_keep ? 16 : 1;
    const int least = is_long ? kBucketCapLong / 8 : kBucketCap / 4;
    auto image_bytes = [&](int cap) { return targets * (cap * entry + pl.cnt_stride * sizeof(int32_t)); };
    const bool few = p.corr_src == FICOCO_C_ATTN && edges <= 2 * (int64_t)p.n_keep;
    int cap = is_long ? kBucketCapLong : std::min(few ? kBucketCap / 2 : kBucketCap, (pl.n_disc + 7) / 8 * 8);
    while (cap > least && image_bytes(cap) > kBucketBytes) cap /= 2;
    const size_t used = off + 3 * 256;                // (each region is rounded up)
    while (cap >= least && (used > scratch || B * image_bytes(cap) > scratch - used)) cap /= 2;
    pl.bkt_cap = cap >= least ? cap : 0;
    const size_t before = off;
    pl.bkt_cnt = take(pl.bkt_cap ? B * targets * pl.cnt_stride * sizeof(int32_t) : 0);
    pl.bkt_src = take(B * targets * pl.bkt_cap * sizeof(int32_t));
    pl.bkt_w = take(B * targets * pl.bkt_cap * sizeof(double));
    pl.beyond += off - before;
  }
  pl.total = off;
  return FICOCO_OK;
}

static int fail(ficoco_ctx* ctx, int code, const char* what, const char* detail) {
  if (ctx) std::snprintf(ctx->err, sizeof(ctx->err), "%s: %s", what, detail ? detail : "");
  return code;
}

// The calling thread's current device must be the one the ctx was created for: every launch
// goes to the current device, and the caller's pointers and stream belong to it.
static int check_device(ficoco_ctx* ctx, const char* fn) {
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess) return fail(ctx, FICOCO_EHIP, fn, "hipGetDevice failed");
  if (cur != ctx->device) return fail(ctx, FICOCO_EINVAL, fn, "the current device is not the device this ctx was created for");
  return FICOCO_OK;
}

// Do the byte ranges [a, a + na) and [b, b + nb) overlap?
static bool ranges_overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a && b && na && nb && a0 < b0 + nb && b0 < a0 + na;
}

// Bytes from X to the end of its last row, and of the dense X_out.
static size_t x_extent(const ficoco_problem& p) {
  const size_t es = p.dtype == FICOCO_BF16 ? 2 : 4;
  return ((size_t)(p.B - 1) * (size_t)p.x_stride_b + (size_t)(p.n_tot - 1) * (size_t)p.x_stride_n + (size_t)p.D) * es;
}
static size_t x_out_extent(const ficoco_problem& p, const Plan& pl) {
  return (size_t)p.B * (size_t)pl.n_out * (size_t)p.D * (p.dtype == FICOCO_BF16 ? 2 : 4);
}

static int prepare(ficoco_ctx* ctx, const ficoco_problem* p, const void* ws, size_t ws_bytes,
                   Plan& pl, const char* fn, size_t scratch = SIZE_MAX) {
  if (!ctx) return FICOCO_EINVAL;
  if (!p) return fail(ctx, FICOCO_EINVAL, fn, "problem is NULL");
  const int dev_rc = check_device(ctx, fn);
  if (dev_rc != FICOCO_OK) return dev_rc;
  const char* why;
  const int rc = make_plan(*p, pl, &why, scratch);
  if (rc != FICOCO_OK) return fail(ctx, rc, fn, why);
  if (!ws || ((uintptr_t)ws & 255)) return fail(ctx, FICOCO_EINVAL, fn, "workspace is NULL or not 256-byte aligned");
  if (ws_bytes < pl.total) return fail(ctx, FICOCO_ENOMEM, fn, "workspace smaller than ficoco_workspace_bytes()");
  return FICOCO_OK;
}

static int finish(ficoco_ctx* ctx, const char* fn) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(ctx, FICOCO_EHIP, fn, hipGetErrorString(e));
  return FICOCO_OK;
}

static int run_step(ficoco_ctx* ctx, const ficoco_problem* p0, int variant, void* ws, size_t ws_bytes,
                    void* X_out, int32_t* pos_out, int32_t* keep_idx, int32_t* discard_idx,
                    int32_t* edge_cnt, int32_t* edge_tgt, double* edge_alpha, double* scores,
                    int32_t* overflow, void* stream, const char* fn, size_t scratch = SIZE_MAX) {
  if (!ctx) return FICOCO_EINVAL;
  if (!p0) return fail(ctx, FICOCO_EINVAL, fn, "problem is NULL");
  if (p0->variant != variant) return fail(ctx, FICOCO_EINVAL, fn, "problem.variant does not match the entry point");
  Plan pl;
  const int rc = prepare(ctx, p0, ws, ws_bytes, pl, fn, scratch);
  if (rc != FICOCO_OK) return rc;
  if (!X_out || !keep_idx || !scores || !overflow ||
      (pl.n_disc > 0 && (!discard_idx || !edge_cnt || !edge_tgt || !edge_alpha)))
    return fail(ctx, FICOCO_EINVAL, fn, "an output pointer is NULL");
  const ficoco_problem& p = *p0;
  if (ranges_overlap(X_out, x_out_extent(p, pl), p.X, x_extent(p)))
    return fail(ctx, FICOCO_EINVAL, fn, "X_out overlaps X (outputs may not alias inputs)");
  if (ranges_overlap(X_out, x_out_extent(p, pl), ws, pl.total))
    return fail(ctx, FICOCO_EINVAL, fn, "X_out overlaps the workspace");
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)ws;
  const bool pr = ctx->probe_start && ctx->probe_kernel == FICOCO_PROBE_REDUCE;
  const bool pg = ctx->probe_start && ctx->probe_kernel == FICOCO_PROBE_GRAM;
  if (pr) (void)hipEventRecord(ctx->probe_start, s);
  const bool tw = text_with_features(p, pl);
  if (pl.qk) launch_attn_qk(p, pl, w, s); else launch_attn_reduce(p, pl, w, s, tw);
  if (pr) (void)hipEventRecord(ctx->probe_stop, s);
  if (pl.need_features) launch_features(p, pl, w, s, tw, tw);
  launch_select(p, pl, w, scores, true, true, discard_idx, keep_idx, overflow, s, tw, pos_out);
  launch_correlate(p, pl, w, discard_idx, keep_idx, edge_cnt, edge_tgt, edge_alpha, overflow, true,
                   pg ? ctx->probe_start : nullptr, pg ? ctx->probe_stop : nullptr, s);
  // (the position ids of the preserved tokens were written by the filter, beside keep_idx)
  launch_compress(p, pl, w, discard_idx, keep_idx, edge_cnt, edge_tgt, edge_alpha, X_out, nullptr, s, true);
  return finish(ctx, fn);
}

}  // namespace ficoco

using namespace ficoco;

extern "C" {

int ficoco_create(ficoco_ctx** out, int device) {
  if (!out) return FICOCO_EINVAL;
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count) return FICOCO_EHIP;
  if (device < kMaxDevices && g_static_ws[device] == nullptr) {
    // the scratch array's address on this device, asked for with that device current
    int prev = -1;
    if (hipGetDevice(&prev) != hipSuccess) return FICOCO_EHIP;
    if (prev != device && hipSetDevice(device) != hipSuccess) return FICOCO_EHIP;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_static_scratch));
    if (prev != device) (void)hipSetDevice(prev);
    if (e != hipSuccess || ptr == nullptr) return FICOCO_EHIP;
    g_static_ws[device] = ptr;
  }
  ficoco_ctx* c = new (std::nothrow) ficoco_ctx;
  if (!c) return FICOCO_ENOMEM;
  c->device = device;
  c->probe_start = nullptr;
  c->probe_stop = nullptr;
  c->probe_kernel = FICOCO_PROBE_REDUCE;
  c->err[0] = 0;
  *out = c;
  return FICOCO_OK;
}

int ficoco_destroy(ficoco_ctx* ctx) {
  delete ctx;
  return FICOCO_OK;
}

const char* ficoco_last_error(const ficoco_ctx* ctx) { return ctx ? ctx->err : "ctx is NULL"; }

int ficoco_set_probe(ficoco_ctx* ctx, int kernel, void* start_event, void* stop_event) {
  if (!ctx || ((start_event == nullptr) != (stop_event == nullptr)) ||
      (kernel != FICOCO_PROBE_REDUCE && kernel != FICOCO_PROBE_GRAM && kernel != FICOCO_PROBE_GRAM_X16))
    return FICOCO_EINVAL;
  ctx->probe_kernel = kernel;
  ctx->probe_start = (hipEvent_t)start_event;
  ctx->probe_stop = (hipEvent_t)stop_event;
  return FICOCO_OK;
}

const char* ficoco_version(void) { return "ficoco-gfx950 0.1"; }

int ficoco_workspace_bytes(const ficoco_problem* p, size_t* out_bytes) {
  if (!p || !out_bytes) return FICOCO_EINVAL;
  Plan pl;
  const char* why;
  const int rc = make_plan(*p, pl, &why);
  if (rc != FICOCO_OK) return rc;
  *out_bytes = pl.total;
  return FICOCO_OK;
}

int ficoco_out_rows(const ficoco_problem* p, int32_t* out_rows) {
  if (!p || !out_rows) return FICOCO_EINVAL;
  Plan pl;
  const char* why;
  const int rc = make_plan(*p, pl, &why);
  if (rc != FICOCO_OK) return rc;
  *out_rows = pl.n_out;
  return FICOCO_OK;
}

int ficoco_reduce(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes, void* stream) {
  Plan pl;
  const int rc = prepare(ctx, p, ws, ws_bytes, pl, "ficoco_reduce");
  if (rc != FICOCO_OK) return rc;
  const bool pr = ctx->probe_start && ctx->probe_kernel == FICOCO_PROBE_REDUCE;
  if (pr) (void)hipEventRecord(ctx->probe_start, (hipStream_t)stream);
  if (pl.qk) launch_attn_qk(*p, pl, (char*)ws, (hipStream_t)stream);
  else launch_attn_reduce(*p, pl, (char*)ws, (hipStream_t)stream);
  if (pr) (void)hipEventRecord(ctx->probe_stop, (hipStream_t)stream);
  return finish(ctx, "ficoco_reduce");
}

int ficoco_score(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes, double* scores,
                 void* stream) {
  Plan pl;
  const int rc = prepare(ctx, p, ws, ws_bytes, pl, "ficoco_score");
  if (rc != FICOCO_OK) return rc;
  if (!scores) return fail(ctx, FICOCO_EINVAL, "ficoco_score", "scores is NULL");
  const bool tw = text_with_features(*p, pl);
  if (pl.qk) launch_attn_qk(*p, pl, (char*)ws, (hipStream_t)stream);
  else launch_attn_reduce(*p, pl, (char*)ws, (hipStream_t)stream, tw);
  if (pl.need_features) launch_features(*p, pl, (char*)ws, (hipStream_t)stream, tw, false);
  launch_score(*p, pl, (char*)ws, scores, (hipStream_t)stream, tw);
  return finish(ctx, "ficoco_score");
}

int ficoco_filter(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes,
                  const double* scores, int32_t* discard_idx, int32_t* keep_idx, void* stream) {
  Plan pl;
  const int rc = prepare(ctx, p, ws, ws_bytes, pl, "ficoco_filter");
  if (rc != FICOCO_OK) return rc;
  if (!scores || !keep_idx || (pl.n_disc > 0 && !discard_idx))
    return fail(ctx, FICOCO_EINVAL, "ficoco_filter", "a pointer is NULL");
  launch_filter(*p, pl, (char*)ws, scores, discard_idx, keep_idx, (hipStream_t)stream);
  return finish(ctx, "ficoco_filter");
}

int ficoco_correlate(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes,
                     const int32_t* discard_idx, const int32_t* keep_idx, int32_t* edge_cnt,
                     int32_t* edge_tgt, double* edge_alpha, int32_t* overflow, void* stream) {
  Plan pl;
  const int rc = prepare(ctx, p, ws, ws_bytes, pl, "ficoco_correlate");
  if (rc != FICOCO_OK) return rc;
  if (!keep_idx || !overflow || (pl.n_disc > 0 && (!discard_idx || !edge_cnt || !edge_tgt || !edge_alpha)))
    return fail(ctx, FICOCO_EINVAL, "ficoco_correlate", "a pointer is NULL");
  const bool pg = ctx->probe_start && (ctx->probe_kernel == FICOCO_PROBE_GRAM || ctx->probe_kernel == FICOCO_PROBE_GRAM_X16);
  launch_correlate(*p, pl, (char*)ws, discard_idx, keep_idx, edge_cnt, edge_tgt, edge_alpha, overflow,
                   false, pg ? ctx->probe_start : nullptr, pg ? ctx->probe_stop : nullptr,
                   (hipStream_t)stream, pg && ctx->probe_kernel == FICOCO_PROBE_GRAM_X16 ? FICOCO_PROBE_REPEAT : 1);
  return finish(ctx, "ficoco_correlate");
}

int ficoco_correlation_gap(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes,
                           const int32_t* discard_idx, const int32_t* keep_idx, double* gap, void* stream) {
  Plan pl;
  const int rc = prepare(ctx, p, ws, ws_bytes, pl, "ficoco_correlation_gap");
  if (rc != FICOCO_OK) return rc;
  if (!keep_idx || (pl.n_disc > 0 && (!discard_idx || !gap)))
    return fail(ctx, FICOCO_EINVAL, "ficoco_correlation_gap", "a pointer is NULL");
  launch_corr_gap(*p, pl, (char*)ws, discard_idx, keep_idx, gap, (hipStream_t)stream);
  return finish(ctx, "ficoco_correlation_gap");
}

int ficoco_gather_tokens(ficoco_ctx* ctx, const ficoco_problem* p, const int32_t* keep_idx, const void* in,
                         int64_t in_stride_b, int64_t in_stride_n, int32_t row_bytes, void* out, void* stream) {
  if (!ctx) return FICOCO_EINVAL;
  if (!p) return fail(ctx, FICOCO_EINVAL, "ficoco_gather_tokens", "problem is NULL");
  const int dev_rc = check_device(ctx, "ficoco_gather_tokens");
  if (dev_rc != FICOCO_OK) return dev_rc;
  Plan pl;
  const char* why;
  const int rc = make_plan(*p, pl, &why);
  if (rc != FICOCO_OK) return fail(ctx, rc, "ficoco_gather_tokens", why);
  if (pl.extra_token)
    return fail(ctx, FICOCO_EUNSUPPORTED, "ficoco_gather_tokens", "the convergent form's additional token has no row to gather");
  if (!keep_idx || !in || !out) return fail(ctx, FICOCO_EINVAL, "ficoco_gather_tokens", "a pointer is NULL");
  if (row_bytes < 4 || row_bytes % 4 != 0 || in_stride_n < row_bytes || in_stride_n % 4 != 0 || in_stride_b % 4 != 0 ||
      ((uintptr_t)in % 4) != 0 || ((uintptr_t)out % 4) != 0)
    return fail(ctx, FICOCO_EINVAL, "ficoco_gather_tokens", "row_bytes / strides / pointers must be multiples of 4 bytes");
  launch_gather(*p, pl, keep_idx, in, in_stride_b, in_stride_n, row_bytes, out, (hipStream_t)stream);
  return finish(ctx, "ficoco_gather_tokens");
}

int ficoco_compress(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes,
                    const int32_t* discard_idx, const int32_t* keep_idx, const int32_t* edge_cnt,
                    const int32_t* edge_tgt, const double* edge_alpha, void* X_out, int32_t* pos_out,
                    void* stream) {
  Plan pl;
  const int rc = prepare(ctx, p, ws, ws_bytes, pl, "ficoco_compress");
  if (rc != FICOCO_OK) return rc;
  if (!X_out || !keep_idx || (pl.n_disc > 0 && (!discard_idx || !edge_cnt || !edge_tgt || !edge_alpha)))
    return fail(ctx, FICOCO_EINVAL, "ficoco_compress", "a pointer is NULL");
  if (ranges_overlap(X_out, x_out_extent(*p, pl), p->X, x_extent(*p)))
    return fail(ctx, FICOCO_EINVAL, "ficoco_compress", "X_out overlaps X (outputs may not alias inputs)");
  launch_compress(*p, pl, (char*)ws, discard_idx, keep_idx, edge_cnt, edge_tgt, edge_alpha, X_out,
                  pos_out, (hipStream_t)stream);
  return finish(ctx, "ficoco_compress");
}

int ficoco_v_step(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes, void* X_out,
                  int32_t* pos_out, int32_t* keep_idx, int32_t* discard_idx, int32_t* edge_cnt,
                  int32_t* edge_tgt, double* edge_alpha, double* scores, int32_t* overflow,
                  void* stream) {
  return run_step(ctx, p, FICOCO_VARIANT_V, ws, ws_bytes, X_out, pos_out, keep_idx, discard_idx,
                  edge_cnt, edge_tgt, edge_alpha, scores, overflow, stream, "ficoco_v_step");
}

int ficoco_v_step_static(ficoco_ctx* ctx, const ficoco_problem* p, void* X_out, int32_t* pos_out,
                         int32_t* keep_idx, int32_t* discard_idx, int32_t* edge_cnt, int32_t* edge_tgt,
                         double* edge_alpha, double* scores, int32_t* overflow, void* stream) {
  const char* fn = "ficoco_v_step_static";
  if (!ctx) return FICOCO_EINVAL;
  if (!p) return fail(ctx, FICOCO_EINVAL, fn, "problem is NULL");
  Plan pl;
  const char* why;
  const int rc = make_plan(*p, pl, &why, kStaticScratchBytes);
  if (rc != FICOCO_OK) return fail(ctx, rc, fn, why);
  if (pl.total - pl.beyond > FICOCO_STATIC_SCRATCH_BYTES || pl.total > kStaticScratchBytes)
    return fail(ctx, FICOCO_ENOMEM, fn, "the step's workspace exceeds the 32 MiB static scratch: use ficoco_v_step with a caller workspace");
  void* ws = ctx->device < kMaxDevices ? g_static_ws[ctx->device] : nullptr;
  if (!ws) return fail(ctx, FICOCO_EHIP, fn, "no static scratch on this device");
  return run_step(ctx, p, FICOCO_VARIANT_V, ws, kStaticScratchBytes, X_out, pos_out, keep_idx, discard_idx,
                  edge_cnt, edge_tgt, edge_alpha, scores, overflow, stream, fn, kStaticScratchBytes);
}

int ficoco_l_step(ficoco_ctx* ctx, const ficoco_problem* p, void* ws, size_t ws_bytes, void* X_out,
                  int32_t* pos_out, int32_t* keep_idx, int32_t* discard_idx, int32_t* edge_cnt,
                  int32_t* edge_tgt, double* edge_alpha, double* scores, int32_t* overflow,
                  void* stream) {
  return run_step(ctx, p, FICOCO_VARIANT_L, ws, ws_bytes, X_out, pos_out, keep_idx, discard_idx,
                  edge_cnt, edge_tgt, edge_alpha, scores, overflow, stream, "ficoco_l_step");
}

}  // extern "C"
