// Correlate stage: correlation row of every discarded token over the preserved tokens,
// its eps-quantile threshold, the correlated targets and their weights
// (Sec. "Correlation-based Information Recycling", Eq. 4, Algorithm 1/2 stage 3, Eq. 2's
// alpha).  One wavefront per discarded token.  Values are evaluated on the fly in double
// precision and every comparison is on doubles.
//
//   tau_i = v[f] + g (v[f+1] - v[f]),  p = eps (n-1), f = floor(p), g = p - f, v = row sorted
//   J_i = { j : C_ij >= tau_i },  alpha_ij = C_ij / sum_{J_i} C_ij  (sum in ascending j)
//
// Only the m = n - f largest values of a row decide tau.  For m <= kSelMax they are kept in
// registers (per lane, then merged across the wavefront); otherwise the row is written to
// the workspace and the two order statistics are found bit by bit.
#include "common.hpp"
#include "gram_tile.hpp"
#include "text_stats.hpp"

#include <algorithm>

namespace ficoco {

enum CorrMode { kAttnV = 0, kAttnL = 1, kCosV = 2, kCosL = 3 };

struct CorrArgs {
  int B, N, n_keep, n_disc, M, k_max, Df, mode;
  const float* abar;     // [B][N][map_pitch] head-mean map, transposed: abar[b][key token i][query token j]
  int map_pitch;
  const double* ttext;   // [B][N][M]
  const bf16_t* xhat;    // [B][N][Df]
  double gamma, invM;
  const int32_t* S;
  const int32_t* T;
  int sel_m, sel_f;
  double sel_g;
  int dense;
  double* rowbuf;        // [B][n_disc][n_keep]
  int32_t* edge_cnt;
  int32_t* edge_tgt;
  double* edge_alpha;
  int32_t* overflow;
  const int32_t* slot_of; // [B][N] keep slot of a visual token, -1 if discarded
  float* ct;             // [ct_splits][B][n_disc][n_keep] approximate cosines from the matrix cores (partial sums)
  int ct_splits;
  double* cmax;          // [B][M]
  float delta;           // bound of |ct - exact dot|
  int top_k;             // > 0: a row whose top_k-th largest value is clear of the rest has exactly the top_k as targets
  int fixed_k;           // > 0: ablation "fixed K" (sel_m = K, sel_g = 0): of the values equal to the threshold only
                         // the lowest positions are taken, K targets in all; -1: every value >= threshold
  double* gap;           // correlation-gap diagnostic output [B][n_disc] (its own kernel)
  int32_t* bkt_cnt;      // [B][n_keep] edges per target, cleared by the filter stage of a fused step, or null
  int32_t* hub_list;     // [B][n_keep] targets with more than kHubMin sources, as they appear, or null ...
  int32_t* hub_cnt;      // [B] ... and their number
  int32_t* bkt_src;      // [B][n_keep][bkt_cap] the first of them: sources (bucket_entry) ...
  double* bkt_w;         // ... and weights, in order of arrival (the merge orders them)
  int bkt_cap, cnt_stride;
};

// One more edge, from discarded row `row` (token i) to keep slot `tgt` with weight `al`, for the
// target's list that the compress stage of a fused step reads.
__device__ __forceinline__ void emit_edge(const CorrArgs& a, int64_t b, int row, int i, int tgt, double al) {
  if (a.bkt_cnt == nullptr || (unsigned)tgt >= (unsigned)a.n_keep) return;
  const int64_t at = b * a.n_keep + tgt;
  const int slot = atomicAdd(&a.bkt_cnt[at * a.cnt_stride], 1);
  if (slot < a.bkt_cap) {
    a.bkt_src[at * a.bkt_cap + slot] = bucket_entry(row, i);
    a.bkt_w[at * a.bkt_cap + slot] = al;
  }
  if (slot == kHubMin && a.hub_cnt) a.hub_list[b * a.n_keep + atomicAdd(&a.hub_cnt[b], 1)] = tgt;    // (once per target)
}

__device__ __forceinline__ double dot_bf16(const bf16_t* __restrict__ x, const bf16_t* __restrict__ y, int D) {
  double acc = 0.0;
  int d = 0;
  for (; d + kVec <= D; d += kVec) {
    double a[kVec], c[kVec];
    load8<bf16_t>(x + d, a);
    load8<bf16_t>(y + d, c);
#pragma unroll
    for (int k = 0; k < kVec; ++k) acc += a[k] * c[k];
  }
  for (; d < D; ++d) acc += widen(x[d]) * widen(y[d]);
  return acc;
}

// C[i][j] for discarded visual token i and preserved visual token j of image b.
__device__ __forceinline__ double corr_value(const CorrArgs& a, int64_t b, int i, int j) {
  double direct;
  if (a.mode == kAttnV || a.mode == kAttnL) {
    direct = (double)a.abar[(b * a.N + i) * a.map_pitch + j];
  } else {
    const double d = dot_bf16(a.xhat + (b * a.N + i) * a.Df, a.xhat + (b * a.N + j) * a.Df, a.Df);
    direct = d > 0.0 ? d : 0.0;
  }
  if (a.mode == kAttnV || a.mode == kCosV) return direct;
  const double* ti = a.ttext + (b * a.N + i) * a.M;
  const double* tj = a.ttext + (b * a.N + j) * a.M;
  double br = 0.0;
  for (int k = 0; k < a.M; ++k) br += ti[k] * tj[k];
  return a.gamma * direct + (1.0 - a.gamma) * (br * a.invM);
}

__device__ __forceinline__ double wave_max(double v) {
  return wave_reduce(v, [](double x, double y) { return y > x ? y : x; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float x, float y) { return y > x ? y : x; });
}
__device__ __forceinline__ int wave_sum(int v) {
  return wave_reduce(v, [](int x, int y) { return x + y; });
}

__device__ __forceinline__ uint64_t order_key(double x) {   // monotone double -> uint64
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ULL);
}
__device__ __forceinline__ double key_value(uint64_t k) {
  const uint64_t u = (k >> 63) ? (k & 0x7fffffffffffffffULL) : ~k;
  return __longlong_as_double((long long)u);
}

// Value of ascending rank `want` (0-based) among row[0..n): bitwise selection on the
// ordered keys, most significant bit first.  All lanes return the same value.
__device__ double select_rank(const double* __restrict__ row, int n, int want, int lane) {
  uint64_t prefix = 0;
  int rank = want;
  for (int bit = 63; bit >= 0; --bit) {
    const uint64_t hi_mask = bit == 63 ? 0ULL : (~0ULL << (bit + 1));
    int zeros = 0;
    for (int j = lane; j < n; j += kWave) {
      const uint64_t k = order_key(row[j]);
      zeros += ((k & hi_mask) == prefix && !((k >> bit) & 1ULL)) ? 1 : 0;
    }
    zeros = wave_sum(zeros);
    if (rank >= zeros) { rank -= zeros; prefix |= 1ULL << bit; }
  }
  return key_value(prefix);
}

__device__ __forceinline__ double threshold_of(double v_f, double v_f1, double g) {
#pragma clang fp contract(off)
  const double diff = v_f1 - v_f;
  const double step = g * diff;
  return v_f + step;
}

__global__ __launch_bounds__(256) void corr_fill_rows_kernel(CorrArgs a) {
  const int lane = threadIdx.x % kWave;
  const int row = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t b = blockIdx.y;
  if (row >= a.n_disc) return;
  const int i = a.S[b * a.n_disc + row];
  double* dst = a.rowbuf + (b * a.n_disc + row) * a.n_keep;
  for (int jj = lane; jj < a.n_keep; jj += kWave) {
    const int j = a.T[b * a.n_keep + jj];
    const bool ok = (unsigned)i < (unsigned)a.N && (unsigned)j < (unsigned)a.N;  // index sets are device data
    dst[jj] = ok ? corr_value(a, b, i, j) : -__builtin_huge_val();
  }
}

// One discarded row, exactly: every value of the row evaluated in double precision.
__device__ void corr_row_exact(const CorrArgs& a, const int64_t b, const int row, const int lane) {
  const int n = a.n_keep;
  const int i = a.S[b * a.n_disc + row];
  const int32_t* T = a.T + b * n;
  if ((unsigned)i >= (unsigned)a.N) {  // index sets are device data: never index with a bad one
    if (lane == 0) a.edge_cnt[b * a.n_disc + row] = 0;
    return;
  }
  const double* rowv = a.dense ? a.rowbuf + (b * a.n_disc + row) * n : nullptr;
  const double NEG = -__builtin_huge_val();

  double v_f, v_f1;
  int n_gt = 0;                      // values strictly above v_f (used by the fixed-K form only)
  if (a.dense) {
    v_f = select_rank(rowv, n, a.sel_f, lane);
    v_f1 = a.sel_f + 1 <= n - 1 ? select_rank(rowv, n, a.sel_f + 1, lane) : v_f;
    if (a.fixed_k > 0) {
      for (int jj = lane; jj < n; jj += kWave) n_gt += rowv[jj] > v_f ? 1 : 0;
      n_gt = wave_sum(n_gt);
    }
  } else {
    // per-lane descending top list, then m rounds of "pop the wavefront maximum"
    double top[kSelMax];
#pragma unroll
    for (int k = 0; k < kSelMax; ++k) top[k] = NEG;
    for (int jj = lane; jj < n; jj += kWave) {
      const int j = T[jj];
      double c = (unsigned)j < (unsigned)a.N ? corr_value(a, b, i, j) : NEG;
      if (c > top[kSelMax - 1]) {
#pragma unroll
        for (int k = 0; k < kSelMax; ++k) {
          const bool sw = c > top[k];
          const double t = top[k];
          top[k] = sw ? c : t;
          c = sw ? t : c;
        }
      }
    }
    v_f = NEG; v_f1 = NEG;
    for (int r = 0; r < a.sel_m; ++r) {
      const double mx = wave_max(top[0]);
      const unsigned long long who = __ballot(top[0] == mx);
      const int first = __ffsll(who) - 1;
      if (lane == first) {
#pragma unroll
        for (int k = 0; k + 1 < kSelMax; ++k) top[k] = top[k + 1];
        top[kSelMax - 1] = NEG;
      }
      if (r == 0 || mx < v_f) n_gt = r;     // pops so far that are strictly above this one
      v_f1 = v_f;
      v_f = mx;
    }
    if (a.sel_m == 1) v_f1 = v_f;
  }
  const double tau = threshold_of(v_f, v_f1, a.sel_g);
  const int tie_quota = a.fixed_k > 0 ? a.sel_m - n_gt : 0x7fffffff;   // values equal to tau that are taken
  int ties_seen = 0;

  // Emit targets in ascending order; lane e of the wavefront ends up holding edge e.
  int cnt = 0;
  double denom = 0.0;
  int my_tgt = -1;
  double my_c = 0.0;
  const int64_t ebase = (b * a.n_disc + row) * a.k_max;
  for (int base = 0; base < n; base += kWave) {
    const int jj = base + lane;
    double c = NEG;
    if (jj < n) {
      if (a.dense) c = rowv[jj];
      else { const int j = T[jj]; if ((unsigned)j < (unsigned)a.N) c = corr_value(a, b, i, j); }
    }
    const bool is_eq = jj < n && c == tau;
    const unsigned long long eqm = __ballot(is_eq);
    const int eq_rank = ties_seen + __popcll(eqm & ((1ULL << lane) - 1ULL));
    ties_seen += __popcll(eqm);
    unsigned long long hit = __ballot(jj < n && (c > tau || (is_eq && eq_rank < tie_quota)));
    while (hit) {
      const int l = __ffsll(hit) - 1;
      hit &= hit - 1;
      const double cl = lane_value(c, l);
      denom += cl;
      if (a.k_max <= kWave) {
        if (lane == cnt) { my_tgt = base + l; my_c = cl; }
      } else if (lane == 0 && cnt < a.k_max) {
        a.edge_tgt[ebase + cnt] = base + l;
        a.edge_alpha[ebase + cnt] = cl;      // raw value, scaled below
      }
      ++cnt;
    }
  }
  const int stored = cnt < a.k_max ? cnt : a.k_max;
  const bool live = denom > 0.0;
  if (a.k_max <= kWave) {
    if (live && lane < stored) {
      const double al = my_c / denom;
      a.edge_tgt[ebase + lane] = my_tgt;
      a.edge_alpha[ebase + lane] = al;
      emit_edge(a, b, row, i, my_tgt, al);
    }
  } else if (live && lane == 0) {
    for (int e = 0; e < stored; ++e) {
      const double al = a.edge_alpha[ebase + e] / denom;
      a.edge_alpha[ebase + e] = al;
      emit_edge(a, b, row, i, a.edge_tgt[ebase + e], al);
    }
  }
  if (lane == 0) {
    a.edge_cnt[b * a.n_disc + row] = live ? stored : 0;
    if (live && cnt > a.k_max) a.overflow[b] = 1;
  }
}

__global__ __launch_bounds__(256) void corr_rows_kernel(CorrArgs a) {
  const int lane = threadIdx.x % kWave;
  const int row = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (row >= a.n_disc) return;  // whole wavefront leaves together
  corr_row_exact(a, blockIdx.y, row, lane);
}

// ---- cosine correlation through the matrix cores -------------------------------------------
// gram_tile_kernel (bf16 MFMA) has written approximate cosines ct[b][row][j].  They only
// propose candidates.  With |ct - exact dot| <= delta and, for FiCoCo-L, the indirect term of
// Eq. 4 inside [0, bound_i], every C_ij lies in [lo_ij, up_ij]; the m-th largest lo of the
// row is a lower bound of v[f], so a target with up_ij below it can neither be one of the
// order statistics that fix tau nor pass the threshold.  The remaining targets (a handful)
// are evaluated exactly in double precision and the row is finished on those.  A row with
// more than 64 candidates is evaluated exactly in full instead.
constexpr int kCandCap = 64;

__device__ __forceinline__ double wave_sum_f64(double v) {
  return wave_reduce(v, [](double x, double y) { return x + y; });
}

// exact C[i][j], the whole wavefront working on one pair (all lanes return the value)
__device__ __forceinline__ double corr_value_wave(const CorrArgs& a, int64_t b, int i, int j, int lane) {
  double direct;
  if (a.mode == kAttnL) {
    direct = (double)a.abar[(b * a.N + i) * a.map_pitch + j];
  } else {
    const bf16_t* x = a.xhat + (b * a.N + i) * a.Df;
    const bf16_t* y = a.xhat + (b * a.N + j) * a.Df;
    double acc = 0.0;
    const int Dv = a.Df - a.Df % kVec;
    for (int d = lane * kVec; d < Dv; d += kWave * kVec) {
      double u[kVec], w[kVec];
      load8<bf16_t>(x + d, u);
      load8<bf16_t>(y + d, w);
#pragma unroll
      for (int k = 0; k < kVec; ++k) acc += u[k] * w[k];
    }
    for (int d = Dv + lane; d < a.Df; d += kWave) acc += widen(x[d]) * widen(y[d]);
    acc = wave_sum_f64(acc);
    direct = acc > 0.0 ? acc : 0.0;
  }
  if (a.mode == kCosV) return direct;
  const double* ti = a.ttext + (b * a.N + i) * a.M;
  const double* tj = a.ttext + (b * a.N + j) * a.M;
  double br = 0.0;
  for (int k = lane; k < a.M; k += kWave) br += ti[k] * tj[k];
  br = wave_sum_f64(br);
  return a.gamma * direct + (1.0 - a.gamma) * (br * a.invM);
}

// Maxima of the text profiles (bound of Eq. 4's indirect term) where the score stage did not form them: staged calls, and steps
// with fewer text queries than the score stage's launch is worth.  (64 queries and four token groups a workgroup, nine rounds of loads:
// 7.3 us at 8 x 576 tokens, 4.1 so; 69 and 23 at 9216 tokens.)
__global__ __launch_bounds__(256) void text_colmax_kernel(TextStatsArgs t) { text_cmax_block(t, blockIdx.x, blockIdx.y); }

constexpr int kCorrSteps = 2;   // 512-feature steps of the exact dot products loaded together

// Exact C[i][j_q] for up to CB targets at once, the whole wavefront working on them together
// (all lanes return the values).  The loads of all CB rows are issued before the first use, so
// a batch costs one memory round trip per 512 features instead of one per target.  Per target
// the arithmetic and its order are those of corr_value_wave.
template <int CB, int MODE>
__device__ __forceinline__ void corr_values_wave(const CorrArgs& a, int64_t b, int i, const int (&j)[CB], int lane,
                                                 double (&out)[CB]) {
  double direct[CB];
  if (MODE == kAttnL) {
#pragma unroll
    for (int q = 0; q < CB; ++q) direct[q] = (double)a.abar[(b * a.N + i) * a.map_pitch + j[q]];
  } else {
    const bf16_t* x = a.xhat + (b * a.N + i) * a.Df;
    const bf16_t* y[CB];
    double acc[CB];
#pragma unroll
    for (int q = 0; q < CB; ++q) { y[q] = a.xhat + (b * a.N + j[q]) * a.Df; acc[q] = 0.0; }
    const int Dv = a.Df - a.Df % kVec;
    // kCorrSteps steps of 512 features at a time: (1 + CB) * kCorrSteps loads in flight.  A lane
    // past the last whole vector reads vector 0 and clears it (straight-line batch).
    for (int d0 = lane * kVec; d0 - lane * kVec < Dv; d0 += kCorrSteps * kWave * kVec) {
      Raw8<bf16_t> xr[kCorrSteps], yr[kCorrSteps][CB];
#pragma unroll
      for (int t = 0; t < kCorrSteps; ++t) {
        const int d = d0 + t * kWave * kVec;
        const int off = d < Dv ? d : 0;
        load_raw(x + off, xr[t]);
#pragma unroll
        for (int q = 0; q < CB; ++q) load_raw(y[q] + off, yr[t][q]);
      }
      issue_fence();
#pragma unroll
      for (int t = 0; t < kCorrSteps; ++t) {
        keep_raw_if(xr[t], d0 + t * kWave * kVec < Dv);      // a cleared x vector adds zeros for every target
        double u[kVec];
        widen_raw(xr[t], u);
#pragma unroll
        for (int q = 0; q < CB; ++q) {
          double w[kVec];
          widen_raw(yr[t][q], w);
#pragma unroll
          for (int k = 0; k < kVec; ++k) acc[q] += u[k] * w[k];
        }
      }
    }
    for (int d = Dv + lane; d < a.Df; d += kWave) {
#pragma unroll
      for (int q = 0; q < CB; ++q) acc[q] += widen(x[d]) * widen(y[q][d]);
    }
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const double t = wave_sum_f64(acc[q]);
      direct[q] = t > 0.0 ? t : 0.0;
    }
  }
  if (MODE == kCosV) {
#pragma unroll
    for (int q = 0; q < CB; ++q) out[q] = direct[q];
    return;
  }
  const double* ti = a.ttext + (b * a.N + i) * a.M;
  double br[CB];
#pragma unroll
  for (int q = 0; q < CB; ++q) br[q] = 0.0;
  for (int k = lane; k < a.M; k += kWave) {
    const double tik = ti[k];
    double tjk[CB];
#pragma unroll
    for (int q = 0; q < CB; ++q) tjk[q] = a.ttext[(b * a.N + j[q]) * a.M + k];
#pragma unroll
    for (int q = 0; q < CB; ++q) br[q] += tik * tjk[q];
  }
#pragma unroll
  for (int q = 0; q < CB; ++q) out[q] = a.gamma * direct[q] + (1.0 - a.gamma) * (wave_sum_f64(br[q]) * a.invM);
}

constexpr int kCandKeep = 32;                    // approximate values held per lane
constexpr int kCandChunk = kCandKeep * kWave;    // targets per pass over the row
static_assert(kCandChunk <= kCandPad, "the block's padding covers one pass");
constexpr int kCandBatch = 4;                    // targets evaluated exactly at a time

// Bound by each wavefront's chain of dependent loads and, at 1152 targets per row, by the vector unit.
// Rows whose targets are clear from the approximate values skip the exact dot products (K = 1) or take
// them of the K targets only, and the largest values are kept by medians: 31.6 -> 18.1 us at 8 x 432 rows
// of 144 targets and 4096 features (K = 1), 32.5 -> 27.4 us at 8064 rows of 1152 (K = 3, 1024 features).
// One instance per correlation (with the mode a run-time value it held 127 registers and spilled four), no threshold where the
// targets are known, and the text rows of the bound asked for ahead of the row (1353 -> 1098 vector instructions per row of 1152):
// 28.2 -> 25.2 us at 8064 rows of 1152, 18.5 -> 17.6 at 8 x 432 rows of 144, 12.1 -> 10.5 on the map's rows.  What is
// asked of every slot of a row (past its end? of a token?) is worked out where it is used, in branches: kept for all of them, the
// answers went over 51 to 113 lanes of vector registers and back.  Map's rows 9.7 -> 8.7 us, the others 28.9 / 28.9 and
// 17.0 / 16.7.  Exact products of three targets where three are left, not four with one of them twice: no faster, left out.
// Compiled for four wavefronts per SIMD (128 registers): the decoder shape has
// 3456 discarded rows, one wavefront each, and the chip holds 3072 of them at three per SIMD.
template <int MC, int MODE>   // MC: lower bounds kept per lane (>= sel_m: one lane may hold the m largest of the row)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void corr_cand_rows_kernel(CorrArgs a) {
  __shared__ int cand_j[4][kCandCap];
  const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
  const int row = blockIdx.x * (blockDim.x / kWave) + wv;
  const int64_t b = blockIdx.y;
  if (row >= a.n_disc) return;  // whole wavefront leaves together
  const int n = a.n_keep;
  const int i = a.S[b * a.n_disc + row];
  const int32_t* T = a.T + b * n;
  if ((unsigned)i >= (unsigned)a.N) {
    if (lane == 0) a.edge_cnt[b * a.n_disc + row] = 0;
    return;
  }
  // approximate direct term of the row: the matrix-core cosines, or (FiCoCo-L with the
  // attention correlation) the token's row of the exact head-mean map, delta = 0
  constexpr bool from_map = MODE == kAttnL;
  const float* ct = from_map ? a.abar + (b * a.N + i) * a.map_pitch : a.ct + (b * a.n_disc + row) * n;
  constexpr bool L = MODE == kCosL || MODE == kAttnL;
  const float gam = L ? (float)a.gamma : 1.0f;
  double bd = 0.0, bd_max = 0.0;           // first text rows of the indirect term's bound: asked for ahead of the row itself
  if (L && lane < a.M) {
    bd = a.ttext[(b * a.N + i) * a.M + lane];
    bd_max = a.cmax[b * a.M + lane];
  }
  const float delta = from_map ? 0.0f : a.delta;
  const float NEGF = -__builtin_huge_valf();
  const int64_t split_stride = (int64_t)a.B * a.n_disc * n;

  // One pass of the row: element u of a lane is target c0 + u*64 + lane.  All loads of a pass
  // are independent (the map gather takes the token indices first), absent targets read as -inf.
  float val[kCandKeep];
  auto load_pass = [&](int c0) {
    const int n_u = min(kCandKeep, (n - c0 + kWave - 1) / kWave);   // slots of this pass that hold targets (uniform)
    if (from_map) {
      int jt[kCandKeep];
#pragma unroll
      for (int ub = 0; ub < kCandKeep; ub += 8) {
        if (ub < n_u) {                                              // uniform: groups of 8 slots that hold targets
#pragma unroll
          for (int u = ub; u < ub + 8; ++u) jt[u] = T[min(c0 + u * kWave + lane, n - 1)];    // (past the row: its last target, masked below)
        } else {
#pragma unroll
          for (int u = ub; u < ub + 8; ++u) jt[u] = -1;
        }
      }
#pragma unroll
      for (int ub = 0; ub < kCandKeep; ub += 8) {
        if (ub < n_u) {                                              // uniform
#pragma unroll
          for (int u = ub; u < ub + 8; ++u) val[u] = ct[(unsigned)jt[u] < (unsigned)a.N ? jt[u] : 0];
        } else {
#pragma unroll
          for (int u = ub; u < ub + 8; ++u) val[u] = 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < kCandKeep; ++u) {
        asm volatile("" : "+v"(jt[u]));         // (compared again: the answers of all slots take more scalar registers than there are)
        val[u] = (unsigned)jt[u] < (unsigned)a.N ? val[u] : 0.0f;
      }
    } else {
      // The block is followed by kCandChunk floats of padding, so a pass may read past the end
      // of the row (what it reads there is masked below): one address, constant offsets.
      const float* c = ct + c0 + lane;
#pragma unroll
      for (int ub = 0; ub < kCandKeep; ub += 8) {
        if (ub < n_u) {                                              // uniform: groups of 8 slots that hold targets
#pragma unroll
          for (int u = 0; u < 8; ++u) val[ub + u] = c[(ub + u) * kWave];
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) val[ub + u] = 0.0f;
        }
      }
      // partial sums of the further K ranges, added in order; the loads of up to four ranges
      // are issued together (a range past the last one reads the last again and adds zero)
#pragma unroll 1
      for (int sp0 = 1; sp0 < a.ct_splits; sp0 += 4) {
#pragma unroll
        for (int ub = 0; ub < kCandKeep; ub += 8) {
          if (ub < n_u) {                                            // uniform
            float part[4][8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float* cq = c + (int64_t)min(sp0 + q, a.ct_splits - 1) * split_stride;
#pragma unroll
              for (int u = 0; u < 8; ++u) part[q][u] = cq[(ub + u) * kWave];
            }
            issue_fence();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const bool in = sp0 + q < a.ct_splits;
#pragma unroll
              for (int u = 0; u < 8; ++u) val[ub + u] += in ? part[q][u] : 0.0f;
            }
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kCandKeep; ++u) {
      if (c0 + u * kWave >= n) break;         // uniform: no reader looks at slots past the row
      if (c0 + (u + 1) * kWave > n) {         // uniform: the row's last step
        val[u] = c0 + u * kWave + lane < n ? val[u] : NEGF;
        asm volatile("" : "+v"(val[u]));      // (a branch: as selects for every step, the conditions of all of them are kept)
      }
    }
  };

  // The largest approximate values: a descending list per lane (one median per entry and value), then m
  // pops of the wavefront maximum; the m-th as a lower bound of an exact value is lambda.
  float top[MC];
#pragma unroll
  for (int k = 0; k < MC; ++k) top[k] = NEGF;
  for (int c0 = 0; c0 < n; c0 += kCandChunk) {
    load_pass(c0);
#pragma unroll
    for (int u = 0; u < kCandKeep; ++u) {
      if (c0 + u * kWave >= n) break;           // uniform: slots past the row hold nothing
#pragma unroll
      for (int k = MC - 1; k > 0; --k) top[k] = __builtin_amdgcn_fmed3f(top[k - 1], top[k], val[u]);
      top[0] = __builtin_amdgcn_fmed3f(top[0], val[u], __builtin_huge_valf());   // the larger one
    }
  }
  float extra = 0.0f;                      // upper bound of (1 - gamma) * indirect term of this row
  if (L) {
    bd *= bd_max;
    for (int k = lane + kWave; k < a.M; k += kWave) bd += a.ttext[(b * a.N + i) * a.M + k] * a.cmax[b * a.M + k];
    bd = wave_sum_f64(bd) * a.invM * (1.0 - a.gamma);
    extra = (float)bd * 1.000001f + 1e-30f;   // rounded up
  }
  auto lower = [&](float v) { return v == NEGF ? NEGF : gam * fmaxf(v - delta, 0.0f); };     // (grows with v)
  float lambda = NEGF, lambda_k = NEGF;
  for (int r = 0; r < a.sel_m; ++r) {
    const float mx = wave_max(top[0]);
    const unsigned long long who = __ballot(top[0] == mx);
    if (lane == __ffsll(who) - 1) {
#pragma unroll
      for (int k = 0; k + 1 < MC; ++k) top[k] = top[k + 1];
      top[MC - 1] = NEGF;
    }
    lambda = lower(mx);
    if (r + 1 == a.top_k) lambda_k = lambda;
  }
  // Smallest approximate value whose upper bound, gam * max(v + delta, 0) * 1.000001 + extra, reaches
  // `least`: rounded down by more than the roundings on the way can add up to.  (Absent targets hold
  // -inf and never qualify.)
  auto qualifying = [&](float least) {
    const float want = least - extra - 4e-7f * (fabsf(least) + extra);
    if (!(want > 0.0f)) return -3.0e38f;
    const float v = want / (gam * 1.000001f);
    return v - v * 4e-7f - delta * 1.000001f;
  };
  // Candidates in ascending target order (a row of one pass is still in registers): targets whose upper
  // bound reaches a lower bound.  First try: if exactly top_k targets reach the top_k-th largest
  // lower bound (less a margin), every other value of the row lies below theirs by more than the
  // margin: tau falls into that gap and the targets are known without a single exact value.  One
  // target's weight is one whatever its value (positive: its lower bound is); several need their
  // values, but nobody else's.  Otherwise every target that could be among the sel_m largest.
  int n_cand = 0;
  bool known = false;
#pragma unroll 1
  for (int attempt = a.top_k > 0 && lambda_k > 0.0f ? 0 : 1; attempt < 2 && !known; ++attempt) {     // uniform
    const float least = qualifying(attempt == 0 ? lambda_k * 0.99999f : lambda);
    n_cand = 0;
    for (int c0 = 0; c0 < n; c0 += kCandChunk) {
      if (n > kCandChunk) load_pass(c0);
#pragma unroll
      for (int u = 0; u < kCandKeep; ++u) {
        if (c0 + u * kWave >= n) break;           // uniform
        const bool is = val[u] >= least;
        const unsigned long long m = __ballot(is);
        if (m == 0) continue;                     // uniform
        if (is) {
          const int slot = n_cand + __popcll(m & ((1ULL << lane) - 1ULL));
          if (slot < kCandCap) cand_j[wv][slot] = c0 + u * kWave + lane;
        }
        n_cand += __popcll(m);
      }
    }
    known = attempt == 0 && n_cand == a.top_k;
  }
  if (n_cand > kCandCap) {       // uniform per wavefront
    corr_row_exact(a, b, row, lane);
    return;
  }
  // exact values of the candidates: lane c keeps candidate c
  const double NEG = -__builtin_huge_val();
  const int myjj = lane < n_cand ? cand_j[wv][lane] : -1;
  const int myj = myjj >= 0 ? T[myjj] : -1;
  double myv = known && lane == 0 ? 1.0 : NEG;     // (a single target: any positive value gives weight one)
  for (int c = 0; c < (known && a.top_k == 1 ? 0 : n_cand); c += kCandBatch) {
    int j[kCandBatch];
    bool ok[kCandBatch];
#pragma unroll
    for (int q = 0; q < kCandBatch; ++q) {
      const int jq = lane_value(myj, min(c + q, n_cand - 1));
      ok[q] = (unsigned)jq < (unsigned)a.N;
      j[q] = ok[q] ? jq : i;                   // a valid row to read; the value is dropped
    }
    double v[kCandBatch];
    corr_values_wave<kCandBatch, MODE>(a, b, i, j, lane, v);
#pragma unroll
    for (int q = 0; q < kCandBatch; ++q)
      if (lane == c + q && c + q < n_cand) myv = ok[q] ? v[q] : NEG;
  }
  // v[f], v[f+1] = m-th and (m-1)-th largest of the exact candidate values
  double v_f = NEG, v_f1 = NEG;
  int n_gt = 0;
  if (!known) {                    // uniform; (known targets need no threshold)
    double act = myv;
    for (int r = 0; r < a.sel_m; ++r) {
      const double mx = wave_max(act);
      const unsigned long long who = __ballot(act == mx);
      if (lane == __ffsll(who) - 1) act = NEG;
      if (r == 0 || mx < v_f) n_gt = r;
      v_f1 = v_f;
      v_f = mx;
    }
    if (a.sel_m == 1) v_f1 = v_f;
  }
  const double tau = threshold_of(v_f, v_f1, a.sel_g);
  const int tie_quota = a.fixed_k > 0 ? a.sel_m - n_gt : 0x7fffffff;
  const bool is_eq = myjj >= 0 && myv == tau;
  const int eq_rank = __popcll(__ballot(is_eq) & ((1ULL << lane) - 1ULL));   // candidates are in ascending target order
  unsigned long long hit = __ballot(myjj >= 0 && (known || myv > tau || (is_eq && eq_rank < tie_quota)));
  const int cnt = __popcll(hit);
  const int my_pos = __popcll(hit & ((1ULL << lane) - 1ULL));
  const bool mine = (hit >> lane) & 1ULL;
  double denom = 0.0;
  while (hit) {                       // ascending target order
    const int l = __ffsll(hit) - 1;
    hit &= hit - 1;
    denom += lane_value(myv, l);
  }
  const bool live = denom > 0.0;
  const int stored = cnt < a.k_max ? cnt : a.k_max;
  const int64_t ebase = (b * a.n_disc + row) * a.k_max;
  if (live && mine && my_pos < stored) {
    const double al = myv / denom;
    a.edge_tgt[ebase + my_pos] = myjj;
    a.edge_alpha[ebase + my_pos] = al;
    emit_edge(a, b, row, i, myjj, al);
  }
  if (lane == 0) {
    a.edge_cnt[b * a.n_disc + row] = live ? stored : 0;
    if (live && cnt > a.k_max) a.overflow[b] = 1;
  }
}

// ---- FiCoCo-V attention correlation ------------------------------------------------------------
// C[i][j] = Pbar[j][i] (Algorithm 1, stage 2).  The head-mean map is stored transposed, so the
// values of discarded token i are one contiguous row; slot_of tells which of its entries belong
// to preserved tokens.  One wavefront per discarded token: one pass keeps each lane's MC largest
// (value, slot) pairs, the m-th and (m-1)-th largest of the row (with multiplicity) are popped
// off the lanes' lists, and the targets at or above the threshold are taken from the lists in
// ascending order; the row is read a second time only if some lane's list could not hold all
// of its targets.  Values are compared as the floats they are stored as.
// kRowBatch = 64-entry steps of the row loaded together; a row that fits one batch stays in
// registers for the second pass (10 steps: the 576-token grid).  Longer rows take batches of
// kRowWide steps (measured at 2880 tokens: 16 is as good as 24, and 48 -- the whole row in
// registers, at a quarter of the resident wavefronts -- is slower).
constexpr int kRowWide = 16;
template <int MC, int kRowBatch>
__global__ __launch_bounds__(256) void corr_attn_rows_kernel(CorrArgs a) {
  const int lane = threadIdx.x % kWave;
  const int row = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t b = blockIdx.y;
  if (row >= a.n_disc) return;                 // whole wavefront leaves together
  const int i = a.S[b * a.n_disc + row];
  if ((unsigned)i >= (unsigned)a.N) {          // index sets are device data
    if (lane == 0) a.edge_cnt[b * a.n_disc + row] = 0;
    return;
  }
  const float* mrow = a.abar + (b * a.N + i) * a.map_pitch;
  const int32_t* slot_of = a.slot_of + b * a.N;
  const float NEGF = -__builtin_huge_valf();

  // One batch of the row: entry u of a lane is query token r0 + 64 u + lane; entries past the
  // row or of discarded tokens read as -inf with slot -1.
  float vv[kRowBatch];
  int sv[kRowBatch];
  auto load_batch = [&](int r0) {
    // Rows of the map are padded to whole 64-entry steps and the slot table by one step, so the
    // steps that begin inside the row are read as they are (one address, constant offsets) and
    // masked below; steps that begin past the row are skipped.
    const int n_u = min(kRowBatch, (a.N - r0 + kWave - 1) / kWave);      // steps of this batch that begin inside the row
    const float* mp = mrow + r0 + lane;
    const int32_t* sp = slot_of + r0 + lane;
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      vv[u] = 0.0f;
      sv[u] = -1;
      if (u < n_u) {                                       // uniform (a scalar branch): nothing is read past the row's last step
        vv[u] = mp[u * kWave];
        sv[u] = sp[u * kWave];
      }
    }
    issue_fence();
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const bool ok = r0 + u * kWave + lane < a.N && sv[u] >= 0;
      vv[u] = ok ? vv[u] : NEGF;
      sv[u] = ok ? sv[u] : -1;
    }
  };

  float top[MC];
  int topj[MC];
#pragma unroll
  for (int k = 0; k < MC; ++k) { top[k] = NEGF; topj[k] = -1; }
  for (int r0 = 0; r0 < a.N; r0 += kRowBatch * kWave) {
    load_batch(r0);
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      float v = vv[u];
      int jq = sv[u];
#pragma unroll
      for (int k = 0; k < MC; ++k) {
        const bool sw = v > top[k];
        const float t = top[k];
        const int tj = topj[k];
        top[k] = sw ? v : t;
        topj[k] = sw ? jq : tj;
        v = sw ? t : v;
        jq = sw ? tj : jq;
      }
    }
  }
  // v[f], v[f+1]: pop the wavefront maximum m times (MC >= m, so one lane may hold them all)
  float vf = NEGF, vf1 = NEGF;
  int n_gt = 0;                                // pops strictly above vf
  int head = 0;                                // entries of this lane's list popped so far (the lists stay as they are)
  for (int r = 0; r < a.sel_m; ++r) {
    float cur = NEGF;
#pragma unroll
    for (int k = 0; k < MC; ++k) cur = k == head ? top[k] : cur;
    const float mx = wave_max(cur);
    const unsigned long long who = __ballot(cur == mx);
    if (lane == __ffsll(who) - 1) ++head;
    if (r == 0 || mx < vf) n_gt = r;
    vf1 = vf;
    vf = mx;
  }
  if (a.sel_m == 1) vf1 = vf;
  const double tau = threshold_of((double)vf, (double)vf1, a.sel_g);
  const int tie_quota = a.fixed_k > 0 ? a.sel_m - n_gt : 0x7fffffff;   // values equal to tau that are taken
  int ties_seen = 0;
  // a float at or below tau: v >= tau_below is a cheap necessary condition for (double)v >= tau
  float tau_below = (float)tau;
  if ((double)tau_below > tau) {             // rounded up: step to the next float below (finite here)
    const uint32_t u = __float_as_uint(tau_below);
    tau_below = tau_below > 0.0f ? __uint_as_float(u - 1u) : (tau_below < 0.0f ? __uint_as_float(u + 1u) : -1.401298464e-45f);
  }

  // Emit the targets in ascending order; lane e ends up holding edge e (k_max <= 64 on this path).
  int cnt = 0;
  double denom = 0.0;
  int my_tgt = -1;
  double my_c = 0.0;
  // A lane whose whole list is at or above tau may have seen more such values than it kept: only
  // then is the row read again.  Otherwise every target is in some lane's list, and the lists
  // are emptied in ascending slot order (slots are distinct) by repeated minimum search.
  const bool list_full = topj[MC - 1] >= 0 && (double)top[MC - 1] >= tau;
  const bool reread = __any(list_full);
  if (!reread) {
    bool open[MC];
#pragma unroll
    for (int k = 0; k < MC; ++k) open[k] = topj[k] >= 0 && (double)top[k] >= tau;
    for (;;) {
      int mine = 0x7fffffff, mk = 0;
#pragma unroll
      for (int k = 0; k < MC; ++k)
        if (open[k] && topj[k] < mine) { mine = topj[k]; mk = k; }
      const int mn = wave_reduce(mine, [](int x, int y) { return y < x ? y : x; });
      if (mn == 0x7fffffff) break;                               // uniform
      const bool owner = mine == mn;
      float vo = 0.0f;
#pragma unroll
      for (int k = 0; k < MC; ++k) {
        if (owner && k == mk) { vo = top[k]; open[k] = false; }
      }
      const int l = __ffsll(__ballot(owner)) - 1;
      const double cl = (double)lane_value(vo, l);
      const bool is_eq = cl == tau;
      const bool take = cl > tau || (is_eq && ties_seen < tie_quota);
      ties_seen += is_eq ? 1 : 0;
      if (take) {
        denom += cl;
        if (lane == cnt) { my_tgt = mn; my_c = cl; }
        ++cnt;
      }
    }
  }
  for (int r0 = 0; reread && r0 < a.N; r0 += kRowBatch * kWave) {
    if (a.N > kRowBatch * kWave || r0 > 0) load_batch(r0);     // a row of one batch is still in registers
    bool some = false;                                           // most batches hold no target at all
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) some |= sv[u] >= 0 && vv[u] >= tau_below;
    if (!__any(some)) continue;
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      if (r0 + u * kWave >= a.N) break;                          // uniform; nothing is loaded past this point
      const double c = (double)vv[u];
      const bool in = sv[u] >= 0;
      const bool is_eq = in && c == tau;
      const unsigned long long eqm = __ballot(is_eq);
      const int eq_rank = ties_seen + __popcll(eqm & ((1ULL << lane) - 1ULL));
      ties_seen += __popcll(eqm);
      unsigned long long hit = __ballot(in && (c > tau || (is_eq && eq_rank < tie_quota)));
      while (hit) {
        const int l = __ffsll(hit) - 1;
        hit &= hit - 1;
        const double cl = lane_value(c, l);
        const int tl = lane_value(sv[u], l);
        denom += cl;
        if (lane == cnt) { my_tgt = tl; my_c = cl; }
        ++cnt;
      }
    }
  }
  const int stored = cnt < a.k_max ? cnt : a.k_max;
  const bool live = denom > 0.0;
  const int64_t ebase = (b * a.n_disc + row) * a.k_max;
  if (live && lane < stored) {
    const double al = my_c / denom;
    a.edge_tgt[ebase + lane] = my_tgt;
    a.edge_alpha[ebase + lane] = al;
    emit_edge(a, b, row, i, my_tgt, al);
  }
  if (lane == 0) {
    a.edge_cnt[b * a.n_disc + row] = live ? stored : 0;
    if (live && cnt > a.k_max) a.overflow[b] = 1;
  }
}

// Pairwise token correlation gap: top-1 minus top-2 value of every discarded row, values
// evaluated exactly (one target per lane at a time), counted with multiplicity.
__global__ __launch_bounds__(256) void corr_gap_kernel(CorrArgs a) {
  const int lane = threadIdx.x % kWave;
  const int row = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t b = blockIdx.y;
  if (row >= a.n_disc) return;  // whole wavefront leaves together
  const int n = a.n_keep;
  const int i = a.S[b * a.n_disc + row];
  const double NEG = -__builtin_huge_val();
  double t1 = NEG, t2 = NEG;           // this lane's two largest values
  if ((unsigned)i < (unsigned)a.N) {
    for (int jj = lane; jj < n; jj += kWave) {
      const int j = a.T[b * n + jj];
      if ((unsigned)j >= (unsigned)a.N) continue;
      const double c = corr_value(a, b, i, j);
      if (c > t1) { t2 = t1; t1 = c; }
      else if (c > t2) t2 = c;
    }
  }
  const double m1 = wave_max(t1);
  const unsigned long long who = __ballot(t1 == m1);
  const bool owner = lane == __ffsll(who) - 1;
  const double m2 = wave_max(owner ? t2 : t1);   // the runner-up: the owner's second value or another lane's best
  if (lane == 0) a.gap[b * a.n_disc + row] = (n >= 2 && m2 > NEG) ? m1 - m2 : 0.0;
}

__global__ void zero_i32_kernel(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

template <int MODE>
static void launch_cand_rows(int sel_m, dim3 grid, dim3 block, hipStream_t s, const CorrArgs& a) {
  if (sel_m <= 2) hipLaunchKernelGGL((corr_cand_rows_kernel<2, MODE>), grid, block, 0, s, a);
  else if (sel_m <= 4) hipLaunchKernelGGL((corr_cand_rows_kernel<4, MODE>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((corr_cand_rows_kernel<8, MODE>), grid, block, 0, s, a);
}

static void launch_text_colmax(const ficoco_problem& p, const Plan& pl, char* ws, hipStream_t s) {
  TextStatsArgs t{};
  fill_text_stats(p, pl, ws, true, t);
  hipLaunchKernelGGL(text_colmax_kernel, dim3(t.cmax_blocks, p.B), dim3(256), 0, s, t);
}

GramForm gram_form(const ficoco_problem& p, const Plan& pl) {
  // Estimated us of the three forms (sixteen launches in a row), from the tiles and the 32-feature stages of a K range.  A workgroup of
  // the 192- and 256-row forms has a compute unit to itself: rounds of 256 tiles, and a nearly empty last one, or tiles that
  // are mostly padding, cost as much as full ones.  Of the 128 x 128 tiles three share a compute unit.  us with tiles of
  // 128 / 192 / 256 rows: 8064 x 1152 with 1024 features 37 / 27 / 31 (567, 252 and 192 tiles); 10368 x 1152 39 / 45 / 34 (324 tiles of
  // 192: two rounds); 36 images of 768 x 384 38 / 45 / 32, 44 of them 57 / 46 / 58 (264 tiles of 256: two rounds); 260 of 480 x 96, 128
  // features 20 / 40 / 28 and 180 of 200 x 200 12.7 / 26 / 18 (padding); 128 of 432 x 144, 256 features 21 / 25 / 16.  Several K
  // ranges: 16 images of 768 x 384, 1024 features 23 / 20, with 4096 65 / 45; 8 of 432 x 144, 4096 features 17.3 / 18.3.
  // Over 1565 shapes (20 to 400 images of 50 to 700 rows, 1 to 280 of up to 10368, 128 to 4096 features) the estimate lies within 25 %
  // for more than nine of ten, and the form chosen takes 1.2 % longer than the best one on average.  The usual form, 256 rows
  // where their tiles fill half the chip, else 128, is left only for one estimated 8 % faster: then four of the shapes are more than 3 %
  // slower than with the usual form, at most 11 %; without that margin 38, at most 34 %.
  auto rounds = [&](int rows, int cols) {
    const int64_t tiles = (int64_t)pl.gram_splits * p.B * ((pl.n_disc + rows - 1) / rows) * ((p.n_keep + cols - 1) / cols);
    return (int)std::min<int64_t>((tiles + 255) / 256, 1 << 24);
  };
  const float st = (float)pl.gram_st_per_split;
  const int sq = rounds(kGT, kGT);
  const float square = 2.5f + sq / 3 * (5.5f + st) + (sq % 3 == 0 ? 0.0f : sq % 3 == 1 ? 3.5f + 0.55f * st : 4.5f + 0.75f * st);
  const float wide = 2.0f + rounds(kG2M, kG2N) * (7.0f + 0.56f * st);
  if (pl.gram_splits > 1) return 1.08f * wide < square ? kGramWide : kGramSquare;      // (the 256-row form takes all of K at once)
  const float tall = 0.5f + rounds(kTallM, kG2N) * (6.5f + 0.8f * st);
  const bool usual_tall = (int64_t)p.B * ((pl.n_disc + kTallM - 1) / kTallM) * ((p.n_keep + kG2N - 1) / kG2N) >= 128;
  const GramForm usual = usual_tall ? kGramTall : kGramSquare, other = usual_tall ? kGramSquare : kGramTall;
  const float t_usual = usual_tall ? tall : square, t_other = usual_tall ? square : tall;
  if (1.08f * std::min(wide, t_other) >= t_usual) return usual;
  return wide <= t_other ? kGramWide : other;
}

void launch_correlate(const ficoco_problem& p, const Plan& pl, char* ws, const int32_t* discard_idx,
                      const int32_t* keep_idx, int32_t* edge_cnt, int32_t* edge_tgt,
                      double* edge_alpha, int32_t* overflow, bool fused,
                      hipEvent_t gram_start, hipEvent_t gram_stop, hipStream_t s, int gram_repeat) {
  // fused: called from a fused step, whose filter stage cleared the overflow flags and whose
  // score stage formed the column maxima of the text profiles (text_stats_in_score)
  if (!fused)
    hipLaunchKernelGGL(zero_i32_kernel, dim3((p.B + 255) / 256), dim3(256), 0, s, overflow, p.B);
  const bool need_colmax = !(fused && text_stats_in_score(p));
  if (pl.n_disc == 0) return;
  if (pl.fixed_k == 0) {       // pruning / convergent form: no discarded token has a target
    const int n = p.B * pl.n_disc;
    hipLaunchKernelGGL(zero_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, edge_cnt, n);
    return;
  }
  CorrArgs a{};
  a.B = p.B; a.N = p.N; a.n_keep = p.n_keep; a.n_disc = pl.n_disc; a.M = p.M; a.k_max = p.k_max; a.Df = pl.Df;
  const bool L = p.variant == FICOCO_VARIANT_L;
  a.mode = p.corr_src == FICOCO_C_ATTN ? (L ? kAttnL : kAttnV) : (L ? kCosL : kCosV);
  a.abar = (const float*)(ws + pl.abar);
  a.map_pitch = pl.map_pitch;
  a.ttext = (const double*)(ws + pl.ttext);
  a.xhat = (const bf16_t*)(ws + pl.xhat);
  a.gamma = (double)p.gamma;
  a.invM = p.M > 0 ? 1.0 / (double)p.M : 0.0;
  a.S = discard_idx; a.T = keep_idx;
  a.sel_m = pl.sel_m; a.sel_f = pl.sel_f; a.sel_g = pl.sel_g;
  a.dense = pl.dense_rows ? 1 : 0;
  a.rowbuf = (double*)(ws + pl.rowbuf);
  a.edge_cnt = edge_cnt; a.edge_tgt = edge_tgt; a.edge_alpha = edge_alpha; a.overflow = overflow;
  a.slot_of = (const int32_t*)(ws + pl.slot_of);
  a.ct = (float*)(ws + pl.ct);
  a.cmax = (double*)(ws + pl.cmax);
  a.fixed_k = pl.fixed_k;
  a.ct_splits = pl.gram_splits;
  a.delta = gram_delta(pl);
  // J_i is the top_k largest values where the next one is clear of them: the threshold lies strictly
  // between v[f] and v[f+1] (g well inside (0, 1)), or at v[f] itself (g = 0, fixed K)
  a.top_k = pl.sel_g == 0.0 ? pl.sel_m : (pl.sel_g > 1e-6 && pl.sel_g < 1.0 - 1e-6) ? pl.sel_m - 1 : 0;
  if (fused && pl.bkt_cap > 0) {
    a.bkt_cnt = (int32_t*)(ws + pl.bkt_cnt);
    a.bkt_src = (int32_t*)(ws + pl.bkt_src);
    a.bkt_w = (double*)(ws + pl.bkt_w);
    a.bkt_cap = pl.bkt_cap;
    a.cnt_stride = pl.cnt_stride;
    if (edges_inverted(pl)) {
      a.hub_list = (int32_t*)(ws + pl.hub_list);
      a.hub_cnt = (int32_t*)(ws + pl.hub_cnt);
    }
  }
  dim3 grid((pl.n_disc + 3) / 4, p.B), block(256);
  if (a.mode == kAttnV && !pl.dense_rows && p.k_max <= kWave) {
    const bool wide = p.N > 10 * kWave;     // longer rows: wider batches (fewer dependent trips to memory)
    if (wide) {
      if (pl.sel_m <= 2) hipLaunchKernelGGL((corr_attn_rows_kernel<2, kRowWide>), grid, block, 0, s, a);
      else if (pl.sel_m <= 4) hipLaunchKernelGGL((corr_attn_rows_kernel<4, kRowWide>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((corr_attn_rows_kernel<8, kRowWide>), grid, block, 0, s, a);
    } else {
      if (pl.sel_m <= 2) hipLaunchKernelGGL((corr_attn_rows_kernel<2, 10>), grid, block, 0, s, a);
      else if (pl.sel_m <= 4) hipLaunchKernelGGL((corr_attn_rows_kernel<4, 10>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((corr_attn_rows_kernel<8, 10>), grid, block, 0, s, a);
    }
    return;
  }
  if (a.mode == kAttnL && !pl.dense_rows && p.k_max <= 64) {
    if (need_colmax) launch_text_colmax(p, pl, ws, s);
    launch_cand_rows<kAttnL>(pl.sel_m, grid, block, s, a);
    return;
  }
  if (pl.use_gram) {
    GramArgs g{a.xhat, p.B, p.N, pl.Df, pl.n_disc, p.n_keep, discard_idx, keep_idx, a.ct, pl.gram_splits, pl.gram_st_per_split};
    auto tiles = [&](int rows, int cols) { return pl.gram_splits * p.B * ((pl.n_disc + rows - 1) / rows) * ((p.n_keep + cols - 1) / cols); };
    const GramForm form = gram_form(p, pl);
    if (gram_start) (void)hipEventRecord(gram_start, s);
    // gram_repeat > 1 (measurement only): the same launch again and again between the two events
    for (int rep = 0; rep < gram_repeat; ++rep) {
      if (form == kGramTall) {
        constexpr size_t kLds = (size_t)2 * (kTallM + kG2N) * kG2Chunks * sizeof(uint4);
        (void)hipFuncSetAttribute((const void*)gram_tall_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
        hipLaunchKernelGGL(gram_tall_kernel, dim3(xcd_padded_total(tiles(kTallM, kG2N))), dim3(kTallThreads), kLds, s, g);
      }
      else if (form == kGramWide) hipLaunchKernelGGL(gram_tile2_kernel, dim3(xcd_padded_total(tiles(kG2M, kG2N))), dim3(kG2Threads), 0, s, g);
      else hipLaunchKernelGGL(gram_tile_kernel, dim3(xcd_padded_total(tiles(kGT, kGT))), dim3(256), 0, s, g);
    }
    if (gram_stop) (void)hipEventRecord(gram_stop, s);
    if (L && need_colmax) launch_text_colmax(p, pl, ws, s);
    if (L) launch_cand_rows<kCosL>(pl.sel_m, grid, block, s, a);
    else launch_cand_rows<kCosV>(pl.sel_m, grid, block, s, a);
    return;
  }
  if (pl.dense_rows) hipLaunchKernelGGL(corr_fill_rows_kernel, grid, block, 0, s, a);
  hipLaunchKernelGGL(corr_rows_kernel, grid, block, 0, s, a);
}

void launch_corr_gap(const ficoco_problem& p, const Plan& pl, char* ws, const int32_t* discard_idx,
                     const int32_t* keep_idx, double* gap, hipStream_t s) {
  if (pl.n_disc == 0) return;
  CorrArgs a{};
  a.B = p.B; a.N = p.N; a.n_keep = p.n_keep; a.n_disc = pl.n_disc; a.M = p.M; a.k_max = p.k_max; a.Df = pl.Df;
  const bool L = p.variant == FICOCO_VARIANT_L;
  a.mode = p.corr_src == FICOCO_C_ATTN ? (L ? kAttnL : kAttnV) : (L ? kCosL : kCosV);
  a.abar = (const float*)(ws + pl.abar);
  a.map_pitch = pl.map_pitch;
  a.ttext = (const double*)(ws + pl.ttext);
  a.xhat = (const bf16_t*)(ws + pl.xhat);
  a.gamma = (double)p.gamma;
  a.invM = p.M > 0 ? 1.0 / (double)p.M : 0.0;
  a.S = discard_idx; a.T = keep_idx;
  a.gap = gap;
  hipLaunchKernelGGL(corr_gap_kernel, dim3((pl.n_disc + 3) / 4, p.B), dim3(256), 0, s, a);
}

}  // namespace ficoco

