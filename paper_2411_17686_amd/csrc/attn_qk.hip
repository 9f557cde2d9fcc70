// Attention reduction from queries and keys (Sec. "Self-Attention": A = Softmax(Q K^T / sqrt(D))):
// the per-head maps are formed on the matrix cores and reduced on the fly, so the [B,H,n,n]
// maps never exist in memory.  Outputs are those of attn_reduce.hip -- per-tile column partials of
// the received attention (first term of Eq. 1), the [CLS] row (second term), the head-mean map
// in single precision, transposed, for the correlate stage (Algorithm 1, stage 2), and for FiCoCo-L
// (causal maps) the text profiles of Eq. 3 / Eq. 4.
//
// Two kernels (before: one workgroup per 48 query rows that exchanged maxima and sums between its
// wavefronts head by head; whole stage 81 -> 70 us at 16 x 577 tokens, 590 -> 290 us at 4 x 2881, 361 -> 98 us
// at the causal 8 x 675): qk_norm_kernel leaves (reference, 1 / row sum) of every (head, query) row, and
// qk_mean_kernel forms the probabilities of one (query tile, key tile) from them, adds the heads in
// registers and writes the tile's outputs.  The logits are computed twice, but once the normalisers
// are known nothing ties the keys of a row together: wavefronts exchange neither maxima nor sums, and
// the work can be cut to fill the chip whatever the numbers of queries, keys and heads are.
//
// Single precision (products of bfloat16 values are exact in it), row sums and column sums in double.
#include "common.hpp"

#include <algorithm>

namespace ficoco {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kQkWaves = 4;                         // wavefronts side by side on the queries, a tile each
constexpr int kQkQB = kQkTile / 16;                 // 16-query blocks of a wavefront
constexpr int kQkKB = 2;                            // 16-key blocks a wavefront takes together
constexpr int kQkKeys = 64;                         // keys staged together: two such steps, or one of each of two wavefronts
static_assert(kQkKeys == 2 * kQkKB * 16, "two steps of keys");
static_assert(kQkTile % 16 == 0, "whole 16-query blocks");

struct QkArgs {
  const bf16_t* Q;
  const bf16_t* K;
  int64_t sb, sh, sn;
  int H, n;             // heads, rows of the block
  int N;                // visual tokens
  int vis0;             // block row of visual token 0
  // The queries that are needed, numbered 0 .. nq: the n_visq visual ones (all or none), then the
  // others from block row x0 on: the [CLS] query (FiCoCo-V) or the text queries (FiCoCo-L).
  int nq, n_visq, x0;
  float scale_log2e;    // qk_scale * log2(e): exponentials are taken as powers of two
  float2* norm;         // [images of this launch][H][nq]: reference, 1 / (row sum relative to it)
  float* abar;          // [B][N][map_pitch] or null
  int map_pitch;
  double* recv_part;    // [B][n_tiles][N] or null
  double* cls;          // [B][N] or null
  double* ttext;        // FiCoCo-L: [B][N][M] head-mean attention of the text queries on the visual keys, or null
  int M;
  int n_tiles;          // query tiles that hold visual queries
  int b0, nb;           // images of this launch
  int q_groups, k_tiles; // workgroups of one image: query tiles or groups of them, key tiles
  bool share_keys;      // row normalisers: one query tile per workgroup, whose wavefronts share its keys
  __device__ __forceinline__ int row(int v) const { return v < n_visq ? vis0 + v : x0 + (v - n_visq); }
};

// v_mfma_f32_16x16x32_bf16: operand A is 16 rows x 32 features (lane: row lane % 16, features
// 8 (lane / 16) .. + 8), operand B 16 columns x 32 features (same), the result 16 x 16 (lane: column
// lane % 16, rows 4 (lane / 16) + v for its four registers v).  Rows are keys here, columns queries:
// a query's logits sit in the registers of four lanes, and sixteen lanes hold consecutive queries of one
// key, which is a piece of a row of the transposed map.

// A lane's 16-byte operand loads from global memory would touch a row of its own in every lane, and
// the address unit takes such a load apart into 64 accesses (measured: it was busy 74 % of the time
// and bound both kernels).  So rows are brought in whole -- neighbouring lanes on neighbouring 16-byte
// chunks -- and turned into operands through LDS.  CH chunks per row; the chunk of row r lies at
// chunk ^ swizzle, which spreads the sixteen rows of an operand read over all 64 banks.
template <int CH>
__device__ __forceinline__ int lds_chunk(int r, int c) { return r * CH + (c ^ ((r / (16 / CH)) & (CH - 1))); }

// ---- row normalisers ---------------------------------------------------------------------------
// A workgroup takes 4 x 48 queries of one head and walks its keys 64 at a time, the next 64 being
// loaded while the current ones are added (few workgroups: 48 queries, the keys shared by its wavefronts).  The exponentials are taken relative to a whole number
// (units of log2) at the largest logit of the first 32 keys, not of the whole row: any reference
// serves as long as nothing overflows, and then the sums need no running maximum.  A row whose sum
// does overflow (its largest logit more than ~70 above those of the first 32 keys) is seen in the
// sum and done again with its own maximum.
//
// Bound by the vector unit: exponential, multiply-add and add per logit, and by the matrix instructions, which hardly
// run beside them (4 x 2881 tokens, 16 heads of 64: 112 us; with operands straight from memory 165-205 us).
template <int KS, bool DEC>
__global__ __launch_bounds__(kQkWaves * kWave) __attribute__((amdgpu_waves_per_eu(2))) void qk_norm_kernel(QkArgs a) {
  constexpr int CH = KS * 4, T = kQkWaves * kWave, RPI = T / CH, NL = kQkKeys / RPI;
  __shared__ u32x4_t stage[2][kQkKeys * CH];
  // The workgroups of a head share an L2 (its keys).  The last ones of the heads, if they are narrow, come behind all
  // others: in their places between them they left every q_groups-th compute unit without work (a quarter of the chip at
  // 16 x 577 tokens: 29.8 us, and 24.3 with the order of precedence below).
  const bool last_narrow = a.nq - (a.q_groups - 1) * (a.share_keys ? 1 : kQkWaves) * kQkTile <= 16;
  const int groups = a.q_groups - (last_narrow ? 1 : 0), units = a.nb * a.H * groups, first = xcd_padded_total(units);
  const bool behind = (int)blockIdx.x >= first;
  const int unit = xcd_logical_id(behind ? blockIdx.x - first : blockIdx.x, behind ? a.nb * a.H : units);
  if (unit >= (behind ? a.nb * a.H : units)) return;
  const int tid = threadIdx.x, lane = tid % kWave, l16 = lane % 16, lg = lane / 16;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int in_head = behind ? groups : unit % groups, head = behind ? unit : unit / groups;
  const int w0 = in_head * (a.share_keys ? 1 : kQkWaves) * kQkTile;
  const bool narrow = a.nq - w0 <= 16;     // one block of queries in all (the [CLS] query behind 576 visual ones)
  const bool share_keys = a.share_keys || narrow;
  const int v0 = share_keys ? w0 : w0 + wv * kQkTile;
  const int h = head % a.H;
  const int64_t bi = head / a.H;
  const float NEG = -__builtin_huge_valf();
  const bf16_t* Qh = a.Q + (a.b0 + bi) * a.sb + (int64_t)h * a.sh;
  const bf16_t* Kh = a.K + (a.b0 + bi) * a.sb + (int64_t)h * a.sh;
  // keys below full_end count for every query of this wavefront, from k_end on for none
  const bool active = v0 < a.nq;
  const int q_lo = a.row(min(v0, a.nq - 1)), q_hi = a.row(min(v0 + kQkTile, a.nq) - 1);
  const int k_end = !active ? 0 : DEC ? min(a.n, q_hi + 1) : a.n;
  const int full_end = DEC ? min(a.n, q_lo + 1) : a.n;
  const int wg_end = DEC ? min(a.n, a.row(min(w0 + kQkWaves * kQkTile, a.nq) - 1) + 1) : a.n;

  int qrow[kQkQB];
  bf16x8_t qf[kQkQB][KS];
#pragma unroll
  for (int qb = 0; qb < kQkQB; ++qb) {
    qrow[qb] = a.row(min(v0 + qb * 16 + l16, a.nq - 1));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) __builtin_memcpy(&qf[qb][ks], Qh + (int64_t)qrow[qb] * a.sn + lg * 8 + ks * 32, 16);
  }

  u32x4_t next[NL];
  auto load_stage = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      __builtin_memcpy(&next[i], Kh + (int64_t)min(k0 + tid / CH + i * RPI, a.n - 1) * a.sn + tid % CH * 8, 16);
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NL; ++i) stage[buf][lds_chunk<CH>(tid / CH + i * RPI, tid % CH)] = next[i];
  };

  typedef f32x4_t Logits[kQkKB][kQkQB];      // of 32 keys
  Logits S;
  // `key_op(kb, ks)` gives this lane's operand
  auto logits = [&](auto qbn, auto key_op, Logits& S) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
#pragma unroll
    for (int kb = 0; kb < kQkKB; ++kb) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8_t kf = key_op(kb, ks);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          S[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[qb][ks], ks == 0 ? f32x4_t{0.0f, 0.0f, 0.0f, 0.0f} : S[kb][qb], 0, 0, 0);
      }
    }
  };
  auto counts = [&](int key, int qb) { return key < a.n && (!DEC || key <= qrow[qb]); };
  // the largest logit of the 32 keys from k0 on that count, and of the four lanes of a query
  float ref[kQkQB];
  double sum[kQkQB];
  auto max_of = [&](auto qbn, int k0) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int kb = 0; kb < kQkKB; ++kb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          ref[qb] = fmaxf(ref[qb], counts(k0 + kb * 16 + lg * 4 + v, qb) ? S[kb][qb][v] : NEG);
  };
  auto set_ref = [&](auto qbn) __attribute__((always_inline)) {       // (key 0 counts for every query, so the maximum is a logit)
    constexpr int QB = decltype(qbn)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      ref[qb] = fmaxf(ref[qb], __shfl_xor(ref[qb], 16, kWave));
      ref[qb] = fmaxf(ref[qb], __shfl_xor(ref[qb], 32, kWave));
      ref[qb] = ceilf(ref[qb] * a.scale_log2e);
    }
  };
  auto add_whole = [&](auto qbn, const Logits& S) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float part;
#pragma unroll
      for (int kb = 0; kb < kQkKB; ++kb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float e = __builtin_amdgcn_exp2f(fmaf(S[kb][qb][v], a.scale_log2e, -ref[qb]));
          part = kb == 0 && v == 0 ? e : part + e;
        }
      sum[qb] += (double)part;
    }
  };
  auto add_chunk = [&](auto qbn, int k0, const Logits& S) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
    if (k0 + kQkKB * 16 <= full_end) {               // uniform
      add_whole(qbn, S);
    } else {
#pragma unroll
      for (int kb = 0; kb < kQkKB; ++kb)
        if (k0 + kb * 16 < k_end) {                  // uniform
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            float part = 0.0f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const float x = counts(k0 + kb * 16 + lg * 4 + v, qb) ? fmaf(S[kb][qb][v], a.scale_log2e, -ref[qb]) : NEG;
              part += __builtin_amdgcn_exp2f(x);
            }
            sum[qb] += (double)part;
          }
        }
    }
  };
  auto across = [&]() {
#pragma unroll
    for (int qb = 0; qb < kQkQB; ++qb) {
      sum[qb] += __shfl_xor(sum[qb], 16, kWave);
      sum[qb] += __shfl_xor(sum[qb], 32, kWave);
    }
  };
#pragma unroll
  for (int qb = 0; qb < kQkQB; ++qb) { ref[qb] = NEG; sum[qb] = 0.0; }

  const std::integral_constant<int, kQkQB> all{};
  auto direct = [&](int k0) {
    return [&, k0](int kb, int ks) {
      bf16x8_t kf;
      __builtin_memcpy(&kf, Kh + (int64_t)min(k0 + kb * 16 + l16, a.n - 1) * a.sn + lg * 8 + ks * 32, 16);
      return kf;
    };
  };
  bool over = false;
  // Each wavefront every fourth 32 keys, with a reference of its own; the four sums are combined in order.
  __shared__ float part_ref[kQkWaves][kQkTile];
  __shared__ double part_sum[kQkWaves][kQkTile];
  auto shared_keys = [&](auto qbn) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
    const int first = wv * kQkKB * 16;
#pragma unroll 1
    for (int k0 = first; k0 < k_end; k0 += kQkWaves * kQkKB * 16) {
      logits(qbn, direct(k0), S);
      if (k0 == first) { max_of(qbn, k0); set_ref(qbn); }     // (-inf where none of them counts: then none of the later ones does)
      add_chunk(qbn, k0, S);
    }
    across();
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      if (lg == 0) { part_ref[wv][qb * 16 + l16] = ref[qb]; part_sum[wv][qb * 16 + l16] = sum[qb]; }
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      for (int w = 0; w < kQkWaves; ++w) ref[qb] = fmaxf(ref[qb], part_ref[w][qb * 16 + l16]);
      sum[qb] = 0.0;
      for (int w = 0; w < kQkWaves; ++w) {
        const float r = part_ref[w][qb * 16 + l16];
        const double t = part_sum[w][qb * 16 + l16];
        over |= !(t < 0x1p100);
        sum[qb] += r > NEG ? ldexp(t, (int)fmaxf(r - ref[qb], -3000.0f)) : 0.0;
      }
    }
  };
  if (share_keys) {                                  // uniform in the workgroup
    if (narrow) shared_keys(std::integral_constant<int, 1>{});
    else shared_keys(all);
    if (wv != 0) return;
  } else {
    // The oldest wavefront of a SIMD is served first (of the four on one at 4 x 2881 tokens they ended at 58, 80, 104
    // and 128 us), and the last one is left alone with its trips through LDS and the matrix unit.  So the wavefronts with
    // most keys left take precedence, down to an eighth of the keys (110 to 120 us then).  Causal maps: wavefronts differ
    // in length and end one after the other anyway (47 us for 8 x 675 tokens, 54 with precedence).
    int level = 4;
    load_stage(0);
    store_stage(0);
    __syncthreads();
#pragma unroll 1
    for (int k0 = 0; k0 < wg_end; k0 += kQkKeys) {
      const int left = k_end - k0, now = (left > a.n / 2 ? 1 : 0) + (left > a.n / 4 ? 1 : 0) + (left > a.n / 8 ? 1 : 0);
      if (!DEC && now != level) {                      // uniform
        level = now;
        if (now == 3) __builtin_amdgcn_s_setprio(3);
        else if (now == 2) __builtin_amdgcn_s_setprio(2);
        else if (now == 1) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
      const int buf = k0 / kQkKeys % 2;
      load_stage(k0 + kQkKeys);       // on their way while the current keys are added (past the end: the last row)
      issue_fence();
      const bf16x8_t* st = (const bf16x8_t*)stage[buf];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (k0 + half * kQkKB * 16 >= k_end) continue;   // uniform
        logits(all, [&](int kb, int ks) { return st[lds_chunk<CH>((half * kQkKB + kb) * 16 + l16, ks * 4 + lg)]; }, S);
        if (half == 0 && k0 == 0) { max_of(all, 0); set_ref(all); }
        add_chunk(all, k0 + half * kQkKB * 16, S);
      }
      store_stage(1 - buf);
      __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
    if (!active) return;
    across();
#pragma unroll
    for (int qb = 0; qb < kQkQB; ++qb) over |= !(sum[qb] < 0x1p100);
  }
  if (__any(over)) {                                 // rare: with the row's own maximum, keys straight from memory
#pragma unroll
    for (int qb = 0; qb < kQkQB; ++qb) { ref[qb] = NEG; sum[qb] = 0.0; }
#pragma unroll 1
    for (int k0 = 0; k0 < k_end; k0 += kQkKB * 16) { logits(all, direct(k0), S); max_of(all, k0); }
    set_ref(all);
#pragma unroll 1
    for (int k0 = 0; k0 < k_end; k0 += kQkKB * 16) { logits(all, direct(k0), S); add_chunk(all, k0, S); }
    across();
  }
#pragma unroll
  for (int qb = 0; qb < kQkQB; ++qb) {
    const int v = v0 + qb * 16 + l16;
    if (lg == 0 && v < a.nq) a.norm[((int64_t)bi * a.H + h) * a.nq + v] = make_float2(ref[qb], (float)(1.0 / sum[qb]));
  }
}

// The value of lane ^ 4: rows shifted by four lanes up for the first quad of a pair, down for the second.
__device__ __forceinline__ int lane_xor_4(int v) {
  const int up = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false);      // row_shl:4 into quads 0 and 2
  return __builtin_amdgcn_update_dpp(up, v, 0x114, 0xF, 0xA, false);             // row_shr:4 into quads 1 and 3
}
// Eight values of every lane, each summed over the 16 lanes of a row: the tree of the four steps lane ^ 1, ^ 2, ^ 4,
// ^ 8.  Every step hands half of the values to the other lane of the pair, so lane l is left with value
// 4 (l & 1) + (l & 2) + (l >> 2 & 1) alone: 15 additions instead of 32.
__device__ __forceinline__ double row_sums_of_8(const double (&x)[8], int l16) {
  auto pick = [](bool second, double a, double b) { return second ? b : a; };
  double y[4], z[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] = pick(l16 & 1, x[i], x[i + 4]) + dpp_move<0xB1>(pick(l16 & 1, x[i + 4], x[i]));
#pragma unroll
  for (int i = 0; i < 2; ++i) z[i] = pick(l16 & 2, y[i], y[i + 2]) + dpp_move<0x4E>(pick(l16 & 2, y[i + 2], y[i]));
  const double give = pick(l16 & 4, z[1], z[0]);
  const double u = pick(l16 & 4, z[0], z[1]) + __hiloint2double(lane_xor_4(__double2hiint(give)), lane_xor_4(__double2loint(give)));
  return u + dpp_move<0x128>(u);      // rotated by eight: lane ^ 8
}

// ---- probabilities, head mean, outputs -----------------------------------------------------------
// A wavefront forms 48 queries x 32 visual keys of an image, the heads added in order in registers.
// SPLIT = false: the four wavefronts of a workgroup sit two by two on 96 queries x 64 keys and
// share the staged rows.  SPLIT = true (few tiles): 48 x 64 by two wavefronts, and four such pairs
// take consecutive shares of the heads, each with a staging area of its own; their sums are added
// pairwise (a fixed tree) in LDS.  Rows are staged 64 features at a time in two buffers, loaded into
// registers two stages ahead; the exponentials of a head are computed beside the matrix
// instructions and LDS reads of the next one, in a fixed order.  The normalisers of a head come through LDS
// as well (each wavefront reading its own took 30 % of the address unit's time).
//
// Bound by the vector unit (exponential, two multiply-adds per logit) and the trips between
// barriers.  Measured at 4 x 2881 tokens, 16 heads of 64 / 16 x 577, 16 of 64 / 8 x 675 causal, 32
// of 128: operands straight from memory 314 / 70 / 99 us; staged, 192 x 64 by eight wavefronts, each head
// on its own 180 / 44 / 56; the next head's matrix instructions under this head's exponentials, 96 x 64 by
// four wavefronts (three workgroups on a compute unit instead of two) 170 / 40 / 51; normalisers through LDS, whole
// tiles written without tests, exponentials between the other instructions 154 / 33.5 / 49.  With heads of 32 four fit if the
// registers are held to 128 (131 otherwise): step of 16 x 577 tokens, 16 heads 77.9 -> 74.1 us, one head 46.0 -> 43.3.
constexpr int kQkBand = 8;                          // key tiles side by side in the order of the workgroups
constexpr int kQkCols = 2;                          // wavefronts side by side on the keys
constexpr int kQkMB = kQkKeys / 16 / kQkCols;       // 16-key blocks of a wavefront
template <bool SPLIT> struct QkMeanShape {
  static constexpr int kRows = SPLIT ? 1 : 2;         // wavefronts side by side on the queries
  static constexpr int kShares = SPLIT ? 4 : 1;       // shares of the heads
  static constexpr int kThreads = kRows * kQkCols * kShares * kWave;
};
template <int KS, bool DEC, bool SPLIT>
__global__ __launch_bounds__(QkMeanShape<SPLIT>::kThreads) __attribute__((amdgpu_waves_per_eu(SPLIT || KS == 4 ? 2 : KS == 1 ? 4 : 3))) void qk_mean_kernel(QkArgs a) {
  constexpr int KSS = KS > 2 ? 2 : KS, NST = KS / KSS, CH = KSS * 4;     // 32-feature steps of a stage, stages of a head
  using Shape = QkMeanShape<SPLIT>;
  constexpr int QR = Shape::kRows * kQkTile;                              // query rows of a stage
  constexpr int T = Shape::kRows * kQkCols * kWave, RPI = T / CH;
  constexpr int NL = (QR + kQkKeys + RPI - 1) / RPI;                      // rounds of RPI rows (past the last key: that key again)
  extern __shared__ u32x4_t stage_m[];                 // [2][SPLIT ? 4 : 1][rounded-up rows of a stage], then the queries' normalisers
  constexpr int kArea = NL * RPI * CH;
  const int units = a.nb * a.q_groups * a.k_tiles;
  const int unit = xcd_logical_id(blockIdx.x, units);
  if (unit >= units) return;
  const int tid = threadIdx.x, lane = tid % kWave, l16 = lane % 16, lg = lane / 16;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int share = SPLIT ? wv / kQkCols : 0;                // of the heads
  // the tiles of an image in columns kQkBand key tiles wide: the workgroups that run together on an
  // XCD then need few rows of either side, which its L2 holds for all heads
  const int64_t bi = unit / (a.k_tiles * a.q_groups), b = a.b0 + bi;
  const int in_img = unit - (int)bi * a.k_tiles * a.q_groups;
  const int band = in_img / (kQkBand * a.q_groups), in_band = in_img - band * kQkBand * a.q_groups;
  const int band_w = min(kQkBand, a.k_tiles - band * kQkBand);
  const int kt = band * kQkBand + in_band % band_w;
  const int w0 = in_band / band_w * QR;
  const bool narrow = a.nq - w0 <= 16;                 // one block of queries in all (uniform)
  const int v0 = SPLIT || narrow ? w0 : w0 + wv / kQkCols * kQkTile;
  const int wk0 = kt * kQkKeys, ik0 = wk0 + wv % kQkCols * kQkMB * 16;         // first visual key of the stage, of this wavefront
  const int per = (a.H + Shape::kShares - 1) / Shape::kShares;            // heads of a share (the last may have fewer)
  const int h_lo = min(share * per, a.H), h_hi = min(h_lo + per, a.H);
  // (decoder: a tile all of whose keys lie behind its queries is zero)
  const bool wg_dead = DEC && a.vis0 + wk0 > a.row(min(w0 + QR, a.nq) - 1);
  const bool active = v0 < a.nq && !(DEC && a.vis0 + ik0 > a.row(min(v0 + kQkTile, a.nq) - 1));

  f32x4_t P[kQkMB][kQkQB];
#pragma unroll
  for (int kb = 0; kb < kQkMB; ++kb)
#pragma unroll
    for (int qb = 0; qb < kQkQB; ++qb) P[kb][qb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

  auto heads = [&]() __attribute__((always_inline)) {
    constexpr int QB = kQkQB;
    const int t = tid % T;
    u32x4_t* area = stage_m + share * kArea;
    constexpr int kBuf = Shape::kShares * kArea;
    const bf16_t* src[NL];                             // this thread's chunk of the stage's rows: queries, then keys
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = t / CH + i * RPI;
      const int row = r < QR ? a.row(min(w0 + r, a.nq - 1)) : a.vis0 + min(wk0 + r - QR, a.N - 1);
      src[i] = (r < QR ? a.Q : a.K) + b * a.sb + (int64_t)row * a.sn + t % CH * 8;
    }
    // (read before the loop: a scalar load on its way there makes every wait for LDS a wait for all of it)
    float scale = a.scale_log2e;
    asm volatile("" : "+s"(scale));
    const float2* nrm = a.norm + bi * a.H * a.nq;
    const uint32_t nrm_at = (uint32_t)min(w0 + t, a.nq - 1);
    u32x4_t next[NL];
    float2 next_nf;
    float2* nf_area = (float2*)(stage_m + 2 * kBuf) + share * QR;    // [2][shares][QR]
    auto load_stage = [&](int h, int part) {
      const int64_t off = (int64_t)h * a.sh + part * KSS * 32;
      if (part == 0) next_nf = (nrm + (int64_t)h * a.nq)[nrm_at];
#pragma unroll
      for (int i = 0; i < NL; ++i) __builtin_memcpy(&next[i], src[i] + off, 16);
    };
    // rows into buffer `buf`; a head's first stage brings its normalisers (nf_buf: the head's parity)
    auto store_stage = [&](int buf, int part, int nf_buf) {
      if (part == 0 && t < QR) nf_area[nf_buf * Shape::kShares * QR + t] = next_nf;
#pragma unroll
      for (int i = 0; i < NL; ++i) area[buf * kBuf + lds_chunk<CH>(t / CH + i * RPI, t % CH)] = next[i];
    };
    const int cnt = h_hi - h_lo, last = max(cnt - 1, 0), h0 = min(h_lo, a.H - 1);
    auto load_at = [&](int i, int part) { load_stage(h0 + min(i, last), part); };     // (past the last head: that one again)
    auto add = [&](const f32x4_t (&S)[kQkMB][QB], const float2 (&nf)[QB], int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          P[kb][qb][v] = fmaf(__builtin_amdgcn_exp2f(fmaf(S[kb][qb][v], a.scale_log2e, -nf[qb].x)), nf[qb].y, P[kb][qb][v]);
    };
    // Head i: its logits into S, beside the exponentials of head i - 1 from Sp -- the matrix
    // instructions and the trips through LDS run under the vector work of the head before.
    auto step = [&](int i, int par, const f32x4_t (&Sp)[kQkMB][QB], const float2 (&np)[QB], f32x4_t (&S)[kQkMB][QB],
                    float2 (&nf)[QB]) __attribute__((always_inline)) {
#pragma unroll
      for (int part = 0; part < NST; ++part) {
        const int buf = NST == 1 ? par : part % 2;
        store_stage(1 - buf, (part + 1) % NST, 1 - par);    // the stage after this one, loaded a step ago
        load_at(i + (part + 2) / NST, (part + 2) % NST);
        issue_fence();
        if (active) {                                  // uniform in the wavefront
          const bf16x8_t* st = (const bf16x8_t*)(area + buf * kBuf);
          bf16x8_t qf[QB][KSS], kf[kQkMB][KSS];
#pragma unroll
          for (int ks = 0; ks < KSS; ++ks) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) qf[qb][ks] = st[lds_chunk<CH>(v0 - w0 + qb * 16 + l16, ks * 4 + lg)];
#pragma unroll
            for (int kb = 0; kb < kQkMB; ++kb) kf[kb][ks] = st[lds_chunk<CH>(QR + ik0 - wk0 + kb * 16 + l16, ks * 4 + lg)];
          }
          issue_fence();
          // In this very order: an exponential to two other vector instructions, then a matrix instruction every
          // second time.
          constexpr int E = kQkMB * QB * 4 / NST, M = kQkMB * KSS * QB, kLead = 6;
          const int e0 = part * E;
          auto x_of = [&](int i) {
            const int kb = i / (QB * 4), qb = i / 4 % QB, v = i % 4;
            return fmaf(Sp[kb][qb][v], scale, -np[qb].x);
          };
          float x[2] = {x_of(e0), x_of(e0 + 1)}, e_prev = 0.0f;
          issue_fence();
#pragma unroll
          for (int i = 0; i <= E; ++i) {
            float e = 0.0f;
            if (i < E) e = __builtin_amdgcn_exp2f(x[i % 2]);
            if (i + 2 < E) x[i % 2] = x_of(e0 + i + 2);
            if (i > 0) {
              const int j = e0 + i - 1, kb = j / (QB * 4), qb = j / 4 % QB, v = j % 4;
              P[kb][qb][v] = fmaf(e_prev, np[qb].y, P[kb][qb][v]);
            }
#pragma unroll
            for (int m = 0; m < M; ++m)
              if (kLead + m * (E - kLead) / M == i) {
                const int ks = m / (kQkMB * QB), kb = m / QB % kQkMB, qb = m % QB;
                S[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][ks], qf[qb][ks], part == 0 && ks == 0 ? f32x4_t{0.0f, 0.0f, 0.0f, 0.0f} : S[kb][qb], 0, 0, 0);
              }
            issue_fence();
            e_prev = e;
          }
          if (part == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
              nf[qb] = nf_area[par * Shape::kShares * QR + v0 - w0 + qb * 16 + l16];
              if (SPLIT && i >= cnt) nf[qb].y = 0.0f;  // (a shorter share: its last head again, not counted)
            }
          }
        }
        __syncthreads();
      }
    };
    // (nothing before the first head: 2^-inf, times zero)
    f32x4_t Sa[kQkMB][QB], Sb[kQkMB][QB];
    float2 na[QB], nb[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      nb[qb] = make_float2(__builtin_huge_valf(), 0.0f);
#pragma unroll
      for (int kb = 0; kb < kQkMB; ++kb) Sb[kb][qb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
    load_at(0, 0);
    store_stage(0, 0, 0);
    load_at(1 / NST, 1 % NST);
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < per; i += 2) {
      step(i, 0, Sb, nb, Sa, na);
      if (i + 1 < per) step(i + 1, 1, Sa, na, Sb, nb);
    }
    if (active) {
#pragma unroll
      for (int kb = 0; kb < kQkMB; ++kb) {
        if (per % 2) add(Sa, na, kb); else add(Sb, nb, kb);
      }
    }
  };
  // outputs of KB x QB blocks from query v0 and visual key ik0 on, of the sums over the heads
  auto write_out = [&](auto kbn, auto qbn, int ik0, const auto& sums) __attribute__((always_inline)) {
    constexpr int KB = decltype(kbn)::value, QB = decltype(qbn)::value;
    const float invH = 1.0f / (float)a.H;
    const int qt = v0 / kQkTile;
    const bool recv = a.recv_part && qt < a.n_tiles;    // uniform
    // Whole blocks of visual queries that all count (all but the edges): no test per value, the rows' addresses in
    // scalar registers, and the column sums of eight keys halved between the lanes step by step.
    if constexpr (KB == 2) {
      if (a.abar && recv && ik0 + KB * 16 <= a.N && v0 + QB * 16 <= a.n_visq && !(DEC && ik0 + KB * 16 - 1 > v0)) {     // uniform
        double cs[KB * 4];
        const uint32_t at = (uint32_t)(lg * 4 * a.map_pitch + l16);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            float* row = a.abar + (b * a.N + ik0 + kb * 16 + v) * a.map_pitch + v0;
            cs[kb * 4 + v] = 0.0;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
              const float pm = sums[kb][qb][v] * invH;
              row[at + qb * 16] = pm;
              cs[kb * 4 + v] += (double)pm;
            }
          }
        const double mine = row_sums_of_8(cs, l16);
        const int i = (l16 & 1) * 4 + (l16 & 2) + (l16 >> 2 & 1);       // the key whose sum this lane holds
        if (l16 < 8) a.recv_part[(b * a.n_tiles + qt) * a.N + ik0 + i / 4 * 16 + lg * 4 + i % 4] = mine;
        return;
      }
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ik = ik0 + kb * 16 + lg * 4 + v;      // visual key
        const bool k_vis = ik < a.N;
        double cs = 0.0;                                // received from this tile's visual queries
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          const int vq = v0 + qb * 16 + l16;
          float pm = sums[kb][qb][v] * invH;            // head-mean probability
          if (DEC && a.vis0 + ik > a.row(vq)) pm = 0.0f;     // a key behind its query
          const bool q_vis = vq < a.n_visq;
          if (k_vis && q_vis && a.abar) a.abar[(b * a.N + ik) * a.map_pitch + vq] = pm;
          if (k_vis && !q_vis && vq < a.nq) {
            if (DEC) a.ttext[(b * a.N + ik) * a.M + (vq - a.n_visq)] = (double)pm;
            else a.cls[b * a.N + ik] = (double)pm;
          }
          cs += q_vis ? (double)pm : 0.0;
        }
        if (recv) {
          // sum over the 16 lanes that hold the tile's other queries of this key (a fixed tree)
          cs += dpp_move<0xB1>(cs);
          cs += dpp_move<0x4E>(cs);
          cs += dpp_move<0x141>(cs);
          cs += dpp_move<0x140>(cs);
          if (l16 == 0 && k_vis) a.recv_part[(b * a.n_tiles + qt) * a.N + ik] = cs;
        }
      }
    }
  };

  if (narrow) {
    // The wavefronts take consecutive shares of the heads,
    // operands straight from memory, and their sums are added in order.
    constexpr int KB = kQkKeys / 16, W = Shape::kThreads / kWave;
    f32x4_t P1[KB][1];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) P1[kb][0] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const int hs = (a.H + W - 1) / W, lo = min(wv * hs, a.H), hi = min(lo + hs, a.H);
    if (lo < hi && !wg_dead) {
      const int v = min(v0 + l16, a.nq - 1);
      const bf16_t* q_at = a.Q + b * a.sb + (int64_t)a.row(v) * a.sn + lg * 8;
      const bf16_t* k_at[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) k_at[kb] = a.K + b * a.sb + (int64_t)(a.vis0 + min(wk0 + kb * 16 + l16, a.N - 1)) * a.sn + lg * 8;
      bf16x8_t qf[KS], kf[KB][KS];
      float2 nf;
      auto load_head = [&](int h) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          __builtin_memcpy(&qf[ks], q_at + (int64_t)h * a.sh + ks * 32, 16);
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) __builtin_memcpy(&kf[kb][ks], k_at[kb] + (int64_t)h * a.sh + ks * 32, 16);
        }
        nf = a.norm[(bi * a.H + h) * a.nq + v];
      };
      load_head(lo);
#pragma unroll 1
      for (int h = lo; h < hi; ++h) {
        f32x4_t S[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          S[kb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) S[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][ks], qf[ks], S[kb], 0, 0, 0);
        }
        const float2 n = nf;
        load_head(min(h + 1, hi - 1));
        issue_fence();
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4)
            P1[kb][0][v4] = fmaf(__builtin_amdgcn_exp2f(fmaf(S[kb][v4], a.scale_log2e, -n.x)), n.y, P1[kb][0][v4]);
      }
    }
    f32x4_t* sums = (f32x4_t*)stage_m;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      if (wv > 0) sums[((wv - 1) * KB + kb) * kWave + lane] = P1[kb][0];
    __syncthreads();
    if (wv != 0) return;
    for (int w = 0; w < W - 1; ++w)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) P1[kb][0] += sums[(w * KB + kb) * kWave + lane];
    write_out(std::integral_constant<int, KB>{}, std::integral_constant<int, 1>{}, wk0, P1);
    return;
  }

  if (!wg_dead) heads();                                // uniform in the workgroup
  if constexpr (SPLIT) {
    f32x4_t* sums = (f32x4_t*)stage_m;                // (the staging areas are free)
#pragma unroll
    for (int step = Shape::kShares / 2; step >= 1; step /= 2) {
      f32x4_t* slot = sums + (wv % (kQkCols * step)) * kQkMB * kQkQB * kWave + lane;
      if (share >= step && share < 2 * step) {
#pragma unroll
        for (int kb = 0; kb < kQkMB; ++kb)
#pragma unroll
          for (int qb = 0; qb < kQkQB; ++qb) slot[(kb * kQkQB + qb) * kWave] = P[kb][qb];
      }
      __syncthreads();
      if (share < step) {
#pragma unroll
        for (int kb = 0; kb < kQkMB; ++kb)
#pragma unroll
          for (int qb = 0; qb < kQkQB; ++qb) P[kb][qb] += slot[(kb * kQkQB + qb) * kWave];
      }
      __syncthreads();
    }
    if (share != 0) return;
  }
  if (v0 < a.nq) write_out(std::integral_constant<int, kQkMB>{}, std::integral_constant<int, kQkQB>{}, ik0, P);
}

template <int KS, bool DEC>
static void launch_qk(QkArgs a, hipStream_t s) {
  constexpr int CH = (KS > 2 ? 2 : KS) * 4;
  const int tiles = (a.nq + kQkTile - 1) / kQkTile;
  a.q_groups = (tiles + kQkWaves - 1) / kQkWaves;
  // Fewer than one workgroup per compute unit (for heads of 32, whose steps are short, four): one tile each, whose keys
  // the wavefronts share.  Step of 16 x 577 tokens, whole tiles per wavefront and shared: one head of 64
  // 52.7 and 47.6 us, three 55.5 and 54.8, four (256 workgroups) 57.4 and 59.5, twelve 76.6 and 88.4; heads of 32: one 49.5 and
  // 45.9, eight 62.0 and 61.6, twelve 70.1 and 69.6.  One image of 577, one head 38.4 and 34.0; of 626, sixteen of 32
  // 38.8 and 35.0.
  a.share_keys = (int64_t)a.nb * a.H * a.q_groups < (KS == 1 ? 1024 : 256);
  if (a.share_keys) a.q_groups = tiles;
  const bool narrow = a.nq - (a.q_groups - 1) * (a.share_keys ? 1 : kQkWaves) * kQkTile <= 16;      // (as the kernel sees it)
  const int groups = a.q_groups - (narrow ? 1 : 0);
  hipLaunchKernelGGL((qk_norm_kernel<KS, DEC>), dim3(xcd_padded_total(a.nb * a.H * groups) + (narrow ? xcd_padded_total(a.nb * a.H) : 0)), dim3(kQkWaves * kWave), 0, s, a);
  auto mean = [&](auto kern, auto shape) {
    using Shape = decltype(shape);
    // two stages of (queries + keys) rows, in whole rounds of the loader; one pair per share of the heads
    constexpr int kLoaders = Shape::kRows * kQkCols * kWave / CH;
    constexpr int kStageRows = (Shape::kRows * kQkTile + kQkKeys + kLoaders - 1) / kLoaders * kLoaders;
    constexpr size_t kLds = 2 * Shape::kShares * ((size_t)kStageRows * CH * sizeof(u32x4_t) + Shape::kRows * kQkTile * sizeof(float2));
    if (kLds > 32768)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    a.q_groups = (tiles + Shape::kRows - 1) / Shape::kRows;
    hipLaunchKernelGGL(kern, dim3(xcd_padded_total(a.nb * a.q_groups * a.k_tiles)), dim3(Shape::kThreads), kLds, s, a);
  };
  // Fewer than one workgroup of the wide form per compute unit: the heads of a tile are split instead
  // (one image of 577 tokens: step 96 us before, 46 us so).
  const bool split = (int64_t)a.nb * ((tiles + QkMeanShape<false>::kRows - 1) / QkMeanShape<false>::kRows) * a.k_tiles < 256;
  if (split) mean(qk_mean_kernel<KS, DEC, true>, QkMeanShape<true>{});
  else mean(qk_mean_kernel<KS, DEC, false>, QkMeanShape<false>{});
}

void launch_attn_qk(const ficoco_problem& p, const Plan& pl, char* ws, hipStream_t s) {
  const bool L = p.variant == FICOCO_VARIANT_L;
  QkArgs a{};
  a.Q = (const bf16_t*)p.Q; a.K = (const bf16_t*)p.K;
  a.sb = p.qk_stride_b; a.sh = p.qk_stride_h; a.sn = p.qk_stride_n;
  a.H = p.H; a.n = p.qk_n; a.N = p.N;
  a.vis0 = p.vis_begin - p.qk_begin;
  a.nq = pl.qk_nq;
  a.n_visq = pl.qk_visq;
  a.x0 = L ? a.vis0 + p.N : p.cls_index - p.qk_begin;
  a.scale_log2e = p.qk_scale * 1.4426950408889634f;
  a.norm = (float2*)(ws + pl.qk_norm);
  a.abar = (p.corr_src == FICOCO_C_ATTN && pl.n_disc > 0) ? (float*)(ws + pl.abar) : nullptr;
  a.map_pitch = pl.map_pitch;
  a.recv_part = p.red_src == FICOCO_R_ATTN_RECV ? (double*)(ws + pl.recv_part) : nullptr;
  a.cls = (double*)(ws + pl.cls);
  if (L) { a.ttext = (double*)(ws + pl.ttext); a.M = p.M; }
  a.n_tiles = pl.n_chunks;
  a.k_tiles = (p.N + kQkKeys - 1) / kQkKeys;
  if (a.nq == 0) return;
  const int ks = p.d_head / 32;
  for (int b0 = 0; b0 < p.B; b0 += pl.qk_images) {    // as many images at a time as the normalisers have room for
    a.b0 = b0;
    a.nb = std::min(pl.qk_images, p.B - b0);
    if (L) { if (ks == 1) launch_qk<1, true>(a, s); else if (ks == 2) launch_qk<2, true>(a, s); else launch_qk<4, true>(a, s); }
    else { if (ks == 1) launch_qk<1, false>(a, s); else if (ks == 2) launch_qk<2, false>(a, s); else launch_qk<4, false>(a, s); }
  }
}

}  // namespace ficoco
