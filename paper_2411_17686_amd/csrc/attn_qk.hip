// Attention reduction from queries and keys (Sec. "Self-Attention": A = Softmax(Q K^T / sqrt(D))):
// the per-head maps are formed on the matrix cores and reduced on the fly, so the [B,H,n,n]
// maps never exist in memory.  Outputs are those of attn_reduce.hip -- per-tile column partials of
// the received attention (first term of Eq. 1), the [CLS] row (second term), the head-mean map
// in single precision, transposed, for the correlate stage (Algorithm 1, stage 2), and for FiCoCo-L
// (causal maps) the text profiles of Eq. 3 / Eq. 4.
//
// Two kernels (before: one workgroup per 48 query rows that exchanged maxima and sums between its
// wavefronts head by head; whole stage 81 -> 50 us at 16 x 577 tokens, 590 -> 242 us at 4 x 2881, 361 -> 86 us
// at the causal 8 x 675): qk_norm_kernel leaves (reference, 1 / row sum) of every (head, query) row, and
// qk_mean_kernel forms the probabilities of one (query tile, key tile) from them, adds the heads in
// registers and writes the tile's outputs.  The logits are computed twice, but once the normalisers
// are known nothing ties the keys of a row together: wavefronts exchange neither maxima nor sums, and
// the work can be cut to fill the chip whatever the numbers of queries, keys and heads are.
//
// Single precision (products of bfloat16 values are exact in it), row sums and column sums in double.
#include "common.hpp"
#include "causal_tiles.hpp"

#include <algorithm>

namespace ficoco {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kQkWaves = 4;                         // wavefronts of a workgroup (of a share of the heads)
constexpr int kQkB = 32;                            // queries and keys of a block: one matrix instruction
constexpr int kQkKeys = 2 * kQkB;                   // keys staged together: a block of each of two wavefronts
constexpr int kQkE = kQkB * kQkB / kWave;           // logits of a block that a lane holds, all of one query
static_assert(kQkTile == 2 * kQkB, "a column partial covers two blocks of queries");

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
  bool long_first;      // row normalisers: one group of every head after the other, those that see most keys first
  __host__ __device__ __forceinline__ int row(int v) const { return v < n_visq ? vis0 + v : x0 + (v - n_visq); }
};

// Rows of a product are keys here, columns queries.  Head mean: v_mfma_f32_32x32x16_bf16, operand A 32 rows x 16
// features (lane: row lane % 32, features 8 (lane / 32) .. + 8), operand B 32 columns x 16 features (same), the
// result 32 x 32 (lane: column lane % 32, rows key_of(v) + 4 (lane / 32) for its registers v): 32 lanes hold consecutive
// queries of one key, which is a piece of a row of the transposed map.  Row normalisers:
// v_mfma_f32_16x16x32_bf16, operand A 16 rows x 32 features (lane: row lane % 16, features 8 (lane / 16) .. + 8),
// operand B the same, the result 16 x 16 (lane: column lane % 16, rows 4 (lane / 16) + v).
//
// The vector unit works beside the 32 x 32 form, hardly beside the 16 x 16 one: 24 x (exponential, multiply-add, add)
// and the same products in either form, four wavefronts per SIMD, take 179 us without products; with them
// 251 (16 x 16), 199 (32 x 32), and 212 / 188 where the instructions alternate.  The normalisers stay with the
// former: three blocks of 32 queries a wavefront leave three wavefronts per SIMD instead of four (4 x 2881 tokens 120 us
// against 112, 16 x 577 26.8 against 24.3).
__device__ __forceinline__ constexpr int key_of(int v) { return v / 4 * 8 + v % 4; }
__device__ __forceinline__ f32x16_t qk_mfma(bf16x8_t keys, bf16x8_t queries, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(keys, queries, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t qk_zero() { return f32x16_t{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}; }

// A lane's 16-byte operand loads from global memory would touch a row of its own in every lane, and
// the address unit takes such a load apart into 64 accesses (measured: it was busy 74 % of the time
// and bound both kernels).  So rows are brought in whole -- neighbouring lanes on neighbouring 16-byte
// chunks -- and turned into operands through LDS.  CH chunks per row; the chunk of row r lies at
// chunk ^ swizzle, which spreads sixteen rows of an operand read over all 64 banks.
template <int CH>
__device__ __forceinline__ int lds_chunk(int r, int c) { return r * CH + (c ^ ((r / (16 / CH)) & (CH - 1))); }

// 16 bytes per lane on their way from memory into LDS, past the registers: lane l fills the 16 bytes at 16 l behind
// an address of the wavefront.  So it is the source that is swizzled: thread t brings chunk
// (t % CH) ^ ((t / 16) % CH) of row t / CH (+ whole rounds of the workgroup: the same for all of them).
__device__ __forceinline__ void load_to_lds(const bf16_t* src, u32x4_t* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void loaded_to_lds() {      // all of the workgroup's loads have arrived
  __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
  __syncthreads();
}

// ---- row normalisers ---------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));
constexpr int kNormTile = 48;                       // queries of a wavefront
constexpr int kNormQB = kNormTile / 16;             // in blocks of 16
constexpr int kNormKB = 2;                          // 16-key blocks a wavefront takes together
static_assert(kQkKeys == 2 * kNormKB * 16, "two steps of keys");

// Workgroups of the heads' groups, without the narrow last ones.
__host__ __device__ __forceinline__ int norm_grid(const QkArgs& a, int heads, int groups) {
  return a.long_first ? xcd_padded_total(heads) * groups : xcd_padded_total(heads * groups);
}

// A workgroup takes 4 x 48 queries of one head and walks its keys 64 at a time, the next 64 being
// loaded while the current ones are added (few workgroups: 48 queries, the keys shared by its wavefronts).
// (Keys loaded straight into LDS: no change.)  The exponentials are taken relative to a whole number (units of log2) at the
// largest logit of the first 32 keys, not of the whole row: any reference serves as long as nothing overflows, and then the
// sums need no running maximum.  A row whose sum does overflow (its largest logit more than ~70 above those of the first 32
// keys) is seen in the sum and done again with its own maximum.
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
  const bool last_narrow = a.nq - (a.q_groups - 1) * (a.share_keys ? 1 : kQkWaves) * kNormTile <= 16;
  const int groups = a.q_groups - (last_narrow ? 1 : 0), all_heads = a.nb * a.H, first = norm_grid(a, all_heads, groups);
  const bool behind = (int)blockIdx.x >= first;
  int in_head, head;
  if (behind) {
    in_head = groups;
    head = xcd_logical_id(blockIdx.x - first, all_heads);
  } else if (DEC && a.long_first) {
    const int per = (all_heads + kXcds - 1) / kXcds, at = blockIdx.x / kXcds;
    in_head = groups - 1 - at / per;
    head = at % per + blockIdx.x % kXcds * per;
  } else {
    const int unit = xcd_logical_id(blockIdx.x, all_heads * groups);
    in_head = unit % groups;
    head = unit / groups;
  }
  if (head >= all_heads) return;
  const int tid = threadIdx.x, lane = tid % kWave, l16 = lane % 16, lg = lane / 16;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int w0 = in_head * (a.share_keys ? 1 : kQkWaves) * kNormTile;
  const bool narrow = a.nq - w0 <= 16;     // one block of queries in all (the [CLS] query behind 576 visual ones)
  const bool share_keys = a.share_keys || narrow;
  const int v0 = share_keys ? w0 : w0 + wv * kNormTile;
  const int h = head % a.H;
  const int64_t bi = head / a.H;
  const float NEG = -__builtin_huge_valf();
  const bf16_t* Qh = a.Q + (a.b0 + bi) * a.sb + (int64_t)h * a.sh;
  const bf16_t* Kh = a.K + (a.b0 + bi) * a.sb + (int64_t)h * a.sh;
  // keys below full_end count for every query of this wavefront, from k_end on for none
  const bool active = v0 < a.nq;
  const int q_lo = a.row(min(v0, a.nq - 1)), q_hi = a.row(min(v0 + kNormTile, a.nq) - 1);
  const int k_end = !active ? 0 : DEC ? min(a.n, q_hi + 1) : a.n;
  const int full_end = DEC ? min(a.n, q_lo + 1) : a.n;
  const int wg_end = DEC ? min(a.n, a.row(min(w0 + kQkWaves * kNormTile, a.nq) - 1) + 1) : a.n;

  int qrow[kNormQB];
  bf16x8_t qf[kNormQB][KS];
#pragma unroll
  for (int qb = 0; qb < kNormQB; ++qb) {
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

  typedef f32x4_t Logits[kNormKB][kNormQB];      // of 32 keys
  Logits S;
  // `key_op(kb, ks)` gives this lane's operand
  auto logits = [&](auto qbn, auto key_op, Logits& S) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
#pragma unroll
    for (int kb = 0; kb < kNormKB; ++kb) {
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
  float ref[kNormQB];
  double sum[kNormQB];
  auto max_of = [&](auto qbn, int k0) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int kb = 0; kb < kNormKB; ++kb)
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
      for (int kb = 0; kb < kNormKB; ++kb)
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
    if (k0 + kNormKB * 16 <= full_end) {               // uniform
      add_whole(qbn, S);
    } else {
#pragma unroll
      for (int kb = 0; kb < kNormKB; ++kb)
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
    for (int qb = 0; qb < kNormQB; ++qb) {
      sum[qb] += __shfl_xor(sum[qb], 16, kWave);
      sum[qb] += __shfl_xor(sum[qb], 32, kWave);
    }
  };
#pragma unroll
  for (int qb = 0; qb < kNormQB; ++qb) { ref[qb] = NEG; sum[qb] = 0.0; }

  const std::integral_constant<int, kNormQB> all{};
  auto direct = [&](int k0) {
    return [&, k0](int kb, int ks) {
      bf16x8_t kf;
      __builtin_memcpy(&kf, Kh + (int64_t)min(k0 + kb * 16 + l16, a.n - 1) * a.sn + lg * 8 + ks * 32, 16);
      return kf;
    };
  };
  bool over = false;
  // Each wavefront every fourth 32 keys, with a reference of its own; the four sums are combined in order.
  __shared__ float part_ref[kQkWaves][kNormTile];
  __shared__ double part_sum[kQkWaves][kNormTile];
  auto shared_keys = [&](auto qbn) __attribute__((always_inline)) {
    constexpr int QB = decltype(qbn)::value;
    const int first = wv * kNormKB * 16;
#pragma unroll 1
    for (int k0 = first; k0 < k_end; k0 += kQkWaves * kNormKB * 16) {
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
        if (k0 + half * kNormKB * 16 >= k_end) continue;   // uniform
        logits(all, [&](int kb, int ks) { return st[lds_chunk<CH>((half * kNormKB + kb) * 16 + l16, ks * 4 + lg)]; }, S);
        if (half == 0 && k0 == 0) { max_of(all, 0); set_ref(all); }
        add_chunk(all, k0 + half * kNormKB * 16, S);
      }
      store_stage(1 - buf);
      __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
    if (!active) return;
    across();
#pragma unroll
    for (int qb = 0; qb < kNormQB; ++qb) over |= !(sum[qb] < 0x1p100);
  }
  if (__any(over)) {                                 // rare: with the row's own maximum, keys straight from memory
#pragma unroll
    for (int qb = 0; qb < kNormQB; ++qb) { ref[qb] = NEG; sum[qb] = 0.0; }
#pragma unroll 1
    for (int k0 = 0; k0 < k_end; k0 += kNormKB * 16) { logits(all, direct(k0), S); max_of(all, k0); }
    set_ref(all);
#pragma unroll 1
    for (int k0 = 0; k0 < k_end; k0 += kNormKB * 16) { logits(all, direct(k0), S); add_chunk(all, k0, S); }
    across();
  }
#pragma unroll
  for (int qb = 0; qb < kNormQB; ++qb) {
    const int v = v0 + qb * 16 + l16;
    if (lg == 0 && v < a.nq) a.norm[((int64_t)bi * a.H + h) * a.nq + v] = make_float2(ref[qb], (float)(1.0 / sum[qb]));
  }
}

// Sixteen values of every lane, each summed over 32 lanes: the tree of the steps lane ^ 1, ^ 2, ^ 4, ^ 8, ^ 16.
// The first four hand half of the values to the other lane of the pair, so lane l is left with value
// sum_index(l) alone: 16 additions instead of 80.
__device__ __forceinline__ int sum_index(int l) { return (l & 1) * 8 + (l & 2) * 2 + (l >> 1 & 2) + (l >> 3 & 1); }
__device__ __forceinline__ double sums_of_16(const double (&x)[16], int l) {
  auto pick = [](bool second, double a, double b) { return second ? b : a; };
  double y[8], z[4], u[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) y[i] = pick(l & 1, x[i], x[i + 8]) + dpp_move<0xB1>(pick(l & 1, x[i + 8], x[i]));
#pragma unroll
  for (int i = 0; i < 4; ++i) z[i] = pick(l & 2, y[i], y[i + 4]) + dpp_move<0x4E>(pick(l & 2, y[i + 4], y[i]));
#pragma unroll
  for (int i = 0; i < 2; ++i) u[i] = pick(l & 4, z[i], z[i + 2]) + lane_xor_4(pick(l & 4, z[i + 2], z[i]));
  const double t = pick(l & 8, u[0], u[1]) + dpp_move<0x128>(pick(l & 8, u[1], u[0]));      // rotated by eight: lane ^ 8
  return t + __shfl_xor(t, 16, kWave);
}

// ---- probabilities, head mean, outputs -----------------------------------------------------------
constexpr int kQkBand = 8;                          // key tiles side by side in the order of the workgroups
// Tile number `unit` of an image (qr queries x kQkKeys keys): in columns kQkBand key tiles wide, so that the workgroups that run
// together on an XCD need few rows of either side, which its L2 holds for all heads.  live_first: first the tiles that hold a key
// some query sees, then the others, which are zero and took places on the chip from which others were missing in between.
__device__ __forceinline__ void qk_tile(const QkArgs& a, int unit, bool live_first, int qr, int& kt0, int& w0) {
  if (live_first) {
    int g;
    causal_tile(unit, a.q_groups, a.k_tiles, qr / kQkKeys, a.n_visq / qr, g, kt0);
    w0 = g * qr;
  } else {
    const int band = unit / (kQkBand * a.q_groups), in_band = unit - band * kQkBand * a.q_groups;
    const int band_w = min(kQkBand, a.k_tiles - band * kQkBand);
    kt0 = band * kQkBand + in_band % band_w;
    w0 = in_band / band_w * qr;
  }
}
template <bool SPLIT> struct QkMeanShape {
  static constexpr int kBlocks = SPLIT ? 1 : 2;       // of queries per wavefront
  static constexpr int kQueries = 2 * kBlocks * kQkB; // of a workgroup
  static constexpr int kShares = SPLIT ? 4 : 1;       // shares of the heads
  static constexpr int kThreads = kQkWaves * kShares * kWave;
  // Causal maps with heads of 128, not split: only launched with one block of queries in all (qk_mean_deep_kernel takes the others).
  static constexpr bool narrow_only(int ks, bool dec) { return dec && ks == 4 && !SPLIT; }
};
// Outputs of 64 queries (32: one block) from v0 and 32 visual keys from ik0 on, of the sums over the heads.
template <bool DEC, int blocks>
__device__ __forceinline__ void qk_write_out(const QkArgs& a, int64_t b, int v0, int ik0, const f32x16_t& s0, const f32x16_t& s1) {
  // (again from the thread's number: kept over the heads, these took registers that heads of 128, split, do not have)
  int here = threadIdx.x;
  asm volatile("" : "+v"(here));
  const int l32 = here % kQkB, hi = here % kWave / kQkB;
  const float invH = 1.0f / (float)a.H;
  const int qt = v0 / kQkTile;
  const bool recv = a.recv_part && qt < a.n_tiles;    // uniform
  double cs[kQkE];                                    // received from this tile's visual queries
  if (blocks == 2 && a.abar && ik0 + kQkB <= a.N && v0 + kQkTile <= a.n_visq && !(DEC && ik0 + kQkB - 1 > v0)) {     // uniform
    // Whole blocks of visual queries that all count (all but the edges): no test per value, the rows' addresses in
    // scalar registers.
    const uint32_t at = (uint32_t)(hi * 4 * a.map_pitch + l32);
#pragma unroll
    for (int v = 0; v < kQkE; ++v) {
      float* row = a.abar + (b * a.N + ik0 + key_of(v)) * a.map_pitch + v0;
      const float p0 = s0[v] * invH, p1 = s1[v] * invH;      // head-mean probabilities
      row[at] = p0;
      row[at + kQkB] = p1;
      cs[v] = (double)p0 + (double)p1;
    }
  } else {
#pragma unroll
    for (int v = 0; v < kQkE; ++v) cs[v] = 0.0;
#pragma unroll
    for (int m = 0; m < blocks; ++m) {
      const int vq = v0 + m * kQkB + l32, k_first = ik0 + 4 * hi, n_k = a.N - k_first;
      const bool q_vis = vq < a.n_visq, q_in = vq < a.nq;
      const int behind = DEC ? a.row(vq) - a.vis0 - k_first : 0;     // keys from there on lie behind the query
      const int64_t key = b * a.N + k_first;
      float* map = a.abar + key * a.map_pitch + vq;
      double* other = DEC ? a.ttext + key * a.M + (vq - a.n_visq) : a.cls + key;
      const int64_t other_pitch = DEC ? a.M : 1;
#pragma unroll
      for (int v = 0; v < kQkE; ++v) {
        const int k = key_of(v);
        float pm = (m == 0 ? s0[v] : s1[v]) * invH;
        if (DEC && k > behind) pm = 0.0f;
        if (k < n_k) {
          if (q_vis) { if (a.abar) map[k * (int64_t)a.map_pitch] = pm; }
          else if (q_in) other[k * other_pitch] = (double)pm;
        }
        cs[v] += q_vis ? (double)pm : 0.0;
      }
    }
  }
  if (recv) {
    const double mine = sums_of_16(cs, l32);
    const int i = sum_index(l32), ik = ik0 + i / 4 * 8 + i % 4 + 4 * hi;
    if (l32 < 16 && ik < a.N) a.recv_part[(b * a.n_tiles + qt) * a.N + ik] = mine;
  }
}

// One block of queries in all, from w0 on, by W wavefronts: they take consecutive shares of the heads, operands straight from memory, and
// their sums are added pairwise (a fixed tree) in `sums` (W x kWave places).  live: some query sees some key of the tile (from wk0 on).
template <int KS, bool DEC, int W>
__device__ __forceinline__ void qk_mean_narrow(const QkArgs& a, int64_t bi, int64_t b, int w0, int wk0, int wv, bool live, f32x16_t* sums) {
  constexpr int KT = (KS > 2 ? 2 : KS) * 2;            // instructions of a block and of the features taken together
  const int lane = threadIdx.x % kWave, l32 = lane % kQkB, hi = lane / kQkB;
  f32x16_t P1[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) P1[kb] = qk_zero();
  const int hs = (a.H + W - 1) / W, lo = min(wv * hs, a.H), h_end = min(lo + hs, a.H);
  if (live) {
    const int v = min(w0 + l32, a.nq - 1);
    const bf16_t* q_at = a.Q + b * a.sb + (int64_t)a.row(v) * a.sn + hi * 8;
    const bf16_t* k_at[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) k_at[kb] = a.K + b * a.sb + (int64_t)(a.vis0 + min(wk0 + kb * kQkB + l32, a.N - 1)) * a.sn + hi * 8;
#pragma unroll 1
    for (int h = lo; h < h_end; ++h) {
      const float2 n = a.norm[(bi * a.H + h) * a.nq + v];
      f32x16_t S[2];
#pragma unroll
      for (int c = 0; c < KS * 2; c += KT) {         // a stage's features at a time
        bf16x8_t qf[KT], kf[2][KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          __builtin_memcpy(&qf[kt], q_at + (int64_t)h * a.sh + (c + kt) * 16, 16);
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) __builtin_memcpy(&kf[kb][kt], k_at[kb] + (int64_t)h * a.sh + (c + kt) * 16, 16);
        }
        issue_fence();
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) S[kb] = qk_mfma(kf[kb][kt], qf[kt], c + kt == 0 ? qk_zero() : S[kb]);
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < kQkE; ++e) P1[kb][e] = fmaf(__builtin_amdgcn_exp2f(fmaf(S[kb][e], a.scale_log2e, -n.x)), n.y, P1[kb][e]);
    }
  }
#pragma unroll
  for (int step = W / 2; step >= 2; step /= 2) {
    f32x16_t* slot = sums + wv % step * 2 * kWave + lane;
    if (wv >= step && wv < 2 * step) { slot[0] = P1[0]; slot[kWave] = P1[1]; }
    __syncthreads();
    if (wv < step) { P1[0] += slot[0]; P1[1] += slot[kWave]; }
    __syncthreads();
  }
  // the last two wavefronts write a block of keys each
  if (wv < 2) sums[wv * kWave + lane] = wv == 0 ? P1[1] : P1[0];
  __syncthreads();
  if (wv >= 2) return;
  const f32x16_t mine = wv == 0 ? P1[0] + sums[kWave + lane] : sums[lane] + P1[1];
  qk_write_out<DEC, 1>(a, b, w0, wk0 + wv * kQkB, mine, mine);
}

// A wavefront forms 64 queries x 32 visual keys of an image, the heads added in order in registers.
// SPLIT = false: the four wavefronts of a workgroup sit two by two on 128 queries x 64 keys and
// share the staged rows.  SPLIT = true (few tiles): 64 x 64 by four wavefronts of one block each, and four such groups
// take consecutive shares of the heads, each with a staging area of its own; their sums are added
// pairwise (a fixed tree) in LDS.  Rows are staged 64 features at a time in two buffers, loaded straight into LDS
// a stage ahead; the normalisers of a head come through LDS as well; the exponentials of a block are computed beside
// the matrix instructions and LDS reads of the next one, in a fixed order.
//
// Bound by the vector unit (exponential, two multiply-adds per logit) and the trips between
// barriers.  Measured at 4 x 2881 tokens, 16 heads of 64 / 16 x 577, 16 of 64 / 8 x 675 causal, 32
// of 128: operands straight from memory 314 / 70 / 99 us; staged through registers, 192 x 64 by eight wavefronts, each head
// on its own 180 / 44 / 56; 96 x 64 by four wavefronts with 16 x 16 products, the next head's beside this head's
// exponentials 170 / 40 / 51; normalisers through LDS, whole tiles written without tests 158 / 34 / 49; 32 x 32 products
// 157 / 33 / 51; rows straight into LDS, order of precedence among the wavefronts 142 / 28.6 / 48.
template <int KS, bool DEC, bool SPLIT>
__global__ __launch_bounds__(QkMeanShape<SPLIT>::kThreads) __attribute__((amdgpu_waves_per_eu(SPLIT ? 4 : KS == 4 ? 2 : 3))) void qk_mean_kernel(QkArgs a) {
  constexpr int KSS = KS > 2 ? 2 : KS, NST = KS / KSS, CH = KSS * 4, KT = KSS * 2;     // 32-feature steps of a stage, stages of a head, instructions of a block and stage
  using Shape = QkMeanShape<SPLIT>;
  constexpr int MB = Shape::kBlocks, QR = Shape::kQueries, kWaves = Shape::kThreads / kWave;    // QR: query rows of a stage
  constexpr int T = kQkWaves * kWave, RPI = T / CH, NL = (QR + kQkKeys) / RPI;   // rounds of RPI rows
  static_assert((QR + kQkKeys) % RPI == 0 && QR % RPI == 0, "whole rounds of queries and of keys");
  extern __shared__ u32x4_t stage_m[];                 // [2][shares][rows of a stage], then the queries' normalisers
  constexpr int kArea = NL * RPI * CH;
  const int units = a.nb * a.q_groups * a.k_tiles;
  const int unit = xcd_logical_id(blockIdx.x, units);
  if (unit >= units) return;
  const int tid = threadIdx.x, lane = tid % kWave, l32 = lane % kQkB, hi = lane / kQkB;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int share = wv / kQkWaves, wq = wv % kQkWaves / 2, wk = wv % 2;
  const int64_t bi = unit / (a.k_tiles * a.q_groups), b = a.b0 + bi;
  const int in_img = unit - (int)bi * a.k_tiles * a.q_groups;
  int kt0, w0;
  qk_tile(a, in_img, DEC && !SPLIT && causal_live_first(units, a.k_tiles), QR, kt0, w0);
  // One block of queries in all (uniform): the wavefronts share its heads, with operands straight from memory, unless the tile is
  // split anyway and a wavefront's share is four 32-feature steps or more: then rows through LDS are faster.  us, so and
  // as any other tile: 8 x 16 text queries, 32 heads of 128 25.3 / 21.4, 24 queries 26.7 / 21.5, one image of 16 and 16 heads 15.6 / 13.9, 8 x 20 and
  // 32 heads of 64 16.0 / 15.6; but 8 x 24 and 16 heads of 64 12.3 / 12.6, 8 heads 9.1 / 10.7, and not split 16 x 401 queries 19.9 / 20.9.
  const bool narrow = a.nq - w0 <= kQkB && !(SPLIT && KS * ((a.H + kWaves - 1) / kWaves) >= 4);
  const int q0 = narrow ? 0 : wq * MB * kQkB, v0 = w0 + q0;
  const int wk0 = kt0 * kQkKeys, ik0 = wk0 + wk * kQkB;       // first visual key of the stage, of this wavefront
  const int per = (a.H + Shape::kShares - 1) / Shape::kShares;            // heads of a share (the last may have fewer)
  const int h_lo = min(share * per, a.H), h_hi = min(h_lo + per, a.H);
  // (decoder: a tile all of whose keys lie behind its queries is zero)
  const bool wg_dead = DEC && a.vis0 + wk0 > a.row(min(w0 + QR, a.nq) - 1);
  // Wavefronts of a last tile that have one block of queries (of 65 to 96: behind 576 visual ones the [CLS] query) add the heads up in
  // quarters: the sums so far are kept in the registers of the other block, where nothing else is added.  With all heads one
  // after the other in single precision the [CLS] row, which weighs most, had more error than in the forms before, where its heads
  // were shared by wavefronts: scores against 64 bits, 16 heads of 64, 577 tokens 1.40e-7, before 1.23e-7, so 1.13e-7; 2881 1.57, 1.26 and
  // 1.26e-7.  (That block as a tile of its own is a fifth more workgroups at 577 tokens: 16 images 27 -> 36 us instead of 27.4.)
  const bool with_lone = !SPLIT && !DEC && !narrow && a.nq - w0 > kQkTile && a.nq - w0 <= kQkTile + kQkB;      // uniform in the workgroup
  const bool lone = with_lone && q0 > 0;
  const bool active = v0 < a.nq && !(DEC && a.vis0 + ik0 > a.row(min(v0 + MB * kQkB, a.nq) - 1));

  f32x16_t P[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) P[m] = qk_zero();

  auto heads = [&](auto fold) __attribute__((always_inline)) {
    constexpr bool kFold = decltype(fold)::value;
    const int t = tid % T;
    u32x4_t* area = stage_m + share * kArea;
    constexpr int kBuf = Shape::kShares * kArea;
    const bf16_t* src[NL];                             // this thread's chunk of the stage's rows: queries, then keys
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = t / CH + i * RPI;
      const int row = r < QR ? a.row(min(w0 + r, a.nq - 1)) : a.vis0 + min(wk0 + r - QR, a.N - 1);
      src[i] = (i * RPI < QR ? a.Q : a.K) + b * a.sb + (int64_t)row * a.sn + (t % CH ^ (t / 16 & (CH - 1))) * 8;
    }
    // (read before the loop: a scalar load on its way there makes every wait for LDS a wait for all of it)
    float scale = a.scale_log2e;
    asm volatile("" : "+s"(scale));
    const float2* nrm = a.norm + bi * a.H * a.nq;
    const uint32_t nrm_at = (uint32_t)min(w0 + t, a.nq - 1);
    float2 next_nf;
    float2* nf_area = (float2*)(stage_m + 2 * kBuf) + share * QR;    // [2][shares][QR]
    // the rows of head h's stage `part` on their way into buffer `buf`
    auto load_stage = [&](int h, int part, int buf) __attribute__((always_inline)) {
      const int64_t off = (int64_t)h * a.sh + part * KSS * 32;
#pragma unroll
      for (int i = 0; i < NL; ++i)
        load_to_lds(src[i] + off, area + buf * kBuf + i * T + wv % kQkWaves * kWave);
    };
    auto load_nf = [&](int h) { next_nf = (nrm + (int64_t)h * a.nq)[nrm_at]; };
    const int counted = w0 + t < a.nq ? -1 : 0;        // (rows past the last query, staged as that one again, add nothing)
    auto store_nf = [&](int par) {
      if (t < QR) {
        float2 v = next_nf;
        if (kFold) v.y = __int_as_float(__float_as_int(v.y) & counted);
        nf_area[par * Shape::kShares * QR + t] = v;
      }
    };
    const int cnt = h_hi - h_lo, last = max(cnt - 1, 0), h0 = min(h_lo, a.H - 1);
    auto head = [&](int i) { return h0 + min(i, last); };               // (past the last head: that one again)

    // Logits: heads of one stage block by block (S[0] and S[1] in turn), else a head's blocks side by side (S of even
    // and odd heads).  The block whose exponentials are due is the one before.
    constexpr int SB = NST > 1 ? MB : 1;
    f32x16_t S[2][SB];
    float2 nf[MB];                                     // of the head whose exponentials are due
#pragma unroll
    for (int m = 0; m < MB; ++m) nf[m] = make_float2(__builtin_huge_valf(), 0.0f);    // (nothing before the first head: 2^-inf, times zero)
#pragma unroll
    for (int m = 0; m < SB; ++m) S[1][m] = qk_zero();
    auto x_of = [&](const f32x16_t& Sd, float2 n, int v) { return fmaf(Sd[v], scale, -n.x); };
    auto add = [&](const f32x16_t& Sd, float2 n, f32x16_t& Pd) __attribute__((always_inline)) {
#pragma unroll
      for (int v = 0; v < kQkE; ++v) Pd[v] = fmaf(__builtin_amdgcn_exp2f(x_of(Sd, n, v)), n.y, Pd[v]);
    };
    // exponentials e0 .. e0 + E of one block beside the NB * KT matrix instructions of the next: an exponential to two
    // other vector instructions, the matrix instructions spread between them
    auto mix = [&](auto count, int e0, const f32x16_t& Sd, float2 n, f32x16_t& Pd, auto nb, const bf16x8_t (&kf)[KT],
                   const auto& qf, auto& Sn, bool fresh) __attribute__((always_inline)) {
      constexpr int E = decltype(count)::value, NB = decltype(nb)::value, M = NB * KT, kLead = 5;
      float x[2] = {x_of(Sd, n, e0), x_of(Sd, n, e0 + 1)}, e_prev = 0.0f;
      issue_fence();
#pragma unroll
      for (int i = 0; i <= E; ++i) {
        float e = 0.0f;
        if (i < E) e = __builtin_amdgcn_exp2f(x[i % 2]);
        if (i + 2 < E) x[i % 2] = x_of(Sd, n, e0 + i + 2);
        if (i > 0) Pd[e0 + i - 1] = fmaf(e_prev, n.y, Pd[e0 + i - 1]);
#pragma unroll
        for (int m = 0; m < M; ++m)
          if (kLead + m * (E - kLead) / M == i) {
            const int kt = m / NB, blk = m % NB;
            Sn[blk] = qk_mfma(kf[kt], qf[blk][kt], fresh && kt == 0 ? qk_zero() : Sn[blk]);
          }
        issue_fence();
        e_prev = e;
      }
    };
    auto step = [&](int i, auto par_c) __attribute__((always_inline)) {
      constexpr int par = decltype(par_c)::value;
#pragma unroll
      for (int part = 0; part < NST; ++part) {
        const int buf = NST == 1 ? par : part % 2;
        if (part == NST - 1) store_nf(1 - par);
        auto load_next = [&]() __attribute__((always_inline)) {
          issue_fence();
          if (part == NST - 1) load_nf(head(i + 2));
          load_stage(head(i + (part + 1) / NST), (part + 1) % NST, 1 - buf);
          issue_fence();
        };
        if (active) {                                  // uniform in the wavefront
          const bf16x8_t* st = (const bf16x8_t*)(area + buf * kBuf);
          auto read_queries = [&](int m, bf16x8_t (&qf)[KT]) __attribute__((always_inline)) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) qf[kt] = st[lds_chunk<CH>(q0 + m * kQkB + l32, kt * 2 + hi)];
          };
          bf16x8_t kf[KT];
          auto read_keys = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) kf[kt] = st[lds_chunk<CH>(QR + wk * kQkB + l32, kt * 2 + hi)];
          };
          float2 mine[MB];
          auto read_nf = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < MB; ++m) {
              mine[m] = nf_area[par * Shape::kShares * QR + q0 + m * kQkB + l32];
              if (SPLIT && i >= cnt) mine[m].y = 0.0f;   // (a shorter share: its last head again, not counted)
            }
          };
          bf16x8_t qf[MB][KT];
          read_keys();
#pragma unroll
          for (int m = 0; m < MB; ++m) read_queries(m, qf[m]);
          if (part == NST - 1) read_nf();
          load_next();                                 // (behind the reads: the compiler has a read wait for every load into LDS before it)
          if constexpr (NST == 1) {
#pragma unroll
            for (int m = 0; m < MB; ++m) {
              const int cur = MB == 1 ? par : m % 2, due = m == 0 ? MB - 1 : m - 1;
              mix(std::integral_constant<int, kQkE>{}, 0, S[1 - cur][0], nf[due], P[due], std::integral_constant<int, 1>{}, kf, &qf[m], S[cur], true);
              if (m == 0) {
#pragma unroll
                for (int q = 0; q < MB; ++q) nf[q] = mine[q];
              }
            }
          } else {
            constexpr int E = MB * kQkE / NST;
            const int due = part * E / kQkE, e0 = part * E % kQkE;
            mix(std::integral_constant<int, E>{}, e0, S[1 - par][due], nf[due], P[due], std::integral_constant<int, MB>{}, kf, qf, S[par], part == 0);
            if (part == NST - 1) {
#pragma unroll
              for (int q = 0; q < MB; ++q) nf[q] = mine[q];
            }
          }
        } else {
          load_next();
        }
        loaded_to_lds();
      }
    };
    load_nf(head(0));
    load_stage(head(0), 0, 0);
    store_nf(0);
    load_nf(head(1));
    loaded_to_lds();
    const int quarter = kFold ? (per + 7) / 8 * 2 : per;      // even
    int i = 0;
#pragma unroll 1
    do {
      const int to = min(i + quarter, per);
#pragma unroll 1
      for (; i < to; i += 2) {
        if (DEC) { }                                   // (as in the normalisers; causal maps 48.5 us without, 49.9 with)
        else if (i == 0) __builtin_amdgcn_s_setprio(3);
        else if (i == per / 4 * 2) __builtin_amdgcn_s_setprio(2);
        else if (i == per * 3 / 8 * 2) __builtin_amdgcn_s_setprio(1);
        else if (i == per * 7 / 16 * 2) __builtin_amdgcn_s_setprio(0);
        step(i, std::integral_constant<int, 0>{});
        if (i + 1 < per) step(i + 1, std::integral_constant<int, 1>{});
      }
      if (kFold && lone) { P[MB - 1] += P[0]; P[0] = qk_zero(); }      // uniform in the wavefront
    } while (i < per);
    if (active) {                                      // what is left: the last block, or the last head's blocks
      if constexpr (NST == 1 && MB == 2) {
        add(S[1][0], nf[1], P[1]);
      } else {
#pragma unroll
        for (int m = 0; m < SB; ++m) {
          if (per % 2) add(S[0][m], nf[m], P[m]); else add(S[1][m], nf[m], P[m]);
        }
      }
    }
  };
  if (narrow) {
    qk_mean_narrow<KS, DEC, kWaves>(a, bi, b, w0, wk0, wv, !wg_dead, (f32x16_t*)stage_m);
    return;
  }
  if constexpr (QkMeanShape<SPLIT>::narrow_only(KS, DEC)) return;

  if (!wg_dead) {                                       // uniform in the workgroup
    if constexpr (!SPLIT && !DEC) {
      if (with_lone) heads(std::integral_constant<bool, true>{});      // (a copy of the loop: what it needs cost all others 4 % of the kernel)
      else heads(std::integral_constant<bool, false>{});
    } else {
      heads(std::integral_constant<bool, false>{});
    }
  }
  if constexpr (SPLIT) {
    f32x16_t* sums = (f32x16_t*)stage_m;              // (the staging areas are free)
#pragma unroll
    for (int step = Shape::kShares / 2; step >= 1; step /= 2) {
      f32x16_t* slot = sums + (wv % (kQkWaves * step)) * kWave + lane;
      if (share >= step && share < 2 * step) *slot = P[0];
      __syncthreads();
      if (share < step) P[0] += *slot;
      __syncthreads();
    }
    // the upper block of a tile's queries goes to the wavefront that has the lower one
    if (share == 0 && wq == 1) sums[wk * kWave + lane] = P[0];
    __syncthreads();
    if (share != 0 || wq != 0) return;
    qk_write_out<DEC, 2>(a, b, w0, ik0, P[0], sums[wk * kWave + lane]);
  } else {
    if (lone) P[0] += P[MB - 1];
    if (v0 < a.nq) qk_write_out<DEC, 2>(a, b, v0, ik0, P[0], P[MB - 1]);
  }
}

// ---- the same for causal maps with heads of 128 -----------------------------------------------------
// Tiles, products and sums of the kernel above in its wide form, in the same order (the same bits; a last tile of at most 32 queries is
// qk_mean_narrow's here too: with its 32 heads all in line the row of one text query behind 512 others has an error of 9.5e-8 against 64 bits, so 5.8e-8).  Few wavefronts share a SIMD: 232 of
// the 360 tiles of 8 x 675 tokens hold a key that some query sees, fewer than there are compute units, and then nothing
// hides a wavefront's trips.  So the fragments of a stage are read into a second set of registers while the products of the one
// before are formed, rows are loaded three stages ahead (three buffers, one barrier a stage, no wait for loads just issued),
// and reads and loads are spread over the stage's products and exponentials.  The buffers are arrays of their own: the
// compiler then knows that a read of one need not wait for the loads into the others.
//
// 8 x 675 tokens, 32 heads (64 stages a workgroup): kernel above 47.2 us; this one with all reads and loads at the head of a stage
// 34.8, spread 30.8.  Bound by what one wavefront issues per stage (850 cycles), loads alone take 540.  With the heads in two
// shares of four wavefronts each (two a SIMD) 37.7 and 33.0: LDS, and the zero tiles wait for a place.
constexpr int kDeepRows = 2 * 2 * kQkB + kQkKeys, kDeepCh = 8;      // queries, then keys, of a stage of 64 features
__global__ __launch_bounds__(kQkWaves * kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void qk_mean_deep_kernel(QkArgs a) {
  constexpr int QR = 4 * kQkB, CH = kDeepCh, T = kQkWaves * kWave, RPI = T / CH, NL = kDeepRows / RPI, KT = 4;
  static_assert(kDeepRows % RPI == 0 && QR % RPI == 0 && NL == 6, "whole rounds of queries and of keys; the loads that are waited for");
  __shared__ u32x4_t buf0[kDeepRows * CH], buf1[kDeepRows * CH], buf2[kDeepRows * CH];
  const int units = a.nb * a.q_groups * a.k_tiles;
  const int unit = xcd_logical_id(blockIdx.x, units);
  if (unit >= units) return;
  const int tid = threadIdx.x, lane = tid % kWave, l32 = lane % kQkB, hi = lane / kQkB;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave), wq = wv / 2, wk = wv % 2;
  const int64_t bi = unit / (a.k_tiles * a.q_groups), b = a.b0 + bi;
  int kt0, w0;
  qk_tile(a, unit - (int)bi * a.k_tiles * a.q_groups, causal_live_first(units, a.k_tiles), QR, kt0, w0);
  const int q0 = wq * 2 * kQkB, v0 = w0 + q0, wk0 = kt0 * kQkKeys, ik0 = wk0 + wk * kQkB;
  const bool live = a.vis0 + wk0 <= a.row(min(w0 + QR, a.nq) - 1);      // uniform in the workgroup: some query sees some key
  if (a.nq - w0 <= kQkB) {                             // uniform in the workgroup
    static_assert(sizeof(buf0) >= kQkWaves * kWave * sizeof(f32x16_t), "the wavefronts' sums");
    qk_mean_narrow<4, true, kQkWaves>(a, bi, b, w0, wk0, wv, live, (f32x16_t*)buf0);
    return;
  }
  f32x16_t P[2] = {qk_zero(), qk_zero()};
  if (live) {
    const bf16_t* src[NL];                             // this thread's chunk of the stage's rows: queries, then keys
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = tid / CH + i * RPI;
      const int row = r < QR ? a.row(min(w0 + r, a.nq - 1)) : a.vis0 + min(wk0 + r - QR, a.N - 1);
      src[i] = (i * RPI < QR ? a.Q : a.K) + b * a.sb + (int64_t)row * a.sn + (tid % CH ^ (tid / 16 & (CH - 1))) * 8;
    }
    float scale = a.scale_log2e;
    asm volatile("" : "+s"(scale));
    const float2* nrm = a.norm + bi * a.H * a.nq;
    uint32_t nrm_at[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) nrm_at[m] = (uint32_t)min(v0 + m * kQkB + l32, a.nq - 1);
    auto load_stage = [&](int h, int part, u32x4_t* buf, int only = -1) __attribute__((always_inline)) {
      int64_t off = (int64_t)min(h, a.H - 1) * a.sh + part * 64;      // (past the last head: that one again)
      asm volatile("" : "+s"(off));
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        if (only >= 0 && i != only) continue;
        asm volatile("" : "+v"(src[i]));
        load_to_lds(src[i] + off, buf + i * T + wv * kWave);
      }
    };
    auto load_nf = [&](int h, float2 (&n)[2]) __attribute__((always_inline)) {
#pragma unroll
      for (int m = 0; m < 2; ++m) n[m] = (nrm + (int64_t)min(h, a.H - 1) * a.nq)[nrm_at[m]];
      issue_fence();
    };
    // Where a lane's fragments lie in a buffer: with the same swizzle for every 32 rows they differ by constants.  (Taken anew for
    // every stage: formed ahead of the loop for each buffer, the addresses spill.)
    int at_q[KT], at_k[KT];                            // in bytes
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      at_q[kt] = lds_chunk<CH>(q0 + l32, kt * 2 + hi) * 16;
      at_k[kt] = lds_chunk<CH>(QR + wk * kQkB + l32, kt * 2 + hi) * 16;
    }
    struct Frags { bf16x8_t k[KT], q[2][KT]; };
    auto read = [&](const u32x4_t* buf, Frags& f, int only = -1) __attribute__((always_inline)) {
      const char* st = (const char*)buf;
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          if (only >= 0 && kt * 3 + r != only) continue;
          if (r == 0) {
            asm volatile("" : "+v"(at_k[kt]));
            f.k[kt] = *(const bf16x8_t*)(st + at_k[kt]);
          } else {
            asm volatile("" : "+v"(at_q[kt]));
            f.q[r - 1][kt] = *(const bf16x8_t*)(st + at_q[kt] + (r - 1) * kQkB * CH * 16);
          }
        }
      }
    };
    f32x16_t S[2][2];                                  // logits of even and odd heads
    S[1][0] = S[1][1] = qk_zero();
    float2 nf[3][2];                                   // normalisers of three heads in turn
#pragma unroll
    for (int m = 0; m < 2; ++m) nf[2][m] = make_float2(__builtin_huge_valf(), 0.0f);    // (nothing before the first head: 2^-inf, times zero)
    auto x_of = [&](const f32x16_t& Sd, float2 n, int v) { return fmaf(Sd[v], scale, -n.x); };
    // The products of one stage beside the exponentials of one block of the head before, the reads of the next stage's
    // fragments and the loads of a stage further on (`side`, in seventeen parts): all in one stream, as a wavefront whose reads
    // stand at the head waits there until LDS has taken those of the others.
    auto multiply = [&](const Frags& f, f32x16_t (&Sn)[2], bool fresh, const f32x16_t& Sd, float2 n, f32x16_t& Pd, auto side) __attribute__((always_inline)) {
      constexpr int E = kQkE, M = 2 * KT;
      float x[2] = {x_of(Sd, n, 0), x_of(Sd, n, 1)}, e_prev = 0.0f;
      issue_fence();
#pragma unroll
      for (int i = 0; i <= E; ++i) {
        float e = 0.0f;
#pragma unroll
        for (int m = 0; m < M; ++m)
          if (m * E / M == i) {
            const int kt = m / 2, blk = m % 2;
            Sn[blk] = qk_mfma(f.k[kt], f.q[blk][kt], fresh && kt == 0 ? qk_zero() : Sn[blk]);
          }
        if (i < E) e = __builtin_amdgcn_exp2f(x[i % 2]);
        if (i + 2 < E) x[i % 2] = x_of(Sd, n, i + 2);
        side(i);
        if (i > 0) Pd[i - 1] = fmaf(e_prev, n.y, Pd[i - 1]);
        issue_fence();
        e_prev = e;
      }
    };
    Frags fr[2];
    // Stage 2 h + part (j: h modulo 6, the turn of buffers and registers): its fragments have been read.  The next stage's rows
    // have arrived once all but the last eight loads have (the six of the stage after it and two normalisers); the buffer of this
    // stage, whose fragments every wavefront has by the barrier, is filled three stages ahead.
    auto buf = [&](auto s_c) { constexpr int s = decltype(s_c)::value % 3; return s == 0 ? buf0 : s == 1 ? buf1 : buf2; };
    auto stage = [&](int h, auto j_c, auto part_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value, part = decltype(part_c)::value, s = 2 * j + part;
      issue_fence();
      __builtin_amdgcn_s_waitcnt(0x0078);              // lgkmcnt(0), vmcnt(8)
      asm volatile("s_barrier" ::: "memory");
      const u32x4_t* after = buf(std::integral_constant<int, s + 1>{});
      u32x4_t* own = buf(std::integral_constant<int, s>{});
      multiply(fr[part], S[j % 2], part == 0, S[1 - j % 2][part], nf[(j + 2) % 3][part], P[part], [&](int i) __attribute__((always_inline)) {
        if (i < 12) read(after, fr[1 - part], i);
        if (i >= 1 && i <= 11 && i % 2 == 1) load_stage(h + (part + 3) / 2, (part + 1) % 2, own, i / 2);
        if (part == 1 && i == 13) load_nf(h + 1, nf[(j + 1) % 3]);
      });
    };
    auto head = [&](int h, auto j_c) __attribute__((always_inline)) {
      stage(h, j_c, std::integral_constant<int, 0>{});
      stage(h, j_c, std::integral_constant<int, 1>{});
    };
    load_stage(0, 0, buf0);
    load_stage(0, 1, buf1);
    load_stage(1, 0, buf2);
    load_nf(0, nf[0]);
    __builtin_amdgcn_s_waitcnt(0x0f7e);                // vmcnt(14): the first stage's loads
    asm volatile("s_barrier" ::: "memory");
    read(buf0, fr[0]);
    int h = 0;
    // Whole turns with no way out in between: the compiler would wait for every load at the loop's head.
#pragma unroll 1
    for (; h + 6 <= a.H; h += 6) {
      head(h, std::integral_constant<int, 0>{});
      head(h + 1, std::integral_constant<int, 1>{});
      head(h + 2, std::integral_constant<int, 2>{});
      head(h + 3, std::integral_constant<int, 3>{});
      head(h + 4, std::integral_constant<int, 4>{});
      head(h + 5, std::integral_constant<int, 5>{});
    }
    if (h < a.H) head(h, std::integral_constant<int, 0>{});
    if (h + 1 < a.H) head(h + 1, std::integral_constant<int, 1>{});
    if (h + 2 < a.H) head(h + 2, std::integral_constant<int, 2>{});
    if (h + 3 < a.H) head(h + 3, std::integral_constant<int, 3>{});
    if (h + 4 < a.H) head(h + 4, std::integral_constant<int, 4>{});
    __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt(0): nothing may arrive in LDS after the workgroup's end
    auto last = [&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value;
      if ((a.H - 1) % 6 != j) return;                  // uniform
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < kQkE; ++v) P[m][v] = fmaf(__builtin_amdgcn_exp2f(x_of(S[j % 2][m], nf[j % 3][m], v)), nf[j % 3][m].y, P[m][v]);
    };
    last(std::integral_constant<int, 0>{});
    last(std::integral_constant<int, 1>{});
    last(std::integral_constant<int, 2>{});
    last(std::integral_constant<int, 3>{});
    last(std::integral_constant<int, 4>{});
    last(std::integral_constant<int, 5>{});
  }
  if (v0 < a.nq) qk_write_out<true, 2>(a, b, v0, ik0, P[0], P[1]);
}

template <int KS, bool DEC>
static void launch_qk(QkArgs a, hipStream_t s) {
  constexpr int CH = (KS > 2 ? 2 : KS) * 4;
  const int tiles = (a.nq + kNormTile - 1) / kNormTile;
  a.q_groups = (tiles + kQkWaves - 1) / kQkWaves;
  // Few workgroups: one tile each, whose keys the wavefronts share.  Fewer than one per compute unit for heads of 64, 192 for heads
  // of 128, whose steps are longer, 640 for heads of 32.  us of the two kernels, whole tiles per wavefront and shared:
  // heads of 64, 1 image of 577 tokens and 2 heads 20.0 / 14.6, 12 and 1 21.1 / 15.6, 16 of 197 and 6 (192 workgroups)
  // 16.4 / 15.8, 12 of 577 and 12 (576) 35.4 / 43.8; of 128, 16 of 197 and 4 (128) 18.2 / 17.6, 12 of 577 and 4 (192) 34.3 / 38.0,
  // 12 of 1025 and 3 (216) 54 / 69; of 32, 12 of 1025 and 4 (288) 39.4 / 34.3, 12 of 577 and 12 (576) 29.9 / 30.1, 20 (960) 39.4 / 43.0.
  // Over 700 shapes, shared relative to whole by the number of workgroups: heads of 64 0.98 at 192 to 256 and 1.03 at 256 to 320; of
  // 128 1.00 at 128 to 192 and 1.09 at 192 to 256; of 32 0.995 at 448 to 640 and 1.05 at 640 to 1024.
  a.share_keys = (int64_t)a.nb * a.H * a.q_groups < (KS == 1 ? 640 : KS == 2 ? 256 : 192);
  if (a.share_keys) a.q_groups = tiles;
  const bool narrow = a.nq - (a.q_groups - 1) * (a.share_keys ? 1 : kQkWaves) * kNormTile <= 16;      // (as the kernel sees it)
  const int groups = a.q_groups - (narrow ? 1 : 0);
  // Causal maps: the groups that see most keys come first, one group of every head after the other.  (Group by group of a head
  // the workgroups that meet on a compute unit are of one length wherever the groups divide the 32 units of an XCD: 8 x 675 tokens, 32
  // heads of 128 45.7 us, and 38.3 so.  With shared keys the short ones go first: 16 heads, one image of 675 32.3, else 36.2 for the stage.)
  auto keys_seen = [&](int g) { return a.row(std::min((g + 1) * kQkWaves * kNormTile, a.nq) - 1) + 1; };
  a.long_first = DEC && !a.share_keys && groups > 1 && causal_long_first(keys_seen(0), keys_seen(groups - 1));
  hipLaunchKernelGGL((qk_norm_kernel<KS, DEC>), dim3(norm_grid(a, a.nb * a.H, groups) + (narrow ? xcd_padded_total(a.nb * a.H) : 0)), dim3(kQkWaves * kWave), 0, s, a);
  auto mean = [&](auto kern, auto shape) {
    using Shape = decltype(shape);
    // two stages of (queries + keys) rows per share of the heads, and the queries' normalisers of two heads
    constexpr size_t kStages = 2 * Shape::kShares * ((size_t)(Shape::kQueries + kQkKeys) * CH * sizeof(u32x4_t) + Shape::kQueries * sizeof(float2));
    constexpr size_t kSums = (size_t)Shape::kThreads * sizeof(f32x16_t);      // (of a narrow tile, at most)
    constexpr size_t kLds = kStages > kSums && !Shape::narrow_only(KS, DEC) ? kStages : kSums;
    if (kLds > 32768)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    a.q_groups = (a.nq + Shape::kQueries - 1) / Shape::kQueries;
    hipLaunchKernelGGL(kern, dim3(xcd_padded_total(a.nb * a.q_groups * a.k_tiles)), dim3(Shape::kThreads), kLds, s, a);
  };
  // Fewer than a workgroup of the wide form for every other compute unit: the heads of a tile are split instead, eight or more
  // (with fewer, the sixteen wavefronts of a split tile cost more than the heads they share).  us of the two kernels, split and wide:
  // one image of 577 tokens, 45 workgroups, 2 heads of 64 14.5 / 13.1, 8 15.8 / 16.7, 12 of 32 14.6 / 16.1; two images, 32 of 32
  // 21.0 / 27.8; three, 135 workgroups, 8 of 64 25.6 / 19.2, 32 of 32 34.1 / 30.9.  Over 700 shapes, split relative to wide below 64 and
  // at 64 to 128 workgroups: one head 1.20, 1.20; four 1.08, 1.08; six 1.06, 1.05; eight 1.00, 0.98; twelve 0.93, 0.90; 32 0.81, 0.77; at
  // 160 and more wide is the better one up to twenty heads.
  const int wide = QkMeanShape<false>::kQueries, q_tiles = (a.nq + wide - 1) / wide;
  const bool split = a.H >= 8 && (int64_t)a.nb * q_tiles * a.k_tiles < 128;
  if constexpr (DEC && KS == 4) {
    // Heads of 128: the form with rows three stages ahead in place of the wide one, the same bits, but for one block of queries, whose heads
    // the wavefronts share.  us of the two kernels, this form and the wide one: 32 heads, 8 x (576 + 64) queries 61.3 / 87.5, 4
    // images (180 tiles) 44.5 / 68.0, 2 x (630 + 200) (140) 46.4 / 71.3; 16 heads, 8 x (576 + 64) 38.0 / 50.6.  Not in place of split
    // heads: about as fast there (32 heads, one image of 576 + 64 38.0 / 39.0, 8 x (96 + 17) 31.9 / 29.1), but all heads in line take the
    // error of the scores against 64 bits from 3.20e-8 to 3.56e-8 (32 heads, 576 + 64), and with sums of three heads, which keep it, 42.9 us
    // instead of 40.9 at one image and 44.7 instead of 43.0 at two.
    if (a.nq > kQkB && !split) {
      a.q_groups = q_tiles;
      hipLaunchKernelGGL(qk_mean_deep_kernel, dim3(xcd_padded_total(a.nb * a.q_groups * a.k_tiles)), dim3(kQkWaves * kWave), 0, s, a);
      return;
    }
  }
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
