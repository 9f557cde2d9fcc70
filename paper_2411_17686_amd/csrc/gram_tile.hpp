// bf16 MFMA tile kernel for the cosine correlation (the one dense contraction of the path):
//   Ct[b][a][j] = xh[b][S[b][a]] . xh[b][T[b][j]]      (float accumulation)
// for the discarded rows a and preserved columns j of every image, xh = unit rows rounded to
// bfloat16.  The result only PROPOSES candidates: every value that can decide a threshold
// is afterwards recomputed in double precision, so the order in which the matrix core adds
// does not matter for the outcome.
//
// 128 x 128 output tile per workgroup (4 wavefronts, 64 x 64 each = 2 x 2 blocks of
// v_mfma_f32_32x32x16_bf16), K staged through LDS 32 at a time,
// double buffered, rows gathered by index.  LDS rows are padded by 16 bytes so that the
// 16-byte fragment reads of a quarter wavefront fall on distinct banks.
//
// What bounds it: with few tiles the chain of a stage (fragments, eight products, stores to LDS, barrier: 850 cycles of a lone
// workgroup), with many the rows and the partial blocks, about 7 TB/s between 8 and 16 images of 432 x 144 with 4096 features
// (17.2 and 25.0 us).  Of 1 image, in 16 ranges of K: 8.7 us; in 8 ranges 11.6, and 12.7 while its loads were under a condition.
#pragma once
#include "common.hpp"

namespace ficoco {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kGT = 128;           // tile rows = tile columns
constexpr int kGK = kGramStage;    // K elements per stage (32 measured best at 4096 tokens; 64 halves LDS occupancy)
constexpr int kGChunks = kGK / 16;  // 16-byte chunks per thread, operand and stage
constexpr int kGStride = kGK + 8;  // LDS row pitch in elements (row + 16 bytes)
constexpr int kGStages = 2;   // K-stages in flight per thread (register ring)

static __device__ const uint4 g_zero_chunk = {0, 0, 0, 0};

struct GramArgs {
  const bf16_t* xhat;  // [B][N][Df]
  int B, N, Df, n_disc, n_keep;
  const int32_t* S;    // [B][n_disc]
  const int32_t* T;    // [B][n_keep]
  float* ct;           // [splits][B][n_disc][n_keep]: partial sums over the K ranges of the splits
  int splits, st_per_split;   // K is cut into `splits` ranges of st_per_split stages (the last may be shorter)
};

__global__ __launch_bounds__(256) void gram_tile_kernel(GramArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t As[2][kGT * kGStride];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[2][kGT * kGStride];
  __shared__ int rowA[kGT];
  __shared__ int rowB[kGT];
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int tiles_m = (a.n_disc + kGT - 1) / kGT, tiles_n = (a.n_keep + kGT - 1) / kGT;
  const int per_split = a.B * tiles_m * tiles_n;
  const int total = per_split * a.splits;
  int logical = xcd_logical_id(blockIdx.x, total);
  if (logical >= total) return;   // padding workgroup
  const int split = logical / per_split;
  logical %= per_split;
  const int64_t b = logical / (tiles_m * tiles_n);
  const int tm = (logical % (tiles_m * tiles_n)) / tiles_n, tn = logical % tiles_n;

  if (tid < kGT) {
    const int r = tm * kGT + tid;
    const int i = r < a.n_disc ? a.S[b * a.n_disc + r] : -1;
    rowA[tid] = (unsigned)i < (unsigned)a.N ? i : -1;      // index sets are device data
  } else {
    const int c = tn * kGT + tid - kGT;
    const int j = c < a.n_keep ? a.T[b * a.n_keep + c] : -1;
    rowB[tid - kGT] = (unsigned)j < (unsigned)a.N ? j : -1;
  }
  __syncthreads();

  // this split's K range, [k_begin, k_begin + k_len)
  const int k_begin = split * a.st_per_split * kGK;
  const int k_len = max(min(a.Df - k_begin, a.st_per_split * kGK), 0);
  // loader: the stage is 128 rows x kGK/8 chunks of 8 elements per operand; thread -> one chunk of kGChunks rows each.
  // A row of no token, and a chunk past the range, is loaded from a chunk of zeros: with the loads under a condition the compiler
  // waited for each where its values joined the zeros of the other way, one latency of memory a stage.
  const uint64_t xb = (uint64_t)(a.xhat + b * a.N * (int64_t)a.Df + k_begin), zeros = (uint64_t)&g_zero_chunk;
  const int lkc = tid % (kGK / 8) * 8;
  int lrow[kGChunks];
  uint64_t srcA[kGChunks], srcB[kGChunks];        // of the next stage to fetch
  uint32_t stepA[kGChunks], stepB[kGChunks];
#pragma unroll
  for (int u = 0; u < kGChunks; ++u) {
    lrow[u] = (tid + 256 * u) / (kGK / 8);
    const int ia = rowA[lrow[u]], ib = rowB[lrow[u]];
    srcA[u] = ia >= 0 ? xb + 2 * ((int64_t)ia * a.Df + lkc) : zeros;
    srcB[u] = ib >= 0 ? xb + 2 * ((int64_t)ib * a.Df + lkc) : zeros;
    stepA[u] = ia >= 0 ? 2 * kGK : 0;
    stepB[u] = ib >= 0 ? 2 * kGK : 0;
  }
  // Register ring of kGStages K-stages in flight per thread: a stage is fetched kGStages
  // iterations before it is stashed into LDS.
  u32x4_t ra[kGStages][kGChunks], rb[kGStages][kGChunks];
  const int n_st = (k_len + kGK - 1) / kGK;
  auto get = [](uint64_t at) { return *(const __attribute__((address_space(1))) u32x4_t*)at; };
  auto fetch = [&](int slot, int st) {
    const bool in = st * kGK + lkc + 8 <= k_len;   // Df is a multiple of 8 on this path
#pragma unroll
    for (int u = 0; u < kGChunks; ++u) {
      ra[slot][u] = get(in ? srcA[u] : zeros);
      rb[slot][u] = get(in ? srcB[u] : zeros);
      srcA[u] += stepA[u];
      srcB[u] += stepB[u];
    }
  };
  auto stash = [&](int slot, int buf) {
#pragma unroll
    for (int u = 0; u < kGChunks; ++u) {
      *reinterpret_cast<u32x4_t*>(&As[buf][lrow[u] * kGStride + lkc]) = ra[slot][u];
      *reinterpret_cast<u32x4_t*>(&Bs[buf][lrow[u] * kGStride + lkc]) = rb[slot][u];
    }
  };

  f32x16_t acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;

  const int wm = wv / 2, wn = wv % 2;
  const int frow = lane % 32, fk = (lane / 32) * 8;   // fragment: row / column within the block, k offset
#pragma unroll
  for (int sl = 0; sl < kGStages; ++sl) fetch(sl, sl);
  stash(0, 0);
  __syncthreads();
  int cur = 0;
  for (int base = 0; base < n_st; base += kGStages) {
#pragma unroll
    for (int sl = 0; sl < kGStages; ++sl) {
      const int it = base + sl;
      if (it < n_st) {                          // uniform over the workgroup
        fetch(sl, it + kGStages);               // slot sl was stashed one iteration ago
#pragma unroll
        for (int kk = 0; kk < kGK; kk += 16) {
          bf16x8_t fa[2], fb[2];
#pragma unroll
          for (int mi = 0; mi < 2; ++mi)
            fa[mi] = *reinterpret_cast<const bf16x8_t*>(&As[cur][(wm * 64 + mi * 32 + frow) * kGStride + kk + fk]);
#pragma unroll
          for (int ni = 0; ni < 2; ++ni)
            fb[ni] = *reinterpret_cast<const bf16x8_t*>(&Bs[cur][(wn * 64 + ni * 32 + frow) * kGStride + kk + fk]);
#pragma unroll
          for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
              acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mi], fb[ni], acc[mi][ni], 0, 0, 0);
        }
        if (it + 1 < n_st) {
          stash((sl + 1) % kGStages, cur ^ 1);  // the other buffer was last read before the previous barrier
          __syncthreads();
          cur ^= 1;
        }
      }
    }
  }

  // C block layout of the 32x32 MFMA: lane holds column lane%32; register v holds row
  // 8*(v/4) + 4*(lane/32) + v%4.
  float* ctb = a.ct + ((int64_t)split * a.B + b) * a.n_disc * (int64_t)a.n_keep;   // this split's block of image b
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      const int col = tn * kGT + wn * 64 + ni * 32 + lane % 32;
      const int row0 = tm * kGT + wm * 64 + mi * 32 + 4 * (lane / 32);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + 8 * (v / 4) + v % 4;
        if (row < a.n_disc && col < a.n_keep) ctb[row * a.n_keep + col] = acc[mi][ni][v];   // below 2^31: n_disc * n_keep < 12288^2
      }
    }
}

// ---- the same product for large blocks ---------------------------------------------------------
// 192 x 192 output tile per workgroup of four wavefronts (2 x 2), 96 x 96 per wavefront = 3 x 3 blocks of
// v_mfma_f32_32x32x16_bf16, one wavefront per SIMD: six fragment reads feed nine matrix instructions.
// Whole rows go from memory straight into LDS, 64 features at a time, three stages ahead (144 KB);
// the fragments of the next sixteen features are read while the matrix cores work on the ones before, across the one barrier of
// a stage too.  LDS rows are the 128 bytes of a stage with no padding; the eight 16-byte chunks of row r sit at
// chunk ^ ((r >> 1) & 7), which keeps the fragment reads (sixteen consecutive rows, one chunk) free of bank conflicts; a
// load fills LDS in the order of the lanes, so it is its source that is permuted.
//
// What bounds it: the matrix cores and, since all workgroups end together, the output.  8064 x 1152 x 1024 (252 tiles, one
// round): 28.3 us; without the stores 21.8, without the loads inside the loop 24, without both 16.5; the 37 MB of output alone
// are 7 us at the rate of a large copy, the product 15.5 us at the rate of a large library product.  Before (256 x 192 tiles of eight
// wavefronts through registers into LDS, one stage ahead): 34.2 us; 8064 x 1152 x 3584: 90 us before, 69 now; two images of
// it: 59.5 before, 50 now.  Two buffers in place of three: 27.8 us here, but 64 images of 768 x 384 x 1024
// (rows out of HBM) 74 us instead of 64.
constexpr int kG2M = 192, kG2N = 192, kG2K = 64;
constexpr int kG2Threads = 256;
constexpr int kG2Chunks = kG2K / 8;        // 16-byte chunks per operand row and stage
__device__ __forceinline__ int g2_slot(int row, int chunk) { return row * kG2Chunks + (chunk ^ ((row >> 1) & 7)); }

__global__ __launch_bounds__(kG2Threads) __attribute__((amdgpu_waves_per_eu(1, 1))) void gram_tile2_kernel(GramArgs a) {
  static_assert(kG2Chunks == 8 && kG2K == 64, "the swizzle spreads eight chunks; four products of sixteen features a stage");
  constexpr int MB = kG2M / 64, kRows = kG2M + kG2N;
  constexpr int kLoads = kRows * kG2Chunks / kG2Threads;  // per thread and stage: rows of A, then of B
  __shared__ uint4 buf0[kRows * kG2Chunks], buf1[kRows * kG2Chunks], buf2[kRows * kG2Chunks];
  __shared__ int tok[kRows];                              // of the rows of A, then of B
  const int tid = threadIdx.x, lane = tid % kWave, l32 = lane % 32, hi = lane / 32;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave), wm = wv / 2, wn = wv % 2;
  const int tiles_m = (a.n_disc + kG2M - 1) / kG2M, tiles_n = (a.n_keep + kG2N - 1) / kG2N;
  const int per_split = a.B * tiles_m * tiles_n, total = per_split * a.splits;
  int logical = xcd_logical_id(blockIdx.x, total);           // the column tiles of the same rows share an XCD
  if (logical >= total) return;   // padding workgroup
  const int split = logical / per_split;
  logical %= per_split;
  const int64_t b = logical / (tiles_m * tiles_n);
  const int tm = (logical % (tiles_m * tiles_n)) / tiles_n, tn = logical % tiles_n;
  bool mine = true;
  for (int q = tid; q < kRows; q += kG2Threads) {
    const int r = q < kG2M ? tm * kG2M + q : tn * kG2N + q - kG2M;
    const int t = q < kG2M ? (r < a.n_disc ? a.S[b * a.n_disc + r] : -1) : (r < a.n_keep ? a.T[b * a.n_keep + r] : -1);
    tok[q] = (unsigned)t < (unsigned)a.N ? t : -1;         // index sets are device data
    mine &= tok[q] >= 0;
  }
  const bool whole = __syncthreads_and(mine);              // every row and column of the tile is a token's

  const int k_begin = split * a.st_per_split * kGramStage;
  const int k_len = max(min(a.Df - k_begin, a.st_per_split * kGramStage), 0);
  const int n_st = k_len / kG2K;                            // whole stages; what is left is a stage of its own
  // A row past the block, or of no token, reads token 0 (its values are not used).
  const bf16_t* xb = a.xhat + b * a.N * (int64_t)a.Df + k_begin;
  int64_t src[kLoads];                                    // in bytes
  const int chunk = (tid % kG2Chunks ^ (tid / 16 % kG2Chunks)) * 8;
#pragma unroll
  for (int i = 0; i < kLoads; ++i)
    src[i] = ((int64_t)max(tok[tid / kG2Chunks + i * (kG2Threads / kG2Chunks)], 0) * a.Df + chunk) * 2;
  auto load = [&](int i, const void* from, uint4* buf) __attribute__((always_inline)) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from,
                                     (__attribute__((address_space(3))) void*)(buf + i * kG2Threads + wv * kWave), 16, 0, 0);
  };
  auto fetch = [&](int st, uint4* buf) __attribute__((always_inline)) {
    const char* at = (const char*)(xb + min(st, n_st - 1) * kG2K);   // past the last stage: that one again, so that the counts below hold
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(i, at + src[i], buf);
    issue_fence();                                          // the loads of the stages stay in their order
  };

  f32x16_t acc[MB][3];
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int ni = 0; ni < 3; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;

  bf16x8_t fr[2][MB + 3];                                   // fragments of sixteen features, of A and then of B; the next ones ahead
  auto read = [&](const uint4* buf, int kk, bf16x8_t (&f)[MB + 3]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < MB + 3; ++q)
      f[q] = ((const bf16x8_t*)buf)[g2_slot((q < MB ? wm * kG2M / 2 + q * 32 : kG2M + wn * 96 + (q - MB) * 32) + l32, kk * 2 + hi)];
  };
  auto multiply = [&](const bf16x8_t (&f)[MB + 3]) __attribute__((always_inline)) {
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
      for (int ni = 0; ni < 3; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[mi], f[MB + ni], acc[mi][ni], 0, 0, 0);
    issue_fence();
  };
  // One stage, its first fragments already read: before its last nine products the wavefronts meet, all done with `buf`
  // and the next stage arrived (the twelve loads of the one after may be on their way); `buf` is filled three stages ahead.
  auto stage = [&](int st, uint4* buf, const uint4* next) __attribute__((always_inline)) {
    // the fragments asked for a group of products ago are waited for before the next ones are asked for
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
      __builtin_amdgcn_s_waitcnt(0xc07f);                    // lgkmcnt(0)
      read(buf, kk + 1, fr[(kk + 1) & 1]);
      issue_fence();
      multiply(fr[kk & 1]);
    }
    __builtin_amdgcn_s_waitcnt(0x0070 | kLoads);          // lgkmcnt(0), vmcnt: all but the loads of the stage after the next
    asm volatile("s_barrier" ::: "memory");
    read(next, 0, fr[0]);
    issue_fence();
    fetch(st + 3, buf);
    multiply(fr[1]);
  };
  if (n_st > 0) {                                           // uniform over the workgroup
    issue_fence();
    fetch(0, buf0);
    fetch(1, buf1);
    fetch(2, buf2);
    __builtin_amdgcn_s_waitcnt(0x4070 | (2 * kLoads & 15)); // lgkmcnt(0), vmcnt: all but the later two stages' loads
    asm volatile("s_barrier" ::: "memory");
    read(buf0, 0, fr[0]);
    int st = 0;
    // Whole turns of the buffers with no way out in between: the compiler would wait for every load at the loop's head.
    for (; st + 2 < n_st; st += 3) {
      stage(st, buf0, buf1);
      stage(st + 1, buf1, buf2);
      stage(st + 2, buf2, buf0);
    }
    if (st < n_st) stage(st, buf0, buf1);
    if (st + 1 < n_st) stage(st + 1, buf1, buf2);
    __builtin_amdgcn_s_waitcnt(0x0f70);                     // vmcnt(0): nothing may arrive in LDS after the workgroup's end
  }
  if (n_st * kG2K < k_len) {                                // less than a stage left: chunks past the range are zeros
    __syncthreads();
    const bool in = n_st * kG2K + chunk + 8 <= k_len;       // Df is a multiple of 8 on this path
    const char* at = (const char*)(xb + n_st * kG2K);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(i, in ? at + src[i] : (const char*)&g_zero_chunk, buf0);
    __builtin_amdgcn_s_waitcnt(0x0f70);                     // vmcnt(0)
    __syncthreads();
#pragma unroll 1
    for (int kk = 0; kk < kG2K / 16; ++kk) {
      read(buf0, kk, fr[0]);
      multiply(fr[0]);
    }
  }

  // C block layout of the 32x32 MFMA: lane holds column lane%32; register v holds row
  // 8*(v/4) + 4*(lane/32) + v%4.
  float* ctb = a.ct + ((int64_t)split * a.B + b) * a.n_disc * (int64_t)a.n_keep;
  if (whole) {                                              // uniform over the workgroup
    const int row0 = tm * kG2M + wm * (kG2M / 2), col0 = tn * kG2N + wn * 96;
    const uint32_t at = (uint32_t)(4 * hi * a.n_keep + l32);
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float* dst = ctb + (int64_t)(row0 + mi * 32 + 8 * (v / 4) + v % 4) * a.n_keep + col0;
#pragma unroll
        for (int ni = 0; ni < 3; ++ni) dst[at + ni * 32] = acc[mi][ni][v];
      }
    return;
  }
  // An edge: whole groups of eight rows without a check of each.  (With a look at the rows' tokens before every group of
  // stores, 260 images of 98 x 98, all edges, took 22.8 us instead of 18.8.)
#pragma unroll
  for (int ni = 0; ni < 3; ++ni) {
    const int lc = wn * 96 + ni * 32 + l32, col = tn * kG2N + lc;
    if (col >= a.n_keep) continue;
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int lr = wm * (kG2M / 2) + mi * 32 + 8 * g, row = tm * kG2M + lr;
        if (row >= a.n_disc) break;                         // uniform, as is the next one
        float* dst = ctb + (int64_t)row * a.n_keep + (uint32_t)(4 * hi * a.n_keep + col);
        const float c0 = acc[mi][ni][4 * g], c1 = acc[mi][ni][4 * g + 1];
        const float c2 = acc[mi][ni][4 * g + 2], c3 = acc[mi][ni][4 * g + 3];
        if (row + 8 <= a.n_disc) {
          dst[0] = c0, dst[a.n_keep] = c1, dst[2 * (int64_t)a.n_keep] = c2, dst[3 * (int64_t)a.n_keep] = c3;
        } else {
          const int left = a.n_disc - row - 4 * hi;
          if (left > 0) dst[0] = c0;
          if (left > 1) dst[a.n_keep] = c1;
          if (left > 2) dst[2 * (int64_t)a.n_keep] = c2;
          if (left > 3) dst[3 * (int64_t)a.n_keep] = c3;
        }
      }
  }
  // Zeros where a row or column of the block is of no token (rare), behind the stores above, of all wavefronts.
  const int rows = min(kG2M, a.n_disc - tm * kG2M), cols = min(kG2N, a.n_keep - tn * kG2N);
  bool none = false;
  for (int q = tid; q < kRows; q += kG2Threads) none |= tok[q] < 0 && (q < kG2M ? q < rows : q - kG2M < cols);
  __builtin_amdgcn_s_waitcnt(0x0f70);                       // vmcnt(0)
  if (!__syncthreads_or(none)) return;
  for (int q = tid; q < rows * cols; q += kG2Threads) {
    const int r = q / cols, c = q % cols;
    if (tok[r] < 0 || tok[kG2M + c] < 0) ctb[(int64_t)(tm * kG2M + r) * a.n_keep + tn * kG2N + c] = 0.0f;
  }
}

// ---- a taller tile ---------------------------------------------------------------------------------
// 256 x 192 output tile per workgroup of 8 wavefronts (4 x 2), 64 x 96 per wavefront = 2 x 3 blocks
// of v_mfma_f32_32x32x16_bf16: five fragment reads feed six matrix instructions.  Rows come through registers, a stage of
// 64 features ahead, into LDS laid out as above; the loader's stores (consecutive lanes = consecutive chunks of consecutive
// rows) are free of bank conflicts too.  Two wavefronts per SIMD hide each other's waits at the head of a tile and its stores at the
// end, so it is the better one where tiles are short or come in several rounds.  us with 256 rows by four wavefronts as above
// and by these eight: 36 images of 768 x 384, 4096 features 126 and 117; 64 of 1000 x 150, 4096 170 and 154; 128 of
// 432 x 144, 256 features 20.8 and 15.7.
constexpr int kTallM = 256, kTallThreads = 512;
__global__ __launch_bounds__(kTallThreads) void gram_tall_kernel(GramArgs a) {
  static_assert(kG2Chunks == 8, "the swizzle spreads eight chunks");
  extern __shared__ uint4 rows_lds[];
  uint4* Abuf = rows_lds;                                 // [2][256 rows][8 chunks]
  uint4* Bbuf = rows_lds + 2 * kTallM * kG2Chunks;        // [2][192 rows][8 chunks]
  __shared__ int rowA[kTallM];
  __shared__ int rowB[kG2N];
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int tiles_m = (a.n_disc + kTallM - 1) / kTallM, tiles_n = (a.n_keep + kG2N - 1) / kG2N;
  const int total = a.B * tiles_m * tiles_n;
  const int logical = xcd_logical_id(blockIdx.x, total);     // the column tiles of the same rows share an XCD
  if (logical >= total) return;   // padding workgroup
  const int64_t b = logical / (tiles_m * tiles_n);
  const int tm = (logical % (tiles_m * tiles_n)) / tiles_n, tn = logical % tiles_n;

  if (tid < kTallM) {
    const int r = tm * kTallM + tid;
    const int i = r < a.n_disc ? a.S[b * a.n_disc + r] : -1;
    rowA[tid] = (unsigned)i < (unsigned)a.N ? i : -1;      // index sets are device data
  } else if (tid < kTallM + kG2N) {
    const int c = tn * kG2N + tid - kTallM;
    const int j = c < a.n_keep ? a.T[b * a.n_keep + c] : -1;
    rowB[tid - kTallM] = (unsigned)j < (unsigned)a.N ? j : -1;
  }
  __syncthreads();

  // loader: per stage 2048 chunks of A (four per thread) and 1536 of B (three per thread);
  // chunk q = (row q / 8, 16 bytes q % 8)
  const bf16_t* Xb = a.xhat + b * a.N * (int64_t)a.Df;
  constexpr int kSlotsA = kTallM * kG2Chunks / kTallThreads, kSlotsB = kG2N * kG2Chunks / kTallThreads;
  constexpr int kSlots = kSlotsA + kSlotsB;
  static_assert(kSlotsA * kTallThreads == kTallM * kG2Chunks && kSlotsB * kTallThreads == kG2N * kG2Chunks, "whole slots");
  // Every load of the loader is unconditional: a row past the block reads token 0 and a chunk past
  // the K range reads the row's first chunk (both valid addresses: N >= 1, Df >= 8), and what was
  // read is cleared when it is put into LDS.  Under a per-lane condition the loads sit in
  // branches, and the compiler then waits for ALL outstanding loads before it issues the next
  // stage's -- one stage in flight instead of two, and the wait at the head of every stage
  // (measured here: 33-35 -> 30-33 us; the 128 x 128 kernel above, with four loads per stage, is
  // no faster for it and keeps its conditional loads).
  const bf16_t* src[kSlots];
  bool row_ok[kSlots];
  int lds_at[kSlots], kc[kSlots];
#pragma unroll
  for (int u = 0; u < kSlots; ++u) {
    const bool aop = u < kSlotsA;
    const int q = tid + kTallThreads * (aop ? u : u - kSlotsA);
    const int row = q / kG2Chunks, chunk = q % kG2Chunks;
    const int tok = aop ? rowA[row] : rowB[row];
    kc[u] = chunk * 8;
    lds_at[u] = g2_slot(row, chunk);
    row_ok[u] = tok >= 0;
    src[u] = Xb + (int64_t)max(tok, 0) * a.Df;
  }
  uint4 rg[kGStages][kSlots];
  const int n_st = (a.Df + kG2K - 1) / kG2K;
  auto in_range = [&](int st, int u) { return st < n_st && st * kG2K + kc[u] + 8 <= a.Df; };   // Df is a multiple of 8 on this path
  auto fetch = [&](int slot, int st) {
#pragma unroll
    for (int u = 0; u < kSlots; ++u) __builtin_memcpy(&rg[slot][u], src[u] + (in_range(st, u) ? st * kG2K + kc[u] : 0), 16);
  };
  auto stash = [&](int slot, int buf, int st) {      // st: the stage that slot holds
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const uint4 v = row_ok[u] && in_range(st, u) ? rg[slot][u] : make_uint4(0, 0, 0, 0);
      if (u < kSlotsA) Abuf[buf * kTallM * kG2Chunks + lds_at[u]] = v;
      else Bbuf[buf * kG2N * kG2Chunks + lds_at[u]] = v;
    }
  };

  f32x16_t acc[2][3];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 3; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;

  const int wm = wv / 2, wn = wv % 2;
  const int frow = lane % 32, fch = lane / 32;     // fragment: row within the block, 16-byte chunk within a 16-feature step
#pragma unroll
  for (int sl = 0; sl < kGStages; ++sl) fetch(sl, sl);
  stash(0, 0, 0);
  __syncthreads();
  int cur = 0;
  for (int base = 0; base < n_st; base += kGStages) {
#pragma unroll
    for (int sl = 0; sl < kGStages; ++sl) {
      const int it = base + sl;
      if (it < n_st) {                          // uniform over the workgroup
        fetch(sl, it + kGStages);               // slot sl was stashed one iteration ago
#pragma unroll
        for (int kk = 0; kk < kG2K / 16; ++kk) {
          bf16x8_t fa[2], fb[3];
#pragma unroll
          for (int mi = 0; mi < 2; ++mi) {
            const uint4 t = Abuf[cur * kTallM * kG2Chunks + g2_slot(wm * 64 + mi * 32 + frow, kk * 2 + fch)];
            __builtin_memcpy(&fa[mi], &t, 16);
          }
#pragma unroll
          for (int ni = 0; ni < 3; ++ni) {
            const uint4 t = Bbuf[cur * kG2N * kG2Chunks + g2_slot(wn * 96 + ni * 32 + frow, kk * 2 + fch)];
            __builtin_memcpy(&fb[ni], &t, 16);
          }
#pragma unroll
          for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 3; ++ni)
              acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mi], fb[ni], acc[mi][ni], 0, 0, 0);
        }
        if (it + 1 < n_st) {
          stash((sl + 1) % kGStages, cur ^ 1, it + 1);  // the other buffer was last read before the previous barrier
          __syncthreads();
          cur ^= 1;
        }
      }
    }
  }

  // C block layout of the 32x32 MFMA: lane holds column lane%32; register v holds row
  // 8*(v/4) + 4*(lane/32) + v%4.
  float* ctb = a.ct + b * a.n_disc * (int64_t)a.n_keep;
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 3; ++ni) {
      const int col = tn * kG2N + wn * 96 + ni * 32 + lane % 32;
      const int row0 = tm * kTallM + wm * 64 + mi * 32 + 4 * (lane / 32);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + 8 * (v / 4) + v % 4;
        if (row < a.n_disc && col < a.n_keep) ctb[(int64_t)row * a.n_keep + col] = acc[mi][ni][v];
      }
    }
}

}  // namespace ficoco
