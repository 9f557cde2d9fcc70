// Statistics of the tokens' text profiles (FiCoCo-L): the body shared by select.hip (its own launch
// before the filter kernel) and features.hip (the fused step lets it ride in the launch of the
// column-sum kernel, which does not depend on it).
#pragma once
#include "common.hpp"

namespace ficoco {

// From 32 text queries on: the task term of Eq. 3, the mean of a token's text profile, is formed
// by one wavefront per token on the whole chip (lane sums over k = lane, lane + 64, ..., then a
// fixed tree), so the per-image workgroup of select_kernel reads one value.  A thread of that
// workgroup walking its token's profile touches a cache line per lane and load, all on one
// compute unit (64 queries: 17 us for the select kernel against 9 + 4 us this way).
// In the fused step the same launch also forms cmax[b][k], the maximum over the visual tokens of
// profile entry k (the bound of Eq. 4's indirect term that the correlate stage needs).  The first workgroups take
// kCmaxQueries text queries of one image each, thread (k, g) walking the tokens g, g + 16, ... with 16 independent
// loads per round, the sixteen token groups meeting in LDS: three rounds at 576 tokens, and the cache lines of a row are read whole.
// (64 queries and four token groups a workgroup were nine rounds, one after the other: 7.2 us for the launch at 8 x 576 tokens
// and 64 queries, 4.8 so.)
struct TextStatsArgs {
  const double* ttext;   // [B][N][M]
  int N, M;
  double* out_g;         // [B][N]
  double* cmax;          // [B][M]
  int cmax_blocks, mean_blocks;      // workgroups per image (cmax_blocks = 0: no maxima)
};
constexpr int kCmaxQueries = 16;
void fill_text_stats(const ficoco_problem& p, const Plan& pl, char* ws, bool with_cmax, TextStatsArgs& t);

// mean of the profiles of tokens 4 bx .. 4 bx + 4, a wavefront each
__device__ __forceinline__ void text_mean_block(const TextStatsArgs& a, int bx, int64_t b) {
  const int lane = threadIdx.x % kWave;
  const int i = bx * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (i >= a.N) return;      // whole wavefront leaves together
  const double* __restrict__ p = a.ttext + (b * a.N + i) * a.M;
  double acc = 0.0;
  for (int k = lane; k < a.M; k += kWave) acc += p[k];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (lane == 0) a.out_g[b * a.N + i] = acc / (double)a.M;
}

// maxima of the profile entries kCmaxQueries bx and on (256 threads)
__device__ __forceinline__ void text_cmax_block(const TextStatsArgs& a, int bx, int64_t b) {
  constexpr int kGroups = 256 / kCmaxQueries;
  __shared__ double part[kGroups][kCmaxQueries];
  const int kl = threadIdx.x % kCmaxQueries, g = threadIdx.x / kCmaxQueries, k = bx * kCmaxQueries + kl;
  const double* __restrict__ p = a.ttext + b * a.N * a.M + min(k, a.M - 1);
  double mx = 0.0;
  for (int i0 = g; i0 < a.N; i0 += 16 * kGroups) {     // past the last token that one again
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(int64_t)min(i0 + u * kGroups, a.N - 1) * a.M];
    issue_fence();
#pragma unroll
    for (int u = 0; u < 16; ++u) mx = v[u] > mx ? v[u] : mx;
  }
  part[g][kl] = mx;
  __syncthreads();
  if (g == 0 && k < a.M) {
#pragma unroll
    for (int q = 1; q < kGroups; ++q) { const double t = part[q][kl]; mx = t > mx ? t : mx; }
    a.cmax[b * a.M + k] = mx;
  }
}

}  // namespace ficoco
