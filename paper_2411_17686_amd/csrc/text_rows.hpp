// Text-query block of FiCoCo-L: the body of the kernel that forms the tokens' text profiles, shared
// by attn_reduce.hip (the launch that reads the maps, or its own) and features.hip (the fused step lets
// it ride in the launch of the row-norm kernel, which does not depend on it).
#pragma once
#include "common.hpp"

namespace ficoco {

constexpr int kHeadBatch = 8;

struct AttnArgs {
  const void* A;
  int64_t sb, sh, sq;
  int H;
  int row0, nrows;  // rows [row0, row0+nrows) of the block are visited
  int col0;         // column of visual key 0
  int N;
  int vis_r0, n_vis;  // rows of the visual queries (n_vis = 0: none)
  int cls_r;          // row of the [CLS] query or -1
  int M;              // text queries (text block only)
  float* abar;
  double* recv_part;
  double* cls;
  double* ttext;
  int rows_per_wg, n_chunks, row_lanes, strip_groups, col_strips, B;
  int shift;          // rows by which chunk 0 is shortened (visual row 0 starts a chunk)
  int map_pitch;      // floats per row of abar
  double invH;
};

// The text block of a problem as AttnArgs (the fields text_reduce_block reads), and its grid.
void fill_text_args(const ficoco_problem& p, const Plan& pl, char* ws, AttnArgs& a);
inline dim3 text_grid(const ficoco_problem& p);

// The next heads of eight columns of one row, the first of them `at` elements behind base; moves on.  The offset is opaque: where
// the compiler forms it from the head's number, each load of a batch has a multiplication of its own, and the first one of a
// float32 batch comes apart into three.  The map kernel alone, float32 and 32 heads: 7.6 us with such loads and 7.2 so (three
// maps of 144 tokens), with eight text rows 6.2 and 5.85 (one map).
template <typename T, int HEADS>
__device__ __forceinline__ void load_heads(const T* base, int64_t& at, int64_t sh, Raw8<T> (&raw)[HEADS]) {
  asm volatile("" : "+s"(at));
#pragma unroll
  for (int u = 0; u < HEADS; ++u) load_raw(base + (at + u * sh), raw[u]);
  at += HEADS * sh;
}

// Text-query block of FiCoCo-L (task term of Eq. 3, profiles of Eq. 4): the head mean of
// A_text[b][h][k][i], stored TRANSPOSED as the token's profile ttext[b][i][k].  A workgroup
// owns 8 consecutive text rows x 256 key columns: a thread forms the head mean of one row and
// 8 columns exactly as the kernel above does (heads added in order, in double), the tile is
// turned in LDS, and each thread then writes the 8 rows of one column as one 64-byte piece.
constexpr int kTextHeadBatch = 16;
constexpr int kTextRows = 8;
using TextTile = double[kTextRows + 1];           // one column's rows; +1: the rows of one column in different banks
constexpr int kTextGroups = 256 / kTextRows;      // 8-column groups per workgroup
constexpr int kTextTiles = kTextGroups * kVec + kVec;    // the LDS it needs: TextTile[kTextTiles], the first kVec for columns before the strip
template <typename T>
__device__ __forceinline__ void text_reduce_block(const AttnArgs& a, int chunk, int strip, int64_t b, TextTile* tile) {
  const int tid = threadIdx.x;
  const int cg = tid % kTextGroups, rl = tid / kTextGroups;
  const int row = chunk * kTextRows + rl;
  const int col0 = strip * kTextGroups * kVec;
  // (the last group of a ragged block takes the last eight columns, as in the kernel above)
  const int col_own = col0 + cg * kVec;
  const int col = a.N >= kVec && col_own < a.N ? min(col_own, a.N - kVec) : col_own;
  const int ncol = max(min(kVec, a.N - col), 0);
  tile += kVec;
  if (row < a.M && ncol > 0) {
    const T* base = (const T*)a.A + b * a.sb + (int64_t)row * a.sq + a.col0 + col;
    double p[kVec];
#pragma unroll
    for (int k = 0; k < kVec; ++k) p[k] = 0.0;
    if (ncol == kVec) {
      int h0 = 0;
      // the grid of this kernel is small (8 rows x 256 keys per workgroup), so each thread keeps
      // more loads in flight than the map kernel does: kTextHeadBatch heads at a time
      int64_t at = 0;
      for (; h0 + kTextHeadBatch <= a.H; h0 += kTextHeadBatch) {
        Raw8<T> raw[kTextHeadBatch];
        load_heads(base, at, a.sh, raw);
        issue_fence();
#pragma unroll
        for (int u = 0; u < kTextHeadBatch; ++u) add_raw(raw[u], p);
      }
      for (; h0 + kHeadBatch <= a.H; h0 += kHeadBatch) {
        Raw8<T> raw[kHeadBatch];
        load_heads(base, at, a.sh, raw);
#pragma unroll
        for (int u = 0; u < kHeadBatch; ++u) add_raw(raw[u], p);
      }
      for (; h0 < a.H; ++h0) {
        Raw8<T> raw[1];
        load_heads(base, at, a.sh, raw);
        add_raw(raw[0], p);
      }
    } else {
      for (int h = 0; h < a.H; ++h)
        for (int k = 0; k < ncol; ++k) p[k] += widen(base[(int64_t)h * a.sh + k]);
    }
#pragma unroll
    for (int k = 0; k < kVec; ++k) tile[col - col0 + k][rl] = p[k] * a.invH;
  }
  __syncthreads();
  const int c = col0 + tid;                        // this thread's column
  if (c >= a.N) return;
  const int r0 = chunk * kTextRows;
  const int nr = min(kTextRows, a.M - r0);
  double* dst = a.ttext + ((int64_t)b * a.N + c) * a.M + r0;
  if (nr == kTextRows && a.M % 2 == 0) {           // 16-byte aligned pieces
#pragma unroll
    for (int k = 0; k < kTextRows; k += 2) {
      double2 v = make_double2(tile[tid][k], tile[tid][k + 1]);
      *reinterpret_cast<double2*>(dst + k) = v;
    }
  } else {
    for (int k = 0; k < nr; ++k) dst[k] = tile[tid][k];
  }
}

inline dim3 text_grid(const ficoco_problem& p) {
  return dim3((p.M + kTextRows - 1) / kTextRows, (p.N + kTextGroups * kVec - 1) / (kTextGroups * kVec), p.B);
}

}  // namespace ficoco
