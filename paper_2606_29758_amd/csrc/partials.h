// Merging the per-vocabulary-tile softmax partials of the logit products.
//
// A product leaves, for every column (token) and vocabulary tile k < ntv, the
// tile's maximum at part_m[k * ldp + col] and its sums relative to it.  They
// are merged by blocks that take kMergeCols columns with kSlices threads each;
// slice s takes the tiles s, s + kSlices, ... in order and the slices are joined
// in a fixed order (the loss's finalize adds the scaled sums in tile order
// instead), so the result depends on the partials alone.  What bounds a merge is
// the latency of its loads: one thread per column walked the 396 tiles of
// V = 152064 twice, with 1 block in flight per 256 tokens (294 us for 2,048 tokens,
// 306 us for 200, 402 us for the proxy of 1,501).  With 32 slices the loss call of
// 200 tokens takes 284 us less and the proxy of 1,501 396 us less; at V = 152064,
// 113,926 tokens of a loss call take 118 us (343 before), 165,881 of a proxy 185 us
// (544 before).  Few tiles leave most of 32 slices idle (merge_variant).
#pragma once

#include "common.h"
#include "gemm.h"

namespace pspo {
namespace {

constexpr int kMergeCols = 32;

// f(Const<kSlices>{}) with the slices for ntv tiles.  A score proxy of 100,000 tokens
// at d = 64, one thread per column / 32 slices / this: V = 384 (1 tile) 59 / 76 /
// 60 us, V = 1000 (3 tiles) 123 / 112 / 96, V = 2000 (6) 174 / 173 / 157.  At 11
// tiles 4 slices are 6% faster there but 1% slower at 4,000 tokens, at 32 tiles 32
// slices are 2% of a loss call of one token faster.
template <class F>
auto merge_variant(int ntv, F&& f) {
  if (ntv == 1) return f(Const<1>{});
  if (ntv <= 8) return f(Const<4>{});
  return f(Const<32>{});
}

// LDS of a merge: one value per (slice, column).
typedef float MergeRow[kMergeCols];

// op over the kSlices values of the thread's column, in a fixed tree; every
// thread of the block calls it and gets its column's result.
template <int kSlices, class Op>
__device__ __forceinline__ float merge_slices(float x, MergeRow* sh, Op op) {
  if constexpr (kSlices == 1) return x;
  const int c = threadIdx.x % kMergeCols, s = threadIdx.x / kMergeCols;
  sh[s][c] = x;
  __syncthreads();
#pragma unroll
  for (int h = kSlices / 2; h > 0; h >>= 1) {
    if (s < h) sh[s][c] = op(sh[s][c], sh[s + h][c]);
    __syncthreads();
  }
  x = sh[0][c];
  __syncthreads();
  return x;
}

// The maximum of column `col` over its tiles (-inf where col < 0).
template <int kSlices>
__device__ __forceinline__ float merge_max(const float* __restrict__ part_m, int ntv, int64_t ldp, int col,
                                           MergeRow* sh) {
  float m = -INFINITY;
  if (col >= 0) {
#pragma unroll 8
    for (int k = threadIdx.x / kMergeCols; k < ntv; k += kSlices) m = fmaxf(m, part_m[k * ldp + col]);
  }
  return merge_slices<kSlices>(m, sh, [](float a, float b) { return fmaxf(a, b); });
}

template <int kSlices>
__device__ __forceinline__ float merge_sum(float x, MergeRow* sh) {
  return merge_slices<kSlices>(x, sh, [](float a, float b) { return a + b; });
}

}  // namespace
}  // namespace pspo
