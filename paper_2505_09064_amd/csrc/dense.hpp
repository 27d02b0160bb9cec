// The small levels of the V-cycle as dense operators.
//
// Below some level the multiplicative cycle is a fixed linear map of a few
// thousand unknowns whose evaluation level by level is a chain of hundreds of
// dependent steps (colours, transfers), each a few microseconds whatever its
// size. The map is tabulated once per handle by running the cycle itself, in the
// cycle's precision, on the columns of the identity (block kernels, 16 columns
// per batch, all batches of a chunk in one launch), and a visit is then one
// matrix-vector product per table:
//   B  (level lo, where the fused bottom starts): x_lo = B b_lo;
//   R, [S Q] (levels ld .. lo - 1 above it): b_lo = R b_ld and
//      x_ld = S b_ld + Q x_lo.
// A product streams its table once: 2,187 unknowns in FP32 are 19 MB, a few
// microseconds, where the level's 19 launches took 115. One wavefront per row;
// the input vector is staged in LDS while the row's first 16-byte chunks are in
// flight. Packed problems are independent, so every part has its own tables
// (segments); a run of the packed cycle on the sum of the parts' j-th unit
// vectors gives column j of every part at once.
#pragma once

#include "kernels.hpp"

namespace vasmg {
namespace dev {

constexpr int kDenseCols = 16;      // columns per batch of a table's construction
constexpr int kDenseWaves = 4;      // rows per workgroup of a product

// One part's table: rows of nr vertices, columns of na (first input) and nc
// (second input) vertices, each input's columns padded to 16 bytes; row stride
// ld elements. r0, a0, c0: the part's first vertex in the level's part order.
struct DenseSeg {
  int64_t m0 = 0;
  int r0 = 0, nr = 0, a0 = 0, na = 0, c0 = 0, nc = 0, ld = 0;
};

template <typename T>
struct DenseShape {
  static constexpr int Q = 16 / sizeof(T);   // values per 16-byte chunk
  __host__ __device__ static int pad(int n) { return (n + Q - 1) / Q * Q; }
};

// A level's vertices in part order: list[i] = device row; loc / seg: a device
// row's index inside its part and its part. Null for a single problem (identity).
struct DenseMap {
  const int* list = nullptr;
  const int* loc = nullptr;
  const int* seg = nullptr;
};

template <typename T, int Q>
struct alignas(16) Chunk {
  T v[Q];
};

// out = M [v1; v2]; one wavefront per row, segment blockIdx.y (one: the only
// segment, by value).
template <typename T, int D>
__global__ __launch_bounds__(64 * kDenseWaves) void k_dense(
    DenseSeg one, const DenseSeg* __restrict__ segs, const T* __restrict__ M,
    const T* __restrict__ v1, const int* __restrict__ list1, const T* __restrict__ v2,
    const int* __restrict__ list2, T* __restrict__ out, const int* __restrict__ list_out) {
  constexpr int DP = Pad<D>::value, Q = DenseShape<T>::Q, NP = 8;
  using C = Chunk<T, Q>;
  extern __shared__ __align__(16) unsigned char dense_smem[];
  T* xs = reinterpret_cast<T*>(dense_smem);
  const DenseSeg s = segs ? segs[blockIdx.y] : one;
  const int rows = s.nr * D;
  if (static_cast<int>(blockIdx.x) * kDenseWaves >= rows) return;
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kDenseWaves + (threadIdx.x >> 6);
  const int nch = s.ld / Q;
  const C* Mr = reinterpret_cast<const C*>(M + s.m0 + static_cast<int64_t>(min(row, rows - 1)) * s.ld);
  C pre[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int t = lane + 64 * i;
    if (t < nch) pre[i] = Mr[t];
  }
  const int c1 = DenseShape<T>::pad(s.na * D);
  for (int i = threadIdx.x; i < s.na; i += blockDim.x) {
    T v[D];
    VecIO<T, D>::load(v1 + static_cast<int64_t>(list1 ? list1[s.a0 + i] : s.a0 + i) * DP, v);
#pragma unroll
    for (int a = 0; a < D; ++a) xs[i * D + a] = v[a];
  }
  for (int i = threadIdx.x; i < s.nc; i += blockDim.x) {
    T v[D];
    VecIO<T, D>::load(v2 + static_cast<int64_t>(list2 ? list2[s.c0 + i] : s.c0 + i) * DP, v);
#pragma unroll
    for (int a = 0; a < D; ++a) xs[c1 + i * D + a] = v[a];
  }
  if (threadIdx.x < c1 - s.na * D) xs[s.na * D + threadIdx.x] = T(0);
  if (threadIdx.x < s.ld - c1 - s.nc * D) xs[c1 + s.nc * D + threadIdx.x] = T(0);
  __syncthreads();
  T acc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) acc[q] = T(0);
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int t = lane + 64 * i;
    if (t < nch) {
      const C x = reinterpret_cast<const C*>(xs)[t];
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[q] += pre[i].v[q] * x.v[q];
    }
  }
#pragma unroll 4
  for (int t = lane + 64 * NP; t < nch; t += 64) {
    const C m = Mr[t], x = reinterpret_cast<const C*>(xs)[t];
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] += m.v[q] * x.v[q];
  }
  T sum = acc[0];
#pragma unroll
  for (int q = 1; q < Q; ++q) sum += acc[q];
  sum = group_sum<T, 64>(sum);
  if (lane == 0 && row < rows) {
    const int i = s.r0 + row / D;
    out[static_cast<int64_t>(list_out ? list_out[i] : i) * DP + row % D] = sum;
  }
}

// ---- construction ---------------------------------------------------------
// Vectors [batch][n][kDenseCols][D]: column c = col0 + batch * kDenseCols + k.
// v = 1 where the row's unknown in its part, plus shift, is the column.
template <typename T, int D>
__global__ __launch_bounds__(kBlock) void k_dense_unit(int n, const int* __restrict__ loc, int col0,
                                                       int shift, T* __restrict__ v) {
  const int64_t e = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  if (e >= static_cast<int64_t>(n) * kDenseCols * D) return;
  const int a = static_cast<int>(e % D), k = static_cast<int>(e / D % kDenseCols);
  const int row = static_cast<int>(e / (D * kDenseCols));
  const int u = (loc ? loc[row] : row) * D + a + shift;
  v[static_cast<int64_t>(blockIdx.y) * n * kDenseCols * D + e] =
      u == col0 + static_cast<int>(blockIdx.y) * kDenseCols + k ? T(1) : T(0);
}

// Table columns from a batch of results v: column c - shift of every part, where
// c - shift lies inside the part's first (second = 0) or second (1) input.
template <typename T, int D>
__global__ __launch_bounds__(kBlock) void k_dense_extract(int n, DenseMap map, DenseSeg one,
                                                          const DenseSeg* __restrict__ segs, int col0,
                                                          int shift, int second,
                                                          const T* __restrict__ v, T* __restrict__ M) {
  const int64_t e = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  if (e >= static_cast<int64_t>(n) * kDenseCols * D) return;
  const int k = static_cast<int>(e % kDenseCols), a = static_cast<int>(e / kDenseCols % D);
  const int row = static_cast<int>(e / (D * kDenseCols));
  const DenseSeg s = segs ? segs[map.seg[row]] : one;
  const int c = col0 + static_cast<int>(blockIdx.y) * kDenseCols + k - shift;
  if (c < 0 || c >= (second ? s.nc : s.na) * D) return;
  const int i = map.loc ? map.loc[row] : row;
  M[s.m0 + static_cast<int64_t>(i * D + a) * s.ld + (second ? DenseShape<T>::pad(s.na * D) : 0) + c] =
      v[(static_cast<int64_t>(blockIdx.y) * n + row) * kDenseCols * D + k * D + a];
}

}  // namespace dev
}  // namespace vasmg
