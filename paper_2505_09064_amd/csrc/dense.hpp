// The small levels of the V-cycle as dense operators.
//
// Below some level the multiplicative cycle is a fixed linear map of a few
// thousand unknowns whose evaluation level by level is a chain of hundreds of
// dependent steps (colours, transfers), each a few microseconds whatever its
// size. The map is tabulated once per handle by running the cycle itself on the
// columns of the identity (block kernels, 16 columns per batch, all batches of a
// chunk in one launch), and a visit is then one matrix-vector product per table:
//   B  (level lo, where the fused bottom starts): x_lo = B b_lo;
//   R, [S Q] (levels ld .. lo - 1 above it): b_lo = R b_ld and
//      x_ld = S b_ld + Q x_lo.
// B holds the coarsest solve, which is FP64 in every cycle: B is built from FP64
// levels, kept and applied in FP64 also where the vectors and the other tables are
// FP32 (375 unknowns at 65^3: 1.1 MB).
// A product streams its table once: 2,187 unknowns in FP32 are 19 MB, a few
// microseconds, where the level's 19 launches took 115. One wavefront per row;
// the input vector is staged in LDS while the row's first 16-byte chunks are in
// flight. Packed problems are independent, so every part has its own tables
// (segments); a run of the packed cycle on the sum of the parts' j-th unit
// vectors gives column j of every part at once.
#pragma once

#include "block.hpp"

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

// out = M [v1; v2], table and sums in T, vectors in V; one wavefront per row, segment
// blockIdx.y (one: the only segment, by value).
template <typename V, typename T, int D>
__global__ __launch_bounds__(64 * kDenseWaves) void k_dense(
    DenseSeg one, const DenseSeg* __restrict__ segs, const T* __restrict__ M,
    const V* __restrict__ v1, const int* __restrict__ list1, const V* __restrict__ v2,
    const int* __restrict__ list2, V* __restrict__ out, const int* __restrict__ list_out) {
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
    V v[D];
    VecIO<V, D>::load(v1 + static_cast<int64_t>(list1 ? list1[s.a0 + i] : s.a0 + i) * DP, v);
#pragma unroll
    for (int a = 0; a < D; ++a) xs[i * D + a] = static_cast<T>(v[a]);
  }
  for (int i = threadIdx.x; i < s.nc; i += blockDim.x) {
    V v[D];
    VecIO<V, D>::load(v2 + static_cast<int64_t>(list2 ? list2[s.c0 + i] : s.c0 + i) * DP, v);
#pragma unroll
    for (int a = 0; a < D; ++a) xs[c1 + i * D + a] = static_cast<T>(v[a]);
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
    out[static_cast<int64_t>(list_out ? list_out[i] : i) * DP + row % D] = static_cast<V>(sum);
  }
}

// ---- several columns -------------------------------------------------------
// The same product for the K columns of a block solve, vectors [vertex][K][D].
// A contraction of 16 rows x cols x K columns: matrix instructions, 16 x 16
// output values per workgroup, its wavefronts taking turns over groups of four
// vertices (their D components are the D steps of the group: a lane loads a
// vertex's components of its matrix row and of its column in one go, both
// contiguous over the wavefront); their partial results meet in LDS and are
// added in wavefront order. The table streams once for all columns.
constexpr int kDenseMcWaves = 8;

typedef float dfloat4 __attribute__((ext_vector_type(4)));
typedef double ddouble4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Mfma16;
template <>
struct Mfma16<float> {
  using Acc = dfloat4;
  static __device__ __forceinline__ Acc step(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int q) { return 4 * (lane >> 4) + q; }
};
template <>
struct Mfma16<double> {
  using Acc = ddouble4;
  static __device__ __forceinline__ Acc step(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int q) { return (lane >> 4) + 4 * q; }
};

// acc += M[row][cols of one input] v: nv vertices, the first at index v0 of v,
// matrix row m (this lane's). Groups of four vertices wave, wave + waves, ...
template <typename V, typename T, int D, int K>
__device__ __forceinline__ void dense_mc_input(const T* __restrict__ m, const V* __restrict__ v, int v0,
                                               int nv, int wave, int lane,
                                               typename Mfma16<T>::Acc& acc) {
  constexpr int UN = sizeof(T) == 4 ? 4 : 2;
  const int n = lane & 15, g = lane >> 4;
  const int groups = (nv + 3) / 4;
  for (int q0 = wave; q0 < groups; q0 += UN * kDenseMcWaves) {
    T a[UN][D], b[UN][D];
    V vb[UN][D];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int i = 4 * (q0 + u * kDenseMcWaves) + g;
      const bool in = i < nv;
      const int ic = in ? i : nv - 1;
      BlockVecIO<T, D, D>::load(m + ic * D, a[u]);
      BlockVecIO<V, D, D>::load(v + (static_cast<int64_t>(v0 + ic) * K + n % K) * D, vb[u]);
#pragma unroll
      for (int c = 0; c < D; ++c) {
        b[u][c] = static_cast<T>(vb[u][c]);
        if (!in) a[u][c] = T(0);
        if (!in || n >= K) b[u][c] = T(0);
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int c = 0; c < D; ++c) acc = Mfma16<T>::step(a[u][c], b[u][c], acc);
    }
  }
}

// out = M [v1; v2] for K columns of a single problem (segment s).
template <typename V, typename T, int D, int K>
__global__ __launch_bounds__(64 * kDenseMcWaves) void k_dense_mc(DenseSeg s, const T* __restrict__ M,
                                                                 const V* __restrict__ v1,
                                                                 const V* __restrict__ v2,
                                                                 V* __restrict__ out) {
  static_assert(K <= 16, "one column per matrix column");
  __shared__ T part[kDenseMcWaves][16][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rows = s.nr * D, row0 = blockIdx.x * 16;
  const T* m = M + s.m0 + static_cast<int64_t>(min(row0 + (lane & 15), rows - 1)) * s.ld;
  typename Mfma16<T>::Acc acc = {T(0), T(0), T(0), T(0)};
  dense_mc_input<V, T, D, K>(m, v1, s.a0, s.na, wave, lane, acc);
  if (s.nc > 0)
    dense_mc_input<V, T, D, K>(m + DenseShape<T>::pad(s.na * D), v2, s.c0, s.nc, wave, lane, acc);
#pragma unroll
  for (int q = 0; q < 4; ++q) part[wave][Mfma16<T>::row(lane, q)][lane & 15] = acc[q];
  __syncthreads();
  const int r = threadIdx.x >> 4, n = threadIdx.x & 15, row = row0 + r;
  if (r >= 16 || n >= K || row >= rows) return;
  T sum = part[0][r][n];
#pragma unroll
  for (int w = 1; w < kDenseMcWaves; ++w) sum += part[w][r][n];
  out[(static_cast<int64_t>(s.r0 + row / D) * K + n) * D + row % D] = static_cast<V>(sum);
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
