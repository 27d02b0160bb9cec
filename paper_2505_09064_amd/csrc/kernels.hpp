// HIP kernels of the V-ASMG-PCG solve phase for gfx950 (CDNA4, wave64).
//
// Data layout (per level, device numbering = vertices sorted by colour, then
// cell, then canonical index):
//   * the blocks coupling a row to earlier colours (L) and to later colours (U)
//     are two separate CSR matrices, each with ascending columns and values
//     stored component-plane-major, val[(a*D+b)*nnz + k]: lanes walking a row
//     read consecutive addresses, and a sweep or residual that needs only one
//     of the two streams one contiguous array;
//   * fine level: diagonal blocks dense, diag[i*D*D + a*D + b]; coarse levels:
//     the blocks inside a Gauss-Seidel cell (diagonal included) as a dense
//     matrix per cell;
//   * vectors vertex-major with a padded stride DP (2 in 2D, 4 in 3D) so a
//     neighbour's components come in one 8/16-byte (FP32) or 16/32-byte (FP64)
//     load; pad entries are kept at zero.
// A block row is handled by a group of G lanes (G divides 64) that stride over
// its blocks (3D cell levels: a cell's threads walk all its rows together);
// partial sums are combined across the group's lanes and lane 0 of the group (or
// wavefront 0 of a cell) finishes the row.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace vasmg {
namespace dev {

constexpr int kBlock = 256;

template <int D>
struct Pad {
  static constexpr int value = (D == 3) ? 4 : 2;
};

// One of the two off-diagonal block matrices (L or U) of a level.
template <typename T>
struct Part {
  const int* __restrict__ ptr;   // [n+1]
  const int* __restrict__ col;   // [nnz]
  const T* __restrict__ val;     // [D*D][nnz]
  int64_t nnz;
};

// ---- padded vector loads/stores -------------------------------------------
template <typename T, int D>
struct VecIO;

template <>
struct VecIO<float, 2> {
  static __device__ __forceinline__ void load(const float* p, float* v) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    v[0] = t.x; v[1] = t.y;
  }
  static __device__ __forceinline__ void store(float* p, const float* v) {
    *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
  }
};
template <>
struct VecIO<float, 3> {
  static __device__ __forceinline__ void load(const float* p, float* v) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z;
  }
  static __device__ __forceinline__ void store(float* p, const float* v) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], 0.0f);
  }
};
template <>
struct VecIO<double, 2> {
  static __device__ __forceinline__ void load(const double* p, double* v) {
    const double2 t = *reinterpret_cast<const double2*>(p);
    v[0] = t.x; v[1] = t.y;
  }
  static __device__ __forceinline__ void store(double* p, const double* v) {
    *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
  }
};
template <>
struct VecIO<double, 3> {
  static __device__ __forceinline__ void load(const double* p, double* v) {
    const double2 t0 = *reinterpret_cast<const double2*>(p);
    const double2 t1 = *reinterpret_cast<const double2*>(p + 2);
    v[0] = t0.x; v[1] = t0.y; v[2] = t1.x;
  }
  static __device__ __forceinline__ void store(double* p, const double* v) {
    *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
    *reinterpret_cast<double2*>(p + 2) = make_double2(v[2], 0.0);
  }
};

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).
// Renumber them so each XCD walks one contiguous range of rows or cells:
// neighbouring rows then gather the same vector lines through the same L2.
__device__ __forceinline__ int xcd_block() {
  const int g = gridDim.x, b = blockIdx.x;
  const int q = g >> 3, r = g & 7;
  const int k = b & 7, j = b >> 3;
  return (k < r) ? k * (q + 1) + j : r * (q + 1) + (k - r) * q + j;
}

// LDS written by some lanes of a wavefront is read by others of it (a wavefront's
// LDS accesses run in program order; the compiler must keep them so).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>).
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>());
}

// v of the lane that CTRL names, kept from `old` where there is none or the row of
// 16 is not in ROWS.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_from(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_from(float old, float v) {
  return __int_as_float(dpp_from<CTRL, ROWS>(__float_as_int(old), __float_as_int(v)));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_from(double old, double v) {
  const long long o = __double_as_longlong(old), b = __double_as_longlong(v);
  const int lo = dpp_from<CTRL, ROWS>(static_cast<int>(o), static_cast<int>(b));
  const int hi = dpp_from<CTRL, ROWS>(static_cast<int>(o >> 32), static_cast<int>(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
constexpr int kDppRowShr = 0x110;      // + n: lane i of 16 <- i - n
constexpr int kDppBcast15 = 0x142;     // last lane of a row of 16 to the next row
constexpr int kDppBcast31 = 0x143;     // lane 31 to the upper half

// One step of the scan below: add the fetched values where the keys agree.
template <int CTRL, int ROWS, typename T, int D>
__device__ __forceinline__ void segment_step(int key, T (&v)[D]) {
  const bool same = dpp_from<CTRL, ROWS>(-1, key) == key;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const T o = dpp_from<CTRL, ROWS>(T(0), v[a]);
    v[a] += same ? o : T(0);
  }
}

// Inclusive sums over runs of equal keys (ascending over the wavefront, >= 0):
// a run's last lane ends with the run's sum. All lanes take part.
template <typename T, int D>
__device__ __forceinline__ void segment_scan(int key, T (&v)[D]) {
  segment_step<kDppRowShr + 1, 0xf>(key, v);
  segment_step<kDppRowShr + 2, 0xf>(key, v);
  segment_step<kDppRowShr + 4, 0xf>(key, v);
  segment_step<kDppRowShr + 8, 0xf>(key, v);
  segment_step<kDppBcast15, 0xa>(key, v);
  segment_step<kDppBcast31, 0xc>(key, v);
}

// v moved between the lanes of a row of 16 (data-parallel primitive CTRL): a few
// cycles, where a shuffle goes through LDS (about 100).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp(static_cast<int>(b), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(static_cast<int>(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
constexpr int kDppXor1 = 0xB1;         // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2, 3, 0, 1]
constexpr int kDppRowShl = 0x100;      // + n: lane i of 16 <- i + n
constexpr int kDppRowRor = 0x120;      // + n: lane i of 16 <- i - n, around the row
constexpr int kDppBcast = 0x150;       // + u: lane u of the row to all 16

// v of lane i ^ 4: up in the even quads of a row, down in the odd ones.
__device__ __forceinline__ int dpp_xor4(int v) {
  const int o = __builtin_amdgcn_update_dpp(0, v, kDppRowShl + 4, 0xf, 0x5, false);
  return __builtin_amdgcn_update_dpp(o, v, kDppRowShr + 4, 0xf, 0xa, false);
}
__device__ __forceinline__ float dpp_xor4(float v) { return __int_as_float(dpp_xor4(__float_as_int(v))); }
__device__ __forceinline__ double dpp_xor4(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_xor4(static_cast<int>(b)), hi = dpp_xor4(static_cast<int>(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// Sum over groups of G lanes, the same in every lane: a butterfly from the widest
// distance to the nearest lane, whose order FP32 results depend on. Rows of 16 meet
// by shuffles, lanes of a row by moves (after the step over 8 lanes, a value
// repeats every 8, so that a rotation by 4 fetches lane i ^ 4's).
template <typename T, int G>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
  for (int off = G / 2; off >= 16; off >>= 1) v += __shfl_xor(v, off, G);
  if constexpr (G > 8) v += dpp<kDppRowRor + 8>(v);
  if constexpr (G > 8) v += dpp<kDppRowRor + 4>(v);
  else if constexpr (G > 4) v += dpp_xor4(v);
  if constexpr (G > 2) v += dpp<kDppXor2>(v);
  if constexpr (G > 1) v += dpp<kDppXor1>(v);
  return v;
}

// Lane 0: the sum over the wavefront by a tree (lane i adds lane i + 32's, ..., i + 1's).
__device__ __forceinline__ double wave_tree(double v) {
  v += __shfl_down(v, 32, 64);
  v += __shfl_down(v, 16, 64);
  v += dpp<kDppRowShl + 8>(v);
  v += dpp<kDppRowShl + 4>(v);
  v += dpp<kDppRowShl + 2>(v);
  return v + dpp<kDppRowShl + 1>(v);
}

// Block-wide deterministic sum of one value per thread (fixed tree order).
__device__ __forceinline__ double block_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Broadcast of lane l's value to the wavefront (l uniform, all lanes active).
__device__ __forceinline__ float bcast(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double bcast(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), l);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), l);
  return __longlong_as_double((static_cast<long long>(hi) << 32) |
                              static_cast<unsigned int>(lo));
}

template <typename T>
__device__ __forceinline__ T ld_stream(const T* p) {
  return *p;
}

template <typename T, int D>
__device__ __forceinline__ void block_fma(const T* __restrict__ val, int64_t nnz, int k,
                                          const T* xj, T* acc) {
#pragma unroll
  for (int a = 0; a < D; ++a) {
#pragma unroll
    for (int b = 0; b < D; ++b) acc[a] += ld_stream(val + (a * D + b) * nnz + k) * xj[b];
  }
}

// Off-diagonal block row product over positions [kb, ke): acc += sum A_k x_col(k).
// UN blocks per lane are loaded before any is used (4 in FP32, so a whole row of
// a coarse level is in flight at once; 2 in FP64 to keep the register budget).
template <typename T, int D, int G>
__device__ __forceinline__ void row_product(int kb, int ke, int lane, const int* __restrict__ col,
                                            const T* __restrict__ val, int64_t nnz,
                                            const T* __restrict__ x, T* acc) {
  constexpr int DP = Pad<D>::value;
  constexpr int UN = sizeof(T) == 4 ? 4 : 2;
  int k = kb + lane;
  for (; k + (UN - 1) * G < ke; k += UN * G) {
    int j[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) j[u] = col[k + u * G];
    T xv[UN][D];
#pragma unroll
    for (int u = 0; u < UN; ++u) VecIO<T, D>::load(x + static_cast<int64_t>(j[u]) * DP, xv[u]);
#pragma unroll
    for (int u = 0; u < UN; ++u) block_fma<T, D>(val, nnz, k + u * G, xv[u], acc);
  }
  for (; k < ke; k += G) {
    const int jj = col[k];
    T xj[D];
    VecIO<T, D>::load(x + static_cast<int64_t>(jj) * DP, xj);
    block_fma<T, D>(val, nnz, k, xj, acc);
  }
}

// Cell levels store every row's L and U blocks padded to whole quads of kQuad
// consecutive blocks (padding: zero blocks pointing at the row itself), so a lane
// takes a quad per step: one 16-byte load of its 4 columns, 4 neighbour
// gathers, and per matrix plane one 16-byte (FP32) or two (FP64) loads. Rows
// and plane strides are multiples of kQuad, so every such load is aligned.
constexpr int kQuad = 4;

template <typename T>
struct Quad;
template <>
struct Quad<float> {
  static __device__ __forceinline__ void load(const float* p, float* v) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
};
template <>
struct Quad<double> {
  static __device__ __forceinline__ void load(const double* p, double* v) {
    const double2 a = *reinterpret_cast<const double2*>(p);
    const double2 b = *reinterpret_cast<const double2*>(p + 2);
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
  }
};

// acc += sum over the quads of positions [kb, ke) (multiples of kQuad).
template <typename T, int D, int G>
__device__ __forceinline__ void quad_product(int kb, int ke, int lane, const int* __restrict__ col,
                                             const T* __restrict__ val, int64_t nnz,
                                             const T* __restrict__ x, T* acc) {
  constexpr int DP = Pad<D>::value;
  for (int q = kb / kQuad + lane; q < ke / kQuad; q += G) {
    const int4 j = reinterpret_cast<const int4*>(col)[q];
    T xv[kQuad][D];
    VecIO<T, D>::load(x + static_cast<int64_t>(j.x) * DP, xv[0]);
    VecIO<T, D>::load(x + static_cast<int64_t>(j.y) * DP, xv[1]);
    VecIO<T, D>::load(x + static_cast<int64_t>(j.z) * DP, xv[2]);
    VecIO<T, D>::load(x + static_cast<int64_t>(j.w) * DP, xv[3]);
#pragma unroll
    for (int a = 0; a < D; ++a) {
#pragma unroll
      for (int b = 0; b < D; ++b) {
        T v[kQuad];
        Quad<T>::load(val + static_cast<int64_t>(a * D + b) * nnz + static_cast<int64_t>(q) * kQuad, v);
        acc[a] += v[0] * xv[0][b] + v[1] * xv[1][b] + v[2] * xv[2][b] + v[3] * xv[3][b];
      }
    }
  }
}

// FP32 takes the quad step; FP64 keeps the per-block step on the same padded
// rows (padding blocks are zeros): a quad of doubles costs more registers than it
// saves in loads (occupancy 3-4 waves per SIMD, measured 20% slower).
template <typename T, int D, int G>
__device__ __forceinline__ void part_quad_product(const Part<T>& p, int i, int lane,
                                                  const T* __restrict__ x, T* acc) {
  if constexpr (sizeof(T) == 4)
    quad_product<T, D, G>(p.ptr[i], p.ptr[i + 1], lane, p.col, p.val, p.nnz, x, acc);
  else
    row_product<T, D, G>(p.ptr[i], p.ptr[i + 1], lane, p.col, p.val, p.nnz, x, acc);
}

// A row's diagonal block and (x != NULL, else zero) its own entry.
template <typename T, int D>
__device__ __forceinline__ void load_own(const T* __restrict__ diag, const T* __restrict__ x, int i, T* dg,
                                         T* xi) {
#pragma unroll
  for (int e = 0; e < D * D; ++e) dg[e] = diag[static_cast<int64_t>(i) * D * D + e];
  if (x) {
    VecIO<T, D>::load(x + static_cast<int64_t>(i) * Pad<D>::value, xi);
  } else {
#pragma unroll
    for (int a = 0; a < D; ++a) xi[a] = T(0);
  }
}

// Off-diagonal products of a point-level row (LO / UP: which parts), a lane group of
// G taking the blocks of each part in order (lane l: blocks l, l + G, ... of L, then
// of U). Rows hold about 7 blocks per part, unevenly (a colour's rows have most of
// theirs in one part), so a row is a chain of three dependent loads (row ranges ->
// columns -> neighbours): the ranges of both parts come together, and columns and
// values of a lane's first UN blocks, whichever part they are in, go out before the
// first neighbour is waited for; only longer rows loop. A lane without a block reads
// the last one there is (or, in an empty row, the block before; an empty part has one
// zero block) times zero.
// lo and up get the parts' sums, in every lane of the group. BOTH: lo gets one sum over
// L's blocks, then U's; in 3D (LIST) dealt to the lanes as one list, which spares uneven
// rows a round (point-Jacobi PCG at 65^3 126 us an iteration, part by part 135); in 2D
// part by part, the order of the operations being part of the result (CellSums).
template <typename T, int D, int G, bool LO, bool UP, bool BOTH = false>
struct PointRow {
  static constexpr int DP = Pad<D>::value, UN = LO && UP ? 2 : 1;
  static constexpr bool LIST = BOTH && D == 3;
  int l0 = 0, le = 0, u0 = 0, ue = 0;
  __device__ __forceinline__ void ranges(const Part<T>& L, const Part<T>& U, int i) {
    if (LO) { l0 = L.ptr[i]; le = L.ptr[i + 1]; }
    if (UP) { u0 = U.ptr[i]; ue = U.ptr[i + 1]; }
  }
  // acc += block m times xv, where `in`
  static __device__ __forceinline__ void add(const T* m, const T* xv, bool in, T* acc) {
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const T xb = in ? xv[b] : T(0);
#pragma unroll
      for (int a = 0; a < D; ++a) acc[a] += m[a * D + b] * xb;
    }
  }
  // The lane's blocks t0 .. t0 + UN - 1.
  __device__ __forceinline__ void round(const Part<T>& L, const Part<T>& U, int lane, int t0,
                                        const T* __restrict__ x, T* lo, T* up) const {
    T m[UN][D * D], xv[UN][D];
    int j[UN];
    bool isu[UN], in[UN];
#pragma unroll
    for (int t = 0; t < UN; ++t) {
      int k;
      if constexpr (LIST) {
        const int nl = le - l0, total = nl + ue - u0, f = lane + (t0 + t) * G;
        const int fc = max(min(f, total - 1), 0);
        isu[t] = fc >= nl;
        in[t] = f < total;
        k = isu[t] ? u0 + fc - nl : l0 + fc;
        if (total == 0) k = max(k - 1, 0);
      } else {
        const int kl = l0 + lane, nl = LO ? max(le - kl + G - 1, 0) / G : 0;   // nl blocks of L
        isu[t] = !LO || (UP && t0 + t >= nl);
        k = isu[t] ? u0 + lane + (t0 + t - nl) * G : kl + (t0 + t) * G;
        const int end = isu[t] ? ue : le;
        in[t] = k < end;
        k = max(min(k, end - 1), 0);
      }
      const int* col = isu[t] ? U.col : L.col;
      const T* val = isu[t] ? U.val : L.val;
      const int64_t nnz = isu[t] ? U.nnz : L.nnz;
      j[t] = col[k];
#pragma unroll
      for (int e = 0; e < D * D; ++e) m[t][e] = val[e * nnz + k];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < UN; ++t) VecIO<T, D>::load(x + static_cast<int64_t>(j[t]) * DP, xv[t]);
    // (pinned here: the compiler would sink a load whose value is only selected)
#pragma unroll
    for (int t = 0; t < UN; ++t) {
#pragma unroll
      for (int b = 0; b < D; ++b) asm volatile("" : "+v"(xv[t][b]));
    }
#pragma unroll
    for (int t = 0; t < UN; ++t) {
      if (BOTH || !UP) {
        add(m[t], xv[t], in[t], lo);
      } else if (!LO) {
        add(m[t], xv[t], in[t], up);
      } else {
        add(m[t], xv[t], in[t] && !isu[t], lo);
        add(m[t], xv[t], in[t] && isu[t], up);
      }
    }
  }
  __device__ __forceinline__ void rest(const Part<T>& p, int k, int ke, const T* __restrict__ x, T* acc) const {
    for (; k < ke; k += G) {
      T xj[D];
      VecIO<T, D>::load(x + static_cast<int64_t>(p.col[k]) * DP, xj);
      block_fma<T, D>(p.val, p.nnz, k, xj, acc);
    }
  }
  __device__ __forceinline__ void sum(const Part<T>& L, const Part<T>& U, int lane,
                                      const T* __restrict__ x, T* lo, T* up) const {
#pragma unroll
    for (int a = 0; a < D; ++a) {
      if (LO) lo[a] = T(0);
      if (UP && !BOTH) up[a] = T(0);
    }
    round(L, U, lane, 0, x, lo, up);
    if constexpr (LIST) {
      for (int t = UN; lane + t * G < le - l0 + ue - u0; t += UN) round(L, U, lane, t, x, lo, up);
    } else {
      const int kl = l0 + lane, nl = LO ? max(le - kl + G - 1, 0) / G : 0;
      if (LO) rest(L, kl + UN * G, le, x, lo);
      if (UP) rest(U, u0 + lane + max(UN - nl, 0) * G, ue, x, BOTH ? lo : up);
    }
#pragma unroll
    for (int a = 0; a < D; ++a) {
      if (LO) lo[a] = group_sum<T, G>(lo[a]);
      if (UP && !BOTH) up[a] = group_sum<T, G>(up[a]);
    }
  }
};

// ---------------------------------------------------------------------------
// K1: y = A x (diag + off-diagonal), optional partial dot x.y per workgroup.
// ---------------------------------------------------------------------------
template <typename T, int D, int G, bool DOT>
__global__ __launch_bounds__(kBlock) void k_spmv(int n, Part<T> L, Part<T> U,
                                                 const T* __restrict__ diag,
                                                 const T* __restrict__ x, T* __restrict__ y,
                                                 double* __restrict__ partial) {
  constexpr int DP = Pad<D>::value;
  const int lane = threadIdx.x % G;
  const int i = xcd_block() * (kBlock / G) + threadIdx.x / G;
  double dot = 0.0;
  if (i < n) {
    PointRow<T, D, G, true, true, true> row;
    row.ranges(L, U, i);
    T acc[D], xi[D], dg[D * D];
    load_own<T, D>(diag, x, i, dg, xi);
    row.sum(L, U, lane, x, acc, nullptr);
    if (lane == 0) {
      T yi[D];
#pragma unroll
      for (int a = 0; a < D; ++a) {
        T s = acc[a];
#pragma unroll
        for (int b = 0; b < D; ++b) s += dg[a * D + b] * xi[b];
        yi[a] = s;
        if (DOT) dot += static_cast<double>(xi[a]) * static_cast<double>(s);
      }
      VecIO<T, D>::store(y + static_cast<int64_t>(i) * DP, yi);
    }
  }
  if (DOT) {
    __shared__ double sh[kBlock];
    const double s = block_sum(dot, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
  }
}

// r = b - A x (full row), used when no saved lower-part sums exist.
template <typename T, int D, int G>
__global__ __launch_bounds__(kBlock) void k_residual_full(
    int n, Part<T> L, Part<T> U, const T* __restrict__ diag, const T* __restrict__ b,
    const T* __restrict__ x, T* __restrict__ r) {
  constexpr int DP = Pad<D>::value;
  const int lane = threadIdx.x % G;
  const int i = xcd_block() * (kBlock / G) + threadIdx.x / G;
  if (i >= n) return;
  PointRow<T, D, G, true, true, true> row;
  row.ranges(L, U, i);
  T acc[D], xi[D], bi[D], dg[D * D];
  load_own<T, D>(diag, x, i, dg, xi);
  VecIO<T, D>::load(b + static_cast<int64_t>(i) * DP, bi);
  row.sum(L, U, lane, x, acc, nullptr);
  if (lane == 0) {
    T ri[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
      T s = bi[a] - acc[a];
#pragma unroll
      for (int c = 0; c < D; ++c) s -= dg[a * D + c] * xi[c];
      ri[a] = s;
    }
    VecIO<T, D>::store(r + static_cast<int64_t>(i) * DP, ri);
  }
}

// ---------------------------------------------------------------------------
// K3: one colour of a point Gauss-Seidel sweep (Algorithm 1 in colour order).
//   MODE 0: forward from a zero guess (only earlier colours are nonzero, so
//           only L is read); saves s_i = b_i - sum_{j<i} A_ij x_j
//   MODE 1: forward from a nonzero guess; saves s_i as well
//   MODE 2: backward (components in reverse order)
// ---------------------------------------------------------------------------
template <typename T, int D, int G, int MODE>
__global__ __launch_bounds__(kBlock) void k_gs_color(
    int row0, int nrows, Part<T> L, Part<T> U, const T* __restrict__ diag,
    const T* __restrict__ b, T* x, T* __restrict__ s_save) {
  constexpr int DP = Pad<D>::value;
  const int lane = threadIdx.x % G;
  const int g = xcd_block() * (kBlock / G) + threadIdx.x / G;
  if (g >= nrows) return;
  const int i = row0 + g;
  // 3D: the backward sweep, which does not want s = b - L x on its own, takes one
  // sum over both parts (2D: two, the order of the operations is part of the result)
  constexpr bool BOTH = D == 3 && MODE == 2;
  PointRow<T, D, G, true, MODE != 0, BOTH> row;
  row.ranges(L, U, i);
  // what finishes the row, before the products
  T dg[D * D], xi[D], bi[D];
  load_own<T, D>(diag, MODE == 0 ? nullptr : x, i, dg, xi);
  VecIO<T, D>::load(b + static_cast<int64_t>(i) * DP, bi);
  T lo[D], up[D];
#pragma unroll
  for (int a = 0; a < D; ++a) up[a] = T(0);
  row.sum(L, U, lane, x, lo, up);
  if (lane != 0) return;
  T s[D], rhs[D];
#pragma unroll
  for (int a = 0; a < D; ++a) {
    s[a] = bi[a] - lo[a];
    rhs[a] = s[a] - up[a];
  }
  if (MODE != 2 && s_save) VecIO<T, D>::store(s_save + static_cast<int64_t>(i) * DP, s);
  if (MODE != 2) {
#pragma unroll
    for (int a = 0; a < D; ++a) {
      T t = rhs[a];
#pragma unroll
      for (int c = 0; c < D; ++c)
        if (c != a) t -= dg[a * D + c] * xi[c];
      xi[a] = t / dg[a * D + a];
    }
  } else {
#pragma unroll
    for (int a = D - 1; a >= 0; --a) {
      T t = rhs[a];
#pragma unroll
      for (int c = 0; c < D; ++c)
        if (c != a) t -= dg[a * D + c] * xi[c];
      xi[a] = t / dg[a * D + a];
    }
  }
  VecIO<T, D>::store(x + static_cast<int64_t>(i) * DP, xi);
}

// K2: r = s - D x - sum_{j > i} A_ij x_j after a forward sweep that saved s.
template <typename T, int D, int G>
__global__ __launch_bounds__(kBlock) void k_residual_upper(
    int n, Part<T> U, const T* __restrict__ diag, const T* __restrict__ s_save,
    const T* __restrict__ x, T* __restrict__ r) {
  constexpr int DP = Pad<D>::value;
  const int lane = threadIdx.x % G;
  const int i = xcd_block() * (kBlock / G) + threadIdx.x / G;
  if (i >= n) return;
  PointRow<T, D, G, false, true> row;
  row.ranges(U, U, i);
  T acc[D], xi[D], si[D], dg[D * D];
  load_own<T, D>(diag, x, i, dg, xi);
  VecIO<T, D>::load(s_save + static_cast<int64_t>(i) * DP, si);
  row.sum(U, U, lane, x, nullptr, acc);
  if (lane == 0) {
    T ri[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
      T s = si[a] - acc[a];
#pragma unroll
      for (int c = 0; c < D; ++c) s -= dg[a * D + c] * xi[c];
      ri[a] = s;
    }
    VecIO<T, D>::store(r + static_cast<int64_t>(i) * DP, ri);
  }
}

// ---------------------------------------------------------------------------
// Coarse lattice levels: Gauss-Seidel over cells of at most NV = 2^D vertices.
// Device rows of a cell are contiguous ([cell_ptr[c], cell_ptr[c+1])); L and U
// hold only blocks coupling to other cells (earlier / later colours); the blocks
// inside a cell, diagonal included, are a dense NU x NU matrix per cell
// (NU = NV * D, column-major: cellM[c*NU*NU + u*NU + t] = M[t][u]).
// One workgroup handles one cell: lane group g sums the off-cell part of the
// cell's g-th row, then lane t of wavefront 0 owns unknown t (vertex t / D,
// component t % D) for the sequential sweep inside the cell, which broadcasts
// each new value with a shuffle.
// ---------------------------------------------------------------------------
template <int D>
struct CellShape {
  static constexpr int NV = 1 << D;
  static constexpr int NU = NV * D;
};

// A cell's record: first device row, rows, then the NV + 1 row ranges' ends in L and
// in U (in blocks; rows beyond the cell's last are empty). One cache line and one
// load, where cell -> rows -> row ranges were two dependent ones: a launch is a
// chain of dependent loads of about 6 us on most levels. Solve of a graded 513 x 513
// mesh, FP32 cycle, 193.1 -> 184.0 ms; of a 65^3 mesh 16.2 -> 15.8 ms.
template <int D>
struct CellRec {
  static constexpr int NV = CellShape<D>::NV;
  static constexpr int L = 2, U = L + NV + 1, ints = D == 2 ? 16 : 32;
  static_assert(U + NV + 1 <= ints, "record too small");
};

// The records of all cells, one int per thread (on the host, and uploaded, they took
// 6 ms of the set-up of a graded 513 x 513 mesh).
template <int D>
__global__ __launch_bounds__(kBlock) void k_cell_records(int ncells, const int* __restrict__ cell_ptr,
                                                         const int* __restrict__ Lptr,
                                                         const int* __restrict__ Uptr, int* __restrict__ rec) {
  using R = CellRec<D>;
  const int64_t e = blockIdx.x * int64_t(kBlock) + threadIdx.x;
  if (e >= static_cast<int64_t>(ncells) * R::ints) return;
  const int c = static_cast<int>(e / R::ints), k = static_cast<int>(e % R::ints);
  const int v0 = cell_ptr[c], m = cell_ptr[c + 1] - v0;
  int v = 0;
  if (k == 0) v = v0;
  else if (k == 1) v = m;
  else if (k < R::U) v = Lptr[v0 + min(k - R::L, m)];
  else if (k <= R::U + R::NV) v = Uptr[v0 + min(k - R::U, m)];
  rec[e] = v;
}

// Cells per workgroup: one per workgroup when a cell's NV * GR lanes fill a
// wavefront or more (its wavefront 0 runs the in-cell sweep); otherwise as many
// as share one wavefront (2D cells with 4 or 8 lanes per row), each with its own
// lane segment for the off-cell sums and the in-cell sweep.
template <int D, int GR>
struct CellPack {
  static constexpr int CT = (1 << D) * GR;                 // lanes per cell
  static constexpr int CPW = CT >= 64 ? 1 : 64 / CT;
  static constexpr int threads = CT * CPW;
};

// Value of lane u of the calling lane's cell segment (CT lanes; several cells
// share a wavefront where CPW > 1); every lane of the wavefront calls it.
template <int CPW, int CT, int U, typename T>
__device__ __forceinline__ T cell_bcast(T v) {
  if constexpr (CPW == 1)
    return bcast(v, U);
  else if constexpr (CT == 16)
    return dpp<kDppBcast + U>(v);
  else
    return __shfl(v, U, CT);
}

// Reciprocal of the lane's own diagonal entry Mrow[t] (1 for lanes without a
// row), taken once before the sequential in-cell sweep: each of its steps then
// costs a multiply instead of a division on the dependent chain.
template <typename T, int NU>
__device__ __forceinline__ T own_reciprocal(const T* Mrow, int t, bool own) {
  T dg = T(1);
#pragma unroll
  for (int u = 0; u < NU; ++u)
    if (u == t) dg = Mrow[u];
  return own ? T(1) / dg : T(1);
}

// One lane's share of a row of a cell level, positions [kb, ke) of a part: steps
// of kStep consecutive blocks, one 16-byte load per matrix plane (FP32: a quad,
// FP64: a pair; rows are padded to quads) and the columns in one load.
template <typename T>
struct CellStep {
  static constexpr int B = 16 / sizeof(T);
  using Cols = std::conditional_t<B == 4, int4, int2>;
  static __device__ __forceinline__ Cols cols(const int* col, int q) {
    return reinterpret_cast<const Cols*>(col)[q];
  }
  static __device__ __forceinline__ int at(const Cols& j, int k) {
    if constexpr (B == 4)
      return k == 0 ? j.x : k == 1 ? j.y : k == 2 ? j.z : j.w;
    else
      return k == 0 ? j.x : j.y;
  }
};

typedef int Vec16 __attribute__((ext_vector_type(4)));   // 16 bytes on the way through registers

template <typename T>
struct alignas(16) StepVals {
  T v[16 / sizeof(T)];
};

// A lane's walk over its steps of a row part. The first step is unconditional
// and taken in pieces (open: columns and matrix values as soon as the row's range
// is known; then its neighbours; then the products), so that the caller can put
// all loads that need no other load's answer in flight before it waits: behind a
// branch the compiler sinks and serialises them. A lane without a step reads the
// row's last one (the part's first where there is none before: allocated even for
// an empty part), which its neighbours fetch anyway, and multiplies it by zeros.
template <typename T, int D, int G>
struct RowWalk {
  static constexpr int DP = Pad<D>::value, B = CellStep<T>::B;
  int q, qe, q0;
  typename CellStep<T>::Cols j;
  StepVals<T> m[D * D];
  __device__ __forceinline__ void columns(const Part<T>& p, int kb, int ke, int lane) {
    q = kb / B + lane;
    qe = ke / B;
    q0 = max(min(q, qe - 1), 0);
    j = CellStep<T>::cols(p.col, q0);
  }
  __device__ __forceinline__ void values(const Part<T>& p, int qq) {
#pragma unroll
    for (int e = 0; e < D * D; ++e)
      m[e] = reinterpret_cast<const StepVals<T>*>(p.val + static_cast<int64_t>(e) * p.nnz)[qq];
  }
  // a step's blocks are summed per component pair and then added, as in the quad
  // steps of the fused bottom
  __device__ __forceinline__ void product(const T* __restrict__ x, T* acc) {
    T xv[B][D];
#pragma unroll
    for (int k = 0; k < B; ++k)
      VecIO<T, D>::load(x + static_cast<int64_t>(CellStep<T>::at(j, k)) * DP, xv[k]);
    __builtin_amdgcn_sched_barrier(0);
    const bool in = q < qe;
#pragma unroll
    for (int k = 0; k < B; ++k) {
#pragma unroll
      for (int b = 0; b < D; ++b)
        if (!in) xv[k][b] = T(0);
    }
#pragma unroll
    for (int a = 0; a < D; ++a) {
#pragma unroll
      for (int b = 0; b < D; ++b) {
        const T* mv = m[a * D + b].v;
        T v = __builtin_elementwise_fma(mv[0], xv[0][b], mv[1] * xv[1][b]);
#pragma unroll
        for (int k = 2; k < B; ++k) v = __builtin_elementwise_fma(mv[k], xv[k][b], v);
        acc[a] = acc[a] + v;
      }
    }
  }
  __device__ __forceinline__ void rest(const Part<T>& p, const T* __restrict__ x, T* acc) {
    for (q += G; q < qe; q += G) {
      j = CellStep<T>::cols(p.col, q);
      values(p, q);
      __builtin_amdgcn_sched_barrier(0);
      product(x, acc);
    }
  }
};

// What the sweeps and the residual of a cell have in common: the off-cell products
// of its rows (their sums end in LDS) and the cell matrix (staged in LDS);
// wavefront 0 then owns the cell's unknowns, one per lane. A launch of a small
// level is one pass through a chain of dependent loads (the cell's record ->
// columns -> neighbours), so nothing waits that need not: both parts' ranges are
// in the record, then come columns and matrix values; the cell matrix goes
// to LDS in 16-byte pieces by all threads.
//
// One cell per workgroup (3D): the rows of a cell are one contiguous run of steps
// in each part, and the workgroup's threads take the steps of both runs in order,
// whichever row they belong to: every lane has a step and every load of a
// wavefront is one contiguous kilobyte. A step's row is found among the cell's row
// ranges (scalars); the sums of a wavefront's rows come from a segmented scan.
// With a group of lanes per row a cell waited for its longest row (up to six
// rounds of 16 lanes where the mean row has one) with half its lanes idle:
// backward launch of level 1 of a 65^3 mesh (1,331 cells a colour, 42.6 MB) FP32
// 17.4 us at the start of this form, 15.5 with a group of lanes per row and the
// loads first, 13.7 flat (3.1 TB/s; the launch itself and the cell's own chain
// are about 5 us of it); 4,092 cells a colour 30.1 -> 26.6 us (4.8 TB/s; a plain
// read of ten such planes streams at 6.1); its residual 194 -> 176 us.
//
// 2D (rows of a few steps, several cells per wavefront): a group of GR lanes per
// row, and the in-cell arithmetic (SEQ below) in one running sum per unknown. The
// order of the FP32 operations is part of the result there: a 2D iteration with
// materials 1:100 takes 15 to 50 products and amplifies another rounding of its
// preconditioner to 1e-9 .. 1e-8 of the solution (4 of 60 such problems above 1e-9
// with this order changed; 3D: none of 1,700, the largest 9.5e-10).
template <typename T, int D, int GR>
struct CellSums {
  static constexpr int NV = CellShape<D>::NV, NU = CellShape<D>::NU;
  static constexpr int CPW = CellPack<D, GR>::CPW, CT = CellPack<D, GR>::CT;
  using Rec = CellRec<D>;
  static constexpr int PC = NU * NU * static_cast<int>(sizeof(T)) / 16;   // 16-byte pieces of M
  static constexpr int PR = (PC + CT - 1) / CT;
  static constexpr bool FLAT = D == 3 && CPW == 1;
  static constexpr int NW = FLAT ? CT / 64 : 1;   // partial sums of a row
  struct Lds {
    T M[CPW][NU * NU];
    T sum[CPW][NW][2 * NV][D];   // lower parts of the rows, then upper parts
    __device__ __forceinline__ T total(int slot, int row, int a) const {
      T v = sum[slot][0][row][a];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += sum[slot][w][row][a];
      return v;
    }
    __device__ __forceinline__ T lo(int slot, int k, int a) const { return total(slot, k, a); }
    __device__ __forceinline__ T up(int slot, int k, int a) const { return total(slot, NV + k, a); }
  };

  // The cell's record: an int per lane for the flat walk, else only its first two.
  struct Head {
    int rec, v0, m;
  };
  static __device__ __forceinline__ Head head(const int* __restrict__ rec, int c, bool live) {
    const int* r = rec + static_cast<int64_t>(c) * Rec::ints;
    if constexpr (FLAT) {
      const int v = r[threadIdx.x & (Rec::ints - 1)];
      return {v, __builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 1)};
    } else {
      const int2 h = *reinterpret_cast<const int2*>(r);
      return {0, h.x, live ? h.y : 0};
    }
  }

  // One step of the flat walk over both parts of a cell.
  template <bool LO, bool UP>
  struct Flat {
    static constexpr int B = CellStep<T>::B, DP = Pad<D>::value;
    int pl[NV + 1], pu[NV + 1];   // row ranges in steps (uniform)
    int nl, total;
    int key, end, q;
    bool in;
    typename CellStep<T>::Cols j;
    StepVals<T> m[D * D];
    // rec: the cell's record, an int per lane, read into scalars lane by lane (as
    // 18 scalar loads per wavefront the ranges missed the scalar cache: the
    // backward launch of 1,331 cells took 56 us instead of 15)
    __device__ __forceinline__ void ranges(int rec) {
      static_for<NV + 1>([&](auto ri) {
        constexpr int r = decltype(ri)::value;
        pl[r] = LO ? __builtin_amdgcn_readlane(rec, Rec::L + r) / B : 0;
        pu[r] = UP ? __builtin_amdgcn_readlane(rec, Rec::U + r) / B : 0;
      });
      nl = pl[NV] - pl[0];
      total = nl + pu[NV] - pu[0];
    }
    __device__ __forceinline__ void fetch(const Part<T>& L, const Part<T>& U, int f) {
      in = f < total;
      const int fc = max(min(f, total - 1), 0);
      const bool u = !LO || (UP && fc >= nl);
      q = u ? pu[0] + fc - nl : pl[0] + fc;
      // a cell without off-cell blocks reads the step before its (empty) run, or
      // the part's first (present and zero even in an empty part)
      if (total == 0) q = max(q - 1, 0);
      // row: the row ranges at or below the step (either part's, constant indices:
      // arrays chosen between at run time would go to scratch memory)
      int kl = 0, ku = 0, el = pl[NV], eu = pu[NV];
      static_for<NV - 1>([&](auto ri) {
        constexpr int r = NV - 1 - decltype(ri)::value;
        if constexpr (LO) {
          kl += q >= pl[r];
          el = q < pl[r] ? pl[r] : el;
        }
        if constexpr (UP) {
          ku += q >= pu[r];
          eu = q < pu[r] ? pu[r] : eu;
        }
      });
      end = u ? eu : el;
      key = in ? (u ? ku + NV : kl) : 2 * NV;
      const int* col = u ? U.col : L.col;
      const T* val = u ? U.val : L.val;
      const int64_t nnz = u ? U.nnz : L.nnz;
      j = CellStep<T>::cols(col, q);
#pragma unroll
      for (int e = 0; e < D * D; ++e)
        m[e] = reinterpret_cast<const StepVals<T>*>(val + static_cast<int64_t>(e) * nnz)[q];
    }
    __device__ __forceinline__ void add(const T* __restrict__ x, T (*sum)[D]) {
      T xv[B][D];
#pragma unroll
      for (int k = 0; k < B; ++k)
        VecIO<T, D>::load(x + static_cast<int64_t>(CellStep<T>::at(j, k)) * DP, xv[k]);
      __builtin_amdgcn_sched_barrier(0);
      T acc[D];
#pragma unroll
      for (int a = 0; a < D; ++a) acc[a] = T(0);
#pragma unroll
      for (int k = 0; k < B; ++k) {
#pragma unroll
        for (int b = 0; b < D; ++b) {
#pragma unroll
          for (int a = 0; a < D; ++a) acc[a] += m[a * D + b].v[k] * xv[k][b];
        }
      }
      segment_scan<T, D>(key, acc);
      if (in && (q + 1 == end || (threadIdx.x & 63) == 63)) {
#pragma unroll
        for (int a = 0; a < D; ++a) sum[key][a] += acc[a];
      }
      wave_sync();   // the next step's tail lanes are others
    }
  };

  // t: thread inside its cell; LO / UP: which parts to sum; own(): loads of the
  // caller's, issued after the row ranges'. Ends in a barrier. E, F (colour-block
  // levels): taken with L and U.
  template <bool LO, bool UP, class Own>
  static __device__ __forceinline__ void run(Lds& sh, int slot, int t, int c, const Head& hd,
                                             const int* __restrict__ rec, const Part<T>& L, const Part<T>& U, const Part<T>* E,
                                             const Part<T>* F, const T* __restrict__ cellM,
                                             const T* __restrict__ x, Own&& own) {
    const int v0 = hd.v0, m = hd.m;
    Vec16 piece[PR];
    const Vec16* Mc = reinterpret_cast<const Vec16*>(cellM + static_cast<int64_t>(c) * NU * NU);
    if constexpr (FLAT) {
      const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
      T(*sum)[D] = sh.sum[0][w];
      Flat<LO, UP> fl;
      static_for<PR>([&](auto ri) {
        constexpr int r = decltype(ri)::value;
        piece[r] = Mc[min(t + r * CT, PC - 1)];
      });
      own();
      __builtin_amdgcn_sched_barrier(0);
      fl.ranges(hd.rec);
      if (lane < 2 * NV) {   // each wavefront its own sums
#pragma unroll
        for (int a = 0; a < D; ++a) sum[lane][a] = T(0);
      }
      wave_sync();
      fl.fetch(L, U, t);
      __builtin_amdgcn_sched_barrier(0);
      static_for<PR>([&](auto ri) {
        constexpr int r = decltype(ri)::value;
        reinterpret_cast<Vec16*>(sh.M[0])[min(t + r * CT, PC - 1)] = piece[r];
      });
      fl.add(x, sum);
      for (int f = CT; f + w * 64 < fl.total; f += CT) {   // uniform over the wavefront
        fl.fetch(L, U, f + t);
        __builtin_amdgcn_sched_barrier(0);
        fl.add(x, sum);
      }
      if (E || F) {
        // colour-block levels: a group of GR lanes per row
        const int g = t / GR, gl = t % GR;
        T lo[D], up[D];
#pragma unroll
        for (int a = 0; a < D; ++a) { lo[a] = T(0); up[a] = T(0); }
        if (g < m) {
          if (LO && E) part_quad_product<T, D, GR>(*E, v0 + g, gl, x, lo);
          if (UP && F) part_quad_product<T, D, GR>(*F, v0 + g, gl, x, up);
        }
#pragma unroll
        for (int a = 0; a < D; ++a) {
          lo[a] = group_sum<T, GR>(lo[a]);
          up[a] = group_sum<T, GR>(up[a]);
        }
        if (gl == 0) {
#pragma unroll
          for (int a = 0; a < D; ++a) {
            sum[g][a] += lo[a];
            sum[NV + g][a] += up[a];
          }
        }
      }
    } else {
      const int g = t / GR, gl = t % GR;
      const bool has = g < m;
      const int* rg = rec + static_cast<int64_t>(c) * Rec::ints + g;
      int lb = 0, le = 0, ub = 0, ue = 0;
      if constexpr (LO) { lb = rg[Rec::L]; le = rg[Rec::L + 1]; }
      if constexpr (UP) { ub = rg[Rec::U]; ue = rg[Rec::U + 1]; }
      static_for<PR>([&](auto ri) {
        constexpr int r = decltype(ri)::value;
        piece[r] = Mc[min(t + r * CT, PC - 1)];
      });
      own();
      __builtin_amdgcn_sched_barrier(0);
      T lo[D], up[D];
#pragma unroll
      for (int a = 0; a < D; ++a) { lo[a] = T(0); up[a] = T(0); }
      RowWalk<T, D, GR> wl, wu;
      if constexpr (LO) wl.columns(L, lb, has ? le : lb, gl);
      if constexpr (UP) wu.columns(U, ub, has ? ue : ub, gl);
      if constexpr (LO) wl.values(L, wl.q0);
      else wu.values(U, wu.q0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < PR; ++r)
        reinterpret_cast<Vec16*>(sh.M[slot])[min(t + r * CT, PC - 1)] = piece[r];
      if constexpr (LO) {
        wl.product(x, lo);
        wl.rest(L, x, lo);
        if constexpr (UP) wu.values(U, wu.q0);
      }
      if constexpr (UP) {
        wu.product(x, up);
        wu.rest(U, x, up);
      }
#pragma unroll
      for (int a = 0; a < D; ++a) {
        if (LO) lo[a] = group_sum<T, GR>(lo[a]);
        if (UP) up[a] = group_sum<T, GR>(up[a]);
      }
      if (gl == 0) {
#pragma unroll
        for (int a = 0; a < D; ++a) {
          if (LO) sh.sum[slot][0][g][a] = lo[a];
          if (UP) sh.sum[slot][0][NV + g][a] = up[a];
        }
      }
    }
    __syncthreads();
  }
};

template <typename T, int D, int GR, int MODE>
__global__ __launch_bounds__((CellPack<D, GR>::threads)) void k_gs_cell(
    int cell0, int ncell, const int* __restrict__ rec, Part<T> L, Part<T> U,
    const T* __restrict__ cellM, const T* __restrict__ b, T* x, T* __restrict__ s_save) {
  constexpr int DP = Pad<D>::value;
  using Sums = CellSums<T, D, GR>;
  constexpr int NV = Sums::NV, NU = Sums::NU, CT = Sums::CT, CPW = Sums::CPW;
  __shared__ __align__(16) typename Sums::Lds sh;
  const int slot = CPW == 1 ? 0 : threadIdx.x / CT;
  const int t = CPW == 1 ? threadIdx.x : threadIdx.x % CT;
  const int ci = xcd_block() * CPW + slot;
  const bool live = CPW == 1 || ci < ncell;   // the last workgroup may hold fewer cells
  const int c = cell0 + (live ? ci : 0);
  const typename Sums::Head hd = Sums::head(rec, c, live);
  const int v0 = hd.v0, m = hd.m, n = m * D;
  const bool own = t < n;
  const int k = own ? t / D : 0, a = own ? t % D : 0;
  const int64_t xi = static_cast<int64_t>(v0 + k) * DP + a;
  T bt = T(0), xc = T(0);
  Sums::template run<true, MODE != 0>(sh, slot, t, c, hd, rec, L, U, nullptr, nullptr, cellM, x, [&] {
    bt = b[xi];
    if (MODE != 0) xc = x[xi];
  });
  if (threadIdx.x >= 64) return;          // wavefront 0 finishes the cell(s)
  if (!own) xc = T(0);
  const int tc = min(t, NU - 1);
  T Mrow[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) Mrow[u] = sh.M[slot][u * NU + tc];
  const T rdg = own ? T(1) / sh.M[slot][tc * NU + tc] : T(1);
  const T s_t = own ? bt - sh.lo(slot, k, a) : T(0);
  if (MODE != 2 && s_save && own) s_save[xi] = s_t;
  T acc = own && MODE != 0 ? s_t - sh.up(slot, k, a) : s_t;
  if constexpr (D == 2) {
    // SEQ. acc: the unknown's right-hand side minus all other unknowns' products.
    // Each unknown in turn is acc / diagonal and the others follow its change.
    // Lanes without an unknown hold zeros (the cell matrix is zero outside the
    // cell's unknowns).
#pragma unroll
    for (int u = 0; u < NU; ++u) Mrow[u] = u == t ? T(0) : Mrow[u];
    if (MODE != 0)
      static_for<NU>([&](auto ui) {
        constexpr int u = decltype(ui)::value;
        acc = __builtin_elementwise_fma(-Mrow[u], cell_bcast<CPW, CT, u>(xc), acc);
      });
    static_for<NU>([&](auto ui) {
      constexpr int u = MODE == 2 ? NU - 1 - decltype(ui)::value : decltype(ui)::value;
      const T delta = __builtin_elementwise_fma(acc, rdg, -xc);
      if (t == u) xc = acc * rdg;
      acc = __builtin_elementwise_fma(-Mrow[u], cell_bcast<CPW, CT, u>(delta), acc);
    });
    if (own) x[xi] = xc;
    return;
  }
  // acc: the unknown's residual. Each unknown in turn moves by residual /
  // diagonal and the others' residuals follow: one multiply, one broadcast and
  // one multiply-add on the chain per step. Lanes without an unknown hold zeros.
  if (MODE != 0) {
    T mx[2] = {T(0), T(0)};
    static_for<NV>([&](auto vi) {
      constexpr int v = decltype(vi)::value;
      if (CPW > 1 || v < m)
        static_for<D>([&](auto ai) {
          constexpr int u = v * D + decltype(ai)::value;
          mx[u % 2] += Mrow[u] * cell_bcast<CPW, CT, u>(xc);
        });
    });
    acc = own ? acc - (mx[0] + mx[1]) : T(0);
  }
  static_for<NV>([&](auto vi) {
    constexpr int v = MODE == 2 ? NV - 1 - decltype(vi)::value : decltype(vi)::value;
    if (CPW > 1 || v < m)
      static_for<D>([&](auto ai) {
        constexpr int u = v * D + (MODE == 2 ? D - 1 - decltype(ai)::value : decltype(ai)::value);
        const T step = acc * rdg;
        if (t == u) xc += step;
        acc -= Mrow[u] * cell_bcast<CPW, CT, u>(step);
      });
  });
  if (own) x[xi] = xc;
}

// ---------------------------------------------------------------------------
// Colour-block levels (3D): cells are grouped into colour blocks of up to
// NB = 2^D cells (a colour is given to a block; the cells of a block are swept
// one after the other, in canonical order). A block's device rows are
// contiguous, its cells in canonical order. Besides L and U (blocks to earlier
// / later colours) a row has E and F: blocks to the earlier / later cells of
// its own colour block.
// One workgroup sweeps one colour block, wavefront w its cell w (GR = 64 / NV
// lanes per row):
//   phase A, all wavefronts at once: the products whose operand is final or
//     old for the whole sweep of this colour, from x in HBM before any cell of
//     the block is written: L (earlier colours: final) and, from a nonzero
//     guess, F and U (forward: later cells and colours still old) or E and U
//     (backward: earlier cells old, later colours new). Meanwhile the part the
//     cells need at their turn (forward: E, backward: F) is staged in LDS for
//     the whole block (it is contiguous in every plane), as is the block's x;
//   phase B, cell by cell in sweep order: the turn part's products with the
//     block's iterate in LDS, where the cells swept before hold their new
//     values, then the sequential sweep inside the cell (as k_gs_cell); the new
//     values go to LDS and HBM; a workgroup barrier closes each step.
// The forward sweeps save s = b - L x - E x (final values) for the residual.
// ---------------------------------------------------------------------------
template <int D>
struct BlockShape {
  static constexpr int NB = 1 << D;           // cells per colour block
  static constexpr int GR = 64 / (1 << D);    // lanes per row: one wavefront per cell
  static constexpr int threads = NB * 64;
};

// Entries of the turn part staged in LDS per colour block (a multiple of kQuad;
// entries beyond it are read from HBM at the turn).
template <typename T>
struct BlockStage {
  static constexpr int cap = sizeof(T) == 4 ? 1408 : 704;
};

// acc += products of the turn part's positions [kb, ke) (relative to the
// block's first entry; multiples of kQuad on cell levels) with the block's LDS
// iterate xs (device rows from r0); entries below `staged` come from the LDS
// stage (tcol, tval planes of stride CAP), the rest from the part in HBM.
template <typename T, int D, int G, int CAP>
__device__ __forceinline__ void block_turn_product(int kb, int ke, int lane, const Part<T>& P,
                                                   int base, int staged, const int* tcol,
                                                   const T* tval, const T* xs, int r0, T* acc) {
  constexpr int DP = Pad<D>::value;
  if constexpr (sizeof(T) == 4) {
    for (int q = kb / kQuad + lane; q < ke / kQuad; q += G) {
      const int e = q * kQuad;
      int4 j;
      T v[D * D][kQuad];
      if (e < staged) {
        j = *reinterpret_cast<const int4*>(tcol + e);
#pragma unroll
        for (int pl = 0; pl < D * D; ++pl) Quad<T>::load(tval + pl * CAP + e, v[pl]);
      } else {
        j = reinterpret_cast<const int4*>(P.col + base)[q];
#pragma unroll
        for (int pl = 0; pl < D * D; ++pl)
          Quad<T>::load(P.val + static_cast<int64_t>(pl) * P.nnz + base + e, v[pl]);
      }
      const int jj[kQuad] = {(j.x - r0) * DP, (j.y - r0) * DP, (j.z - r0) * DP, (j.w - r0) * DP};
#pragma unroll
      for (int a = 0; a < D; ++a) {
#pragma unroll
        for (int b = 0; b < D; ++b) {
          const T* vv = v[a * D + b];
          acc[a] += vv[0] * xs[jj[0] + b] + vv[1] * xs[jj[1] + b] + vv[2] * xs[jj[2] + b] +
                    vv[3] * xs[jj[3] + b];
        }
      }
    }
  } else {
    for (int e = kb + lane; e < ke; e += G) {
      const bool st = e < staged;
      const int j = ((st ? tcol[e] : P.col[base + e]) - r0) * DP;
#pragma unroll
      for (int a = 0; a < D; ++a) {
#pragma unroll
        for (int b = 0; b < D; ++b) {
          const int pl = a * D + b;
          const T v = st ? tval[pl * CAP + e] : P.val[static_cast<int64_t>(pl) * P.nnz + base + e];
          acc[a] += v * xs[j + b];
        }
      }
    }
  }
}

// Two workgroups per compute unit (4 waves per SIMD: at most 128 VGPRs).
template <typename T, int D, int MODE>
__global__ __launch_bounds__(BlockShape<D>::threads, 4) void k_gs_block(
    int blk0, const int* __restrict__ block_ptr, const int* __restrict__ cell_ptr, Part<T> L,
    Part<T> U, Part<T> E, Part<T> F, const T* __restrict__ cellM, const T* __restrict__ b, T* x,
    T* __restrict__ s_save) {
  constexpr int DP = Pad<D>::value, DD = D * D;
  constexpr int NV = CellShape<D>::NV, NU = CellShape<D>::NU;
  constexpr int NB = BlockShape<D>::NB, GR = BlockShape<D>::GR;
  constexpr int CAP = BlockStage<T>::cap;
  __shared__ __align__(16) T xs[NB * NV * DP];
  __shared__ __align__(16) int tcol[CAP];
  __shared__ __align__(16) T tval[DD * CAP];
  const Part<T>& TP = MODE == 2 ? F : E;   // the part taken at each cell's turn
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int bk = blk0 + xcd_block();
  const int cb = block_ptr[bk], nc = block_ptr[bk + 1] - cb;
  const int r0 = cell_ptr[cb], nrow = cell_ptr[cb + nc] - r0;
  // stage the block's turn part (contiguous in each plane, 16-byte aligned)
  const int tbase = TP.ptr[r0];
  const int staged = min(TP.ptr[r0 + nrow] - tbase, CAP);
  {
    constexpr int VW = 16 / sizeof(T);   // elements per 16-byte copy
    for (int e = threadIdx.x * 4; e < staged; e += blockDim.x * 4)
      *reinterpret_cast<int4*>(tcol + e) = *reinterpret_cast<const int4*>(TP.col + tbase + e);
    for (int pl = 0; pl < DD; ++pl) {
      const T* src = TP.val + static_cast<int64_t>(pl) * TP.nnz + tbase;
      for (int e = threadIdx.x * VW; e < staged; e += blockDim.x * VW)
        *reinterpret_cast<int4*>(tval + pl * CAP + e) = *reinterpret_cast<const int4*>(src + e);
    }
    for (int e = threadIdx.x; e < nrow * DP; e += blockDim.x)
      xs[e] = MODE != 0 ? x[static_cast<int64_t>(r0) * DP + e] : T(0);
  }
  // this wavefront's cell: the owned unknown t = lane (vertex t / D, component t % D)
  const bool has = w < nc;
  const int c = cb + (has ? w : 0);
  const int v0 = cell_ptr[c], m = has ? cell_ptr[c + 1] - v0 : 0, n = m * D;
  const int t = lane;
  const bool own = t < n;
  const int k = own ? t / D : 0, a = own ? t % D : 0;
  const int64_t xi = static_cast<int64_t>(v0 + k) * DP + a;
  T Mrow[NU];
  const T* Mc = cellM + static_cast<int64_t>(c) * NU * NU;
#pragma unroll
  for (int u = 0; u < NU; ++u) Mrow[u] = (own && u < n) ? Mc[u * NU + t] : T(0);
  const T bt = own ? b[xi] : T(0);
  T xc = (own && MODE != 0) ? x[xi] : T(0);
  // phase A (the turn part's row bounds are loaded now: at the turn only LDS is read)
  const int g = lane / GR, gl = lane % GR;
  const int tkb = g < m ? TP.ptr[v0 + g] - tbase : 0, tke = g < m ? TP.ptr[v0 + g + 1] - tbase : 0;
  T pa[D], pu[D];
#pragma unroll
  for (int q = 0; q < D; ++q) { pa[q] = T(0); pu[q] = T(0); }
  if (g < m) {
    const int i = v0 + g;
    part_quad_product<T, D, GR>(L, i, gl, x, pa);
    if (MODE == 1) {
      part_quad_product<T, D, GR>(F, i, gl, x, pu);
      part_quad_product<T, D, GR>(U, i, gl, x, pu);
    }
    if (MODE == 2) {
      part_quad_product<T, D, GR>(E, i, gl, x, pa);
      part_quad_product<T, D, GR>(U, i, gl, x, pa);
    }
  }
  T my_pa = T(0), my_pu = T(0);
#pragma unroll
  for (int q = 0; q < D; ++q) {   // every lane takes part in each shuffle
    const T s1 = __shfl(group_sum<T, GR>(pa[q]), k * GR, 64);
    const T s2 = MODE == 1 ? __shfl(group_sum<T, GR>(pu[q]), k * GR, 64) : T(0);
    if (q == a) { my_pa = s1; my_pu = s2; }
  }
  const T rdg = own_reciprocal<T, NU>(Mrow, t, own);
  __syncthreads();   // stage and block iterate in LDS
  // phase B: the cells in sweep order
  for (int step = 0; step < nc; ++step) {
    const int kk = MODE == 2 ? nc - 1 - step : step;
    if (w == kk) {
      T pt[D];
#pragma unroll
      for (int q = 0; q < D; ++q) pt[q] = T(0);
      if (g < m)
        block_turn_product<T, D, GR, CAP>(tkb, tke, gl, TP, tbase, staged, tcol, tval, xs, r0, pt);
      T my_pt = T(0);
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const T s1 = __shfl(group_sum<T, GR>(pt[q]), k * GR, 64);
        if (q == a) my_pt = s1;
      }
      T acc;
      if (MODE != 2) {
        const T s_t = own ? bt - my_pa - my_pt : T(0);
        if (s_save && own) s_save[xi] = s_t;
        acc = s_t - my_pu;
      } else {
        acc = own ? bt - my_pa - my_pt : T(0);
      }
      if (MODE != 0) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          if (u < n) {
            const T xu = bcast(xc, u);
            if (u != t) acc -= Mrow[u] * xu;
          }
        }
      }
#pragma unroll
      for (int uu = 0; uu < NU; ++uu) {
        const int u = MODE == 2 ? NU - 1 - uu : uu;
        if (u < n) {
          T delta = T(0);
          if (t == u) {
            const T xn = acc * rdg;
            delta = xn - xc;
            xc = xn;
          }
          delta = bcast(delta, u);
          if (t != u) acc -= Mrow[u] * delta;
        }
      }
      if (own) {
        xs[(v0 + k - r0) * DP + a] = xc;
        x[xi] = xc;
      }
    }
    __syncthreads();
  }
}

// out_t = base_t - (off-cell part)_t - (M x)_t on cell levels.
//   KIND 0: residual after a forward sweep: base = saved s, upper range only
//           (U, and F on colour-block levels: s holds b - L x - E x)
//   KIND 1: full residual: base = b, both ranges
//   KIND 2: SpMV: base = 0, both ranges, result negated (y = A x)
//   BLK: a colour-block level, E (with L) and F (with U) taken as well.
template <typename T, int D, int GR, int KIND, bool BLK>
__global__ __launch_bounds__((CellPack<D, GR>::threads)) void k_cell_apply(
    int ncell, const int* __restrict__ rec, Part<T> L, Part<T> U, Part<T> E, Part<T> F,
    const T* __restrict__ cellM, const T* __restrict__ base, const T* __restrict__ x,
    T* __restrict__ out) {
  constexpr int DP = Pad<D>::value;
  using Sums = CellSums<T, D, GR>;
  constexpr int NV = Sums::NV, NU = Sums::NU, CT = Sums::CT, CPW = Sums::CPW;
  __shared__ __align__(16) typename Sums::Lds sh;
  const int slot = CPW == 1 ? 0 : threadIdx.x / CT;
  const int t = CPW == 1 ? threadIdx.x : threadIdx.x % CT;
  const int ci = xcd_block() * CPW + slot;
  const bool live = CPW == 1 || ci < ncell;
  const int c = live ? ci : 0;
  const typename Sums::Head hd = Sums::head(rec, c, live);
  const int v0 = hd.v0, m = hd.m, n = m * D;
  const bool own = t < n;
  const int k = own ? t / D : 0, a = own ? t % D : 0;
  const int64_t xi = static_cast<int64_t>(v0 + k) * DP + a;
  T xt = T(0), bt = T(0);
  Sums::template run<KIND != 0, true>(sh, slot, t, c, hd, rec, L, U, BLK ? &E : nullptr,
                                      BLK ? &F : nullptr, cellM, x, [&] {
                                        xt = x[xi];
                                        if (KIND != 2) bt = base[xi];
                                      });
  if (threadIdx.x >= 64) return;
  if (!own) xt = T(0);
  const int tc = min(t, NU - 1);
  constexpr int CH = D == 2 ? 1 : 2;   // running sums (2D: one, SEQ)
  T mx[2] = {T(0), T(0)};
  static_for<NV>([&](auto vi) {
    constexpr int v = decltype(vi)::value;
    if (CPW > 1 || v < m)
      static_for<D>([&](auto ai) {
        constexpr int u = v * D + decltype(ai)::value;
        mx[u % CH] += sh.M[slot][u * NU + tc] * cell_bcast<CPW, CT, u>(xt);
      });
  });
  if (!own) return;
  const T off = (KIND != 0 ? sh.lo(slot, k, a) : T(0)) + sh.up(slot, k, a);
  out[xi] = KIND == 2 ? off + (mx[0] + mx[1]) : bt - off - (mx[0] + mx[1]);
}

// ---------------------------------------------------------------------------
// Damped vertex-block Jacobi step: x = omega D^{-1} v (FIRST, from a zero guess,
// v = b) or x += omega D^{-1} v (v = the residual b - A x).
// ---------------------------------------------------------------------------
template <typename T, int D, bool FIRST>
__global__ __launch_bounds__(kBlock) void k_jacobi_step(int n, const T* __restrict__ dinv, T omega,
                                                        const T* __restrict__ v, T* __restrict__ x) {
  constexpr int DP = Pad<D>::value;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  T vi[D], xi[D];
  VecIO<T, D>::load(v + static_cast<int64_t>(i) * DP, vi);
  if (!FIRST) VecIO<T, D>::load(x + static_cast<int64_t>(i) * DP, xi);
  const T* Di = dinv + static_cast<int64_t>(i) * D * D;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    T t = T(0);
#pragma unroll
    for (int b = 0; b < D; ++b) t += Di[a * D + b] * vi[b];
    xi[a] = FIRST ? omega * t : xi[a] + omega * t;
  }
  VecIO<T, D>::store(x + static_cast<int64_t>(i) * DP, xi);
}

// ---------------------------------------------------------------------------
// K4: restriction b_c = P^T r (gather over the CSR of P^T); K5: x += P e.
// ---------------------------------------------------------------------------
// Both transfers are gathers over a scalar CSR (weights shared by the
// components); GT lanes share a row so its entries are loaded together.
template <typename T, int D, int GT>
__device__ __forceinline__ void transfer_row(int pb, int pe, int lane, const int* __restrict__ idx,
                                             const T* __restrict__ w, const T* __restrict__ v,
                                             T* acc) {
  constexpr int DP = Pad<D>::value;
  for (int p = pb + lane; p < pe; p += GT) {
    T e[D];
    VecIO<T, D>::load(v + static_cast<int64_t>(idx[p]) * DP, e);
    const T wp = w[p];
#pragma unroll
    for (int a = 0; a < D; ++a) acc[a] += wp * e[a];
  }
#pragma unroll
  for (int a = 0; a < D; ++a) acc[a] = group_sum<T, GT>(acc[a]);
}

template <typename T, int D, int GT>
__global__ __launch_bounds__(kBlock) void k_restrict(int nc, const int* __restrict__ ptr,
                                                     const int* __restrict__ idx,
                                                     const T* __restrict__ w,
                                                     const T* __restrict__ r, T* __restrict__ bc) {
  constexpr int DP = Pad<D>::value;
  const int lane = threadIdx.x % GT;
  const int I = xcd_block() * (kBlock / GT) + threadIdx.x / GT;
  if (I >= nc) return;
  T acc[D];
#pragma unroll
  for (int a = 0; a < D; ++a) acc[a] = T(0);
  transfer_row<T, D, GT>(ptr[I], ptr[I + 1], lane, idx, w, r, acc);
  if (lane == 0) VecIO<T, D>::store(bc + static_cast<int64_t>(I) * DP, acc);
}

// fixed (optional): constrained components of the fine rows, whose
// prolongation rows are zero.
template <typename T, int D, int GT>
__global__ __launch_bounds__(kBlock) void k_prolong_add(int nf, const int* __restrict__ ptr,
                                                        const int* __restrict__ idx,
                                                        const T* __restrict__ w,
                                                        const T* __restrict__ e, T* x,
                                                        const uint8_t* __restrict__ fixed) {
  constexpr int DP = Pad<D>::value;
  const int lane = threadIdx.x % GT;
  const int i = xcd_block() * (kBlock / GT) + threadIdx.x / GT;
  if (i >= nf) return;
  T xi[D];
  if (lane == 0) VecIO<T, D>::load(x + static_cast<int64_t>(i) * DP, xi);
  T acc[D];
#pragma unroll
  for (int a = 0; a < D; ++a) acc[a] = T(0);
  transfer_row<T, D, GT>(ptr[i], ptr[i + 1], lane, idx, w, e, acc);
  if (lane == 0) {
    const int fx = fixed ? fixed[i] : 0;
#pragma unroll
    for (int a = 0; a < D; ++a) xi[a] += ((fx >> a) & 1) ? T(0) : acc[a];
    VecIO<T, D>::store(x + static_cast<int64_t>(i) * DP, xi);
  }
}

// ---------------------------------------------------------------------------
// K6: coarsest solve L L^T e = b in FP64 (one workgroup; n <= kCoarseMax).
// ---------------------------------------------------------------------------
constexpr int kCoarseMax = 4096;

template <typename T, int D>
__global__ __launch_bounds__(kBlock) void k_coarse_solve(int n, const double* __restrict__ L,
                                                         const T* __restrict__ b, T* __restrict__ x) {
  constexpr int DP = Pad<D>::value;
  __shared__ double y[kCoarseMax];
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    y[i] = static_cast<double>(b[(i / D) * DP + (i % D)]);
  __syncthreads();
  for (int j = 0; j < n; ++j) {           // L y = b, column by column
    if (threadIdx.x == 0) y[j] /= L[static_cast<int64_t>(j) * n + j];
    __syncthreads();
    const double yj = y[j];
    for (int i = j + 1 + threadIdx.x; i < n; i += blockDim.x)
      y[i] -= L[static_cast<int64_t>(i) * n + j] * yj;
    __syncthreads();
  }
  for (int j = n - 1; j >= 0; --j) {      // L^T x = y
    if (threadIdx.x == 0) y[j] /= L[static_cast<int64_t>(j) * n + j];
    __syncthreads();
    const double yj = y[j];
    for (int i = threadIdx.x; i < j; i += blockDim.x)
      y[i] -= L[static_cast<int64_t>(j) * n + i] * yj;
    __syncthreads();
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) x[(i / D) * DP + (i % D)] = static_cast<T>(y[i]);
}

// K6, small coarsest levels (n <= kCoarseInvMax): x = A_c^{-1} b with the inverse
// formed at setup from the same Cholesky factor; one pass instead of 2n
// dependent steps. Row i is one thread's sum in ascending column order.
constexpr int kCoarseInvMax = 256;
template <typename T, int D>
__global__ __launch_bounds__(kBlock) void k_coarse_apply(int n, const double* __restrict__ Minv,
                                                         const T* __restrict__ b, T* __restrict__ x) {
  constexpr int DP = Pad<D>::value;
  __shared__ double y[kCoarseInvMax];
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    y[i] = static_cast<double>(b[(i / D) * DP + (i % D)]);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double* row = Minv + static_cast<int64_t>(i) * n;
    double s = 0.0;
    for (int j = 0; j < n; ++j) s += row[j] * y[j];
    x[(i / D) * DP + (i % D)] = static_cast<T>(s);
  }
}

// ---------------------------------------------------------------------------
// The bottom of the cycle in one workgroup: the last few cell levels above a
// small coarsest level (smoothing, residual, restriction, prolongation) and the
// coarsest solve by the inverse, which would otherwise take 2 x colours + 3
// launches per level, each too small to fill the chip. The levels' vectors
// live in LDS; each wavefront updates one cell of the current colour (GR =
// 64 / 2^d lanes per row) with the arithmetic of k_gs_cell / k_cell_apply, and
// colours and phases are separated by workgroup barriers. Several levels are
// fused only for the V-cycle (one visit per level); the first level may start
// from a nonzero iterate (second visit of a W-cycle).
// ---------------------------------------------------------------------------
constexpr int kBottomThreads = 512;
constexpr int kBottomLevels = 4;
constexpr int kBottomLds = 56 * 1024;   // dynamic LDS: the levels' vectors and pointer copies

// Pointers that k_bottom reads from its level table (device memory, not kernel
// arguments) are generic to the compiler, which then emits flat loads: counted
// against both the memory and the LDS wait counters, so LDS reads also wait for
// the matrix loads in flight. Its matrix loads go through pointers in the global
// address space instead.
template <typename T>
using gptr = const __attribute__((address_space(1))) T*;
typedef int gint4 __attribute__((ext_vector_type(4)));
typedef float gfloat4 __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ gptr<T> to_global(const T* p) {
  return (gptr<T>)p;
}

template <typename T>
struct BottomLevel {
  int n = 0, ncolors = 0, ncells = 0, nnext = 0;
  const int* color_ptr = nullptr;   // cells of each colour, [ncolors + 1]
  const int* cell_ptr = nullptr;
  Part<T> L{}, U{};
  const T* cellM = nullptr;
  const int *p_ptr = nullptr, *p_idx = nullptr;
  const T* p_w = nullptr;
  const int *pt_ptr = nullptr, *pt_idx = nullptr;
  const T* pt_w = nullptr;
  const uint8_t* fixed = nullptr;   // constrained components (zero prolongation rows), or null
};

template <typename T>
struct BottomArgs {
  int nlev = 0, ncoarse = 0;
  int npre = 1, npost = 1, zero_guess = 1;
  const BottomLevel<T>* lev = nullptr;   // device array [nlev]
  const double* Minv = nullptr;
  const T* b = nullptr;   // first fused level's right-hand side (in)
  T* x = nullptr;         // first fused level's iterate (in unless zero_guess, out)
};

// One level in LDS: right-hand side, iterate, saved s, residual, and copies of
// the colour, cell and row pointers (the sweeps' dependent index loads).
template <typename T>
struct BottomVecs {
  T *b, *x, *s, *r;
  int *color_ptr, *cell_ptr, *Lptr, *Uptr;
};

// LDS elements of one level: four padded vectors (T) and its pointers (int).
__host__ __device__ inline int bottom_vec_elems(int n, int dp) { return 4 * n * dp; }
__host__ __device__ inline int bottom_int_elems(int n, int ncolors, int ncells) {
  return (ncolors + 1) + (ncells + 1) + 2 * (n + 1);
}

// acc += the products of positions [kb, ke) of one part with the LDS iterate x:
// quads of 4 blocks (FP32, one 16-byte load per plane) or single blocks (FP64),
// loaded through global-address-space pointers.
template <typename T, int D, int G>
__device__ __forceinline__ void bottom_part(int kb, int ke, int lane, const int* col, const T* val,
                                            int64_t nnz, const T* x, T* acc) {
  constexpr int DP = Pad<D>::value;
  const gptr<int> gc = to_global(col);
  const gptr<T> gv = to_global(val);
  if constexpr (sizeof(T) == 4) {
    for (int q = kb / kQuad + lane; q < ke / kQuad; q += G) {
      const gint4 j = *reinterpret_cast<gptr<gint4>>(gc + q * kQuad);
      const int jj[kQuad] = {j.x, j.y, j.z, j.w};
#pragma unroll
      for (int a = 0; a < D; ++a) {
#pragma unroll
        for (int b = 0; b < D; ++b) {
          const gfloat4 v = *reinterpret_cast<gptr<gfloat4>>(
              gv + static_cast<int64_t>(a * D + b) * nnz + static_cast<int64_t>(q) * kQuad);
          acc[a] += v.x * x[jj[0] * DP + b] + v.y * x[jj[1] * DP + b] + v.z * x[jj[2] * DP + b] +
                    v.w * x[jj[3] * DP + b];
        }
      }
    }
  } else {
    for (int k = kb + lane; k < ke; k += G) {
      const int j = gc[k];
#pragma unroll
      for (int a = 0; a < D; ++a) {
#pragma unroll
        for (int b = 0; b < D; ++b) acc[a] += gv[static_cast<int64_t>(a * D + b) * nnz + k] * x[j * DP + b];
      }
    }
  }
}

// One cell by one wavefront (MODE as k_gs_cell: 0 zero-guess forward, 1 forward,
// 2 backward); RES: compute r = s - U x - M x instead of a sweep.
template <typename T, int D, int MODE, bool RES>
__device__ __forceinline__ void bottom_cell(const BottomLevel<T>& lv, int c, const BottomVecs<T>& v) {
  constexpr int DP = Pad<D>::value;
  constexpr int NV = CellShape<D>::NV, NU = CellShape<D>::NU;
  constexpr int GR = 64 / NV;
  const int lane = threadIdx.x & 63;
  const int v0 = v.cell_ptr[c], m = v.cell_ptr[c + 1] - v0, n = m * D;
  // the in-cell block row first, so its loads overlap the off-cell products
  const int t = lane;
  const bool own = t < n;
  const int k = own ? t / D : 0, comp = own ? t % D : 0;
  T Mrow[NU];
  const gptr<T> Mc = to_global(lv.cellM) + static_cast<int64_t>(c) * NU * NU;
#pragma unroll
  for (int u = 0; u < NU; ++u) Mrow[u] = (own && u < n) ? Mc[u * NU + t] : T(0);
  const int g = lane / GR, gl = lane % GR;
  T lo[D], up[D];
#pragma unroll
  for (int q = 0; q < D; ++q) { lo[q] = T(0); up[q] = T(0); }
  const bool want_lo = !RES, want_up = RES || MODE != 0;
  if (g < m) {
    const int i = v0 + g;
    if (want_lo) bottom_part<T, D, GR>(v.Lptr[i], v.Lptr[i + 1], gl, lv.L.col, lv.L.val, lv.L.nnz, v.x, lo);
    if (want_up) bottom_part<T, D, GR>(v.Uptr[i], v.Uptr[i + 1], gl, lv.U.col, lv.U.val, lv.U.nnz, v.x, up);
  }
#pragma unroll
  for (int q = 0; q < D; ++q) {
    lo[q] = group_sum<T, GR>(lo[q]);
    up[q] = group_sum<T, GR>(up[q]);
  }
  T my_lo = T(0), my_up = T(0);
#pragma unroll
  for (int q = 0; q < D; ++q) {   // every lane takes part in each shuffle
    const T l1 = __shfl(lo[q], k * GR, 64), u1 = __shfl(up[q], k * GR, 64);
    if (q == comp) { my_lo = l1; my_up = u1; }
  }
  const int xi = (v0 + k) * DP + comp;
  T xc = (own && (MODE != 0 || RES)) ? v.x[xi] : T(0);
  if (RES) {
    T mx = T(0);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      if (u < n) mx += Mrow[u] * bcast(xc, u);
    }
    if (own) v.r[xi] = v.s[xi] - my_up - mx;
    return;
  }
  const T s_t = own ? v.b[xi] - my_lo : T(0);
  if (MODE != 2 && own) v.s[xi] = s_t;
  T acc = s_t - (MODE != 0 ? my_up : T(0));
  const T rdg = own_reciprocal<T, NU>(Mrow, t, own);
  if (MODE != 0) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      if (u < n) {
        const T xu = bcast(xc, u);
        if (u != t) acc -= Mrow[u] * xu;
      }
    }
  }
#pragma unroll
  for (int uu = 0; uu < NU; ++uu) {
    const int u = MODE == 2 ? NU - 1 - uu : uu;
    if (u < n) {
      T delta = T(0);
      if (t == u) {
        const T xn = acc * rdg;
        delta = xn - xc;
        xc = xn;
      }
      delta = bcast(delta, u);
      if (t != u) acc -= Mrow[u] * delta;
    }
  }
  if (own) v.x[xi] = xc;
}

template <typename T, int D, int MODE>
__device__ __forceinline__ void bottom_sweep(const BottomLevel<T>& lv, const BottomVecs<T>& v) {
  const int w = threadIdx.x >> 6, nw = kBottomThreads / 64;
  for (int q = 0; q < lv.ncolors; ++q) {
    const int col = MODE == 2 ? lv.ncolors - 1 - q : q;
    for (int c = v.color_ptr[col] + w; c < v.color_ptr[col + 1]; c += nw)
      bottom_cell<T, D, MODE, false>(lv, c, v);
    __syncthreads();
  }
}

// Gather over a scalar CSR (rows [0, nrows), weights shared by the components)
// from the padded vector src into dst (ADD: dst += ...).
template <typename T, int D, bool ADD, typename TD>
__device__ __forceinline__ void bottom_transfer(int nrows, const int* ptr, const int* idx,
                                                const T* w, const T* src, int sstride, TD* dst,
                                                int dstride, const uint8_t* fixed = nullptr) {
  for (int i = threadIdx.x; i < nrows; i += blockDim.x) {
    T acc[D];
#pragma unroll
    for (int q = 0; q < D; ++q) acc[q] = T(0);
    for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
      const T wp = w[p];
      const T* e = src + idx[p] * sstride;
#pragma unroll
      for (int q = 0; q < D; ++q) acc[q] += wp * e[q];
    }
    const int fx = (ADD && fixed) ? fixed[i] : 0;
#pragma unroll
    for (int q = 0; q < D; ++q) {
      if (ADD)
        dst[i * dstride + q] += ((fx >> q) & 1) ? T(0) : acc[q];
      else
        dst[i * dstride + q] = static_cast<TD>(acc[q]);
    }
  }
}

template <typename T, int D>
__global__ __launch_bounds__(kBottomThreads) void k_bottom(BottomArgs<T> a) {
  constexpr int DP = Pad<D>::value;
  extern __shared__ __align__(16) unsigned char bottom_smem[];
  __shared__ double cy[kCoarseInvMax];
  __shared__ T cx[kCoarseInvMax];
  // LDS: every level's vectors (T), then every level's pointers (int)
  T* base = reinterpret_cast<T*>(bottom_smem);
  int total = 0;
  for (int j = 0; j < a.nlev; ++j) total += bottom_vec_elems(a.lev[j].n, DP);
  int* ibase = reinterpret_cast<int*>(base + total);
  auto vecs = [&](int k) {   // level k's LDS arrays
    int off = 0, ioff = 0;
    for (int j = 0; j < k; ++j) {
      off += bottom_vec_elems(a.lev[j].n, DP);
      ioff += bottom_int_elems(a.lev[j].n, a.lev[j].ncolors, a.lev[j].ncells);
    }
    const BottomLevel<T>& lv = a.lev[k];
    const int len = lv.n * DP;
    int* cp = ibase + ioff;
    int* cl = cp + lv.ncolors + 1;
    int* lp = cl + lv.ncells + 1;
    return BottomVecs<T>{base + off, base + off + len, base + off + 2 * len, base + off + 3 * len,
                         cp, cl, lp, lp + lv.n + 1};
  };
  // zero vectors, pointer copies; first level: b and (second W-cycle visit) x
  // from HBM; deeper levels start at zero
  {
    for (int e = threadIdx.x; e < total; e += blockDim.x) base[e] = T(0);
    for (int k = 0; k < a.nlev; ++k) {
      const BottomLevel<T>& lv = a.lev[k];
      const BottomVecs<T> v = vecs(k);
      for (int e = threadIdx.x; e <= lv.ncolors; e += blockDim.x) v.color_ptr[e] = lv.color_ptr[e];
      for (int e = threadIdx.x; e <= lv.ncells; e += blockDim.x) v.cell_ptr[e] = lv.cell_ptr[e];
      for (int e = threadIdx.x; e <= lv.n; e += blockDim.x) {
        v.Lptr[e] = lv.L.ptr[e];
        v.Uptr[e] = lv.U.ptr[e];
      }
    }
    __syncthreads();
    const BottomVecs<T> v = vecs(0);
    const int len = a.lev[0].n * DP;
    for (int e = threadIdx.x; e < len; e += blockDim.x) {
      v.b[e] = a.b[e];
      if (!a.zero_guess) v.x[e] = a.x[e];
    }
    __syncthreads();
  }
  // down: pre-smoothing, residual r = s - U x - M x, restriction
  for (int k = 0; k < a.nlev; ++k) {
    const BottomLevel<T>& lv = a.lev[k];
    const BottomVecs<T> v = vecs(k);
    for (int it = 0; it < a.npre; ++it) {
      if (it == 0 && (k > 0 || a.zero_guess))
        bottom_sweep<T, D, 0>(lv, v);
      else
        bottom_sweep<T, D, 1>(lv, v);
    }
    const int w = threadIdx.x >> 6, nw = kBottomThreads / 64;
    for (int c = w; c < lv.ncells; c += nw) bottom_cell<T, D, 1, true>(lv, c, v);
    __syncthreads();
    if (k + 1 < a.nlev)
      bottom_transfer<T, D, false, T>(lv.nnext, lv.pt_ptr, lv.pt_idx, lv.pt_w, v.r, DP, vecs(k + 1).b, DP);
    else   // the coarsest right-hand side, rounded to T as in the level vectors
      bottom_transfer<T, D, false, double>(lv.nnext, lv.pt_ptr, lv.pt_idx, lv.pt_w, v.r, DP, cy, D);
    __syncthreads();
  }
  // coarsest: x = A_c^{-1} b, rows in ascending column order (FP64)
  for (int i = threadIdx.x; i < a.ncoarse; i += blockDim.x) {
    const gptr<double> row = to_global(a.Minv) + static_cast<int64_t>(i) * a.ncoarse;
    double s = 0.0;
    for (int j = 0; j < a.ncoarse; ++j) s += row[j] * cy[j];
    cx[i] = static_cast<T>(s);
  }
  __syncthreads();
  // up: prolongation x += P e, post-smoothing
  for (int k = a.nlev - 1; k >= 0; --k) {
    const BottomLevel<T>& lv = a.lev[k];
    const BottomVecs<T> v = vecs(k);
    if (k + 1 < a.nlev)
      bottom_transfer<T, D, true, T>(lv.n, lv.p_ptr, lv.p_idx, lv.p_w, vecs(k + 1).x, DP, v.x, DP,
                                     lv.fixed);
    else
      bottom_transfer<T, D, true, T>(lv.n, lv.p_ptr, lv.p_idx, lv.p_w, cx, D, v.x, DP, lv.fixed);
    __syncthreads();
    for (int it = 0; it < a.npost; ++it) bottom_sweep<T, D, 2>(lv, v);
  }
  const BottomVecs<T> v = vecs(0);
  for (int e = threadIdx.x; e < a.lev[0].n * DP; e += blockDim.x) a.x[e] = v.x[e];
}

// ---------------------------------------------------------------------------
// K7/K8: PCG vector kernels and device-side scalars (FP64, deterministic).
// ---------------------------------------------------------------------------
struct Scalars {
  double rho;       // r^T z of the current direction
  double pq;        // p^T A p
  double alpha, beta;
  double res;       // ||r||
  double normF;     // ||F||
  double rtol;
  double res_true;  // ||F - A x||
  int done;         // 1 = stop (converged or breakdown)
  int status;       // 0 running/converged, 5 breakdown
  int first;        // next beta finalisation is the first one
  int iters;        // products A p so far
};

enum FinMode { FIN_NORMF = 0, FIN_ALPHA = 1, FIN_RES = 2, FIN_BETA = 3, FIN_TRUE = 4 };

// Scalar steps of Algorithm 2 from a finished reduction `tot`.
template <int MODE>
__device__ __forceinline__ void finalize_scalar(double tot, Scalars* s) {
  if (MODE == FIN_NORMF) {
    s->normF = sqrt(tot);
    s->res = s->normF;
    s->done = 0;
    s->status = 0;
    s->first = 1;
    s->iters = 0;
    s->alpha = s->beta = 0.0;
  } else if (MODE == FIN_ALPHA) {
    s->pq = tot;
    if (!(tot > 0.0) || !isfinite(tot)) {
      s->status = 5;
      s->done = 1;
    } else {
      s->alpha = s->rho / tot;
    }
  } else if (MODE == FIN_RES) {
    s->res = sqrt(tot);
    s->iters += 1;
    if (!isfinite(s->res)) {
      s->status = 5;
      s->done = 1;
    } else if (s->res / s->normF < s->rtol) {
      s->done = 1;
    }
  } else if (MODE == FIN_BETA) {
    if (s->first) {
      s->beta = 0.0;
      s->first = 0;
    } else {
      s->beta = tot / s->rho;
    }
    s->rho = tot;
    if (!isfinite(tot)) {
      s->status = 5;
      s->done = 1;
    }
  } else {
    s->res_true = sqrt(tot);
  }
}

// The iteration's report to the host: products so far and the stop flag, written
// to pinned host memory that the host polls (a copy and a stream synchronisation
// per iteration left the device idle for 8 to 12 us).
__device__ __forceinline__ void report(int* mail, const Scalars* s) {
  __hip_atomic_store(mail, s->iters * 2 + (s->done ? 1 : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// mail (FIN_RES): where to report.
template <int MODE>
__global__ __launch_bounds__(1024) void k_finalize(const double* __restrict__ partial, int np,
                                                   Scalars* s, int* mail) {
  __shared__ double sh[1024];
  if (MODE != FIN_NORMF && MODE != FIN_TRUE && s->done) {
    if (MODE == FIN_RES && threadIdx.x == 0) report(mail, s);
    return;
  }
  double v = 0.0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) v += partial[i];
  const double tot = block_sum(v, sh);
  if (threadIdx.x == 0) {
    finalize_scalar<MODE>(tot, s);
    if (MODE == FIN_RES) report(mail, s);
  }
}

// partial sums of a.b over a flat vector (grid-stride, fixed grid)
template <typename TB>
__global__ __launch_bounds__(kBlock) void k_dot(int64_t n, const double* __restrict__ a,
                                                const TB* __restrict__ b,
                                                double* __restrict__ partial,
                                                const int* __restrict__ done) {
  if (done && *done) return;
  __shared__ double sh[kBlock];
  double v = 0.0;
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock)
    v += a[i] * static_cast<double>(b[i]);
  const double s = block_sum(v, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// x += alpha p; r -= alpha q; partial ||r||^2; b0 = (T) r (V-cycle input)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_update_xr(int64_t n, const Scalars* __restrict__ s,
                                                      const double* __restrict__ p,
                                                      const double* __restrict__ q,
                                                      double* __restrict__ x,
                                                      double* __restrict__ r, T* __restrict__ b0,
                                                      double* __restrict__ partial) {
  __shared__ double sh[kBlock];
  if (s->done) return;
  const double alpha = s->alpha;
  double v = 0.0;
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock) {
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    if (b0) b0[i] = static_cast<T>(ri);
    v += ri * ri;
  }
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// p = z + beta p with z = (double) the V-cycle output
template <typename T>
__global__ __launch_bounds__(kBlock) void k_update_p(int64_t n, const Scalars* __restrict__ s,
                                                     const T* __restrict__ z,
                                                     double* __restrict__ p) {
  if (s->done) return;
  const double beta = s->beta;
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock)
    p[i] = static_cast<double>(z[i]) + beta * p[i];
}

// Small problems (n <= kSmallFlat entries): the vector steps of an iteration are
// launches that do next to nothing, so one workgroup takes a run of them. After the
// SpMV: alpha from its partial sums, x += alpha p, r -= alpha q, ||r||, the stopping
// test and the report. FP32-cycle iteration, separate launches and this way: 968
// entries 73 and 68 us, 4,232 79 and 76, 5,832 82 and 81, 8,112 110 and 114.
constexpr int kSmallFlat = 6144;
constexpr int kSmallRounds = kSmallFlat / 1024;   // entries per thread

// Sum over the workgroup, thread t holding entries t, t + 1024, ...: in the order of
// k_dot's workgroups of 256 entries and k_finalize's tree over them, so that a
// problem's iterates do not depend on which form its size takes (PCG in FP32-cycle
// 2D problems amplifies one flipped rounding of r to 1e-9 of the solution). A
// workgroup of 256 entries is four wavefronts here: the first adds the others'
// values as the tree's two widest steps do, and goes on inside itself.
struct SmallSum {
  double w[kSmallRounds][4][3][64];
  double part[kSmallFlat / kBlock];
};

__device__ __forceinline__ double small_sum(int n, double (&v)[kSmallRounds], SmallSum& sh) {
#pragma unroll
  for (int j = 0; j < kSmallRounds; ++j) asm volatile("" : "+v"(v[j]));   // products rounded before the sums
  const int g = threadIdx.x >> 8, w = (threadIdx.x >> 6) & 3, l = threadIdx.x & 63;
  if (w > 0) {
#pragma unroll
    for (int j = 0; j < kSmallRounds; ++j)
      if (1024 * j < n) sh.w[j][g][w - 1][l] = v[j];
  }
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int j = 0; j < kSmallRounds; ++j) {
      double c = 0.0;
      if (1024 * j < n)
        c = wave_tree((v[j] + sh.w[j][g][1][l]) + (sh.w[j][g][0][l] + sh.w[j][g][2][l]));
      if (l == 0) sh.part[4 * j + g] = c;
    }
  }
  __syncthreads();
  constexpr int NP = kSmallFlat / kBlock;
  return bcast(wave_tree(l < NP ? sh.part[l] : 0.0), 0);
}

template <typename T>
__global__ __launch_bounds__(1024) void k_small_xr(int n, Scalars* s, const double* __restrict__ partial,
                                                   int np, const double* __restrict__ p,
                                                   const double* __restrict__ q, double* __restrict__ x,
                                                   double* __restrict__ r, T* __restrict__ b0, int* mail) {
  __shared__ double sh[1024];
  __shared__ SmallSum ss;
  if (s->done) {
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double rho = s->rho;
  double v = 0.0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) v += partial[i];
  const double pq = block_sum(v, sh);
  if (threadIdx.x == 0) finalize_scalar<FIN_ALPHA>(pq, s);
  if (!(pq > 0.0) || !isfinite(pq)) {   // breakdown: finalize_scalar has stopped the iteration
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double alpha = rho / pq;
  double e[kSmallRounds];
#pragma unroll
  for (int j = 0; j < kSmallRounds; ++j) {
    const int i = threadIdx.x + 1024 * j;
    e[j] = 0.0;
    if (i < n) {
      x[i] += alpha * p[i];
      const double ri = r[i] - alpha * q[i];
      r[i] = ri;
      if (b0) b0[i] = static_cast<T>(ri);
      e[j] = ri * ri;
    }
  }
  const double rr = small_sum(n, e, ss);
  if (threadIdx.x == 0) {
    finalize_scalar<FIN_RES>(rr, s);
    report(mail, s);
  }
}

// After the preconditioner: rho = r.z, beta, p = z + beta p.
template <typename T>
__global__ __launch_bounds__(1024) void k_small_p(int n, Scalars* s, const double* __restrict__ r,
                                                  const T* __restrict__ z, double* __restrict__ p) {
  __shared__ SmallSum ss;
  if (s->done) return;
  const double rho = s->rho;
  const bool first = s->first != 0;
  double e[kSmallRounds];
#pragma unroll
  for (int j = 0; j < kSmallRounds; ++j) {
    const int i = threadIdx.x + 1024 * j;
    e[j] = i < n ? r[i] * static_cast<double>(z[i]) : 0.0;
  }
  const double tot = small_sum(n, e, ss);   // (its barriers keep the reads of s before the write)
  if (threadIdx.x == 0) finalize_scalar<FIN_BETA>(tot, s);
  if (!isfinite(tot)) return;
  const double beta = first ? 0.0 : tot / rho;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) p[i] = static_cast<double>(z[i]) + beta * p[i];
}

// point Jacobi z = r / a_ii (a context preconditioner, not the paper's)
template <int D>
__global__ __launch_bounds__(kBlock) void k_jacobi(int n, const double* __restrict__ diag,
                                                   const double* __restrict__ r,
                                                   double* __restrict__ z,
                                                   const int* __restrict__ done) {
  if (done && *done) return;
  constexpr int DP = Pad<D>::value;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int a = 0; a < D; ++a)
    z[static_cast<int64_t>(i) * DP + a] =
        r[static_cast<int64_t>(i) * DP + a] / diag[static_cast<int64_t>(i) * D * D + a * D + a];
}

// flat conversions and fills
template <typename TA, typename TB>
__global__ __launch_bounds__(kBlock) void k_convert(int64_t n, const TA* __restrict__ a,
                                                    TB* __restrict__ b) {
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock)
    b[i] = static_cast<TB>(a[i]);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill(int64_t n, T* __restrict__ a, T v) {
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock)
    a[i] = v;
}

// r = F - q (flat), partial ||r||^2
__global__ __launch_bounds__(kBlock) void k_sub_norm(int64_t n, const double* __restrict__ F,
                                                     const double* __restrict__ q,
                                                     double* __restrict__ r,
                                                     double* __restrict__ partial) {
  __shared__ double sh[kBlock];
  double v = 0.0;
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock) {
    const double t = F[i] - q[i];
    if (r) r[i] = t;
    v += t * t;
  }
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// user layout [nv][D] <-> device numbering (padded) through a vertex map
// fixed (optional): constrained components of the rows, read as 0.
template <typename TS, typename TD, int D>
__global__ __launch_bounds__(kBlock) void k_gather_user(int n, const int* __restrict__ map,
                                                        const TS* __restrict__ src,
                                                        TD* __restrict__ dst,
                                                        const uint8_t* __restrict__ fixed) {
  constexpr int DP = Pad<D>::value;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int64_t v = map[i];
  const int fx = fixed ? fixed[i] : 0;
#pragma unroll
  for (int a = 0; a < DP; ++a)
    dst[static_cast<int64_t>(i) * DP + a] =
        (a < D && !((fx >> a) & 1)) ? static_cast<TD>(src[v * D + a]) : TD(0);
}

template <typename TS, typename TD, int D>
__global__ __launch_bounds__(kBlock) void k_scatter_user(int n, const int* __restrict__ map,
                                                         const TS* __restrict__ src,
                                                         TD* __restrict__ dst) {
  constexpr int DP = Pad<D>::value;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int64_t v = map[i];
#pragma unroll
  for (int a = 0; a < D; ++a) dst[v * D + a] = static_cast<TD>(src[static_cast<int64_t>(i) * DP + a]);
}

}  // namespace dev
}  // namespace vasmg
