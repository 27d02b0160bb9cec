// Packed solves: several independent problems in one block-diagonal hierarchy,
// each with its own PCG recurrence (Section 2.2, Algorithm 2): its own dot
// products, alpha, beta and stopping test, so every problem runs the iteration
// it would run alone (to rounding) while the V-cycle and the SpMV launches are
// shared. A problem is a segment of the fine level: seg_rows[seg_ptr[s] ..
// seg_ptr[s + 1]) are its device rows, ascending.
// Included by vasmg.hip (uses kBlock, block_sum, Scalars, finalize_scalar).
#pragma once

namespace vasmg {
namespace dev {

// One workgroup per segment sums over its entries (DP per row). The order is that of
// 256 threads, each taking every 256th entry, and a tree over them (so that a part's
// iterates stay what they are whatever fetches the entries); all 1,024 threads fetch,
// for the loads in flight, and hand the factors over in LDS.
constexpr int kSegBlock = 1024, kSegChunk = 2 * kSegBlock;

struct SegSum {
  double a[kSegChunk], b[kSegChunk], t[kBlock];
};

// Sum of a b over the entries e < n, f(e, a, b) giving entry e's factors (called
// once per entry, by one thread); the same in every thread.
template <class F>
__device__ __forceinline__ double seg_sum(int64_t n, SegSum& sh, F&& f) {
  const int t = threadIdx.x;
  double a[2], b[2], v = 0.0;
  auto fetch = [&](int64_t c0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t e = c0 + t + u * kSegBlock;
      a[u] = b[u] = 0.0;
      if (e < n) f(e, a[u], b[u]);
    }
  };
  fetch(0);
  for (int64_t c0 = 0; c0 < n; c0 += kSegChunk) {
    __syncthreads();   // the chunk before has been added
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sh.a[t + u * kSegBlock] = a[u];
      sh.b[t + u * kSegBlock] = b[u];
    }
    __syncthreads();
    fetch(c0 + kSegChunk);
    if (t < kBlock) {
#pragma unroll
      for (int i = 0; i < kSegChunk / kBlock; ++i)
        v = __builtin_fma(sh.a[t + i * kBlock], sh.b[t + i * kBlock], v);
    }
  }
  if (t < kBlock) sh.t[t] = v;
  __syncthreads();
#pragma unroll
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (t < s) sh.t[t] += sh.t[t + s];
    __syncthreads();
  }
  const double r = sh.t[0];
  __syncthreads();
  return r;
}

// The segment's dot product (DIFF: of a - b with itself), then the scalar step MODE
// (the norms of the right-hand side and the true residual) on its own scalars.
template <int MODE, bool DIFF, int DP>
__global__ __launch_bounds__(kSegBlock) void k_seg_dot(const int* __restrict__ seg_ptr,
                                                       const int* __restrict__ seg_rows,
                                                       const double* __restrict__ a,
                                                       const double* __restrict__ b,
                                                       Scalars* __restrict__ ss) {
  __shared__ SegSum sh;
  const int s = blockIdx.x, lo = seg_ptr[s];
  const int64_t n = static_cast<int64_t>(seg_ptr[s + 1] - lo) * DP;
  const double tot = seg_sum(n, sh, [&](int64_t e, double& u, double& v) {
    const int64_t i = static_cast<int64_t>(seg_rows[lo + e / DP]) * DP + e % DP;
    if (DIFF) {
      u = v = a[i] - b[i];
    } else {
      u = a[i];
      v = b[i];
    }
  });
  if (threadIdx.x == 0) finalize_scalar<MODE>(tot, &ss[s]);
}

// After ||F||: rtol, and segments with nothing to solve (F = 0, or not finite:
// breakdown) finish at once.
__global__ void k_seg_start(int nseg, Scalars* __restrict__ ss, double rtol, int* mail) {
  const int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= nseg) return;
  ss[s].rtol = rtol;
  const double f = ss[s].normF;
  if (!isfinite(f)) {
    ss[s].status = 5;
    ss[s].done = 1;
  } else if (f == 0.0) {
    ss[s].done = 1;
  }
  report(mail + s, &ss[s]);
}

// The vector work of an iteration, one workgroup per part: all of it between the
// SpMV and the preconditioner (p.q, alpha, x += alpha p, r -= alpha q, b0 = (T) r,
// ||r||, the stopping test, the report) and all of it after (r.z, beta,
// p = z + beta p).
template <typename T, int DP>
__global__ __launch_bounds__(kSegBlock) void k_seg_xr(const int* __restrict__ seg_ptr,
                                                      const int* __restrict__ seg_rows,
                                                      Scalars* __restrict__ ss,
                                                      const double* __restrict__ p,
                                                      const double* __restrict__ q,
                                                      double* __restrict__ x, double* __restrict__ r,
                                                      T* __restrict__ b0, int* mail) {
  __shared__ SegSum sh;
  Scalars* s = ss + blockIdx.x;
  mail += blockIdx.x;
  if (s->done) {
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double rho = s->rho;
  const int lo = seg_ptr[blockIdx.x];
  const int64_t n = static_cast<int64_t>(seg_ptr[blockIdx.x + 1] - lo) * DP;
  auto at = [&](int64_t e) { return static_cast<int64_t>(seg_rows[lo + e / DP]) * DP + e % DP; };
  const double pq = seg_sum(n, sh, [&](int64_t e, double& u, double& v) {
    const int64_t i = at(e);
    u = p[i];
    v = q[i];
  });
  if (threadIdx.x == 0) finalize_scalar<FIN_ALPHA>(pq, s);
  if (!(pq > 0.0) || !isfinite(pq)) {   // breakdown: this part has stopped
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double alpha = rho / pq;
  const double rr = seg_sum(n, sh, [&](int64_t e, double& u, double& v) {
    const int64_t i = at(e);
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    if (b0) b0[i] = static_cast<T>(ri);
    u = v = ri;
  });
  if (threadIdx.x == 0) {
    finalize_scalar<FIN_RES>(rr, s);
    report(mail, s);
  }
}

template <typename T, int DP>
__global__ __launch_bounds__(kSegBlock) void k_seg_p(const int* __restrict__ seg_ptr,
                                                     const int* __restrict__ seg_rows,
                                                     Scalars* __restrict__ ss,
                                                     const double* __restrict__ r,
                                                     const T* __restrict__ z, double* __restrict__ p) {
  __shared__ SegSum sh;
  Scalars* s = ss + blockIdx.x;
  if (s->done) return;
  const double rho = s->rho;
  const bool first = s->first != 0;
  const int lo = seg_ptr[blockIdx.x];
  const int64_t n = static_cast<int64_t>(seg_ptr[blockIdx.x + 1] - lo) * DP;
  auto at = [&](int64_t e) { return static_cast<int64_t>(seg_rows[lo + e / DP]) * DP + e % DP; };
  const double tot = seg_sum(n, sh, [&](int64_t e, double& u, double& v) {
    const int64_t i = at(e);
    u = r[i];
    v = static_cast<double>(z[i]);
  });   // (its barriers keep the reads of s before the write)
  if (threadIdx.x == 0) finalize_scalar<FIN_BETA>(tot, s);
  if (!isfinite(tot)) return;
  const double beta = first ? 0.0 : tot / rho;
#pragma unroll 4
  for (int64_t e = threadIdx.x; e < n; e += kSegBlock) {
    const int64_t i = at(e);
    p[i] = static_cast<double>(z[i]) + beta * p[i];
  }
}

}  // namespace dev
}  // namespace vasmg
