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

// A segment's entries (DP per row) by one workgroup: thread t takes entries t,
// t + 256, ..., UN of them per round, whose rows are known a round before and whose
// loads are all in flight before the first is used; body(i, s, v) then takes entry i
// with what load(i) fetched, in ascending order. Returns the tree sum of the threads'
// v. (The order of the sum is part of the result: see CellSums.)
template <int DP, int UN, class Load, class Body>
__device__ __forceinline__ double seg_walk(const int* __restrict__ rows, int64_t n, double* sh, Load&& load,
                                           Body&& body) {
  using S = decltype(load(int64_t(0)));
  const int64_t step = int64_t(kBlock) * UN;
  double v = 0.0;
  int row[UN];
  auto fetch_rows = [&](int64_t e0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t e = e0 + u * kBlock;
      row[u] = rows[(e < n ? e : n - 1) / DP];
    }
  };
  const int64_t first = threadIdx.x;
  if (first < n) fetch_rows(first);
  for (int64_t e0 = first; e0 < n; e0 += step) {
    int64_t i[UN];
    S s[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      // (past the end: the last row's, unused)
      i[u] = static_cast<int64_t>(row[u]) * DP + (e0 + u * kBlock) % DP;
      s[u] = load(i[u]);
    }
    if (e0 + step < n) fetch_rows(e0 + step);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (e0 + u * kBlock < n) body(i[u], s[u], v);
  }
  return block_sum(v, sh);
}

struct SegPair {
  double a, b;
};
struct SegUpdate {
  double p, q, x, r;
};

// The segment's dot product (DIFF: of a - b with itself), then the scalar step MODE
// (the norms of the right-hand side and the true residual) on its own scalars.
template <int MODE, bool DIFF, int DP>
__global__ __launch_bounds__(kBlock) void k_seg_dot(const int* __restrict__ seg_ptr,
                                                    const int* __restrict__ seg_rows,
                                                    const double* __restrict__ a,
                                                    const double* __restrict__ b,
                                                    Scalars* __restrict__ ss) {
  __shared__ double sh[kBlock];
  const int s = blockIdx.x, lo = seg_ptr[s];
  const int64_t n = static_cast<int64_t>(seg_ptr[s + 1] - lo) * DP;
  const double tot = seg_walk<DP, 16>(
      seg_rows + lo, n, sh, [&](int64_t i) { return SegPair{a[i], b[i]}; },
      [&](int64_t, const SegPair& e, double& v) {
        const double t = e.a - e.b;
        v += DIFF ? t * t : e.a * e.b;
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
// p = z + beta p). The vector work of an iteration this way, and as separate launches
// whose sums also ran in one workgroup per part, with few loads in flight, and whose
// updates were spread over the chip: 2 parts of 62,500 2D rows 190 and 812 us, 8 of
// them 257 and 1,061, 2 of 250,000 1,035 and 4,253, 2 of 91,125 3D rows 787 and 3,134.
// (A part's 13 array passes run in one workgroup here, its sums need 6 of them: these
// sums with the updates spread over the chip were not measured.)
template <typename T, int DP>
__global__ __launch_bounds__(kBlock) void k_seg_xr(const int* __restrict__ seg_ptr,
                                                   const int* __restrict__ seg_rows,
                                                   Scalars* __restrict__ ss,
                                                   const double* __restrict__ p,
                                                   const double* __restrict__ q,
                                                   double* __restrict__ x, double* __restrict__ r,
                                                   T* __restrict__ b0, int* mail) {
  __shared__ double sh[kBlock];
  Scalars* s = ss + blockIdx.x;
  mail += blockIdx.x;
  if (s->done) {
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double rho = s->rho;
  const int lo = seg_ptr[blockIdx.x];
  const int64_t n = static_cast<int64_t>(seg_ptr[blockIdx.x + 1] - lo) * DP;
  const double pq = seg_walk<DP, 16>(
      seg_rows + lo, n, sh, [&](int64_t i) { return SegPair{p[i], q[i]}; },
      [&](int64_t, const SegPair& e, double& v) { v += e.a * e.b; });
  if (threadIdx.x == 0) finalize_scalar<FIN_ALPHA>(pq, s);
  if (!(pq > 0.0) || !isfinite(pq)) {   // breakdown: this part has stopped
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double alpha = rho / pq;
  const double rr = seg_walk<DP, 8>(
      seg_rows + lo, n, sh, [&](int64_t i) { return SegUpdate{p[i], q[i], x[i], r[i]}; },
      [&](int64_t i, const SegUpdate& e, double& v) {
        x[i] = e.x + alpha * e.p;
        const double ri = e.r - alpha * e.q;
        r[i] = ri;
        if (b0) b0[i] = static_cast<T>(ri);
        v += ri * ri;
      });
  if (threadIdx.x == 0) {
    finalize_scalar<FIN_RES>(rr, s);
    report(mail, s);
  }
}

template <typename T, int DP>
__global__ __launch_bounds__(kBlock) void k_seg_p(const int* __restrict__ seg_ptr,
                                                  const int* __restrict__ seg_rows,
                                                  Scalars* __restrict__ ss,
                                                  const double* __restrict__ r,
                                                  const T* __restrict__ z, double* __restrict__ p) {
  __shared__ double sh[kBlock];
  Scalars* s = ss + blockIdx.x;
  if (s->done) return;
  const double rho = s->rho;
  const bool first = s->first != 0;
  const int lo = seg_ptr[blockIdx.x];
  const int64_t n = static_cast<int64_t>(seg_ptr[blockIdx.x + 1] - lo) * DP;
  const double tot = seg_walk<DP, 16>(
      seg_rows + lo, n, sh, [&](int64_t i) { return SegPair{r[i], static_cast<double>(z[i])}; },
      [&](int64_t, const SegPair& e, double& v) { v += e.a * e.b; });
  // (its barriers keep the reads of s before the write)
  if (threadIdx.x == 0) finalize_scalar<FIN_BETA>(tot, s);
  if (!isfinite(tot)) return;
  const double beta = first ? 0.0 : tot / rho;
  seg_walk<DP, 16>(
      seg_rows + lo, n, sh, [&](int64_t i) { return SegPair{static_cast<double>(z[i]), p[i]}; },
      [&](int64_t i, const SegPair& e, double&) { p[i] = e.a + beta * e.b; });
}

}  // namespace dev
}  // namespace vasmg
