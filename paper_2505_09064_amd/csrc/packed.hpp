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

// One workgroup per segment: the segment's dot product over its rows (DP
// entries each; DIFF: of a - b with itself), summed in a fixed order, then the
// scalar step MODE (the norms of the right-hand side and the true residual) on
// the segment's own scalars.
constexpr int kSegBlock = 1024;

template <int MODE, bool DIFF>
__global__ __launch_bounds__(kSegBlock) void k_seg_dot(const int* __restrict__ seg_ptr,
                                                       const int* __restrict__ seg_rows, int DP,
                                                       const double* __restrict__ a,
                                                       const double* __restrict__ b,
                                                       Scalars* __restrict__ ss) {
  __shared__ double sh[kSegBlock];
  const int s = blockIdx.x;
  const int lo = seg_ptr[s], hi = seg_ptr[s + 1];
  double v = 0.0;
  for (int64_t q = static_cast<int64_t>(lo) * DP + threadIdx.x; q < static_cast<int64_t>(hi) * DP;
       q += kSegBlock) {
    const int64_t i = static_cast<int64_t>(seg_rows[q / DP]) * DP + q % DP;
    if (DIFF) {
      const double t = a[i] - b[i];
      v += t * t;
    } else {
      v += a[i] * b[i];
    }
  }
  const double tot = block_sum(v, sh);
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
// p = z + beta p). As separate launches, with the sums by 256 threads per part and
// the updates spread over the chip, an iteration of 8 parts of 3,840 rows took
// 509 us, and 424 us this way; of 2 parts of 7,600 rows 536 and 374 us. The sums
// need one workgroup per part in either form, so they bound both at any part size.
template <typename T, int DP>
__global__ __launch_bounds__(kSegBlock) void k_seg_xr(const int* __restrict__ seg_ptr,
                                                      const int* __restrict__ seg_rows,
                                                      Scalars* __restrict__ ss,
                                                      const double* __restrict__ p,
                                                      const double* __restrict__ q,
                                                      double* __restrict__ x, double* __restrict__ r,
                                                      T* __restrict__ b0, int* mail) {
  __shared__ double sh[kSegBlock];
  Scalars* s = ss + blockIdx.x;
  mail += blockIdx.x;
  if (s->done) {
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double rho = s->rho;
  const int64_t lo = static_cast<int64_t>(seg_ptr[blockIdx.x]) * DP;
  const int64_t hi = static_cast<int64_t>(seg_ptr[blockIdx.x + 1]) * DP;
  double v = 0.0;
#pragma unroll 4
  for (int64_t e = lo + threadIdx.x; e < hi; e += kSegBlock) {
    const int64_t i = static_cast<int64_t>(seg_rows[e / DP]) * DP + e % DP;
    v += p[i] * q[i];
  }
  const double pq = block_sum(v, sh);
  if (threadIdx.x == 0) finalize_scalar<FIN_ALPHA>(pq, s);
  if (!(pq > 0.0) || !isfinite(pq)) {   // breakdown: this part has stopped
    if (threadIdx.x == 0) report(mail, s);
    return;
  }
  const double alpha = rho / pq;
  v = 0.0;
#pragma unroll 4
  for (int64_t e = lo + threadIdx.x; e < hi; e += kSegBlock) {
    const int64_t i = static_cast<int64_t>(seg_rows[e / DP]) * DP + e % DP;
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    if (b0) b0[i] = static_cast<T>(ri);
    v += ri * ri;
  }
  const double rr = block_sum(v, sh);
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
  __shared__ double sh[kSegBlock];
  Scalars* s = ss + blockIdx.x;
  if (s->done) return;
  const double rho = s->rho;
  const bool first = s->first != 0;
  const int64_t lo = static_cast<int64_t>(seg_ptr[blockIdx.x]) * DP;
  const int64_t hi = static_cast<int64_t>(seg_ptr[blockIdx.x + 1]) * DP;
  double v = 0.0;
#pragma unroll 4
  for (int64_t e = lo + threadIdx.x; e < hi; e += kSegBlock) {
    const int64_t i = static_cast<int64_t>(seg_rows[e / DP]) * DP + e % DP;
    v += r[i] * static_cast<double>(z[i]);
  }
  const double tot = block_sum(v, sh);   // (its barriers keep the reads of s before the write)
  if (threadIdx.x == 0) finalize_scalar<FIN_BETA>(tot, s);
  if (!isfinite(tot)) return;
  const double beta = first ? 0.0 : tot / rho;
#pragma unroll 4
  for (int64_t e = lo + threadIdx.x; e < hi; e += kSegBlock) {
    const int64_t i = static_cast<int64_t>(seg_rows[e / DP]) * DP + e % DP;
    p[i] = static_cast<double>(z[i]) + beta * p[i];
  }
}

}  // namespace dev
}  // namespace vasmg
