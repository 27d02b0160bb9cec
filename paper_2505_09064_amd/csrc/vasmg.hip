// Device hierarchy, V-cycle schedule, PCG driver and the C ABI of libvasmg.
//
// Solve phase of arXiv 2505.09064: PCG (Section 2.2, Algorithm 2) with one
// V-cycle (Section 3, Algorithm 3 applied recursively) as the preconditioner.
// All steps run in the kernels of kernels.hpp. One PCG iteration is split in
// two captured hipGraphs:
//   graph A: q = A p with p.q partials, alpha, x += alpha p, r -= alpha q with
//            ||r||^2 partials (and the FP32 copy of r), convergence flag;
//   graph B: z = B r (the V-cycle), r.z partials, beta, p = z + beta p.
// Graph A ends in a report to pinned host memory that the host polls (the only
// per-iteration wait).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <chrono>
#include <mutex>
#include <numeric>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "../../include/vasmg.h"
#include "hierarchy.hpp"
#include "kernels.hpp"
#include "block.hpp"
#include "packed.hpp"
#include "dense.hpp"

using namespace vasmg;
using dev::Scalars;

namespace {

thread_local std::string g_last_error;
std::atomic<int> g_galerkin_window{0};   // test hook: device Galerkin window (0 = max)

#define HIP_CHECK(expr)                                                                    \
  do {                                                                                     \
    hipError_t _e = (expr);                                                                \
    if (_e != hipSuccess)                                                                  \
      throw vasmg::Error{VASMG_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(_e)}; \
  } while (0)

inline int pow2_ceil(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

inline int grid_for(int64_t items, int per_block) {
  return static_cast<int>(std::max<int64_t>(1, (items + per_block - 1) / per_block));
}

constexpr int kFlatGrid = 1024;   // fixed grid of the flat reduction kernels

// -------------------------------------------------------------------------
struct DevLevel {
  int n = 0;
  int d = 0;
  int ncolors = 0;
  int64_t nnz = 0;                 // off-diagonal (point) or off-cell (cell) blocks
  int64_t nnz_lo = 0, nnz_up = 0;  // blocks coupling to earlier / later colours
  int64_t Lstride = 0, Ustride = 0; // stored L / U entries (plane stride; rows padded on cell levels)
  int64_t p_nnz = 0;               // entries of P_l
  int G = 8;                       // lanes per block row (Gauss-Seidel, residual)
  int Gspmv = 8;                   // lanes per block row of the fine FP64 SpMV
  int mcGL = 0;                    // block right-hand sides: lanes per block row
  std::vector<int> color_ptr;      // host: device rows (point levels) or cells (cell
                                   // levels) of colour c = [ptr[c], ptr[c+1])
  bool cells = false;              // coarse lattice level: Gauss-Seidel over cells
  int ncells = 0;
  int* cell_ptr = nullptr;         // cell levels: first device row of each cell
  int* cell_rec = nullptr;         // cell levels: each cell's record (CellRec)
  // colour-block levels (cells grouped into blocks of several cells, a colour
  // per block): color_ptr then counts blocks, block_ptr gives each block's
  // first cell, and the off-cell blocks inside a row's colour block form the
  // parts E (earlier cells) and F (later cells)
  bool blocks = false;
  int nblocks = 0;
  int* block_ptr = nullptr;
  int *Eptr = nullptr, *Ecol = nullptr, *Fptr = nullptr, *Fcol = nullptr;
  float *Eval32 = nullptr, *Fval32 = nullptr;
  double *Eval64 = nullptr, *Fval64 = nullptr;
  int64_t nnz_e = 0, nnz_f = 0, Estride = 0, Fstride = 0;
  int* color_ptr_dev = nullptr;    // device copy of color_ptr (fused bottom levels only)
  float* cellM32 = nullptr;        // cell levels: dense in-cell blocks (column-major)
  double* cellM64 = nullptr;
  int* perm = nullptr;             // device row -> canonical index
  uint8_t* fixed = nullptr;        // constrained components per device row (null: none)
  // off-diagonal blocks to earlier colours (L) and to later colours (U)
  int *Lptr = nullptr, *Lcol = nullptr, *Uptr = nullptr, *Ucol = nullptr;
  float *Lval32 = nullptr, *Uval32 = nullptr;
  double *Lval64 = nullptr, *Uval64 = nullptr;
  float* diag32 = nullptr;
  double* diag64 = nullptr;
  // damped vertex-block Jacobi smoother (option smoother = JACOBI)
  float* dinv32 = nullptr;
  double* dinv64 = nullptr;
  double omega = 0.0;
  // prolongation to the next level (device numbering on both sides)
  int nnext = 0;
  int* p_ptr = nullptr;
  int* p_idx = nullptr;
  float* p_w32 = nullptr;
  double* p_w64 = nullptr;
  int* pt_ptr = nullptr;
  int* pt_idx = nullptr;
  float* pt_w32 = nullptr;
  double* pt_w64 = nullptr;
  // V-cycle work vectors (padded, V-cycle precision)
  void* b = nullptr;
  void* x = nullptr;
  void* s = nullptr;
  void* r = nullptr;
  bool has32 = false, has64 = false;
};

}  // namespace

// Pinned host blocks for the per-iteration scalar read-back. Freeing pinned
// memory synchronises the whole device (it would stall every other solve in
// flight), so blocks are recycled through this pool and never freed.
class PinnedPool {
 public:
  static constexpr size_t kBytes = 4096;
  static constexpr int kBatch = 64;
  void* get() {
    std::lock_guard<std::mutex> g(mu_);
    if (!free_.empty()) {
      void* p = free_.back();
      free_.pop_back();
      return p;
    }
    // one allocation per 64 blocks: pinned allocations are rare and early
    char* p = nullptr;
    if (hipHostMalloc(reinterpret_cast<void**>(&p), kBytes * kBatch, hipHostMallocCoherent) != hipSuccess)
      throw vasmg::Error{VASMG_ENOMEM, "pinned host allocation failed"};
    for (int i = kBatch - 1; i > 0; --i) free_.push_back(p + static_cast<size_t>(i) * kBytes);
    return p;
  }
  void put(void* p) {
    if (!p) return;
    std::lock_guard<std::mutex> g(mu_);
    free_.push_back(p);
  }

 private:
  std::mutex mu_;
  std::vector<void*> free_;
};

PinnedPool& pinned_pool() {
  static PinnedPool* pool = new PinnedPool;   // lives until the process ends
  return *pool;
}

constexpr int kMailWords = 512;   // reports in a pinned block

struct vasmg_ctx {
  Hierarchy H;
  vasmg_options opt{};
  int d = 0, DP = 0;
  int L = 0;                        // index of the coarsest level
  bool host_only = true;
  bool vc32 = false;                // V-cycle precision FP32
  int device = 0;
  std::vector<void*> allocs;
  hipStream_t alloc_stream = nullptr;   // set: stream-ordered allocations on it
  int64_t dev_bytes = 0;                // device bytes allocated so far
  void* pinned = nullptr;               // pinned block: h_sc, h_rtol, kh_sc
  std::vector<DevLevel> lev;
  double* chol = nullptr;           // coarsest factor
  double* cinv = nullptr;           // coarsest inverse (small coarsest levels), else null
  // fused bottom (k_bottom): levels bottom_lo..L-1 and the coarsest solve in one
  // workgroup; -1 when the cycle has none
  int bottom_lo = -1;
  int64_t bottom_vec = 0, bottom_int = 0;   // its LDS elements: vectors (T), pointers (int)
  dev::BottomLevel<float>* bottom32 = nullptr;
  dev::BottomLevel<double>* bottom64 = nullptr;
  // dense tables (dense.hpp) of the cycle from level dense_lo down: B of levels
  // bottom_lo.. (dense[0]) and, when dense_lo < bottom_lo, R (dense[1]) and
  // [S Q] (dense[2]) of levels dense_lo .. bottom_lo - 1; -1 when the cycle has none
  struct DenseTable {
    void* M = nullptr;              // dense[0]: FP64, the others: V-cycle precision
    int bytes = 0;                  // per value
    dev::DenseSeg one;              // the only segment of a single problem
    dev::DenseSeg* segs = nullptr;  // packed: one per part
    int nseg = 1, max_rows = 0, max_ld = 0;
    int64_t elems = 0;
  };
  int dense_lo = -1;
  bool dense_off = false;           // not wanted (vasmg_set_dense_tables)
  bool no_dense = false;            // left out (a server's allowance: plan_tables)
  int64_t dense_work = 0;           // bound of their transient vectors (0: kDenseWorkBytes)
  DenseTable dense[3];
  dev::DenseMap dense_map[2];       // vertices of bottom_lo and dense_lo in part order
  int64_t n_coarse = 0;
  double upload_ms[3] = {0.0, 0.0, 0.0};   // last upload's layouts, autotune, graph capture
  // PCG state (FP64, padded, fine device numbering)
  int n0 = 0;
  int64_t n0p = 0;                  // n0 * DP
  int* user_map = nullptr;          // fine device row -> mesh vertex
  double *F = nullptr, *X = nullptr, *R = nullptr, *P = nullptr, *Q = nullptr, *Z = nullptr;
  double* partial = nullptr;
  int n_partial = 0;
  Scalars* sc = nullptr;
  Scalars* h_sc = nullptr;          // pinned host copy
  double* h_rtol = nullptr;         // pinned
  int* mail = nullptr;              // pinned: reports of the iteration (one per column or part)
  int* big_mail = nullptr;          // own allocation, more than kMailWords parts
  hipStream_t cap_stream = nullptr;
  hipGraphExec_t gA = nullptr, gB = nullptr;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  // block right-hand sides: K columns interleaved per vertex (K = 0: none)
  int K = 0;
  std::vector<void*> kb, kx, ks, kr;   // per level V-cycle vectors [n][K][DP]
  double *kF = nullptr, *kX = nullptr, *kR = nullptr, *kP = nullptr, *kQ = nullptr;
  double* kpartial = nullptr;
  int kn_partial = 0;                  // partial sums per column
  Scalars* ksc = nullptr;              // [K]
  Scalars* kh_sc = nullptr;            // pinned host copy [K]
  hipGraphExec_t kgA = nullptr, kgB = nullptr;
  GalerkinDevice* gdev = nullptr;     // setup_device = 1, during the upload only
  GalerkinDevice* gdev_bg = nullptr;  // owned: value downloads still running after setup
  // packed problems (vasmg_pack): nseg segments of the fine level, each with its
  // own PCG scalars (0: one problem)
  int nseg = 0;
  std::vector<int64_t> seg_vertex_off;   // [nseg + 1] mesh-vertex offsets of the parts
  std::vector<int64_t> seg_free_off;     // [nseg + 1] fine canonical vertex offsets
  std::vector<std::vector<int64_t>> seg_level_off;   // the same on every level
  int *seg_ptr = nullptr, *seg_rows = nullptr;
  Scalars* ssc = nullptr;                // [nseg]
  hipGraphExec_t sgA = nullptr, sgB = nullptr;
  mutable std::vector<std::vector<int>> order_cache;   // device numbering per level (setup)

  template <class T>
  T* dalloc(int64_t count) {
    void* p = nullptr;
    if (count <= 0) count = 1;
    const size_t bytes = sizeof(T) * static_cast<size_t>(count);
    hipError_t e;
    if (alloc_stream) {
      e = hipMallocAsync(&p, bytes, alloc_stream);
      if (e == hipSuccess) e = hipStreamSynchronize(alloc_stream);
    } else {
      e = hipMalloc(&p, bytes);
    }
    if (e != hipSuccess)
      throw vasmg::Error{VASMG_ENOMEM, "device allocation of " + std::to_string(bytes) +
                                           " bytes failed: " + hipGetErrorString(e)};
    allocs.push_back(p);
    dev_bytes += static_cast<int64_t>(bytes);
    return static_cast<T*>(p);
  }
  // Setup-time copies and clears: on the allocation stream when there is one
  // (a server's handle must not touch the legacy null stream while other
  // handles capture graphs), else the synchronous calls.
  void copy(void* dst, const void* src, size_t bytes, hipMemcpyKind kind) {
    if (alloc_stream) {
      HIP_CHECK(hipMemcpyAsync(dst, src, bytes, kind, alloc_stream));
      HIP_CHECK(hipStreamSynchronize(alloc_stream));
    } else {
      HIP_CHECK(hipMemcpy(dst, src, bytes, kind));
    }
  }
  void clear(void* p, size_t bytes) {
    if (alloc_stream) {
      HIP_CHECK(hipMemsetAsync(p, 0, bytes, alloc_stream));
      HIP_CHECK(hipStreamSynchronize(alloc_stream));
    } else {
      HIP_CHECK(hipMemset(p, 0, bytes));
    }
  }
  template <class T>
  T* upload(const std::vector<T>& v) {
    T* p = dalloc<T>(static_cast<int64_t>(v.size()));
    if (!v.empty()) copy(p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice);
    return p;
  }
  // Waits for the background downloads of the level values into H, if any.
  void settle_host_values() {
    if (!gdev_bg) return;
    GalerkinDevice* g = gdev_bg;
    gdev_bg = nullptr;
    std::unique_ptr<GalerkinDevice, void (*)(GalerkinDevice*)> own(g, galerkin_device_destroy);
    galerkin_device_join(g);
  }
  ~vasmg_ctx() {
    if (gdev_bg) galerkin_device_destroy(gdev_bg);   // joins the downloads writing into H
    if (gA) (void)hipGraphExecDestroy(gA);
    if (gB) (void)hipGraphExecDestroy(gB);
    if (kgA) (void)hipGraphExecDestroy(kgA);
    if (kgB) (void)hipGraphExecDestroy(kgB);
    if (sgA) (void)hipGraphExecDestroy(sgA);
    if (sgB) (void)hipGraphExecDestroy(sgB);
    for (auto& e : ev)
      if (e) (void)hipEventDestroy(e);
    if (cap_stream) (void)hipStreamDestroy(cap_stream);
    for (void* p : allocs) {
      if (alloc_stream)
        (void)hipFreeAsync(p, alloc_stream);
      else
        (void)hipFree(p);
    }
    pinned_pool().put(pinned);
    if (big_mail) (void)hipHostFree(big_mail);
  }
};

namespace {

// -------------------------------------------------------------------------
// upload: colour-major renumbering, device-built level layouts, transfers
// -------------------------------------------------------------------------
void upload_transfers(vasmg_ctx& C, int l, bool need32, bool need64, const std::vector<int>& perm,
                      const std::vector<int>& inv_next) {
  const Level& hl = C.H.levels[l];
  DevLevel& dl = C.lev[l];
  const int n = static_cast<int>(hl.n);
  // transfers P_l (rows: this level's device rows; cols: next level's device rows)
  const ScalarCSR& P = hl.P;
  const int nn = static_cast<int>(P.ncols);
  dl.nnext = nn;
  // the canonical P still on the device after its Galerkin product: renumber and
  // transpose it there (the same arrays as below)
  int64_t gn = 0, gnn = 0, gnnz = 0;
  const int64_t* gptr = nullptr;
  const int32_t* gcol = nullptr;
  const double* gval = nullptr;
  if (C.gdev && !C.alloc_stream &&
      galerkin_device_prolongation(C.gdev, l, &gn, &gnn, &gnnz, &gptr, &gcol, &gval) && gn == n &&
      gnn == nn && gnnz == static_cast<int64_t>(P.col.size())) {
    hipStream_t st = static_cast<hipStream_t>(galerkin_device_stream(C.gdev));
    dl.p_nnz = gnnz;
    dl.p_ptr = C.dalloc<int>(n + 1);
    dl.p_idx = C.dalloc<int>(gnnz);
    dl.pt_ptr = C.dalloc<int>(nn + 1);
    dl.pt_idx = C.dalloc<int>(gnnz);
    if (need64) {
      dl.p_w64 = C.dalloc<double>(gnnz);
      dl.pt_w64 = C.dalloc<double>(gnnz);
    }
    if (need32) {
      dl.p_w32 = C.dalloc<float>(gnnz);
      dl.pt_w32 = C.dalloc<float>(gnnz);
    }
    int* d_inv = nullptr;
    HIP_CHECK(hipMallocAsync(reinterpret_cast<void**>(&d_inv), std::max<size_t>(inv_next.size(), 1) * sizeof(int),
                             st));
    HIP_CHECK(hipMemcpyAsync(d_inv, inv_next.data(), inv_next.size() * sizeof(int), hipMemcpyHostToDevice, st));
    transfers_layout_device(st, n, nn, gnnz, gptr, gcol, gval, dl.perm, d_inv, dl.p_ptr, dl.p_idx,
                            dl.p_w64, dl.p_w32, dl.pt_ptr, dl.pt_idx, dl.pt_w64, dl.pt_w32);
    HIP_CHECK(hipFreeAsync(d_inv, st));
    HIP_CHECK(hipStreamSynchronize(st));
    galerkin_device_release_prolongation(C.gdev, l);
    return;
  }
  std::vector<int> pptr(n + 1, 0), pidx(P.col.size());
  std::vector<double> pw(P.col.size());
  for (int i = 0; i < n; ++i) pptr[i + 1] = pptr[i] + static_cast<int>(P.rowptr[perm[i] + 1] - P.rowptr[perm[i]]);
  for (int i = 0; i < n; ++i) {
    int k = pptr[i];
    for (int64_t p = P.rowptr[perm[i]]; p < P.rowptr[perm[i] + 1]; ++p, ++k) {
      pidx[k] = inv_next[P.col[p]];
      pw[k] = P.val[p];
    }
  }
  std::vector<int> tptr(nn + 1, 0), tidx(pidx.size());
  std::vector<double> tw(pidx.size());
  for (int j : pidx) tptr[j + 1]++;
  for (int j = 0; j < nn; ++j) tptr[j + 1] += tptr[j];
  {
    std::vector<int> fill(tptr.begin(), tptr.end() - 1);
    for (int i = 0; i < n; ++i)
      for (int k = pptr[i]; k < pptr[i + 1]; ++k) {
        const int q = fill[pidx[k]]++;
        tidx[q] = i;
        tw[q] = pw[k];
      }
  }
  dl.p_nnz = static_cast<int64_t>(pidx.size());
  dl.p_ptr = C.upload(pptr);
  dl.p_idx = C.upload(pidx);
  dl.pt_ptr = C.upload(tptr);
  dl.pt_idx = C.upload(tidx);
  if (need64) {
    dl.p_w64 = C.upload(pw);
    dl.pt_w64 = C.upload(tw);
  }
  if (need32) {
    dl.p_w32 = C.upload(std::vector<float>(pw.begin(), pw.end()));
    dl.pt_w32 = C.upload(std::vector<float>(tw.begin(), tw.end()));
  }
}

void upload_level_device(vasmg_ctx& C, int l, bool need32, bool need64, const std::vector<int>& inv,
                         const std::vector<int>& cell_lo, const std::vector<int>& cell_hi,
                         const std::vector<int>& cell_ptr, const std::vector<int>& blk_lo,
                         const std::vector<int>& blk_hi);

// Stable counting sort of perm by key[perm[i]] in [0, range).
void counting_sort_by(std::vector<int>& perm, const std::vector<int32_t>& key, int64_t range) {
  std::vector<int64_t> cnt(static_cast<size_t>(range) + 1, 0);
  for (int i : perm) cnt[key[i] + 1]++;
  for (int64_t k = 0; k < range; ++k) cnt[k + 1] += cnt[k];
  std::vector<int> out(perm.size());
  for (int i : perm) out[cnt[key[i]]++] = i;
  perm.swap(out);
}

// Device numbering of level l: canonical rows sorted by colour, colour block,
// cell (ties keep the canonical order); the identity on the coarsest level.
// Three stable counting sorts (cell, then block, then colour), computed once
// per level and kept.
std::vector<int> device_order(const vasmg_ctx& C, int l) {
  if (static_cast<int>(C.order_cache.size()) > l && !C.order_cache[l].empty())
    return C.order_cache[l];
  const Level& hl = C.H.levels[l];
  std::vector<int> perm(static_cast<size_t>(hl.n));
  std::iota(perm.begin(), perm.end(), 0);
  if (l != C.L && hl.n > 0) {
    counting_sort_by(perm, hl.cell, hl.ncells);
    if (hl.block != hl.cell) counting_sort_by(perm, hl.block, hl.nblocks);
    counting_sort_by(perm, hl.color, std::max<int32_t>(hl.ncolors, 1));
  }
  if (static_cast<int>(C.order_cache.size()) <= l) C.order_cache.resize(l + 1);
  C.order_cache[l] = perm;
  return perm;
}

void upload_level(vasmg_ctx& C, int l, bool need32, bool need64, const std::vector<int>& inv_next) {
  const Level& hl = C.H.levels[l];
  DevLevel& dl = C.lev[l];
  const int d = C.d, dd = d * d, n = static_cast<int>(hl.n);
  dl.n = n;
  dl.d = d;
  const bool coarsest = (l == C.L);
  dl.cells = !coarsest && l > 0;
  // device order: colour, colour block, cell, canonical index (identity on the coarsest)
  const std::vector<int> perm = device_order(C, l);
  std::vector<int> inv(n);
  if (coarsest) {
    dl.ncolors = 1;
    dl.color_ptr = {0, n};
  } else {
    dl.ncolors = hl.ncolors;
  }
  for (int i = 0; i < n; ++i) inv[perm[i]] = i;
  dl.perm = C.upload(perm);
  if (!hl.fixed.empty()) {
    std::vector<uint8_t> fx(n);
    for (int i = 0; i < n; ++i) fx[i] = hl.fixed[perm[i]];
    dl.fixed = C.upload(fx);
  }
  if (coarsest && l > 0) return;   // a coarse coarsest level only needs its factor and vectors

  // cell (and colour block) of each device row (single rows on point levels)
  std::vector<int> cell_lo(n), cell_hi(n), cell_ptr, blk_lo, blk_hi, block_ptr;
  if (dl.cells) {
    dl.blocks = hl.block_steps > 2;
    std::vector<int> ccp(dl.ncolors + 1, 0);
    for (int i = 0; i < n; ++i) {
      const bool new_cell = i == 0 || hl.cell[perm[i]] != hl.cell[perm[i - 1]];
      const bool new_block = i == 0 || hl.block[perm[i]] != hl.block[perm[i - 1]];
      if (new_cell) cell_ptr.push_back(i);
      if (new_block) {
        block_ptr.push_back(static_cast<int>(cell_ptr.size()) - 1);
        ccp[hl.color[perm[i]] + 1]++;
      }
    }
    cell_ptr.push_back(n);
    block_ptr.push_back(static_cast<int>(cell_ptr.size()) - 1);
    for (size_t c = 0; c + 1 < cell_ptr.size(); ++c)
      if (cell_ptr[c + 1] - cell_ptr[c] > (1 << d))
        throw vasmg::Error{VASMG_EINVAL, "internal: Gauss-Seidel cell larger than 2^d vertices"};
    for (size_t k = 0; k + 1 < block_ptr.size(); ++k)
      if (block_ptr[k + 1] - block_ptr[k] > (dl.blocks ? (1 << d) : 1))
        throw vasmg::Error{VASMG_EINVAL, "internal: colour block with too many cells"};
    for (int c = 0; c < dl.ncolors; ++c) ccp[c + 1] += ccp[c];
    dl.color_ptr = ccp;   // cells per colour, or colour blocks per colour
    dl.ncells = static_cast<int>(cell_ptr.size()) - 1;
    dl.nblocks = static_cast<int>(block_ptr.size()) - 1;
    for (int c = 0; c < dl.ncells; ++c)
      for (int i = cell_ptr[c]; i < cell_ptr[c + 1]; ++i) {
        cell_lo[i] = cell_ptr[c];
        cell_hi[i] = cell_ptr[c + 1];
      }
    if (dl.blocks) {
      blk_lo.resize(n);
      blk_hi.resize(n);
      for (int k = 0; k < dl.nblocks; ++k)
        for (int i = cell_ptr[block_ptr[k]]; i < cell_ptr[block_ptr[k + 1]]; ++i) {
          blk_lo[i] = cell_ptr[block_ptr[k]];
          blk_hi[i] = cell_ptr[block_ptr[k + 1]];
        }
    }
  } else {
    if (!coarsest) {
      dl.color_ptr.assign(dl.ncolors + 1, 0);
      for (int i = 0; i < n; ++i) dl.color_ptr[hl.color[i] + 1]++;
      for (int c = 0; c < dl.ncolors; ++c) dl.color_ptr[c + 1] += dl.color_ptr[c];
    }
    for (int i = 0; i < n; ++i) {
      cell_lo[i] = i;
      cell_hi[i] = i + 1;
    }
  }
  upload_level_device(C, l, need32, need64, inv, cell_lo, cell_hi, cell_ptr, blk_lo, blk_hi);
  if (dl.blocks) dl.block_ptr = C.upload(block_ptr);
  if (!coarsest) upload_transfers(C, l, need32, need64, perm, inv_next);
  if (!coarsest && C.opt.smoother == VASMG_SMOOTHER_JACOBI) {
    if (C.gdev) galerkin_device_join(C.gdev);   // the host values of the level
    std::vector<double> dinv;
    block_diag_inverse(hl.A, hl.fixed, dinv);
    const double lam = jacobi_lambda_max(hl.A, dinv, 30);
    if (!(lam > 0.0) || !std::isfinite(lam))
      throw vasmg::Error{VASMG_EDEGENERATE, "Jacobi smoother: no positive eigenvalue estimate"};
    dl.omega = (4.0 / 3.0) / lam;
    std::vector<double> dd_dev(dinv.size());
    for (int i = 0; i < n; ++i)
      std::copy(dinv.begin() + static_cast<int64_t>(perm[i]) * dd,
                dinv.begin() + static_cast<int64_t>(perm[i] + 1) * dd,
                dd_dev.begin() + static_cast<int64_t>(i) * dd);
    if (need64) dl.dinv64 = C.upload(dd_dev);
    if (need32) dl.dinv32 = C.upload(std::vector<float>(dd_dev.begin(), dd_dev.end()));
  }
}

// Lanes per block row from the mean off-cell blocks per row. Point levels: about
// two blocks per lane. 3D cell levels (a cell's lanes share its rows' steps): about
// a quad of 4 blocks per lane and part, 16 or 32 (forward sweep + residual +
// backward sweep of a level at 8 / 16 / 32 / 64 lanes: 218,053 rows of 120 blocks
// 0.86 / 0.83 / 0.78 / 1.01 ms in FP32 and 1.49 / 1.44 / 1.34 / 1.36 in FP64, 19,369 rows
// of 90 blocks 0.34 / 0.27 / 0.24 / 0.41). 2D cell levels (short rows): about two
// quads per lane, 4..64, several cells sharing a wavefront below 16 (137,528 rows of
// 22 blocks, 4 / 8 / 16 lanes: 0.169 / 0.197 / 0.268).
void set_lanes(DevLevel& dl) {
  const double avg = dl.n > 0 ? static_cast<double>(dl.nnz) / dl.n : 1.0;
  auto lanes = [&](double blocks, int lo, int hi) {
    return std::min(hi, std::max(lo, pow2_ceil(static_cast<int>(std::ceil(avg / blocks)))));
  };
  dl.G = !dl.cells ? lanes(2.0, 4, 64) : dl.d == 2 ? lanes(8.0, 4, 64) : lanes(4.0, 16, 32);
  dl.Gspmv = dl.G;
}

// Row pointers of the L or U part from per-row block counts; rows padded to
// whole quads of 4 blocks on cell levels.
std::vector<int> padded_ptr(const std::vector<int>& cnt, bool cells) {
  const int Q = cells ? dev::kQuad : 1;
  std::vector<int> ptr(cnt.size() + 1, 0);
  for (size_t i = 0; i < cnt.size(); ++i) {
    const int64_t next = static_cast<int64_t>(ptr[i]) + (cnt[i] + Q - 1) / Q * Q;
    if (next > INT32_MAX) throw vasmg::Error{VASMG_EINVAL, "level too large for int32 row pointers"};
    ptr[i + 1] = static_cast<int>(next);
  }
  return ptr;
}

int cell_rec_ints(int d) { return d == 2 ? dev::CellRec<2>::ints : dev::CellRec<3>::ints; }

// Device memory that lives for one level's layout: stream-ordered on the upload
// stream when there is one (a server slot's), else plain allocations.
struct TempDev {
  hipStream_t st = nullptr;
  bool ordered = false;
  std::vector<void*> p;
  TempDev(hipStream_t s, bool o) : st(s), ordered(o) {}
  TempDev(const TempDev&) = delete;
  TempDev& operator=(const TempDev&) = delete;
  ~TempDev() {
    for (void* q : p) {
      if (ordered)
        (void)hipFreeAsync(q, st);
      else
        (void)hipFree(q);
    }
  }
  template <class T>
  T* get(size_t n) {
    void* q = nullptr;
    const size_t bytes = std::max<size_t>(n, 1) * sizeof(T);
    const hipError_t e = ordered ? hipMallocAsync(&q, bytes, st) : hipMalloc(&q, bytes);
    if (e != hipSuccess)
      throw vasmg::Error{e == hipErrorOutOfMemory ? VASMG_ENOMEM : VASMG_EDEVICE,
                         "transient device allocation of " + std::to_string(bytes) +
                             " bytes failed: " + hipGetErrorString(e)};
    p.push_back(q);
    return static_cast<T*>(q);
  }
  template <class T>
  T* up(const T* src, size_t n) {
    void* q = nullptr;
    const size_t bytes = std::max<size_t>(n, 1) * sizeof(T);
    HIP_CHECK(ordered ? hipMallocAsync(&q, bytes, st) : hipMalloc(&q, bytes));
    p.push_back(q);
    if (n) HIP_CHECK(hipMemcpyAsync(q, src, n * sizeof(T), hipMemcpyHostToDevice, st));
    return static_cast<T*>(q);
  }
  template <class T, class A>
  T* up(const std::vector<T, A>& v) { return up(v.data(), v.size()); }
};

// Device layout of level l: built by the layout kernels from the level's
// canonical FP64 operator, resident from the device Galerkin products
// (setup_device = 1) or copied in from the host hierarchy for the layout only.
// Only the renumbering, the cell ranges and the row pointers travel besides.
void upload_level_device(vasmg_ctx& C, int l, bool need32, bool need64, const std::vector<int>& inv,
                         const std::vector<int>& cell_lo, const std::vector<int>& cell_hi,
                         const std::vector<int>& cell_ptr, const std::vector<int>& blk_lo,
                         const std::vector<int>& blk_hi) {
  const Level& hl = C.H.levels[l];
  DevLevel& dl = C.lev[l];
  const int d = C.d, dd = d * d, n = dl.n, NU = (1 << d) * d;
  hipStream_t st = C.alloc_stream;
  DevOperator A;
  const bool resident = galerkin_device_operator(C.gdev, l, &A);
  if (!st && resident) st = static_cast<hipStream_t>(galerkin_device_stream(C.gdev));
  TempDev tmp(st, C.alloc_stream != nullptr);
  if (!resident) {
    A.n = hl.n;
    A.ptr = tmp.up(hl.A.rowptr);
    A.col = tmp.up(hl.A.col);
    A.val = tmp.up(hl.A.val);
  }
  LayoutArgs a;
  a.d = d;
  a.n = n;
  a.perm = dl.perm;
  a.inv = tmp.up(inv);
  a.lo = tmp.up(cell_lo);
  a.hi = tmp.up(cell_hi);
  if (dl.cells) {
    std::vector<int> cor(n);
    for (int c = 0; c + 1 < static_cast<int>(cell_ptr.size()); ++c)
      for (int i = cell_ptr[c]; i < cell_ptr[c + 1]; ++i) cor[i] = c;
    a.cell_of_row = tmp.up(cor);
  }
  if (dl.blocks) {
    a.blo = tmp.up(blk_lo);
    a.bhi = tmp.up(blk_hi);
  }
  a.fixed = dl.fixed;
  // parts: L (earlier colours), E / F (earlier / later cells of the row's colour
  // block, colour-block levels only), U (later colours)
  const int nparts = dl.blocks ? kParts : 2;
  const int pidx[kParts] = {kPartL, kPartU, kPartE, kPartF};
  std::vector<int> cnt[kParts];
  int* d_cnt[kParts] = {nullptr, nullptr, nullptr, nullptr};
  for (int q = 0; q < nparts; ++q) {
    cnt[pidx[q]].assign(n, 0);
    d_cnt[pidx[q]] = tmp.up(cnt[pidx[q]]);
    a.part[pidx[q]].cnt = d_cnt[pidx[q]];
  }
  layout_count(A, a, st);
  for (int q = 0; q < nparts; ++q)
    HIP_CHECK(hipMemcpyAsync(cnt[pidx[q]].data(), d_cnt[pidx[q]], n * sizeof(int),
                             hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  for (int i = 0; i < n; ++i) {
    dl.nnz_lo += cnt[kPartL][i];
    dl.nnz_up += cnt[kPartU][i];
    if (dl.blocks) {
      dl.nnz_e += cnt[kPartE][i];
      dl.nnz_f += cnt[kPartF][i];
    }
  }
  dl.nnz = dl.nnz_lo + dl.nnz_up + dl.nnz_e + dl.nnz_f;
  set_lanes(dl);
  // every part plane-major over its own blocks; on cell levels every row is
  // padded to whole quads of 4 blocks (zero blocks pointing at the row itself),
  // so a lane reads 4 consecutive blocks with one 16-byte load per plane
  const std::vector<int> Lptr = padded_ptr(cnt[kPartL], dl.cells), Uptr = padded_ptr(cnt[kPartU], dl.cells);
  const int64_t nL = Lptr[n], nU = Uptr[n];
  dl.Lstride = nL;
  dl.Ustride = nU;
  dl.Lptr = C.upload(Lptr);
  dl.Uptr = C.upload(Uptr);
  dl.Lcol = C.dalloc<int>(std::max<int64_t>(nL, dev::kQuad));   // a first step to read (RowWalk)
  dl.Ucol = C.dalloc<int>(std::max<int64_t>(nU, dev::kQuad));
  int64_t nE = 0, nF = 0;
  if (dl.blocks) {
    const std::vector<int> Eptr = padded_ptr(cnt[kPartE], true), Fptr = padded_ptr(cnt[kPartF], true);
    nE = Eptr[n];
    nF = Fptr[n];
    dl.Estride = nE;
    dl.Fstride = nF;
    dl.Eptr = C.upload(Eptr);
    dl.Fptr = C.upload(Fptr);
    dl.Ecol = C.dalloc<int>(nE);
    dl.Fcol = C.dalloc<int>(nF);
  }
  if (dl.cells) {
    dl.cell_ptr = C.upload(cell_ptr);
    const int64_t words = static_cast<int64_t>(dl.ncells) * cell_rec_ints(d);
    dl.cell_rec = C.dalloc<int>(words);
    const dim3 grid((words + dev::kBlock - 1) / dev::kBlock), blk(dev::kBlock);
    if (d == 2)
      hipLaunchKernelGGL((dev::k_cell_records<2>), grid, blk, 0, st, dl.ncells, dl.cell_ptr, dl.Lptr, dl.Uptr,
                         dl.cell_rec);
    else
      hipLaunchKernelGGL((dev::k_cell_records<3>), grid, blk, 0, st, dl.ncells, dl.cell_ptr, dl.Lptr, dl.Uptr,
                         dl.cell_rec);
  }
  const int64_t m_len = dl.cells ? static_cast<int64_t>(dl.ncells) * NU * NU : static_cast<int64_t>(n) * dd;
  if (need64) {
    dl.Lval64 = C.dalloc<double>(std::max<int64_t>(nL * dd, dev::kQuad));
    dl.Uval64 = C.dalloc<double>(std::max<int64_t>(nU * dd, dev::kQuad));
    if (dl.blocks) {
      dl.Eval64 = C.dalloc<double>(nE * dd);
      dl.Fval64 = C.dalloc<double>(nF * dd);
    }
    (dl.cells ? dl.cellM64 : dl.diag64) = C.dalloc<double>(m_len);
    dl.has64 = true;
  }
  if (need32) {
    dl.Lval32 = C.dalloc<float>(std::max<int64_t>(nL * dd, dev::kQuad));
    dl.Uval32 = C.dalloc<float>(std::max<int64_t>(nU * dd, dev::kQuad));
    if (dl.blocks) {
      dl.Eval32 = C.dalloc<float>(nE * dd);
      dl.Fval32 = C.dalloc<float>(nF * dd);
    }
    (dl.cells ? dl.cellM32 : dl.diag32) = C.dalloc<float>(m_len);
    dl.has32 = true;
  }
  // the first step of an empty part (RowWalk, Flat): a zero block of row 0
  auto clear_first = [&](int64_t nnz, int* col, float* v32, double* v64) {
    if (nnz > 0) return;
    C.clear(col, dev::kQuad * sizeof(int));
    if (v32) C.clear(v32, dev::kQuad * sizeof(float));
    if (v64) C.clear(v64, dev::kQuad * sizeof(double));
  };
  clear_first(nL, dl.Lcol, dl.Lval32, dl.Lval64);
  clear_first(nU, dl.Ucol, dl.Uval32, dl.Uval64);
  a.part[kPartL] = {dl.Lptr, d_cnt[kPartL], nL, dl.Lcol, dl.Lval32, dl.Lval64};
  a.part[kPartU] = {dl.Uptr, d_cnt[kPartU], nU, dl.Ucol, dl.Uval32, dl.Uval64};
  if (dl.blocks) {
    a.part[kPartE] = {dl.Eptr, d_cnt[kPartE], nE, dl.Ecol, dl.Eval32, dl.Eval64};
    a.part[kPartF] = {dl.Fptr, d_cnt[kPartF], nF, dl.Fcol, dl.Fval32, dl.Fval64};
  }
  a.M32 = dl.cells ? dl.cellM32 : dl.diag32;
  a.M64 = dl.cells ? dl.cellM64 : dl.diag64;
  a.m_len = m_len;
  layout_fill(A, a, st);
}

// inverse permutation of level l's device numbering (canonical -> device)
std::vector<int> device_inverse(const vasmg_ctx& C, int l) {
  const std::vector<int> perm = device_order(C, l);
  std::vector<int> inv(perm.size());
  for (size_t i = 0; i < perm.size(); ++i) inv[perm[i]] = static_cast<int>(i);
  return inv;
}

// A^{-1} = L^{-T} L^{-1} from the lower Cholesky factor L (row-major n x n), in
// FP64; symmetric by construction (each pair of entries computed once).
std::vector<double> coarse_inverse(const std::vector<double>& Lf, int64_t n) {
  std::vector<double> Li(static_cast<size_t>(n * n), 0.0);   // L^{-1}, lower
  for (int64_t j = 0; j < n; ++j) {
    Li[j * n + j] = 1.0 / Lf[j * n + j];
    for (int64_t i = j + 1; i < n; ++i) {
      double s = 0.0;
      for (int64_t k = j; k < i; ++k) s += Lf[i * n + k] * Li[k * n + j];
      Li[i * n + j] = -s / Lf[i * n + i];
    }
  }
  std::vector<double> M(static_cast<size_t>(n * n), 0.0);
  for (int64_t i = 0; i < n; ++i)
    for (int64_t j = 0; j <= i; ++j) {
      double s = 0.0;
      for (int64_t k = i; k < n; ++k) s += Li[k * n + i] * Li[k * n + j];
      M[i * n + j] = s;
      M[j * n + i] = s;
    }
  return M;
}

void select_bottom(vasmg_ctx& C);
bool table64(const vasmg_ctx& C, int l);

void upload_all(vasmg_ctx& C) {
  const int nl = static_cast<int>(C.H.levels.size());
  C.L = nl - 1;
  C.lev.assign(nl, DevLevel());
  const bool vasmg = C.opt.preconditioner == VASMG_PRECOND_VASMG;
  const int last = vasmg ? C.L : 0;
  for (int l = 0; l <= last; ++l) {
    const bool fine = (l == 0);
    const bool need64 = fine || !C.vc32;
    const bool need32 = C.vc32 && vasmg;
    std::vector<int> inv_next;
    if (l < C.L) inv_next = device_inverse(C, l + 1);
    upload_level(C, l, need32, need64 || table64(C, l), inv_next);
    if (!need64) C.lev[l].has64 = false;   // the FP64 values serve the construction of B only
  }
  const int T = C.vc32 ? 4 : 8;
  for (int l = 0; l <= last; ++l) {
    DevLevel& dl = C.lev[l];
    const int64_t len = static_cast<int64_t>(C.H.levels[l].n) * C.DP;
    dl.b = C.dalloc<char>(len * T);
    dl.x = C.dalloc<char>(len * T);
    dl.s = C.dalloc<char>(len * T);
    dl.r = C.dalloc<char>(len * T);
    C.clear(dl.b, len * T);
    C.clear(dl.x, len * T);
    C.clear(dl.s, len * T);
    C.clear(dl.r, len * T);
  }
  if (vasmg) {
    C.n_coarse = C.H.n_coarse_dofs;
    if (C.n_coarse > dev::kCoarseMax)
      throw vasmg::Error{VASMG_EINVAL, "coarsest level has more than 4096 DOFs"};
    C.chol = C.upload(C.H.chol);
    if (C.n_coarse <= dev::kCoarseInvMax) C.cinv = C.upload(coarse_inverse(C.H.chol, C.n_coarse));
    if (C.cinv && C.L >= 2 && C.opt.smoother == VASMG_SMOOTHER_GS && C.opt.n_pre >= 1)
      select_bottom(C);
  }
  // PCG vectors
  C.n0 = static_cast<int>(C.H.levels[0].n);
  C.n0p = static_cast<int64_t>(C.n0) * C.DP;
  {
    std::vector<int> um(C.n0);
    std::vector<int> perm0(C.n0);
    C.copy(perm0.data(), C.lev[0].perm, sizeof(int) * C.n0, hipMemcpyDeviceToHost);
    for (int i = 0; i < C.n0; ++i) um[i] = C.H.free_vertices[perm0[i]];
    C.user_map = C.upload(um);
  }
  for (double** v : {&C.F, &C.X, &C.R, &C.P, &C.Q, &C.Z}) {
    *v = C.dalloc<double>(C.n0p);
    C.clear(*v, sizeof(double) * C.n0p);
  }
  // FP64 V-cycle: its fine right-hand side is the PCG residual itself
  if (!C.vc32) C.lev[0].b = C.R;
  // partial sums: the flat reduction grid, or one per workgroup of the fine SpMV
  // (sized for the narrowest workgroup row count any lane width can give)
  C.n_partial = std::max(kFlatGrid, grid_for(C.n0, dev::kBlock / 64));
  C.partial = C.dalloc<double>(C.n_partial);
  C.sc = C.dalloc<Scalars>(1);
  C.clear(C.sc, sizeof(Scalars));
  // pinned: Scalars at 0, rtol at 256, block scalars [16] at 512, reports [kMailWords] at 2048
  static_assert(512 + 16 * sizeof(Scalars) <= 2048 && 2048 + kMailWords * sizeof(int) <= PinnedPool::kBytes,
                "pinned block too small");
  C.pinned = pinned_pool().get();
  C.h_sc = static_cast<Scalars*>(C.pinned);
  C.h_rtol = reinterpret_cast<double*>(static_cast<char*>(C.pinned) + 256);
  C.mail = reinterpret_cast<int*>(static_cast<char*>(C.pinned) + 2048);
  if (C.nseg > kMailWords) {
    HIP_CHECK(hipHostMalloc(reinterpret_cast<void**>(&C.big_mail), sizeof(int) * C.nseg,
                            hipHostMallocCoherent));
    C.mail = C.big_mail;
  }
  for (auto& e : C.ev) HIP_CHECK(hipEventCreate(&e));
  HIP_CHECK(hipStreamCreateWithFlags(&C.cap_stream, hipStreamNonBlocking));
  if (C.nseg > 0) {
    // segment of each fine device row, and each segment's rows (ascending)
    const std::vector<int> perm0 = device_order(C, 0);
    std::vector<int> of(C.n0), cnt(C.nseg + 1, 0);
    for (int i = 0; i < C.n0; ++i) {
      const int64_t v = perm0[i];
      of[i] = static_cast<int>(std::upper_bound(C.seg_free_off.begin(), C.seg_free_off.end(), v) -
                               C.seg_free_off.begin()) - 1;
      cnt[of[i] + 1]++;
    }
    for (int k = 0; k < C.nseg; ++k) cnt[k + 1] += cnt[k];
    std::vector<int> rows(C.n0), fill(cnt.begin(), cnt.end() - 1);
    for (int i = 0; i < C.n0; ++i) rows[fill[of[i]]++] = i;
    C.seg_ptr = C.upload(cnt);
    C.seg_rows = C.upload(rows);
    C.ssc = C.dalloc<Scalars>(C.nseg);
    C.clear(C.ssc, sizeof(Scalars) * C.nseg);
  }
  std::vector<std::vector<int>>().swap(C.order_cache);   // numbering no longer needed
}

// -------------------------------------------------------------------------
// kernel launch helpers
// -------------------------------------------------------------------------
#define DISPATCH_G(Gv, ...)                 \
  switch (Gv) {                             \
    case 4: { constexpr int GG = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int GG = 8; __VA_ARGS__; } break;   \
    case 16: { constexpr int GG = 16; __VA_ARGS__; } break; \
    case 32: { constexpr int GG = 32; __VA_ARGS__; } break; \
    default: { constexpr int GG = 64; __VA_ARGS__; } break; \
  }

template <typename T>
struct LevelMats;
template <>
struct LevelMats<float> {
  static dev::Part<float> L(const DevLevel& l) { return {l.Lptr, l.Lcol, l.Lval32, l.Lstride}; }
  static dev::Part<float> U(const DevLevel& l) { return {l.Uptr, l.Ucol, l.Uval32, l.Ustride}; }
  static dev::Part<float> E(const DevLevel& l) { return {l.Eptr, l.Ecol, l.Eval32, l.Estride}; }
  static dev::Part<float> F(const DevLevel& l) { return {l.Fptr, l.Fcol, l.Fval32, l.Fstride}; }
  static const float* diag(const DevLevel& l) { return l.diag32; }
  static const float* pw(const DevLevel& l) { return l.p_w32; }
  static const float* ptw(const DevLevel& l) { return l.pt_w32; }
  static const float* cellM(const DevLevel& l) { return l.cellM32; }
  static const float* dinv(const DevLevel& l) { return l.dinv32; }
  static bool ok(const DevLevel& l) { return l.has32; }
};
template <>
struct LevelMats<double> {
  static dev::Part<double> L(const DevLevel& l) { return {l.Lptr, l.Lcol, l.Lval64, l.Lstride}; }
  static dev::Part<double> U(const DevLevel& l) { return {l.Uptr, l.Ucol, l.Uval64, l.Ustride}; }
  static dev::Part<double> E(const DevLevel& l) { return {l.Eptr, l.Ecol, l.Eval64, l.Estride}; }
  static dev::Part<double> F(const DevLevel& l) { return {l.Fptr, l.Fcol, l.Fval64, l.Fstride}; }
  static const double* diag(const DevLevel& l) { return l.diag64; }
  static const double* pw(const DevLevel& l) { return l.p_w64; }
  static const double* ptw(const DevLevel& l) { return l.pt_w64; }
  static const double* cellM(const DevLevel& l) { return l.cellM64; }
  static const double* dinv(const DevLevel& l) { return l.dinv64; }
  static bool ok(const DevLevel& l) { return l.has64; }
};

// cells per colour that the fused bottom takes in at most two rounds of its wavefronts
constexpr int kBottomCellsPerColour = 2 * dev::kBottomThreads / 64;

template <typename T>
dev::BottomLevel<T>* upload_bottom(vasmg_ctx& C) {
  std::vector<dev::BottomLevel<T>> v;
  for (int l = C.bottom_lo; l < C.L; ++l) {
    const DevLevel& lv = C.lev[l];
    if (!LevelMats<T>::ok(lv)) return nullptr;
    dev::BottomLevel<T> b;
    b.n = lv.n;
    b.ncolors = lv.ncolors;
    b.ncells = lv.ncells;
    b.nnext = lv.nnext;
    b.color_ptr = lv.color_ptr_dev;
    b.cell_ptr = lv.cell_ptr;
    b.L = LevelMats<T>::L(lv);
    b.U = LevelMats<T>::U(lv);
    b.cellM = LevelMats<T>::cellM(lv);
    b.p_ptr = lv.p_ptr;
    b.p_idx = lv.p_idx;
    b.p_w = LevelMats<T>::pw(lv);
    b.pt_ptr = lv.pt_ptr;
    b.pt_idx = lv.pt_idx;
    b.pt_w = LevelMats<T>::ptw(lv);
    b.fixed = lv.fixed;
    v.push_back(b);
  }
  return C.upload(v);
}

// Chooses the levels of the fused bottom: from L-1 upwards, cell levels whose
// colours hold few cells (each colour a round or two of the workgroup's
// wavefronts) and whose LDS vectors fit together; one level for the W-cycle,
// which visits the levels above L-1 twice.
void select_bottom(vasmg_ctx& C) {
  // the kernel restricts into (and prolongs from) the coarsest level's DOFs in LDS
  if (static_cast<int64_t>(C.lev[C.L - 1].nnext) * C.d != C.n_coarse || C.n_coarse > dev::kCoarseInvMax)
    return;
  const int tb = C.vc32 ? 4 : 8;
  const int maxlev = C.opt.cycle == VASMG_CYCLE_W ? 1 : dev::kBottomLevels;
  auto fits = [&](const DevLevel& lv) {
    if (!lv.cells || lv.blocks) return false;
    for (int c = 0; c < lv.ncolors; ++c)
      if (lv.color_ptr[c + 1] - lv.color_ptr[c] > kBottomCellsPerColour) return false;
    return true;
  };
  int lo = C.L;
  int64_t nvec = 0, nint = 0;
  while (lo - 1 >= 1 && C.L - (lo - 1) <= maxlev) {
    const DevLevel& lv = C.lev[lo - 1];
    const int64_t e = dev::bottom_vec_elems(lv.n, C.DP);
    const int64_t ie = dev::bottom_int_elems(lv.n, lv.ncolors, lv.ncells);
    if (!fits(lv) || (nvec + e) * tb + (nint + ie) * 4 > dev::kBottomLds) break;
    nvec += e;
    nint += ie;
    --lo;
  }
  if (lo == C.L) return;
  C.bottom_lo = lo;
  C.bottom_vec = nvec;
  C.bottom_int = nint;
  for (int l = lo; l < C.L; ++l) C.lev[l].color_ptr_dev = C.upload(C.lev[l].color_ptr);
  C.bottom32 = upload_bottom<float>(C);
  C.bottom64 = upload_bottom<double>(C);
}

// Returns the number of workgroups (= partial sums written when partial != NULL).
template <typename T, int D>
int launch_spmv(const DevLevel& lv, const T* x, T* y, double* partial, int n_partial, hipStream_t st) {
  const int G = lv.Gspmv;
  int used = 0;
  DISPATCH_G(G, {
    const int grid = grid_for(lv.n, dev::kBlock / GG);
    if (partial && grid > n_partial)
      throw vasmg::Error{VASMG_EINVAL, "internal: SpMV partial buffer too small"};
    used = grid;
    if (partial)
      hipLaunchKernelGGL((dev::k_spmv<T, D, GG, true>), dim3(grid), dim3(dev::kBlock), 0, st, lv.n,
                         LevelMats<T>::L(lv), LevelMats<T>::U(lv), LevelMats<T>::diag(lv),
                         x, y, partial);
    else
      hipLaunchKernelGGL((dev::k_spmv<T, D, GG, false>), dim3(grid), dim3(dev::kBlock), 0, st,
                         lv.n, LevelMats<T>::L(lv), LevelMats<T>::U(lv), LevelMats<T>::diag(lv),
                         x, y, partial);
  });
  return used;
}


template <typename T, int D>
void launch_gs_color(const DevLevel& lv, int c, int mode, const T* b, T* x, T* s_save, hipStream_t st) {
  const int r0 = lv.color_ptr[c], nr = lv.color_ptr[c + 1] - r0;
  if (nr <= 0) return;
  DISPATCH_G(lv.G, {
    const int grid = grid_for(nr, dev::kBlock / GG);
    if (mode == 0)
      hipLaunchKernelGGL((dev::k_gs_color<T, D, GG, 0>), dim3(grid), dim3(dev::kBlock), 0, st, r0,
                         nr, LevelMats<T>::L(lv), LevelMats<T>::U(lv), LevelMats<T>::diag(lv), b, x,
                         s_save);
    else if (mode == 1)
      hipLaunchKernelGGL((dev::k_gs_color<T, D, GG, 1>), dim3(grid), dim3(dev::kBlock), 0, st, r0,
                         nr, LevelMats<T>::L(lv), LevelMats<T>::U(lv), LevelMats<T>::diag(lv), b, x,
                         s_save);
    else
      hipLaunchKernelGGL((dev::k_gs_color<T, D, GG, 2>), dim3(grid), dim3(dev::kBlock), 0, st, r0,
                         nr, LevelMats<T>::L(lv), LevelMats<T>::U(lv), LevelMats<T>::diag(lv), b, x,
                         s_save);
  });
}

#define DISPATCH_GR(Gv, ...)                                  \
  switch (Gv) {                                               \
    case 4: { constexpr int GR = 4; __VA_ARGS__; } break;     \
    case 8: { constexpr int GR = 8; __VA_ARGS__; } break;     \
    case 16: { constexpr int GR = 16; __VA_ARGS__; } break;   \
    case 32: { constexpr int GR = 32; __VA_ARGS__; } break;   \
    default: { constexpr int GR = 64; __VA_ARGS__; } break;   \
  }

// One colour of a colour-block level: one workgroup per block (k_gs_block).
// The V-cycle kernels do not read the stop flag (see enqueue_iter_B).
template <typename T, int D>
void launch_gs_blocks(const DevLevel& lv, int c, int mode, const T* b, T* x, T* s_save,
                      hipStream_t st) {
  if constexpr (D == 3) {
    const int k0 = lv.color_ptr[c], nk = lv.color_ptr[c + 1] - k0;
    if (nk <= 0) return;
    const T* M = LevelMats<T>::cellM(lv);
    const dev::Part<T> Lp = LevelMats<T>::L(lv), Up = LevelMats<T>::U(lv);
    const dev::Part<T> Ep = LevelMats<T>::E(lv), Fp = LevelMats<T>::F(lv);
    const dim3 grid(nk), blk(dev::BlockShape<D>::threads);
    if (mode == 0)
      hipLaunchKernelGGL((dev::k_gs_block<T, D, 0>), grid, blk, 0, st, k0, lv.block_ptr,
                         lv.cell_ptr, Lp, Up, Ep, Fp, M, b, x, s_save);
    else if (mode == 1)
      hipLaunchKernelGGL((dev::k_gs_block<T, D, 1>), grid, blk, 0, st, k0, lv.block_ptr,
                         lv.cell_ptr, Lp, Up, Ep, Fp, M, b, x, s_save);
    else
      hipLaunchKernelGGL((dev::k_gs_block<T, D, 2>), grid, blk, 0, st, k0, lv.block_ptr,
                         lv.cell_ptr, Lp, Up, Ep, Fp, M, b, x, static_cast<T*>(nullptr));
  } else {
    throw vasmg::Error{VASMG_EINVAL, "internal: colour blocks are built in 3D only"};
  }
}

template <typename T, int D>
void launch_gs_cells(const DevLevel& lv, int c, int mode, const T* b, T* x, T* s_save, hipStream_t st) {
  if (lv.blocks) {
    launch_gs_blocks<T, D>(lv, c, mode, b, x, s_save, st);
    return;
  }
  const int c0 = lv.color_ptr[c], nc = lv.color_ptr[c + 1] - c0;
  if (nc <= 0) return;
  const T* M = LevelMats<T>::cellM(lv);
  const dev::Part<T> Lp = LevelMats<T>::L(lv), Up = LevelMats<T>::U(lv);
  DISPATCH_GR(lv.G, {
    using Pack = dev::CellPack<D, GR>;
    const dim3 blk(Pack::threads), grid((nc + Pack::CPW - 1) / Pack::CPW);
    if (mode == 0)
      hipLaunchKernelGGL((dev::k_gs_cell<T, D, GR, 0>), grid, blk, 0, st, c0, nc, lv.cell_rec,
                         Lp, Up, M, b, x, s_save);
    else if (mode == 1)
      hipLaunchKernelGGL((dev::k_gs_cell<T, D, GR, 1>), grid, blk, 0, st, c0, nc, lv.cell_rec,
                         Lp, Up, M, b, x, s_save);
    else
      hipLaunchKernelGGL((dev::k_gs_cell<T, D, GR, 2>), grid, blk, 0, st, c0, nc, lv.cell_rec,
                         Lp, Up, M, b, x, s_save);
  });
}

template <typename T, int D, int KIND>
void launch_cell_apply(const DevLevel& lv, const T* base, const T* x, T* out,
                       hipStream_t st) {
  const dev::Part<T> Ep = LevelMats<T>::E(lv), Fp = LevelMats<T>::F(lv);
  DISPATCH_GR(lv.G, {
    using Pack = dev::CellPack<D, GR>;
    const dim3 grid((lv.ncells + Pack::CPW - 1) / Pack::CPW), blk(Pack::threads);
    if (lv.blocks)
      hipLaunchKernelGGL((dev::k_cell_apply<T, D, GR, KIND, true>), grid, blk, 0, st, lv.ncells,
                         lv.cell_rec, LevelMats<T>::L(lv), LevelMats<T>::U(lv), Ep, Fp,
                         LevelMats<T>::cellM(lv), base, x, out);
    else
      hipLaunchKernelGGL((dev::k_cell_apply<T, D, GR, KIND, false>), grid, blk, 0, st, lv.ncells,
                         lv.cell_rec, LevelMats<T>::L(lv), LevelMats<T>::U(lv), Ep, Fp,
                         LevelMats<T>::cellM(lv), base, x, out);
  });
}

template <typename T, int D>
void launch_gs_sweep(const DevLevel& lv, bool backward, bool zero_guess, const T* b, T* x,
                     T* s_save, hipStream_t st) {
  if (lv.cells) {
    if (!backward) {
      for (int c = 0; c < lv.ncolors; ++c)
        launch_gs_cells<T, D>(lv, c, zero_guess ? 0 : 1, b, x, s_save, st);
    } else {
      for (int c = lv.ncolors - 1; c >= 0; --c) launch_gs_cells<T, D>(lv, c, 2, b, x, nullptr, st);
    }
    return;
  }
  if (!backward) {
    for (int c = 0; c < lv.ncolors; ++c)
      launch_gs_color<T, D>(lv, c, zero_guess ? 0 : 1, b, x, s_save, st);
  } else {
    for (int c = lv.ncolors - 1; c >= 0; --c) launch_gs_color<T, D>(lv, c, 2, b, x, nullptr, st);
  }
}

template <typename T, int D>
void launch_residual_upper(const DevLevel& lv, const T* s, const T* x, T* r,
                           hipStream_t st) {
  if (lv.cells) {
    launch_cell_apply<T, D, 0>(lv, s, x, r, st);
    return;
  }
  DISPATCH_G(lv.G, {
    hipLaunchKernelGGL((dev::k_residual_upper<T, D, GG>), dim3(grid_for(lv.n, dev::kBlock / GG)),
                       dim3(dev::kBlock), 0, st, lv.n, LevelMats<T>::U(lv), LevelMats<T>::diag(lv),
                       s, x, r);
  });
}

template <typename T, int D>
void launch_residual_full(const DevLevel& lv, const T* b, const T* x, T* r,
                          hipStream_t st) {
  if (lv.cells) {
    launch_cell_apply<T, D, 1>(lv, b, x, r, st);
    return;
  }
  DISPATCH_G(lv.G, {
    hipLaunchKernelGGL((dev::k_residual_full<T, D, GG>), dim3(grid_for(lv.n, dev::kBlock / GG)),
                       dim3(dev::kBlock), 0, st, lv.n, LevelMats<T>::L(lv), LevelMats<T>::U(lv),
                       LevelMats<T>::diag(lv), b, x, r);
  });
}

// restriction rows (P^T) hold up to ~27 entries, prolongation rows up to 2^d
constexpr int kRestrictLanes = 8, kProlongLanes = 4;

template <typename T, int D>
void launch_jacobi(const DevLevel& lv, bool first, const T* v, T* x,
                   hipStream_t st) {
  const dim3 grid(grid_for(lv.n, dev::kBlock)), blk(dev::kBlock);
  const T om = static_cast<T>(lv.omega);
  if (first)
    hipLaunchKernelGGL((dev::k_jacobi_step<T, D, true>), grid, blk, 0, st, lv.n,
                       LevelMats<T>::dinv(lv), om, v, x);
  else
    hipLaunchKernelGGL((dev::k_jacobi_step<T, D, false>), grid, blk, 0, st, lv.n,
                       LevelMats<T>::dinv(lv), om, v, x);
}

template <typename T, int D>
void launch_restrict(const DevLevel& lv, const T* r, T* bc, hipStream_t st) {
  hipLaunchKernelGGL((dev::k_restrict<T, D, kRestrictLanes>),
                     dim3(grid_for(lv.nnext, dev::kBlock / kRestrictLanes)), dim3(dev::kBlock), 0,
                     st, lv.nnext, lv.pt_ptr, lv.pt_idx, LevelMats<T>::ptw(lv), r, bc);
}

template <typename T, int D>
void launch_prolong(const DevLevel& lv, const T* e, T* x, hipStream_t st) {
  hipLaunchKernelGGL((dev::k_prolong_add<T, D, kProlongLanes>),
                     dim3(grid_for(lv.n, dev::kBlock / kProlongLanes)), dim3(dev::kBlock), 0, st,
                     lv.n, lv.p_ptr, lv.p_idx, LevelMats<T>::pw(lv), e, x, lv.fixed);
}

template <typename T>
void launch_fill(T* a, int64_t n, T v, hipStream_t st) {
  hipLaunchKernelGGL((dev::k_fill<T>), dim3(std::min<int64_t>(kFlatGrid, grid_for(n, dev::kBlock))),
                     dim3(dev::kBlock), 0, st, n, a, v);
}

// -------------------------------------------------------------------------
// Phase profiler: brackets each phase of the schedule with events (outside
// graphs) and accumulates launches, device time and algorithmic HBM bytes.
// -------------------------------------------------------------------------
struct PhaseStat {
  std::string name;
  int level;
  int launches;
  double ms;
  double bytes;
};

struct Profiler {
  hipStream_t st;
  std::vector<PhaseStat> stats;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending;
  std::vector<size_t> pending_idx;
  template <class F>
  void phase(const std::string& name, int level, int launches, double bytes, F&& fn) {
    hipEvent_t a, b;
    HIP_CHECK(hipEventCreate(&a));
    HIP_CHECK(hipEventCreate(&b));
    HIP_CHECK(hipEventRecord(a, st));
    fn();
    HIP_CHECK(hipEventRecord(b, st));
    size_t idx = stats.size();
    for (size_t i = 0; i < stats.size(); ++i)
      if (stats[i].name == name && stats[i].level == level) idx = i;
    if (idx == stats.size()) stats.push_back({name, level, 0, 0.0, 0.0});
    stats[idx].launches += launches;
    stats[idx].bytes += bytes;
    pending.emplace_back(a, b);
    pending_idx.push_back(idx);
  }
  void finish() {
    HIP_CHECK(hipStreamSynchronize(st));
    for (size_t i = 0; i < pending.size(); ++i) {
      float ms = 0.f;
      HIP_CHECK(hipEventElapsedTime(&ms, pending[i].first, pending[i].second));
      stats[pending_idx[i]].ms += ms;
      (void)hipEventDestroy(pending[i].first);
      (void)hipEventDestroy(pending[i].second);
    }
    pending.clear();
    pending_idx.clear();
  }
};

template <class F>
void run_phase(Profiler* prof, const char* name, int level, int launches, double bytes, F&& fn) {
  if (prof)
    prof->phase(name, level, launches, bytes, fn);
  else
    fn();
}

// Algorithmic HBM bytes of the phases of one level (each array read or written
// once per launch; the gathered neighbour vector counted once per launch).
struct LevelBytes {
  double gs_fwd0, gs_fwd, residual, gs_bwd, restrict_, prolong;
};

LevelBytes level_bytes(const vasmg_ctx& C, int l, int tb) {
  const DevLevel& lv = C.lev[l];
  const int D = C.d, DP = C.DP, dd = D * D;
  const double blk = dd * tb + 4.0;                 // values + column index
  const double n = lv.n, vec = n * DP * tb;
  const int NU = (1 << D) * D;
  const double own = lv.cells ? lv.ncells * (NU * NU * static_cast<double>(tb) + 4.0)
                              : n * dd * static_cast<double>(tb);
  const double rows = n * (lv.blocks ? 20.0 : 12.0);  // row pointers of the parts
  const int launches_per_sweep = lv.ncolors;
  (void)launches_per_sweep;
  LevelBytes b{};
  const double all = static_cast<double>(lv.nnz_lo + lv.nnz_up + lv.nnz_e + lv.nnz_f);
  b.gs_fwd0 = (lv.nnz_lo + lv.nnz_e) * blk + rows + own + 4 * vec;   // b, x(w), s(w), x gathers
  b.gs_fwd = all * blk + rows + own + 5 * vec;
  b.residual = (lv.nnz_up + lv.nnz_f) * blk + rows + own + 4 * vec;  // s, x, gathers, r(w)
  b.gs_bwd = all * blk + rows + own + 4 * vec;
  const double nn = lv.nnext;
  b.restrict_ = lv.p_nnz * (4.0 + tb) + (nn + 1) * 4 + vec + nn * DP * tb;
  b.prolong = lv.p_nnz * (4.0 + tb) + (n + 1) * 4 + nn * DP * tb + 2 * vec;
  return b;
}

template <typename T>
struct BottomOf;
template <>
struct BottomOf<float> {
  static const dev::BottomLevel<float>* get(const vasmg_ctx& C) { return C.bottom32; }
};
template <>
struct BottomOf<double> {
  static const dev::BottomLevel<double>* get(const vasmg_ctx& C) { return C.bottom64; }
};

// out = table `which` applied to v1 (and v2): levels as in build_dense.
template <typename T, int D>
void launch_dense(const vasmg_ctx& C, int which, const T* v1, const T* v2, T* out, hipStream_t st) {
  const vasmg_ctx::DenseTable& t = C.dense[which];
  const int* lo = C.dense_map[0].list;
  const int* hi = C.dense_map[1].list;
  const dim3 grid(grid_for(t.max_rows, dev::kDenseWaves), t.nseg), blk(64 * dev::kDenseWaves);
  if (which == 0)
    hipLaunchKernelGGL((dev::k_dense<T, double, D>), grid, blk, t.max_ld * sizeof(double), st, t.one,
                       t.segs, static_cast<const double*>(t.M), v1, lo, v2, lo, out, lo);
  else
    hipLaunchKernelGGL((dev::k_dense<T, T, D>), grid, blk, t.max_ld * sizeof(T), st, t.one, t.segs,
                       static_cast<const T*>(t.M), v1, hi, v2, lo, out, which == 2 ? hi : lo);
}

// One V-cycle: lev[0].b -> lev[0].x (Algorithm 3, recursive, zero initial guess).
// One visit of level l of the multiplicative cycle (Algorithm 3, recursive):
// smoothing from zero (zero_guess) or from the current x, residual, restriction,
// `visits` coarse visits (2 for the W-cycle above the coarsest level),
// prolongation and post-smoothing.
template <typename T, int D>
void enqueue_level(vasmg_ctx& C, int l, bool zero_guess, hipStream_t st,
                   Profiler* prof) {
  const int L = C.L;
  const int tb = sizeof(T);
  if (l == L) {
    run_phase(prof, "coarse_solve", L, 1, static_cast<double>(C.n_coarse) * C.n_coarse * 8.0, [&] {
      if (C.cinv)
        hipLaunchKernelGGL((dev::k_coarse_apply<T, D>), dim3(1), dim3(dev::kBlock), 0, st,
                           static_cast<int>(C.n_coarse), C.cinv, static_cast<const T*>(C.lev[L].b),
                           static_cast<T*>(C.lev[L].x));
      else
        hipLaunchKernelGGL((dev::k_coarse_solve<T, D>), dim3(1), dim3(dev::kBlock), 0, st,
                           static_cast<int>(C.n_coarse), C.chol, static_cast<const T*>(C.lev[L].b),
                           static_cast<T*>(C.lev[L].x));
    });
    return;
  }
  const int npre = C.opt.n_pre, npost = C.opt.n_post;
  DevLevel& lv = C.lev[l];
  T* b = static_cast<T*>(lv.b);
  T* x = static_cast<T*>(lv.x);
  T* s = static_cast<T*>(lv.s);
  T* r = static_cast<T*>(lv.r);
  const LevelBytes by = prof ? level_bytes(C, l, tb) : LevelBytes{};
  if (l == C.dense_lo) {
    const int lo = C.bottom_lo;
    T* bl = static_cast<T*>(C.lev[lo].b);
    T* xl = static_cast<T*>(C.lev[lo].x);
    if (l < lo)
      run_phase(prof, "dense_down", l, 1, C.dense[1].elems * static_cast<double>(C.dense[1].bytes),
                [&] { launch_dense<T, D>(C, 1, b, nullptr, bl, st); });
    run_phase(prof, "bottom", lo, 1, C.dense[0].elems * static_cast<double>(C.dense[0].bytes),
              [&] { launch_dense<T, D>(C, 0, bl, nullptr, xl, st); });
    if (l < lo)
      run_phase(prof, "dense_up", l, 1, C.dense[2].elems * static_cast<double>(C.dense[2].bytes),
                [&] { launch_dense<T, D>(C, 2, b, xl, x, st); });
    return;
  }
  const dev::BottomLevel<T>* bottom = BottomOf<T>::get(C);
  if (l == C.bottom_lo && bottom) {
    dev::BottomArgs<T> a;
    a.nlev = L - l;
    a.ncoarse = static_cast<int>(C.n_coarse);
    a.npre = npre;
    a.npost = npost;
    a.zero_guess = zero_guess ? 1 : 0;
    a.lev = bottom;
    a.Minv = C.cinv;
    a.b = b;
    a.x = x;
    double bytes = static_cast<double>(C.n_coarse) * C.n_coarse * 8.0;
    if (prof)
      for (int k = l; k < L; ++k) {
        const LevelBytes bk = level_bytes(C, k, tb);
        bytes += npre * bk.gs_fwd + bk.residual + bk.restrict_ + bk.prolong + npost * bk.gs_bwd;
      }
    const size_t lds = static_cast<size_t>(C.bottom_vec) * sizeof(T) + C.bottom_int * sizeof(int);
    run_phase(prof, "bottom", l, 1, bytes, [&] {
      hipLaunchKernelGGL((dev::k_bottom<T, D>), dim3(1), dim3(dev::kBottomThreads), lds, st, a);
    });
    return;
  }
  const bool jac = C.opt.smoother == VASMG_SMOOTHER_JACOBI;
  if (jac) {
    // damped block Jacobi: x = w D^-1 b from zero, then x += w D^-1 (b - A x)
    run_phase(prof, "jacobi_pre", l, 2 * npre, npre * by.gs_fwd, [&] {
      for (int k = 0; k < npre; ++k) {
        if (zero_guess && k == 0) {
          launch_jacobi<T, D>(lv, true, b, x, st);
        } else {
          launch_residual_full<T, D>(lv, b, x, r, st);
          launch_jacobi<T, D>(lv, false, r, x, st);
        }
      }
    });
    run_phase(prof, "residual_full", l, 2, by.gs_fwd, [&] {
      if (npre == 0 && zero_guess) launch_fill<T>(x, static_cast<int64_t>(lv.n) * C.DP, T(0), st);
      launch_residual_full<T, D>(lv, b, x, r, st);
    });
  } else if (npre == 0) {
    run_phase(prof, "residual_full", l, 2, by.gs_fwd, [&] {
      if (zero_guess) launch_fill<T>(x, static_cast<int64_t>(lv.n) * C.DP, T(0), st);
      launch_residual_full<T, D>(lv, b, x, r, st);
    });
  } else {
    for (int k = 0; k < npre; ++k) {
      const bool z = zero_guess && k == 0;
      run_phase(prof, z ? "gs_fwd_zero" : "gs_fwd", l, lv.ncolors, z ? by.gs_fwd0 : by.gs_fwd,
                [&] { launch_gs_sweep<T, D>(lv, false, z, b, x, s, st); });
    }
    run_phase(prof, "residual", l, 1, by.residual,
              [&] { launch_residual_upper<T, D>(lv, s, x, r, st); });
  }
  run_phase(prof, "restrict", l, 1, by.restrict_,
            [&] { launch_restrict<T, D>(lv, r, static_cast<T*>(C.lev[l + 1].b), st); });
  const int visits = (C.opt.cycle == VASMG_CYCLE_W && l + 1 < L) ? 2 : 1;
  for (int v = 0; v < visits; ++v) enqueue_level<T, D>(C, l + 1, v == 0, st, prof);
  run_phase(prof, "prolong", l, 1, by.prolong, [&] {
    launch_prolong<T, D>(lv, static_cast<const T*>(C.lev[l + 1].x), x, st);
  });
  for (int k = 0; k < npost; ++k) {
    if (jac)
      run_phase(prof, "jacobi_post", l, 2, by.gs_bwd, [&] {
        launch_residual_full<T, D>(lv, b, x, r, st);
        launch_jacobi<T, D>(lv, false, r, x, st);
      });
    else
      run_phase(prof, "gs_bwd", l, lv.ncolors, by.gs_bwd,
                [&] { launch_gs_sweep<T, D>(lv, true, false, b, x, nullptr, st); });
  }
}

// z = B r with r in lev[0].b, z in lev[0].x (V- or W-cycle, or the additive
// two-level form S r + P_0 B_1 P_0^T r with B_1 the V-cycle of levels 1..L).
template <typename T, int D>
void enqueue_vcycle(vasmg_ctx& C, hipStream_t st, Profiler* prof = nullptr) {
  if (C.opt.cycle != VASMG_CYCLE_ADDITIVE || C.L == 0) {
    enqueue_level<T, D>(C, 0, true, st, prof);
    return;
  }
  const int tb = sizeof(T);
  DevLevel& l0 = C.lev[0];
  T* b = static_cast<T*>(l0.b);
  T* x = static_cast<T*>(l0.x);
  T* s = static_cast<T*>(l0.s);
  const LevelBytes by = prof ? level_bytes(C, 0, tb) : LevelBytes{};
  run_phase(prof, "restrict", 0, 1, by.restrict_,
            [&] { launch_restrict<T, D>(l0, b, static_cast<T*>(C.lev[1].b), st); });
  enqueue_level<T, D>(C, 1, true, st, prof);     // V-cycle below (cycle != W)
  if (C.opt.smoother == VASMG_SMOOTHER_JACOBI) {
    T* r = static_cast<T*>(l0.r);
    const int steps = C.opt.n_pre + C.opt.n_post;
    if (steps == 0) launch_fill<T>(x, static_cast<int64_t>(l0.n) * C.DP, T(0), st);
    for (int k = 0; k < steps; ++k)
      run_phase(prof, "jacobi", 0, k == 0 ? 1 : 2, by.gs_fwd, [&] {
        if (k == 0) {
          launch_jacobi<T, D>(l0, true, b, x, st);
        } else {
          launch_residual_full<T, D>(l0, b, x, r, st);
          launch_jacobi<T, D>(l0, false, r, x, st);
        }
      });
  } else {
    for (int k = 0; k < C.opt.n_pre; ++k)
      run_phase(prof, k == 0 ? "gs_fwd_zero" : "gs_fwd", 0, l0.ncolors,
                k == 0 ? by.gs_fwd0 : by.gs_fwd,
                [&] { launch_gs_sweep<T, D>(l0, false, k == 0, b, x, s, st); });
    if (C.opt.n_pre == 0)
      launch_fill<T>(x, static_cast<int64_t>(l0.n) * C.DP, T(0), st);
    for (int k = 0; k < C.opt.n_post; ++k)
      run_phase(prof, "gs_bwd", 0, l0.ncolors, by.gs_bwd,
                [&] { launch_gs_sweep<T, D>(l0, true, false, b, x, nullptr, st); });
  }
  run_phase(prof, "prolong", 0, 1, by.prolong, [&] {
    launch_prolong<T, D>(l0, static_cast<const T*>(C.lev[1].x), x, st);
  });
}

template <int D>
void enqueue_precond(vasmg_ctx& C, hipStream_t st) {
  if (C.vc32)
    enqueue_vcycle<float, D>(C, st);
  else
    enqueue_vcycle<double, D>(C, st);
}

// -------------------------------------------------------------------------
// PCG graphs
// -------------------------------------------------------------------------
// alpha from the SpMV's np partial sums; x, r updates; ||r||, the stopping test and the
// report.
void enqueue_update(vasmg_ctx& C, int np, hipStream_t st) {
  if (C.n0p <= dev::kSmallFlat) {
    const int n = static_cast<int>(C.n0p);
    if (C.vc32)
      hipLaunchKernelGGL((dev::k_small_xr<float>), dim3(1), dim3(1024), 0, st, n, C.sc, C.partial, np,
                         C.P, C.Q, C.X, C.R, static_cast<float*>(C.lev[0].b), C.mail);
    else
      hipLaunchKernelGGL((dev::k_small_xr<double>), dim3(1), dim3(1024), 0, st, n, C.sc, C.partial, np,
                         C.P, C.Q, C.X, C.R, static_cast<double*>(nullptr), C.mail);
    return;
  }
  hipLaunchKernelGGL((dev::k_finalize<dev::FIN_ALPHA>), dim3(1), dim3(1024), 0, st, C.partial, np,
                     C.sc, static_cast<int*>(nullptr));
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_update_xr<float>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st, C.n0p,
                       C.sc, C.P, C.Q, C.X, C.R, static_cast<float*>(C.lev[0].b), C.partial);
  else
    hipLaunchKernelGGL((dev::k_update_xr<double>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st,
                       C.n0p, C.sc, C.P, C.Q, C.X, C.R, static_cast<double*>(nullptr), C.partial);
  hipLaunchKernelGGL((dev::k_finalize<dev::FIN_RES>), dim3(1), dim3(1024), 0, st, C.partial,
                     kFlatGrid, C.sc, C.mail);
}

template <int D>
void enqueue_iter_A(vasmg_ctx& C, hipStream_t st) {
  const int np = launch_spmv<double, D>(C.lev[0], C.P, C.Q, C.partial, C.n_partial, st);
  enqueue_update(C, np, st);
}

// rho = r.z; beta; p = z + beta p
template <typename T>
void enqueue_direction(vasmg_ctx& C, const T* z, hipStream_t st) {
  if (C.n0p <= dev::kSmallFlat) {
    hipLaunchKernelGGL((dev::k_small_p<T>), dim3(1), dim3(1024), 0, st, static_cast<int>(C.n0p), C.sc, C.R,
                       z, C.P);
    return;
  }
  hipLaunchKernelGGL((dev::k_dot<T>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st, C.n0p, C.R, z,
                     C.partial, static_cast<const int*>(&C.sc->done));
  hipLaunchKernelGGL((dev::k_finalize<dev::FIN_BETA>), dim3(1), dim3(1024), 0, st, C.partial, kFlatGrid,
                     C.sc, static_cast<int*>(nullptr));
  hipLaunchKernelGGL((dev::k_update_p<T>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st, C.n0p, C.sc, z,
                     C.P);
}

// z = B r; rho = r.z; beta; p = z + beta p
template <int D>
void enqueue_iter_B(vasmg_ctx& C, hipStream_t st) {
  const int pc = C.opt.preconditioner;
  if (pc == VASMG_PRECOND_VASMG) {
    // the host launches this graph only while the iteration has not stopped, so
    // the V-cycle kernels do not read the flag (it would head their load chains)
    enqueue_precond<D>(C, st);
    if (C.vc32)
      enqueue_direction(C, static_cast<const float*>(C.lev[0].x), st);
    else
      enqueue_direction(C, static_cast<const double*>(C.lev[0].x), st);
  } else if (pc == VASMG_PRECOND_JACOBI) {
    hipLaunchKernelGGL((dev::k_jacobi<D>), dim3(grid_for(C.n0, dev::kBlock)), dim3(dev::kBlock), 0, st,
                       C.n0, C.lev[0].diag64, C.R, C.Z, static_cast<const int*>(&C.sc->done));
    enqueue_direction(C, static_cast<const double*>(C.Z), st);
  } else {
    enqueue_direction(C, static_cast<const double*>(C.R), st);
  }
}

// -------------------------------------------------------------------------
// Autotuner: lanes per block row of each level, by timing the level's own
// kernels (forward zero-guess sweep + residual + backward sweep, and the fine
// FP64 SpMV) with hipEvents; the fastest median of three wins.
// -------------------------------------------------------------------------
template <typename T, int D>
double time_level(vasmg_ctx& C, int l, hipStream_t st) {
  DevLevel& lv = C.lev[l];
  T* b = static_cast<T*>(lv.b);
  T* x = static_cast<T*>(lv.x);
  T* s = static_cast<T*>(lv.s);
  T* r = static_cast<T*>(lv.r);
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  std::vector<float> t;
  for (int rep = 0; rep < 4; ++rep) {
    HIP_CHECK(hipEventRecord(e0, st));
    launch_gs_sweep<T, D>(lv, false, true, b, x, s, st);
    launch_residual_upper<T, D>(lv, s, x, r, st);
    launch_gs_sweep<T, D>(lv, true, false, b, x, nullptr, st);
    HIP_CHECK(hipEventRecord(e1, st));
    HIP_CHECK(hipEventSynchronize(e1));
    float ms = 0.f;
    HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    if (rep > 0) t.push_back(ms);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  std::sort(t.begin(), t.end());
  return t[t.size() / 2];
}

template <int D>
double time_spmv(vasmg_ctx& C, hipStream_t st) {
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  std::vector<float> t;
  for (int rep = 0; rep < 4; ++rep) {
    HIP_CHECK(hipEventRecord(e0, st));
    launch_spmv<double, D>(C.lev[0], C.P, C.Q, C.partial, C.n_partial, st);
    HIP_CHECK(hipEventRecord(e1, st));
    HIP_CHECK(hipEventSynchronize(e1));
    float ms = 0.f;
    HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    if (rep > 0) t.push_back(ms);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  std::sort(t.begin(), t.end());
  return t[t.size() / 2];
}

template <int D>
void autotune(vasmg_ctx& C) {
  hipStream_t st = C.cap_stream;
  const int last = C.opt.preconditioner == VASMG_PRECOND_VASMG ? C.L - 1 : -1;
  for (int l = 0; l <= last; ++l) {
    DevLevel& lv = C.lev[l];
    if (C.dense_lo > 0 && l >= C.dense_lo) break;   // the solve takes these levels as tables
    const int64_t len = static_cast<int64_t>(lv.n) * C.DP;
    if (C.vc32) {
      launch_fill<float>(static_cast<float*>(lv.b), len, 1.0f, st);
      launch_fill<float>(static_cast<float*>(lv.x), len, 0.0f, st);
    } else {
      launch_fill<double>(static_cast<double*>(lv.b), len, 1.0, st);
      launch_fill<double>(static_cast<double*>(lv.x), len, 0.0, st);
    }
    std::vector<int> cand = lv.cells ? (D == 3 ? std::vector<int>{8, 16, 32, 64}
                                               : std::vector<int>{4, 8, 16, 32})
                                     : std::vector<int>{4, 8, 16, 32};
    double best = 1e30;
    int bestG = lv.G;
    for (int g : cand) {
      lv.G = g;
      const double ms = C.vc32 ? time_level<float, D>(C, l, st) : time_level<double, D>(C, l, st);
      if (ms < best) {
        best = ms;
        bestG = g;
      }
    }
    lv.G = bestG;
    if (C.opt.verbose)
      std::fprintf(stderr, "[vasmg] autotune level %d: %d lanes per row (%.3f ms per V(1,1) pass)\n",
                   l, bestG, best);
  }
  launch_fill<double>(C.P, C.n0p, 1.0, st);
  double best = 1e30;
  int bestG = C.lev[0].Gspmv;
  for (int g : {4, 8, 16, 32}) {
    C.lev[0].Gspmv = g;
    const double ms = time_spmv<D>(C, st);
    if (ms < best) {
      best = ms;
      bestG = g;
    }
  }
  C.lev[0].Gspmv = bestG;
  if (C.opt.verbose)
    std::fprintf(stderr, "[vasmg] autotune fine SpMV: %d lanes per row (%.3f ms)\n", bestG, best);
  HIP_CHECK(hipStreamSynchronize(st));
}

std::mutex g_capture_mutex;   // one graph capture at a time in the process

hipGraphExec_t capture(vasmg_ctx& C, void (*fn)(vasmg_ctx&, hipStream_t)) {
  std::lock_guard<std::mutex> lock(g_capture_mutex);
  hipGraph_t g = nullptr;
  hipGraphExec_t ge = nullptr;
  // relaxed: other threads (a server's slots) may upload, copy or free meanwhile;
  // the captured sequence itself is kernel launches only
  HIP_CHECK(hipStreamBeginCapture(C.cap_stream, hipStreamCaptureModeRelaxed));
  fn(C, C.cap_stream);
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipStreamEndCapture(C.cap_stream, &g));
  HIP_CHECK(hipGraphInstantiate(&ge, g, nullptr, nullptr, 0));
  HIP_CHECK(hipGraphDestroy(g));
  return ge;
}

template <int D>
void ensure_graphs(vasmg_ctx& C) {
  if (!C.gA) C.gA = capture(C, &enqueue_iter_A<D>);
  if (!C.gB) C.gB = capture(C, &enqueue_iter_B<D>);
}

// -------------------------------------------------------------------------
// Reports of the iteration (dev::report): pinned words that the host polls, so the
// next graph is launched as soon as the stopping test is known. The stream's work
// up to here has otherwise no effect that the host reads.
// -------------------------------------------------------------------------
void clear_reports(int* mail, int n) {
  for (int k = 0; k < n; ++k) __atomic_store_n(mail + k, -1, __ATOMIC_RELAXED);
}

// Waits until the n words report iteration `it` or a stop; true if all have
// stopped. Polls for up to 2 ms (giving way to other threads after 50 us), then
// waits for the stream (which also returns a launch's error).
bool wait_reports(const int* mail, int n, int it, hipStream_t st) {
  auto reported = [&](int v) { return v >= 0 && ((v & 1) || v >= 2 * it); };
  const auto start = std::chrono::steady_clock::now();
  bool polling = true, all = true;
  for (int k = 0; k < n; ++k) {
    int v = __atomic_load_n(mail + k, __ATOMIC_RELAXED);
    while (!reported(v) && polling) {
      const auto waited = std::chrono::steady_clock::now() - start;
      if (waited > std::chrono::milliseconds(2)) {
        HIP_CHECK(hipStreamSynchronize(st));
        polling = false;
      } else if (waited > std::chrono::microseconds(50)) {
        std::this_thread::yield();
      } else {
        __builtin_ia32_pause();
      }
      v = __atomic_load_n(mail + k, __ATOMIC_RELAXED);
    }
    all = all && v >= 0 && (v & 1);
  }
  return all;
}

// -------------------------------------------------------------------------
// Packed problems: the shared SpMV and V-cycle, per-segment scalars
// -------------------------------------------------------------------------
// alpha_s; x, r updates; ||r||_s, the stopping test and the report
template <int D>
void enqueue_packed_update(vasmg_ctx& C, hipStream_t st) {
  constexpr int DP = dev::Pad<D>::value;
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_seg_xr<float, DP>), dim3(C.nseg), dim3(dev::kBlock), 0, st, C.seg_ptr,
                       C.seg_rows, C.ssc, C.P, C.Q, C.X, C.R, static_cast<float*>(C.lev[0].b), C.mail);
  else
    hipLaunchKernelGGL((dev::k_seg_xr<double, DP>), dim3(C.nseg), dim3(dev::kBlock), 0, st, C.seg_ptr,
                       C.seg_rows, C.ssc, C.P, C.Q, C.X, C.R, static_cast<double*>(nullptr), C.mail);
}

// rho_s, beta_s; p = z + beta_s p
template <int D>
void enqueue_packed_direction(vasmg_ctx& C, hipStream_t st) {
  constexpr int DP = dev::Pad<D>::value;
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_seg_p<float, DP>), dim3(C.nseg), dim3(dev::kBlock), 0, st, C.seg_ptr,
                       C.seg_rows, C.ssc, C.R, static_cast<const float*>(C.lev[0].x), C.P);
  else
    hipLaunchKernelGGL((dev::k_seg_p<double, DP>), dim3(C.nseg), dim3(dev::kBlock), 0, st, C.seg_ptr,
                       C.seg_rows, C.ssc, C.R, static_cast<const double*>(C.lev[0].x), C.P);
}

// q = A p and the update
template <int D>
void enqueue_packed_A(vasmg_ctx& C, hipStream_t st) {
  launch_spmv<double, D>(C.lev[0], C.P, C.Q, nullptr, 0, st);
  enqueue_packed_update<D>(C, st);
}

// z = B r (the whole packed V-cycle) and the direction
template <int D>
void enqueue_packed_B(vasmg_ctx& C, hipStream_t st) {
  enqueue_precond<D>(C, st);
  enqueue_packed_direction<D>(C, st);
}

template <int D>
void ensure_packed_graphs(vasmg_ctx& C) {
  if (!C.sgA) C.sgA = capture(C, &enqueue_packed_A<D>);
  if (!C.sgB) C.sgB = capture(C, &enqueue_packed_B<D>);
}

// All segments from x0 = 0: d_rhs / d_x the parts' user vectors one after the
// other ([sum n_vertices][D], device); info[nseg].
template <int D>
int solve_packed(vasmg_ctx& C, const double* d_rhs, double* d_x, double rtol, hipStream_t st,
                 vasmg_solve_info* info) {
  constexpr int DP = dev::Pad<D>::value;
  ensure_packed_graphs<D>(C);
  const int n0 = C.n0;
  const int64_t n0p = C.n0p;
  const int nseg = C.nseg;
  HIP_CHECK(hipEventRecord(C.ev[0], st));
  hipLaunchKernelGGL((dev::k_gather_user<double, double, D>), dim3(grid_for(n0, dev::kBlock)),
                     dim3(dev::kBlock), 0, st, n0, C.user_map, d_rhs, C.F,
                     static_cast<const uint8_t*>(C.lev[0].fixed));
  hipLaunchKernelGGL((dev::k_seg_dot<dev::FIN_NORMF, false, DP>), dim3(nseg), dim3(dev::kBlock), 0, st,
                     C.seg_ptr, C.seg_rows, C.F, C.F, C.ssc);
  clear_reports(C.mail, nseg);
  hipLaunchKernelGGL(dev::k_seg_start, dim3(grid_for(nseg, dev::kBlock)), dim3(dev::kBlock), 0, st, nseg,
                     C.ssc, rtol, C.mail);
  launch_fill<double>(C.X, n0p, 0.0, st);
  launch_fill<double>(C.P, n0p, 0.0, st);
  hipLaunchKernelGGL((dev::k_convert<double, double>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st, n0p, C.F,
                     C.R);
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_convert<double, float>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st, n0p,
                       C.R, static_cast<float*>(C.lev[0].b));
  HIP_CHECK(hipGetLastError());
  if (!wait_reports(C.mail, nseg, 0, st)) {
    // Algorithm 2 initialisation for every segment: z = B r, p = z, rho = r^T z
    HIP_CHECK(hipGraphLaunch(C.sgB, st));
    for (int k = 0; k < C.opt.max_iters; ++k) {
      HIP_CHECK(hipGraphLaunch(C.sgA, st));
      if (wait_reports(C.mail, nseg, k + 1, st)) break;
      HIP_CHECK(hipGraphLaunch(C.sgB, st));
    }
  }
  // true residuals, scatter
  launch_spmv<double, D>(C.lev[0], C.X, C.Q, nullptr, 0, st);
  hipLaunchKernelGGL((dev::k_seg_dot<dev::FIN_TRUE, true, DP>), dim3(nseg), dim3(dev::kBlock), 0, st,
                     C.seg_ptr, C.seg_rows, C.F, C.Q, C.ssc);
  launch_fill<double>(d_x, C.H.n_mesh_vertices * D, 0.0, st);
  hipLaunchKernelGGL((dev::k_scatter_user<double, double, D>), dim3(grid_for(n0, dev::kBlock)),
                     dim3(dev::kBlock), 0, st, n0, C.user_map, C.X, d_x);
  std::vector<Scalars> hs(nseg);
  HIP_CHECK(hipMemcpyAsync(hs.data(), C.ssc, sizeof(Scalars) * nseg, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipEventRecord(C.ev[1], st));
  HIP_CHECK(hipStreamSynchronize(st));
  HIP_CHECK(hipGetLastError());
  float ms = 0.f;
  HIP_CHECK(hipEventElapsedTime(&ms, C.ev[0], C.ev[1]));
  int worst = VASMG_OK;
  for (int k = 0; k < nseg; ++k) {
    const Scalars& s = hs[k];
    vasmg_solve_info& o = info[k];
    std::memset(&o, 0, sizeof(o));
    const bool conv = s.status != 5 && (s.normF == 0.0 || s.res / s.normF < rtol);
    o.iterations = s.iters;
    o.converged = conv ? 1 : 0;
    o.rel_res = s.normF > 0 ? s.res / s.normF : 0.0;
    o.rel_res_true = s.normF > 0 ? s.res_true / s.normF : 0.0;
    o.t_solve_ms = ms;
    o.status = s.status == 5 ? VASMG_EBREAKDOWN : (conv ? VASMG_OK : VASMG_ENOTCONV);
    if (o.status == VASMG_EBREAKDOWN)
      worst = VASMG_EBREAKDOWN;
    else if (o.status == VASMG_ENOTCONV && worst == VASMG_OK)
      worst = VASMG_ENOTCONV;
  }
  return worst;
}

// -------------------------------------------------------------------------
// one right-hand side: d_rhs/d_x user layout [nv][D] (device), d_x0 may be NULL
// -------------------------------------------------------------------------
template <int D>
int solve_one(vasmg_ctx& C, const double* d_rhs, const double* d_x0, double* d_x, double rtol,
              hipStream_t st, vasmg_solve_info* info) {
  ensure_graphs<D>(C);
  const int n0 = C.n0;
  const int64_t n0p = C.n0p;
  const int gflat = kFlatGrid;
  HIP_CHECK(hipEventRecord(C.ev[0], st));
  hipLaunchKernelGGL((dev::k_gather_user<double, double, D>), dim3(grid_for(n0, dev::kBlock)),
                     dim3(dev::kBlock), 0, st, n0, C.user_map, d_rhs, C.F,
                     static_cast<const uint8_t*>(C.lev[0].fixed));
  // ||F||, then r = F - A x0 (or F), p = 0
  hipLaunchKernelGGL((dev::k_dot<double>), dim3(gflat), dim3(dev::kBlock), 0, st, n0p, C.F, C.F,
                     C.partial, static_cast<const int*>(nullptr));
  hipLaunchKernelGGL((dev::k_finalize<dev::FIN_NORMF>), dim3(1), dim3(1024), 0, st, C.partial, gflat,
                     C.sc, static_cast<int*>(nullptr));
  *C.h_rtol = rtol;
  HIP_CHECK(hipMemcpyAsync(&C.sc->rtol, C.h_rtol, sizeof(double), hipMemcpyHostToDevice, st));
  if (d_x0) {
    hipLaunchKernelGGL((dev::k_gather_user<double, double, D>), dim3(grid_for(n0, dev::kBlock)),
                       dim3(dev::kBlock), 0, st, n0, C.user_map, d_x0, C.X,
                       static_cast<const uint8_t*>(C.lev[0].fixed));
    launch_spmv<double, D>(C.lev[0], C.X, C.Q, nullptr, 0, st);
    hipLaunchKernelGGL(dev::k_sub_norm, dim3(gflat), dim3(dev::kBlock), 0, st, n0p, C.F, C.Q, C.R,
                       C.partial);
    hipLaunchKernelGGL((dev::k_finalize<dev::FIN_TRUE>), dim3(1), dim3(1024), 0, st, C.partial, gflat,
                       C.sc, static_cast<int*>(nullptr));
  } else {
    launch_fill<double>(C.X, n0p, 0.0, st);
    hipLaunchKernelGGL((dev::k_convert<double, double>), dim3(gflat), dim3(dev::kBlock), 0, st, n0p,
                       C.F, C.R);
  }
  launch_fill<double>(C.P, n0p, 0.0, st);
  if (C.vc32 && C.opt.preconditioner == VASMG_PRECOND_VASMG)
    hipLaunchKernelGGL((dev::k_convert<double, float>), dim3(gflat), dim3(dev::kBlock), 0, st, n0p,
                       C.R, static_cast<float*>(C.lev[0].b));
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipMemcpyAsync(C.h_sc, C.sc, sizeof(Scalars), hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  const double normF = C.h_sc->normF;
  int status = VASMG_OK;
  double t_a = 0.0, t_b = 0.0;
  const bool prof = C.opt.profile != 0;
  bool done = false;
  if (!std::isfinite(normF)) {
    status = VASMG_EBREAKDOWN;
    done = true;
  } else if (normF == 0.0) {
    launch_fill<double>(C.X, n0p, 0.0, st);
    done = true;
  } else if (d_x0 && C.h_sc->res_true / normF < rtol) {
    done = true;
  }
  if (!done) {
    // Algorithm 2 initialisation: z = B r, p = z, rho = r^T z
    if (prof) HIP_CHECK(hipEventRecord(C.ev[2], st));
    HIP_CHECK(hipGraphLaunch(C.gB, st));
    if (prof) HIP_CHECK(hipEventRecord(C.ev[3], st));
    int k = 0;
    clear_reports(C.mail, 1);
    while (k < C.opt.max_iters) {
      if (prof) {
        HIP_CHECK(hipEventSynchronize(C.ev[3]));
        float ms = 0.f;
        HIP_CHECK(hipEventElapsedTime(&ms, C.ev[2], C.ev[3]));
        t_b += ms;
        HIP_CHECK(hipEventRecord(C.ev[2], st));
      }
      HIP_CHECK(hipGraphLaunch(C.gA, st));
      if (prof) HIP_CHECK(hipEventRecord(C.ev[3], st));
      const bool stopped = wait_reports(C.mail, 1, k + 1, st);
      if (prof) {
        HIP_CHECK(hipEventSynchronize(C.ev[3]));
        float ms = 0.f;
        HIP_CHECK(hipEventElapsedTime(&ms, C.ev[2], C.ev[3]));
        t_a += ms;
      }
      ++k;
      if (stopped) break;
      if (prof) HIP_CHECK(hipEventRecord(C.ev[2], st));
      HIP_CHECK(hipGraphLaunch(C.gB, st));
      if (prof) HIP_CHECK(hipEventRecord(C.ev[3], st));
    }
  }
  // true residual, scatter
  launch_spmv<double, D>(C.lev[0], C.X, C.Q, nullptr, 0, st);
  hipLaunchKernelGGL(dev::k_sub_norm, dim3(gflat), dim3(dev::kBlock), 0, st, n0p, C.F, C.Q,
                     static_cast<double*>(nullptr), C.partial);
  hipLaunchKernelGGL((dev::k_finalize<dev::FIN_TRUE>), dim3(1), dim3(1024), 0, st, C.partial, gflat,
                     C.sc, static_cast<int*>(nullptr));
  launch_fill<double>(d_x, C.H.n_mesh_vertices * D, 0.0, st);
  hipLaunchKernelGGL((dev::k_scatter_user<double, double, D>), dim3(grid_for(n0, dev::kBlock)),
                     dim3(dev::kBlock), 0, st, n0, C.user_map, C.X, d_x);
  HIP_CHECK(hipMemcpyAsync(C.h_sc, C.sc, sizeof(Scalars), hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipEventRecord(C.ev[1], st));
  HIP_CHECK(hipStreamSynchronize(st));
  HIP_CHECK(hipGetLastError());
  const Scalars& s = *C.h_sc;
  if (status == VASMG_OK) {
    if (s.status == 5)
      status = VASMG_EBREAKDOWN;
    else if (normF != 0.0 && !(s.res / normF < rtol) && !(d_x0 && s.iters == 0))
      status = VASMG_ENOTCONV;
  }
  if (info) {
    float ms = 0.f;
    HIP_CHECK(hipEventElapsedTime(&ms, C.ev[0], C.ev[1]));
    info->iterations = s.iters;
    info->converged = status == VASMG_OK ? 1 : 0;
    info->status = status;
    info->reserved = 0;
    info->rel_res = normF > 0 ? s.res / normF : 0.0;
    info->rel_res_true = normF > 0 ? s.res_true / normF : 0.0;
    info->t_solve_ms = ms;
    info->t_spmv_ms = t_a;
    info->t_precond_ms = t_b;
    info->t_vector_ms = 0.0;
    info->bytes_model = 0.0;
  }
  return status;
}

// -------------------------------------------------------------------------
// Block right-hand sides: K PCG recurrences that share every matrix read
// (vectors [row][K][DP], per-column scalars; kernels in block.hpp).
// -------------------------------------------------------------------------
#define DISPATCH_K(Kv, ...)                                  \
  switch (Kv) {                                              \
    case 4: { constexpr int KK = 4; __VA_ARGS__; } break;    \
    case 8: { constexpr int KK = 8; __VA_ARGS__; } break;    \
    default: { constexpr int KK = 16; __VA_ARGS__; } break;  \
  }

void upload_block(vasmg_ctx& C, int K) {
  if (K != 4 && K != 8 && K != 16)
    throw vasmg::Error{VASMG_EINVAL, "block_rhs must be 0, 4, 8 or 16"};
  if (C.opt.preconditioner != VASMG_PRECOND_VASMG || C.opt.n_pre < 1)
    throw vasmg::Error{VASMG_EINVAL, "block_rhs needs the V-ASMG preconditioner with n_pre >= 1"};
  if (C.n_coarse * K > dev::kCoarseMax)
    throw vasmg::Error{VASMG_EINVAL, "block_rhs: coarsest level too large for K columns"};
  C.K = K;
  const int tb = C.vc32 ? 4 : 8;
  const int nl = C.L + 1;
  C.kb.assign(nl, nullptr);
  C.kx.assign(nl, nullptr);
  C.ks.assign(nl, nullptr);
  C.kr.assign(nl, nullptr);
  for (int l = 0; l < nl; ++l) {
    // the fine level keeps the padded stride; coarse levels store D components
    const int stride = l == 0 ? C.DP : C.d;
    const int64_t bytes = static_cast<int64_t>(C.lev[l].n) * K * stride * tb;
    for (auto* v : {&C.kb, &C.kx, &C.ks, &C.kr}) {
      (*v)[l] = C.dalloc<char>(bytes);
      C.clear((*v)[l], bytes);
    }
  }
  const int64_t n = C.n0p * K;
  for (double** v : {&C.kF, &C.kX, &C.kR, &C.kP, &C.kQ}) {
    *v = C.dalloc<double>(n);
    C.clear(*v, sizeof(double) * n);
  }
  if (!C.vc32) C.kb[0] = C.kR;    // FP64 V-cycle: its fine right-hand side is r
  // one partial per workgroup of the block SpMV: sized for the wide lane groups
  // (fewest rows per workgroup), whichever the heuristic, the tuner or the
  // block_lanes option puts on the fine level
  C.kn_partial = std::max(kFlatGrid, grid_for(C.n0, dev::kBlock / dev::kPointLanesWide));
  // lanes per block row: on the cell levels the narrow groups (their rows go
  // through LDS in chunks, which keeps a long row's loads in flight with few
  // slots, and more cells fit on a compute unit: 65^3, K = 16, 56.8 ms per
  // block solve against 58.3 with the wide groups on the long-row levels); on
  // the point level the wide groups for long rows
  for (int l = 0; l < C.L; ++l) {
    DevLevel& lv = C.lev[l];
    const double avg = lv.n > 0 ? static_cast<double>(lv.nnz) / lv.n : 0.0;
    // (16 columns: the wide groups where a colour has no more cells than the chip
    // compute units, a workgroup each and its chain of chunks all there is: 23x30x26,
    // narrow / wide, FP32 28.0 / 23.9 ms, FP64 34.7 / 30.6; FP32 in 2D keeps one
    // order of the sums, see CellSums)
    if (lv.cells)
      lv.mcGL = K == 16 && lv.ncells <= 256 * lv.ncolors && (C.d == 3 || !C.vc32) ? dev::kCellLanesWide
                                                                                 : dev::kCellLanesNarrow;
    else
      lv.mcGL = avg >= 24.0 ? dev::kPointLanesWide : dev::kPointLanesNarrow;
    if (C.opt.block_lanes != 0) {   // forced: narrow (1) or wide (2) groups everywhere
      const bool wide = C.opt.block_lanes == 2;
      lv.mcGL = lv.cells ? (wide ? dev::kCellLanesWide : dev::kCellLanesNarrow)
                         : (wide ? dev::kPointLanesWide : dev::kPointLanesNarrow);
    }
  }
  C.kpartial = C.dalloc<double>(static_cast<int64_t>(C.kn_partial) * K);
  C.ksc = C.dalloc<Scalars>(K);
  C.clear(C.ksc, sizeof(Scalars) * K);
  C.kh_sc = reinterpret_cast<Scalars*>(static_cast<char*>(C.pinned) + 512);
}

#define DISPATCH_POINT_GL(GLv, ...)                                         \
  if ((GLv) == dev::kPointLanesWide) {                                      \
    constexpr int GL = dev::kPointLanesWide; __VA_ARGS__;                   \
  } else {                                                                  \
    constexpr int GL = dev::kPointLanesNarrow; __VA_ARGS__;                 \
  }
#define DISPATCH_CELL_GL(GLv, ...)                                          \
  if ((GLv) == dev::kCellLanesWide) {                                       \
    constexpr int GL = dev::kCellLanesWide; __VA_ARGS__;                    \
  } else {                                                                  \
    constexpr int GL = dev::kCellLanesNarrow; __VA_ARGS__;                  \
  }

template <int D, int K>
int launch_spmv_mc(const vasmg_ctx& C, const double* x, double* y, double* partial,
                   hipStream_t st) {
  const DevLevel& lv = C.lev[0];
  int grid = 0;
  DISPATCH_POINT_GL(lv.mcGL, {
    grid = grid_for(lv.n, dev::kBlock / GL);
    if (partial && grid > C.kn_partial)
      throw vasmg::Error{VASMG_EINVAL, "internal: block SpMV partial buffer too small"};
    if (partial)
      hipLaunchKernelGGL((dev::k_spmv_mc<D, K, GL, true>), dim3(grid), dim3(dev::kBlock), 0, st,
                         lv.n, LevelMats<double>::L(lv), LevelMats<double>::U(lv), lv.diag64, x, y,
                         partial);
    else
      hipLaunchKernelGGL((dev::k_spmv_mc<D, K, GL, false>), dim3(grid), dim3(dev::kBlock), 0, st,
                         lv.n, LevelMats<double>::L(lv), LevelMats<double>::U(lv), lv.diag64, x, y,
                         partial);
  });
  return grid;
}

// GLv: lanes per block row; nbatch batches of K columns (cell levels only).
template <typename T, int D, int K>
void launch_gs_sweep_mc(const DevLevel& lv, int GLv, int nbatch, bool backward, bool zero_guess,
                        const T* b, T* x, T* s, hipStream_t st) {
  const int64_t batch = static_cast<int64_t>(lv.n) * K * D;
  const dev::Part<T> Lp = LevelMats<T>::L(lv), Up = LevelMats<T>::U(lv);
  for (int q = 0; q < lv.ncolors; ++q) {
    const int c = backward ? lv.ncolors - 1 - q : q;
    const int mode = backward ? 2 : (zero_guess ? 0 : 1);
    const int r0 = lv.color_ptr[c], nr = lv.color_ptr[c + 1] - r0;
    if (nr <= 0) continue;
    if (lv.cells) {
      const T* M = LevelMats<T>::cellM(lv);
      DISPATCH_CELL_GL(GLv, {
        const dim3 grid(nr, nbatch), blk((1 << D) * GL);
        if (mode == 0)
          hipLaunchKernelGGL((dev::k_gs_cell_mc<T, D, K, GL, 0>), grid, blk, 0, st, r0, lv.cell_ptr,
                             Lp, Up, M, b, x, s, batch);
        else if (mode == 1)
          hipLaunchKernelGGL((dev::k_gs_cell_mc<T, D, K, GL, 1>), grid, blk, 0, st, r0, lv.cell_ptr,
                             Lp, Up, M, b, x, s, batch);
        else
          hipLaunchKernelGGL((dev::k_gs_cell_mc<T, D, K, GL, 2>), grid, blk, 0, st, r0, lv.cell_ptr,
                             Lp, Up, M, b, x, static_cast<T*>(nullptr), batch);
      });
    } else {
      const T* dg = LevelMats<T>::diag(lv);
      DISPATCH_POINT_GL(GLv, {
        const dim3 grid(grid_for(nr, dev::kBlock / GL)), blk(dev::kBlock);
        if (mode == 0)
          hipLaunchKernelGGL((dev::k_gs_color_mc<T, D, K, GL, 0>), grid, blk, 0, st, r0, nr, Lp,
                             Up, dg, b, x, s);
        else if (mode == 1)
          hipLaunchKernelGGL((dev::k_gs_color_mc<T, D, K, GL, 1>), grid, blk, 0, st, r0, nr, Lp,
                             Up, dg, b, x, s);
        else
          hipLaunchKernelGGL((dev::k_gs_color_mc<T, D, K, GL, 2>), grid, blk, 0, st, r0, nr, Lp,
                             Up, dg, b, x, static_cast<T*>(nullptr));
      });
    }
  }
}

// r = b - A x of a level from the forward sweep's saved lower sums s
template <typename T, int D, int K>
void launch_residual_mc(const DevLevel& lv, int GLv, int nbatch, const T* s, const T* x, T* r,
                        hipStream_t st) {
  if (lv.cells) {
    DISPATCH_CELL_GL(GLv, {
      hipLaunchKernelGGL((dev::k_cell_residual_mc<T, D, K, GL>), dim3(lv.ncells, nbatch),
                         dim3((1 << D) * GL), 0, st, lv.cell_ptr, LevelMats<T>::L(lv),
                         LevelMats<T>::U(lv), LevelMats<T>::cellM(lv), s, x, r,
                         static_cast<int64_t>(lv.n) * K * D);
    });
  } else {
    DISPATCH_POINT_GL(GLv, {
      hipLaunchKernelGGL((dev::k_residual_upper_mc<T, D, K, GL>), dim3(grid_for(lv.n, dev::kBlock / GL)),
                         dim3(dev::kBlock), 0, st, lv.n, LevelMats<T>::U(lv), LevelMats<T>::diag(lv), s, x,
                         r);
    });
  }
}

// out = table `which` applied to the K columns of v1 (and v2).
template <typename T, int D, int K>
void launch_dense_mc(const vasmg_ctx& C, int which, const void* v1, const void* v2, void* out,
                     hipStream_t st) {
  const vasmg_ctx::DenseTable& t = C.dense[which];
  const dim3 grid(grid_for(t.max_rows, 16)), blk(64 * dev::kDenseMcWaves);
  const T *a = static_cast<const T*>(v1), *b = static_cast<const T*>(v2);
  if (which == 0)
    hipLaunchKernelGGL((dev::k_dense_mc<T, double, D, K>), grid, blk, 0, st, t.one,
                       static_cast<const double*>(t.M), a, b, static_cast<T*>(out));
  else
    hipLaunchKernelGGL((dev::k_dense_mc<T, T, D, K>), grid, blk, 0, st, t.one,
                       static_cast<const T*>(t.M), a, b, static_cast<T*>(out));
}

template <typename T, int D, int K>
void enqueue_vcycle_mc(vasmg_ctx& C, hipStream_t st) {
  const int L = C.L, top = C.dense_lo > 0 ? C.dense_lo : C.L;   // levels smoothed one by one
  for (int l = 0; l < top; ++l) {
    const DevLevel& lv = C.lev[l];
    T* b = static_cast<T*>(C.kb[l]);
    T* x = static_cast<T*>(C.kx[l]);
    T* s = static_cast<T*>(C.ks[l]);
    T* r = static_cast<T*>(C.kr[l]);
    for (int k = 0; k < C.opt.n_pre; ++k)
      launch_gs_sweep_mc<T, D, K>(lv, lv.mcGL, 1, false, k == 0, b, x, s, st);
    launch_residual_mc<T, D, K>(lv, lv.mcGL, 1, s, x, r, st);
    const dim3 rgrid(grid_for(lv.nnext, dev::kBlock / dev::RestrictMc<T, D, K>::lanes));
    if (l == 0)
      hipLaunchKernelGGL((dev::k_restrict_mc<T, D, K, dev::Pad<D>::value>), rgrid, dim3(dev::kBlock),
                         0, st, lv.nnext, lv.pt_ptr, lv.pt_idx, LevelMats<T>::ptw(lv), r,
                         static_cast<T*>(C.kb[l + 1]), int64_t(0));
    else
      hipLaunchKernelGGL((dev::k_restrict_mc<T, D, K, D>), rgrid, dim3(dev::kBlock), 0, st,
                         lv.nnext, lv.pt_ptr, lv.pt_idx, LevelMats<T>::ptw(lv), r,
                         static_cast<T*>(C.kb[l + 1]), int64_t(0));
  }
  const int nco = static_cast<int>(C.n_coarse), lo = C.bottom_lo;
  const T* bL = static_cast<const T*>(C.kb[L]);
  T* xL = static_cast<T*>(C.kx[L]);
  if (top < L) {
    if (top < lo) launch_dense_mc<T, D, K>(C, 1, C.kb[top], nullptr, C.kb[lo], st);
    launch_dense_mc<T, D, K>(C, 0, C.kb[lo], nullptr, C.kx[lo], st);
    if (top < lo) launch_dense_mc<T, D, K>(C, 2, C.kb[top], C.kx[lo], C.kx[top], st);
  } else if (L == 0 && C.cinv)
    hipLaunchKernelGGL((dev::k_coarse_apply_mc<T, D, K, dev::Pad<D>::value>), dim3(1),
                       dim3(dev::kBlock), 0, st, nco, C.cinv, bL, xL);
  else if (L == 0)
    hipLaunchKernelGGL((dev::k_coarse_solve_mc<T, D, K, dev::Pad<D>::value>), dim3(1),
                       dim3(dev::kBlock), 0, st, nco, C.chol, bL, xL);
  else if (C.cinv)
    hipLaunchKernelGGL((dev::k_coarse_apply_mc<T, D, K, D>), dim3(1), dim3(dev::kBlock), 0, st, nco,
                       C.cinv, bL, xL);
  else
    hipLaunchKernelGGL((dev::k_coarse_solve_mc<T, D, K, D>), dim3(1), dim3(dev::kBlock), 0, st, nco,
                       C.chol, bL, xL);
  for (int l = top - 1; l >= 0; --l) {
    const DevLevel& lv = C.lev[l];
    T* b = static_cast<T*>(C.kb[l]);
    T* x = static_cast<T*>(C.kx[l]);
    const dim3 pgrid(grid_for(lv.n, dev::kBlock / K));
    if (l == 0)
      hipLaunchKernelGGL((dev::k_prolong_mc<T, D, K, dev::Pad<D>::value>), pgrid, dim3(dev::kBlock),
                         0, st, lv.n, lv.p_ptr, lv.p_idx, LevelMats<T>::pw(lv),
                         static_cast<const T*>(C.kx[l + 1]), x, static_cast<const uint8_t*>(lv.fixed),
                         int64_t(0));
    else
      hipLaunchKernelGGL((dev::k_prolong_mc<T, D, K, D>), pgrid, dim3(dev::kBlock), 0, st, lv.n,
                         lv.p_ptr, lv.p_idx, LevelMats<T>::pw(lv),
                         static_cast<const T*>(C.kx[l + 1]), x, static_cast<const uint8_t*>(lv.fixed),
                         int64_t(0));
    for (int k = 0; k < C.opt.n_post; ++k)
      launch_gs_sweep_mc<T, D, K>(lv, lv.mcGL, 1, true, false, b, x, nullptr, st);
  }
}

// q = A p, alpha, x += alpha p, r -= alpha q, ||r|| and the stop flags (per column)
template <int D, int K>
void enqueue_iter_A_mc(vasmg_ctx& C, hipStream_t st) {
  constexpr int DP = dev::Pad<D>::value;
  const int64_t n = C.n0p * K;
  const int np = launch_spmv_mc<D, K>(C, C.kP, C.kQ, C.kpartial, st);
  hipLaunchKernelGGL((dev::k_finalize_mc<dev::FIN_ALPHA, K>), dim3(K), dim3(dev::kBlock), 0, st,
                     C.kpartial, np, C.ksc, static_cast<int*>(nullptr));
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_update_xr_mc<float, K, DP>), dim3(kFlatGrid), dim3(dev::kBlock), 0,
                       st, n, C.ksc, C.kP, C.kQ, C.kX, C.kR, static_cast<float*>(C.kb[0]),
                       C.kpartial);
  else
    hipLaunchKernelGGL((dev::k_update_xr_mc<double, K, DP>), dim3(kFlatGrid), dim3(dev::kBlock), 0,
                       st, n, C.ksc, C.kP, C.kQ, C.kX, C.kR, static_cast<double*>(nullptr),
                       C.kpartial);
  hipLaunchKernelGGL((dev::k_finalize_mc<dev::FIN_RES, K>), dim3(K), dim3(dev::kBlock), 0, st,
                     C.kpartial, kFlatGrid, C.ksc, C.mail);
}

// z = B r, rho = r.z, beta, p = z + beta p (per column)
template <int D, int K>
void enqueue_iter_B_mc(vasmg_ctx& C, hipStream_t st) {
  constexpr int DP = dev::Pad<D>::value;
  const int64_t n = C.n0p * K;
  if (C.vc32) {
    enqueue_vcycle_mc<float, D, K>(C, st);
    hipLaunchKernelGGL((dev::k_dot_mc<K, DP, float>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st, n,
                       C.kR, static_cast<const float*>(C.kx[0]), C.kpartial);
  } else {
    enqueue_vcycle_mc<double, D, K>(C, st);
    hipLaunchKernelGGL((dev::k_dot_mc<K, DP, double>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st,
                       n, C.kR, static_cast<const double*>(C.kx[0]), C.kpartial);
  }
  hipLaunchKernelGGL((dev::k_finalize_mc<dev::FIN_BETA, K>), dim3(K), dim3(dev::kBlock), 0, st,
                     C.kpartial, kFlatGrid, C.ksc, static_cast<int*>(nullptr));
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_update_p_mc<float, K, DP>), dim3(kFlatGrid), dim3(dev::kBlock), 0, st,
                       n, C.ksc, static_cast<const float*>(C.kx[0]), C.kP);
  else
    hipLaunchKernelGGL((dev::k_update_p_mc<double, K, DP>), dim3(kFlatGrid), dim3(dev::kBlock), 0,
                       st, n, C.ksc, static_cast<const double*>(C.kx[0]), C.kP);
}

// Columns c0 .. c0+nc-1 (nc <= K) of the user arrays [n_rhs][nv][D]; the
// unused columns of the block are zero and stop at once.
template <int D, int K>
void ensure_block_graphs(vasmg_ctx& C) {
  if (!C.kgA) C.kgA = capture(C, &enqueue_iter_A_mc<D, K>);
  if (!C.kgB) C.kgB = capture(C, &enqueue_iter_B_mc<D, K>);
}

template <int D, int K>
int solve_block(vasmg_ctx& C, const double* d_rhs, const double* d_x0, double* d_x, int c0, int nc,
                double rtol, hipStream_t st, vasmg_solve_info* info) {
  constexpr int DP = dev::Pad<D>::value;
  ensure_block_graphs<D, K>(C);
  const int n0 = C.n0;
  const int64_t n = C.n0p * K;
  const int64_t nv = C.H.n_mesh_vertices;
  const int gflat = kFlatGrid;
  const dim3 gk(grid_for(static_cast<int64_t>(n0) * K, dev::kBlock));
  HIP_CHECK(hipEventRecord(C.ev[0], st));
  hipLaunchKernelGGL((dev::k_gather_user_mc<D, K>), gk, dim3(dev::kBlock), 0, st, n0, C.user_map,
                     d_rhs, nv, c0, nc, C.kF, static_cast<const uint8_t*>(C.lev[0].fixed));
  hipLaunchKernelGGL((dev::k_dot_mc<K, DP, double>), dim3(gflat), dim3(dev::kBlock), 0, st, n, C.kF,
                     C.kF, C.kpartial);
  hipLaunchKernelGGL((dev::k_finalize_mc<dev::FIN_NORMF, K>), dim3(K), dim3(dev::kBlock), 0, st,
                     C.kpartial, gflat, C.ksc, static_cast<int*>(nullptr));
  if (d_x0) {
    hipLaunchKernelGGL((dev::k_gather_user_mc<D, K>), gk, dim3(dev::kBlock), 0, st, n0, C.user_map,
                       d_x0, nv, c0, nc, C.kX, static_cast<const uint8_t*>(C.lev[0].fixed));
    hipLaunchKernelGGL((dev::k_zero_cols_mc<K, DP>), dim3(gflat), dim3(dev::kBlock), 0, st, n, C.ksc,
                       C.kX);
    launch_spmv_mc<D, K>(C, C.kX, C.kQ, nullptr, st);
    hipLaunchKernelGGL((dev::k_sub_norm_mc<K, DP>), dim3(gflat), dim3(dev::kBlock), 0, st, n, C.kF,
                       C.kQ, C.kR, C.kpartial);
    hipLaunchKernelGGL((dev::k_finalize_mc<dev::FIN_TRUE, K>), dim3(K), dim3(dev::kBlock), 0, st,
                       C.kpartial, gflat, C.ksc, static_cast<int*>(nullptr));
  } else {
    launch_fill<double>(C.kX, n, 0.0, st);
    hipLaunchKernelGGL((dev::k_convert<double, double>), dim3(gflat), dim3(dev::kBlock), 0, st, n,
                       C.kF, C.kR);
  }
  hipLaunchKernelGGL((dev::k_start_mc<K>), dim3(1), dim3(64), 0, st, C.ksc, rtol, d_x0 ? 1 : 0);
  launch_fill<double>(C.kP, n, 0.0, st);
  if (C.vc32)
    hipLaunchKernelGGL((dev::k_convert<double, float>), dim3(gflat), dim3(dev::kBlock), 0, st, n,
                       C.kR, static_cast<float*>(C.kb[0]));
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipMemcpyAsync(C.kh_sc, C.ksc, sizeof(Scalars) * K, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  std::vector<double> normF(K);
  bool all_done = true;
  for (int k = 0; k < K; ++k) {
    normF[k] = C.kh_sc[k].normF;
    all_done = all_done && C.kh_sc[k].done;
  }
  if (!all_done) {
    HIP_CHECK(hipGraphLaunch(C.kgB, st));
    clear_reports(C.mail, K);
    for (int it = 0; it < C.opt.max_iters; ++it) {
      HIP_CHECK(hipGraphLaunch(C.kgA, st));
      if (wait_reports(C.mail, K, it + 1, st)) break;
      HIP_CHECK(hipGraphLaunch(C.kgB, st));
    }
  }
  // true residuals, scatter
  launch_spmv_mc<D, K>(C, C.kX, C.kQ, nullptr, st);
  hipLaunchKernelGGL((dev::k_sub_norm_mc<K, DP>), dim3(gflat), dim3(dev::kBlock), 0, st, n, C.kF,
                     C.kQ, static_cast<double*>(nullptr), C.kpartial);
  hipLaunchKernelGGL((dev::k_finalize_mc<dev::FIN_TRUE, K>), dim3(K), dim3(dev::kBlock), 0, st,
                     C.kpartial, gflat, C.ksc, static_cast<int*>(nullptr));
  launch_fill<double>(d_x + static_cast<int64_t>(c0) * nv * D, static_cast<int64_t>(nc) * nv * D, 0.0,
                      st);                                       // fixed DOFs
  hipLaunchKernelGGL((dev::k_scatter_user_mc<D, K>), gk, dim3(dev::kBlock), 0, st, n0, C.user_map,
                     C.kX, nv, c0, nc, d_x);
  HIP_CHECK(hipMemcpyAsync(C.kh_sc, C.ksc, sizeof(Scalars) * K, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipEventRecord(C.ev[1], st));
  HIP_CHECK(hipStreamSynchronize(st));
  HIP_CHECK(hipGetLastError());
  float ms = 0.f;
  HIP_CHECK(hipEventElapsedTime(&ms, C.ev[0], C.ev[1]));
  int worst = VASMG_OK;
  for (int k = 0; k < nc; ++k) {
    const Scalars& sk = C.kh_sc[k];
    int status = VASMG_OK;
    if (!std::isfinite(normF[k]) || sk.status == 5)
      status = VASMG_EBREAKDOWN;
    else if (normF[k] != 0.0 && !(sk.res / normF[k] < rtol) && !(d_x0 && sk.iters == 0))
      status = VASMG_ENOTCONV;
    if (status != VASMG_OK && worst == VASMG_OK) worst = status;
    if (info) {
      vasmg_solve_info& f = info[k];
      f.iterations = sk.iters;
      f.converged = status == VASMG_OK ? 1 : 0;
      f.rel_res = normF[k] > 0 ? sk.res / normF[k] : 0.0;
      f.rel_res_true = normF[k] > 0 ? sk.res_true / normF[k] : 0.0;
      f.t_solve_ms = ms;
      f.t_spmv_ms = f.t_precond_ms = f.t_vector_ms = f.bytes_model = 0.0;
      f.status = status;
      f.reserved = 0;
    }
  }
  return worst;
}

// -------------------------------------------------------------------------
// Dense tables of the small levels (dense.hpp)
// -------------------------------------------------------------------------
// Largest part (DOFs) a table is built for, and largest tables together. A
// level of 2,187 DOFs costs 115 us per visit as colour launches and 6 us as
// tables, which take about 1.3 ms to build: paid back by one solve of a dozen
// iterations. The next level up in 3D has eight times the DOFs, 64 times the
// table: its products would cost what its launches do.
constexpr int64_t kDenseMaxDofs = 2304;
constexpr int64_t kDenseMaxBytes = int64_t(256) << 20;
// Transient vectors of one chunk of columns, and the least worth building with. Building
// takes (ms; bound 384 / 96 / 32 / 16 MiB) 2.8 / 4.1 / 7.2 / 13 for the 1,980 DOFs
// under a 9^3 mesh in FP64, 2.5 / 2.1 / 4.7 / 5.9 in FP32, 5.5 / 8 / 18 / 33 for a
// pack of eight 3D parts.
constexpr int64_t kDenseWorkBytes = int64_t(96) << 20;
constexpr int64_t kDenseLeastWork = int64_t(16) << 20;
// FP32 cycles in 2D take tables only up to this stiffness contrast of the mesh.
// Another rounding of the preconditioner moves the solution of PCG little where it
// converges in 10 to 20 products, and by 1e-9 and more where it takes 15 to 50 (200
// 2D problems of up to 60,000 vertices each, FP32 tables against the level launches,
// largest relative change: contrast 1 1.4e-12, 4 9e-13, 10 3.4e-11, 30 1.3e-9, 100
// 1.2e-8; 1,700 3D problems, contrast 100, 9.5e-10).
constexpr double kDenseMaxContrast2d = 10.0;

bool dense_wanted(const vasmg_ctx& C) {
  return !C.dense_off && !C.no_dense && C.opt.cycle != VASMG_CYCLE_W &&
         !(C.vc32 && C.d == 2 && C.H.contrast > kDenseMaxContrast2d);
}

// Vertex offsets of the parts on level l.
std::vector<int64_t> part_offsets(const vasmg_ctx& C, int l) {
  if (C.nseg > 0) return C.seg_level_off[l];
  return {0, C.H.levels[l].n};
}

// Bytes of the tables that start at level ld over a bottom of vertex offsets `lo`
// (padding included); -1 if a part is too large.
int64_t dense_table_bytes(const vasmg_ctx& C, const std::vector<int64_t>& hi,
                          const std::vector<int64_t>& lo, bool split) {
  const int64_t tb = C.vc32 ? 4 : 8;
  auto row = [](int64_t n, int64_t bytes) { return (n * bytes + 15) / 16 * 16; };
  int64_t b = 0;
  for (size_t p = 0; p + 1 < hi.size(); ++p) {
    const int64_t n = (hi[p + 1] - hi[p]) * C.d, m = (lo[p + 1] - lo[p]) * C.d;
    if (n > kDenseMaxDofs || m > kDenseMaxDofs) return -1;
    b += m * row(m, 8) + (split ? m * row(n, tb) + n * (row(n, tb) + row(m, tb)) : 0);
  }
  return b;
}

// Whether the handle's cycle and size admit tables at all.
bool dense_possible(const vasmg_ctx& C) {
  return dense_wanted(C) && C.opt.preconditioner == VASMG_PRECOND_VASMG &&
         C.opt.smoother == VASMG_SMOOTHER_GS && C.opt.n_pre >= 1 && C.H.levels.size() >= 3 &&
         C.H.n_coarse_dofs <= dev::kCoarseInvMax;
}

// FP32 cycle: whether level l may lie in the fused bottom, whose table is built from
// FP64 values (select_bottom's limits, before the levels are laid out).
bool table64(const vasmg_ctx& C, int l) {
  const int L = static_cast<int>(C.H.levels.size()) - 1;
  return C.vc32 && dense_possible(C) && l >= 1 && l < L && L - l <= dev::kBottomLevels &&
         dev::bottom_vec_elems(static_cast<int>(C.H.levels[l].n), C.DP) * 4 <= dev::kBottomLds;
}

// Vectors of one column batch of levels l0 .. l1 (the last one: b and x only).
int64_t dense_batch_bytes(const vasmg_ctx& C, int l0, int l1, int64_t value) {
  int64_t b = 0;
  for (int l = l0; l <= l1; ++l)
    b += C.H.levels[l].n * dev::kDenseCols * C.d * value * (l == l1 ? 2 : 4);
  return b;
}

// Column batches per chunk, within the transient vectors' bound.
int dense_chunk(const vasmg_ctx& C, int64_t cols, int64_t batch_bytes) {
  const int64_t work = C.dense_work > 0 ? C.dense_work : kDenseWorkBytes;
  return static_cast<int>(std::min<int64_t>((cols + dev::kDenseCols - 1) / dev::kDenseCols,
                                            std::max<int64_t>(1, work / batch_bytes)));
}

// Upper bound of the tables' bytes before the levels are on the device (any
// bottom level at or below the tables' first level), and of the construction's
// transient vectors; 0 when the cycle takes none.
int64_t dense_bytes_bound(const vasmg_ctx& C, int64_t* work) {
  *work = 0;
  if (!dense_possible(C)) return 0;
  const int L = static_cast<int>(C.H.levels.size()) - 1;
  for (int l = 1; l < L; ++l) {
    const std::vector<int64_t> off = part_offsets(C, l), next = part_offsets(C, std::min(l + 1, L - 1));
    const int64_t one = dense_table_bytes(C, off, off, false), split = dense_table_bytes(C, off, next, true);
    if (one < 0 || split < 0) continue;
    int64_t part = 0;
    for (size_t p = 0; p + 1 < off.size(); ++p) part = std::max(part, (off[p + 1] - off[p]) * C.d);
    auto chunk = [&](int l0, int64_t cols, int64_t value) {
      const int64_t batch = dense_batch_bytes(C, l0, L, value);
      return dense_chunk(C, cols, batch) * batch;
    };
    int bottom = l;   // FP32 cycle: the FP64 vectors cover the fused bottom only
    while (C.vc32 && bottom < L - 1 && !table64(C, bottom)) ++bottom;
    *work = std::max(chunk(l, 2 * part, C.vc32 ? 4 : 8), chunk(bottom, part, 8));
    const int64_t rows = C.H.levels[l].n * 12;   // part order, packed only
    return std::min(std::max(one, split), kDenseMaxBytes) + (C.nseg > 0 ? 2 * rows + 1024 * C.nseg : 0);
  }
  return 0;
}

// The cycle on column batches: b of level l0 -> down to level l1's b (levels
// l0 .. l1 - 1), then from level l1's x up to level l0's x. Vectors per level
// in w (b, x, s, r).
struct DenseWork {
  void* v[4] = {nullptr, nullptr, nullptr, nullptr};
};

template <typename T, int D>
void dense_down(vasmg_ctx& C, std::vector<DenseWork>& w, int l0, int l1, int nb, hipStream_t st) {
  constexpr int K = dev::kDenseCols;
  for (int l = l0; l < l1; ++l) {
    const DevLevel& lv = C.lev[l];
    T *b = static_cast<T*>(w[l].v[0]), *x = static_cast<T*>(w[l].v[1]);
    T *s = static_cast<T*>(w[l].v[2]), *r = static_cast<T*>(w[l].v[3]);
    for (int k = 0; k < C.opt.n_pre; ++k)
      launch_gs_sweep_mc<T, D, K>(lv, dev::kCellLanesNarrow, nb, false, k == 0, b, x, s, st);
    launch_residual_mc<T, D, K>(lv, dev::kCellLanesNarrow, nb, s, x, r, st);
    hipLaunchKernelGGL((dev::k_restrict_mc<T, D, K, D>), dim3(grid_for(lv.nnext, dev::kBlock / dev::RestrictMc<T, D, K>::lanes), nb),
                       dim3(dev::kBlock), 0, st, lv.nnext, lv.pt_ptr, lv.pt_idx, LevelMats<T>::ptw(lv), r,
                       static_cast<T*>(w[l + 1].v[0]), static_cast<int64_t>(lv.n) * K * D);
  }
}

template <typename T, int D>
void dense_up(vasmg_ctx& C, std::vector<DenseWork>& w, int l0, int l1, int nb, hipStream_t st) {
  constexpr int K = dev::kDenseCols;
  for (int l = l1 - 1; l >= l0; --l) {
    const DevLevel& lv = C.lev[l];
    T *b = static_cast<T*>(w[l].v[0]), *x = static_cast<T*>(w[l].v[1]);
    hipLaunchKernelGGL((dev::k_prolong_mc<T, D, K, D>), dim3(grid_for(lv.n, dev::kBlock / K), nb),
                       dim3(dev::kBlock), 0, st, lv.n, lv.p_ptr, lv.p_idx, LevelMats<T>::pw(lv),
                       static_cast<const T*>(w[l + 1].v[1]), x, static_cast<const uint8_t*>(lv.fixed),
                       static_cast<int64_t>(lv.nnext) * K * D);
    for (int k = 0; k < C.opt.n_post; ++k)
      launch_gs_sweep_mc<T, D, K>(lv, dev::kCellLanesNarrow, nb, true, false, b, x,
                                  static_cast<T*>(nullptr), st);
  }
}

// A chunk's vectors of levels l0 .. l1 in the slab.
template <typename T, int D>
std::vector<DenseWork> dense_vectors(const vasmg_ctx& C, int l0, int l1, int nb, char* slab, hipStream_t st) {
  std::vector<DenseWork> w(C.L + 1);
  T* p = reinterpret_cast<T*>(slab);
  for (int l = l0; l <= l1; ++l) {
    const int64_t len = static_cast<int64_t>(C.lev[l].n) * dev::kDenseCols * D * nb;
    for (int q = 0; q < (l == l1 ? 2 : 4); ++q) {
      w[l].v[q] = p;
      p += len;
    }
    // the zero padding blocks of a row multiply the row's own entry of x before
    // the first sweep has written it
    launch_fill<T>(static_cast<T*>(w[l].v[1]), len, T(0), st);
  }
  return w;
}

// Unit vectors c0 - shift, ... in vector v of level l (q: its part order).
template <typename T, int D>
void dense_unit(const vasmg_ctx& C, const std::vector<DenseWork>& w, int l, int q, int v, int nb, int col0,
                int shift, hipStream_t st) {
  const int64_t e = static_cast<int64_t>(C.lev[l].n) * dev::kDenseCols * D;
  hipLaunchKernelGGL((dev::k_dense_unit<T, D>), dim3(grid_for(e, dev::kBlock), nb), dim3(dev::kBlock), 0, st,
                     C.lev[l].n, C.dense_map[q].loc, col0, shift, static_cast<T*>(w[l].v[v]));
}

template <typename T, int D>
void dense_extract(const vasmg_ctx& C, const std::vector<DenseWork>& w, int which, int l, int q, int v, int nb,
                   int col0, int shift, int second, hipStream_t st) {
  const int64_t e = static_cast<int64_t>(C.lev[l].n) * dev::kDenseCols * D;
  const vasmg_ctx::DenseTable& t = C.dense[which];
  hipLaunchKernelGGL((dev::k_dense_extract<T, D>), dim3(grid_for(e, dev::kBlock), nb), dim3(dev::kBlock), 0, st,
                     C.lev[l].n, C.dense_map[q], t.one, t.segs, col0, shift, second,
                     static_cast<const T*>(w[l].v[v]), static_cast<T*>(t.M));
}

template <typename T, int D>
void build_dense(vasmg_ctx& C, hipStream_t st) {
  constexpr int K = dev::kDenseCols;
  const int lo = C.bottom_lo, L = C.L;
  const std::vector<int64_t> off_lo = part_offsets(C, lo);
  auto fits = [&](int64_t bytes) { return bytes >= 0 && bytes <= kDenseMaxBytes; };
  if (!fits(dense_table_bytes(C, off_lo, off_lo, false))) return;
  int ld = lo;
  while (ld - 1 >= 1 && C.lev[ld - 1].cells && !C.lev[ld - 1].blocks &&
         fits(dense_table_bytes(C, part_offsets(C, ld - 1), off_lo, true)))
    --ld;
  const std::vector<int64_t> off_hi = part_offsets(C, ld);
  const int np = static_cast<int>(off_lo.size()) - 1;
  // part order of the two levels' vertices (canonical order is part by part)
  if (C.nseg > 0) {
    for (int q = 0; q < 2; ++q) {
      const int l = q == 0 ? lo : ld;
      const std::vector<int64_t>& off = q == 0 ? off_lo : off_hi;
      const int n = C.lev[l].n;
      std::vector<int> perm(n), list(n), loc(n), seg(n);
      C.copy(perm.data(), C.lev[l].perm, sizeof(int) * n, hipMemcpyDeviceToHost);
      for (int i = 0; i < n; ++i) {
        const int p = static_cast<int>(std::upper_bound(off.begin(), off.end(), perm[i]) - off.begin()) - 1;
        list[perm[i]] = i;
        loc[i] = static_cast<int>(perm[i] - off[p]);
        seg[i] = p;
      }
      C.dense_map[q].list = C.upload(list);
      C.dense_map[q].loc = C.upload(loc);
      C.dense_map[q].seg = C.upload(seg);
    }
  }
  auto table = [&](int which, int bytes, const std::vector<int64_t>& ro, const std::vector<int64_t>& ao,
                   const std::vector<int64_t>* co) {
    vasmg_ctx::DenseTable& t = C.dense[which];
    std::vector<dev::DenseSeg> segs(np);
    auto pad = [&](int n) { return (n * bytes + 15) / 16 * 16 / bytes; };
    int64_t m = 0;
    for (int p = 0; p < np; ++p) {
      dev::DenseSeg& g = segs[p];
      g.m0 = m;
      g.r0 = static_cast<int>(ro[p]);
      g.nr = static_cast<int>(ro[p + 1] - ro[p]);
      g.a0 = static_cast<int>(ao[p]);
      g.na = static_cast<int>(ao[p + 1] - ao[p]);
      g.c0 = co ? static_cast<int>((*co)[p]) : 0;
      g.nc = co ? static_cast<int>((*co)[p + 1] - (*co)[p]) : 0;
      g.ld = pad(g.na * D) + pad(g.nc * D);
      m += static_cast<int64_t>(g.nr) * D * g.ld;
      t.max_rows = std::max(t.max_rows, g.nr * D);
      t.max_ld = std::max(t.max_ld, g.ld);
    }
    t.one = segs[0];
    t.nseg = np;
    t.elems = m;
    t.bytes = bytes;
    if (C.nseg > 0) t.segs = C.upload(segs);
    t.M = C.dalloc<char>(m * bytes);
    if (bytes == 8)   // the row padding
      launch_fill<double>(static_cast<double*>(t.M), m, 0.0, st);
    else
      launch_fill<float>(static_cast<float*>(t.M), m, 0.0f, st);
  };
  table(0, 8, off_lo, off_lo, nullptr);
  if (ld < lo) {
    table(1, sizeof(T), off_lo, off_hi, nullptr);
    table(2, sizeof(T), off_hi, off_hi, &off_lo);
  }
  auto max_part = [&](const std::vector<int64_t>& off) {
    int64_t m = 0;
    for (int p = 0; p < np; ++p) m = std::max(m, off[p + 1] - off[p]);
    return static_cast<int>(m) * D;
  };
  const int n_lo = max_part(off_lo), n_hi = max_part(off_hi), n_up = ld < lo ? n_hi + n_lo : 0;
  const int64_t batch_lo = dense_batch_bytes(C, lo, L, 8), batch_up = dense_batch_bytes(C, ld, lo, sizeof(T));
  const int nb_lo = dense_chunk(C, n_lo, batch_lo), nb_up = n_up ? dense_chunk(C, n_up, batch_up) : 0;
  TempDev tmp(st, C.alloc_stream != nullptr);
  // one slab: freeing the vectors one by one takes longer
  char* slab = tmp.get<char>(std::max(batch_lo * nb_lo, batch_up * nb_up));
  {
    std::vector<DenseWork> w = dense_vectors<double, D>(C, lo, L, nb_lo, slab, st);
    for (int c0 = 0; c0 < n_lo; c0 += nb_lo * K) {   // B: the cycle from level lo on unit vectors
      const int nb = std::min(nb_lo, (n_lo - c0 + K - 1) / K);
      dense_unit<double, D>(C, w, lo, 0, 0, nb, c0, 0, st);
      dense_down<double, D>(C, w, lo, L, nb, st);
      hipLaunchKernelGGL((dev::k_coarse_apply_mc<double, D, K, D>), dim3(1, nb), dim3(dev::kBlock), 0, st,
                         static_cast<int>(C.n_coarse), C.cinv, static_cast<const double*>(w[L].v[0]),
                         static_cast<double*>(w[L].v[1]));
      dense_up<double, D>(C, w, lo, L, nb, st);
      dense_extract<double, D>(C, w, 0, lo, 0, 1, nb, c0, 0, 0, st);
    }
  }
  if (ld < lo) {
    // R and S: unit vectors in b_ld with x_lo = 0; Q: unit vectors in x_lo with b_ld = 0
    std::vector<DenseWork> w = dense_vectors<T, D>(C, ld, lo, nb_up, slab, st);
    for (int c0 = 0; c0 < n_up; c0 += nb_up * K) {
      const int nb = std::min(nb_up, (n_up - c0 + K - 1) / K);
      dense_unit<T, D>(C, w, ld, 1, 0, nb, c0, 0, st);
      dense_down<T, D>(C, w, ld, lo, nb, st);
      dense_extract<T, D>(C, w, 1, lo, 0, 0, nb, c0, 0, 0, st);
      dense_unit<T, D>(C, w, lo, 0, 1, nb, c0, n_hi, st);
      dense_up<T, D>(C, w, ld, lo, nb, st);
      dense_extract<T, D>(C, w, 2, ld, 1, 1, nb, c0, 0, 0, st);
      dense_extract<T, D>(C, w, 2, ld, 1, 1, nb, c0, n_hi, 1, st);
    }
  }
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipStreamSynchronize(st));
  C.dense_lo = ld;
}

// Tables where the cycle has a fused bottom to extend (Gauss-Seidel V-cycle or
// the additive form, whose coarse part is one; the W-cycle revisits its levels
// from a nonzero iterate and keeps k_bottom). Without memory for them the
// handle goes on without.
void make_dense(vasmg_ctx& C) {
  if (C.bottom_lo < 0 || !dense_wanted(C)) return;
  hipStream_t st = C.alloc_stream;
  if (!st && C.gdev) {   // the level layouts are still being written on the setup's stream
    st = static_cast<hipStream_t>(galerkin_device_stream(C.gdev));
    HIP_CHECK(hipStreamSynchronize(nullptr));
  }
  const size_t kept = C.allocs.size();
  const int64_t bytes = C.dev_bytes;
  try {
    if (C.d == 2)
      C.vc32 ? build_dense<float, 2>(C, st) : build_dense<double, 2>(C, st);
    else
      C.vc32 ? build_dense<float, 3>(C, st) : build_dense<double, 3>(C, st);
  } catch (const vasmg::Error& e) {
    if (e.status != VASMG_ENOMEM) throw;
    (void)hipGetLastError();
    for (; C.allocs.size() > kept; C.allocs.pop_back()) {
      if (C.alloc_stream)
        (void)hipFreeAsync(C.allocs.back(), C.alloc_stream);
      else
        (void)hipFree(C.allocs.back());
    }
    C.dev_bytes = bytes;
    for (auto& t : C.dense) t = {};
    for (auto& m : C.dense_map) m = {};
  }
}

bool device_available();

// Device upload of a host-built hierarchy (+ block vectors, autotuning).
// alloc_stream != NULL: allocations are stream-ordered on it.
// Block right-hand sides: lanes per block row of each level (narrow or wide
// groups) by timing the level's own block kernels (forward zero-guess sweep,
// residual, backward sweep; on the fine level also the block SpMV, which shares
// the setting); the fastest median of three wins.
template <typename T, int D, int K>
double time_level_mc(vasmg_ctx& C, int l, hipStream_t st) {
  DevLevel& lv = C.lev[l];
  T* b = static_cast<T*>(C.kb[l]);
  T* x = static_cast<T*>(C.kx[l]);
  T* s = static_cast<T*>(C.ks[l]);
  T* r = static_cast<T*>(C.kr[l]);
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  std::vector<float> t;
  for (int rep = 0; rep < 4; ++rep) {
    HIP_CHECK(hipEventRecord(e0, st));
    launch_gs_sweep_mc<T, D, K>(lv, lv.mcGL, 1, false, true, b, x, s, st);
    launch_residual_mc<T, D, K>(lv, lv.mcGL, 1, s, x, r, st);
    launch_gs_sweep_mc<T, D, K>(lv, lv.mcGL, 1, true, false, b, x, s, st);
    if (l == 0) launch_spmv_mc<D, K>(C, C.kP, C.kQ, nullptr, st);
    HIP_CHECK(hipEventRecord(e1, st));
    HIP_CHECK(hipEventSynchronize(e1));
    float ms = 0.f;
    HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    if (rep > 0) t.push_back(ms);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  std::sort(t.begin(), t.end());
  return t[t.size() / 2];
}

template <int D, int K>
void autotune_block(vasmg_ctx& C) {
  hipStream_t st = C.cap_stream;
  for (int l = 0; l < (C.dense_lo > 0 ? C.dense_lo : C.L); ++l) {
    DevLevel& lv = C.lev[l];
    const bool fine64 = l == 0 && !C.vc32;
    int best_gl = lv.mcGL;
    double best = 1e30;
    const int opts[2] = {lv.cells ? dev::kCellLanesNarrow : dev::kPointLanesNarrow,
                         lv.cells ? dev::kCellLanesWide : dev::kPointLanesWide};
    for (int gl : opts) {
      lv.mcGL = gl;
      const double ms = (C.vc32 && !fine64) ? time_level_mc<float, D, K>(C, l, st)
                                            : time_level_mc<double, D, K>(C, l, st);
      if (ms < best) {
        best = ms;
        best_gl = gl;
      }
    }
    lv.mcGL = best_gl;
    if (C.opt.verbose)
      std::fprintf(stderr, "[vasmg] autotune block level %d: %d lanes per row (%.3f ms)\n", l, best_gl,
                   best);
  }
  HIP_CHECK(hipStreamSynchronize(st));
}

void upload_device(vasmg_ctx& C, hipStream_t alloc_stream) {
  if (!device_available()) throw vasmg::Error{VASMG_EDEVICE, "no HIP device available"};
  HIP_CHECK(hipGetDevice(&C.device));
  C.alloc_stream = alloc_stream;
  using Clock = std::chrono::steady_clock;
  auto ms_since = [](Clock::time_point t) {
    return std::chrono::duration<double, std::milli>(Clock::now() - t).count();
  };
  auto t = Clock::now();
  upload_all(C);
  if (C.opt.block_rhs != 0) upload_block(C, C.opt.block_rhs);
  make_dense(C);
  C.upload_ms[0] = ms_since(t);
  t = Clock::now();
  if (C.opt.autotune) {
    if (C.d == 2)
      autotune<2>(C);
    else
      autotune<3>(C);
    if (C.K > 0 && C.opt.block_lanes == 0) {
      if (C.d == 2) {
        DISPATCH_K(C.K, { autotune_block<2, KK>(C); });
      } else {
        DISPATCH_K(C.K, { autotune_block<3, KK>(C); });
      }
    }
  }
  C.upload_ms[1] = ms_since(t);
  t = Clock::now();
  // The PCG graphs are captured here, after the lanes per row are final, and not
  // at the first solve: a solve then instantiates and allocates nothing.
  auto graphs = [&](auto dtag) {
    constexpr int D = decltype(dtag)::value;
    if (C.nseg > 0) {
      ensure_packed_graphs<D>(C);
      return;
    }
    ensure_graphs<D>(C);
    if (C.K > 0) DISPATCH_K(C.K, { ensure_block_graphs<D, KK>(C); });
  };
  if (C.d == 2)
    graphs(std::integral_constant<int, 2>());
  else
    graphs(std::integral_constant<int, 3>());
  C.upload_ms[2] = ms_since(t);
  C.host_only = false;
}

// Upper bound of the device bytes upload_device will allocate, from the host
// hierarchy (every stored block counted as off-diagonal, the transient copy of
// the largest level's canonical operator included, 5% + 1 MiB margin).
int64_t estimate_device_bytes(const vasmg_ctx& C, bool tables = true) {
  const Hierarchy& H = C.H;
  const int d = C.d, dd = d * d, DP = C.DP, NU = (1 << d) * d;
  const bool vasmg = C.opt.preconditioner == VASMG_PRECOND_VASMG;
  const int L = static_cast<int>(H.levels.size()) - 1;
  const int last = vasmg ? L : 0;
  const int64_t tbv = C.vc32 ? 4 : 8;
  const int64_t K = C.opt.block_rhs;
  int64_t b = 0;
  for (int l = 0; l <= last; ++l) {
    const Level& lv = H.levels[l];
    const int64_t n = lv.n, nb = lv.A.nnzb();
    const bool need64 = l == 0 || !C.vc32 || (tables && table64(C, l)), need32 = C.vc32 && vasmg;
    const int64_t vb = (need64 ? 8 : 0) + (need32 ? 4 : 0);
    b += n * 4 + 2 * (n + 1) * 4 + nb * (4 + dd * vb);
    if (l > 0 && l < L)
      b += lv.ncells * (NU * NU * vb + 4 + 4 * cell_rec_ints(d)) + 4 * (lv.ncolors + 2);
    else
      b += n * dd * vb;
    if (l < L) {
      const int64_t pn = static_cast<int64_t>(lv.P.col.size());
      b += (n + 1) * 4 + (H.levels[l + 1].n + 1) * 4 + 2 * pn * (4 + vb);
    }
    b += 4 * n * DP * tbv * (1 + K);
  }
  // the largest level's canonical operator, copied in for its layout only, and the
  // layout's per-row arrays
  int64_t transient = 0;
  for (int l = 0; l <= last; ++l) {
    const Level& lv = H.levels[l];
    transient = std::max(transient, lv.A.nnzb() * (4 + dd * 8) + (lv.n + 1) * 8 + 6 * lv.n * 4);
  }
  if (tables) {
    int64_t dense_work = 0;
    b += dense_bytes_bound(C, &dense_work);
    transient = std::max(transient, dense_work);
  }
  b += transient;
  const int64_t n0p = H.levels[0].n * DP;
  b += 6 * n0p * 8 + H.levels[0].n * 4 + H.n_coarse_dofs * H.n_coarse_dofs * 16;   // factor + inverse
  b += (std::max<int64_t>(kFlatGrid, H.levels[0].n / 4 + 1)) * 8 * (1 + K);
  b += 5 * n0p * 8 * K;
  if (C.nseg > 0) b += H.levels[0].n * 12 + static_cast<int64_t>(C.nseg + 1) * (4 + sizeof(Scalars));
  return b + b / 20 + (1 << 20);
}

vasmg_status fail_with(const vasmg::Error& e) {
  g_last_error = e.msg;
  return static_cast<vasmg_status>(e.status);
}

bool device_available() {
  int n = 0;
  return hipGetDeviceCount(&n) == hipSuccess && n > 0;
}

}  // namespace

namespace vasmg {
// Device bytes of a host-built handle without dense tables.
int64_t plain_bytes(vasmg_handle h) { return estimate_device_bytes(*h, false); }

// What the tables and their construction add to them; with more than `allowance`
// the upload leaves the tables out (0). The construction's vectors shrink to fit:
// the tables' values do not depend on them.
int64_t plan_tables(vasmg_handle h, int64_t allowance) {
  const int64_t plain = plain_bytes(h);
  h->dense_work = kDenseLeastWork;
  int64_t extra = estimate_device_bytes(*h) - plain;
  if (extra > allowance) {
    h->no_dense = true;
    return 0;
  }
  h->dense_work = std::min(kDenseWorkBytes, kDenseLeastWork + (allowance - extra) / 10 * 9);
  extra = estimate_device_bytes(*h) - plain;
  return extra;
}
}  // namespace vasmg

// ---------------------------------------------------------------------------
// Staging of the no-allocation host-pointer solve (vasmg_solve_noalloc): one
// fixed array of this library per GPU, in place of the device buffers
// vasmg_solve allocates per call. In host code `scratch` names a host-side
// stand-in, not device memory: its device address on each GPU comes from
// hipGetSymbolAddress (with that GPU current) and only that address is used.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = static_cast<size_t>(64) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;                   // guards g_scratch_ptr
void* g_scratch_ptr[kMaxDevices] = {};        // device address of `scratch` per GPU
std::mutex g_scratch_use[kMaxDevices];        // one no-allocation solve per GPU at a time

// Device address of this GPU's copy of `scratch`; dev must be the current device.
unsigned char* scratch_address(int dev) {
  if (dev < 0 || dev >= kMaxDevices)
    throw vasmg::Error{VASMG_EDEVICE, "device index beyond the no-allocation table"};
  std::lock_guard<std::mutex> g(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      throw vasmg::Error{VASMG_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") +
                                            hipGetErrorString(e)};
    g_scratch_ptr[dev] = p;
  }
  return static_cast<unsigned char*>(g_scratch_ptr[dev]);
}

// masked: the level's constrained components read as 0 (the restriction's
// zero prolongation rows)
template <typename T, int D>
void debug_gather(vasmg_ctx& C, int l, const double* src, T* dst, hipStream_t st,
                  bool masked = false) {
  const int n = static_cast<int>(C.H.levels[l].n);
  hipLaunchKernelGGL((dev::k_gather_user<double, T, D>), dim3(grid_for(n, dev::kBlock)),
                     dim3(dev::kBlock), 0, st, n, C.lev[l].perm, src, dst,
                     masked ? static_cast<const uint8_t*>(C.lev[l].fixed) : nullptr);
}
template <typename T, int D>
void debug_scatter(vasmg_ctx& C, int l, const T* src, double* dst, hipStream_t st) {
  const int n = static_cast<int>(C.H.levels[l].n);
  hipLaunchKernelGGL((dev::k_scatter_user<T, double, D>), dim3(grid_for(n, dev::kBlock)),
                     dim3(dev::kBlock), 0, st, n, C.lev[l].perm, src, dst);
}

void check_handle(vasmg_handle h) {
  if (!h) throw vasmg::Error{VASMG_EINVAL, "null handle"};
  if (h->host_only) throw vasmg::Error{VASMG_EDEVICE, "handle was set up host-only"};
  HIP_CHECK(hipSetDevice(h->device));
}

void check_level(vasmg_handle h, int level, bool need_transfer) {
  if (level < 0 || level > h->L) throw vasmg::Error{VASMG_EINVAL, "level out of range"};
  if (need_transfer && level >= h->L) throw vasmg::Error{VASMG_EINVAL, "no transfer on the coarsest level"};
  if (h->opt.preconditioner != VASMG_PRECOND_VASMG && level > 0)
    throw vasmg::Error{VASMG_EINVAL, "hierarchy not uploaded (non-V-ASMG preconditioner)"};
}

template <typename T>
void check_prec(vasmg_handle h, int level) {
  if (level == h->L && level > 0) throw vasmg::Error{VASMG_EINVAL, "coarsest level has no operator on the device"};
  if (!LevelMats<T>::ok(h->lev[level]))
    throw vasmg::Error{VASMG_EINVAL, "requested precision not resident for this level"};
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* vasmg_last_error(void) { return g_last_error.c_str(); }

vasmg_status vasmg_set_galerkin_window(int32_t cols) {
  if (cols < 0) {
    g_last_error = "vasmg_set_galerkin_window: cols must be >= 0";
    return VASMG_EINVAL;
  }
  g_galerkin_window.store(cols);
  return VASMG_OK;
}

vasmg_status vasmg_default_options(int32_t dim, vasmg_options* out) {
  if (!out || (dim != 2 && dim != 3)) {
    g_last_error = "vasmg_default_options: dim must be 2 or 3 and out non-null";
    return VASMG_EINVAL;
  }
  std::memset(out, 0, sizeof(*out));
  out->leaf_capacity = dim == 2 ? 4 : 8;
  out->n_pre = 1;
  out->n_post = 1;
  out->precision = VASMG_FP64;
  out->tree_vertices = VASMG_TREE_ALL;
  out->coarsest_max_dofs = 0;
  out->max_iters = 10000;
  out->preconditioner = VASMG_PRECOND_VASMG;
  return VASMG_OK;
}

vasmg_status vasmg_setup(const vasmg_mesh* mesh, const vasmg_options* opt, vasmg_handle* out) {
  if (out) *out = nullptr;
  try {
    if (!mesh || !out) throw vasmg::Error{VASMG_EINVAL, "null mesh or output pointer"};
    std::unique_ptr<vasmg_ctx> C(new vasmg_ctx());
    if (opt) {
      C->opt = *opt;
    } else if (vasmg_default_options(mesh->dim, &C->opt) != VASMG_OK) {
      throw vasmg::Error{VASMG_EINVAL, "dim must be 2 or 3"};
    }
    vasmg_options& o = C->opt;
    if (o.leaf_capacity == 0) o.leaf_capacity = mesh->dim == 2 ? 4 : 8;
    if (o.leaf_capacity < 1) throw vasmg::Error{VASMG_EINVAL, "leaf_capacity must be >= 1"};
    if (o.n_pre < 0 || o.n_post < 0 || o.n_pre > 16 || o.n_post > 16)
      throw vasmg::Error{VASMG_EINVAL, "n_pre/n_post must be in [0, 16]"};
    if (o.precision != VASMG_FP64 && o.precision != VASMG_FP32_PRECOND)
      throw vasmg::Error{VASMG_EINVAL, "unknown precision"};
    if (o.tree_vertices != VASMG_TREE_ALL && o.tree_vertices != VASMG_TREE_FREE)
      throw vasmg::Error{VASMG_EINVAL, "unknown tree_vertices"};
    if (o.preconditioner < 0 || o.preconditioner > 2)
      throw vasmg::Error{VASMG_EINVAL, "unknown preconditioner"};
    if (o.max_iters <= 0) o.max_iters = 10000;
    if (o.coarsest_max_dofs < 0) throw vasmg::Error{VASMG_EINVAL, "coarsest_max_dofs < 0"};
    if (o.block_rhs != 0 && o.block_rhs != 4 && o.block_rhs != 8 && o.block_rhs != 16)
      throw vasmg::Error{VASMG_EINVAL, "block_rhs must be 0, 4, 8 or 16"};
    if (o.cycle < VASMG_CYCLE_V || o.cycle > VASMG_CYCLE_ADDITIVE)
      throw vasmg::Error{VASMG_EINVAL, "unknown cycle"};
    if (o.smoother != VASMG_SMOOTHER_GS && o.smoother != VASMG_SMOOTHER_JACOBI)
      throw vasmg::Error{VASMG_EINVAL, "unknown smoother"};
    if (o.block_rhs != 0 && (o.cycle != VASMG_CYCLE_V || o.smoother != VASMG_SMOOTHER_GS))
      throw vasmg::Error{VASMG_EINVAL, "block_rhs supports the Gauss-Seidel V-cycle only"};
    if (o.setup_device != 0 && o.setup_device != 1)
      throw vasmg::Error{VASMG_EINVAL, "setup_device must be 0 or 1"};
    MeshView mv{mesh->dim, mesh->n_vertices, mesh->coords, mesh->n_elements, mesh->elems,
                mesh->E, mesh->nu, mesh->fixed};
    if (o.color_blocks != 0 && o.color_blocks != 1)
      throw vasmg::Error{VASMG_EINVAL, "color_blocks must be 0 (off) or 1 (on)"};
    if (o.block_lanes < 0 || o.block_lanes > 2)
      throw vasmg::Error{VASMG_EINVAL, "block_lanes must be 0, 1 (narrow) or 2 (wide)"};
    SetupParams prm{o.leaf_capacity, o.tree_vertices == VASMG_TREE_FREE, o.coarsest_max_dofs};
    // the block right-hand-side kernels sweep one cell per workgroup: no colour blocks
    prm.color_blocks = o.color_blocks == 1 && o.block_rhs == 0;
    std::unique_ptr<GalerkinDevice, void (*)(GalerkinDevice*)> gdev(nullptr, galerkin_device_destroy);
    if (o.setup_device == 1) {
      if (!device_available()) throw vasmg::Error{VASMG_EDEVICE, "no HIP device for setup_device = 1"};
      gdev.reset(galerkin_device_create(g_galerkin_window.load()));
      prm.galerkin = galerkin_device;
      prm.assemble = assemble_device;
      prm.settle = galerkin_device_settle;
      prm.wait_structure = galerkin_device_wait_structure;
      prm.transfers = transfers_device;
      prm.galerkin_ctx = gdev.get();
    }
    build_hierarchy(mv, prm, C->H);
    if (gdev && o.host_only) {   // every value back on the host, no device memory kept
      galerkin_device_join(gdev.get());
      gdev.reset();
    }
    C->d = mesh->dim;
    C->DP = mesh->dim == 3 ? 4 : 2;
    C->L = static_cast<int>(C->H.levels.size()) - 1;
    C->vc32 = o.precision == VASMG_FP32_PRECOND;
    C->host_only = o.host_only != 0;
    if (o.verbose) {
      for (size_t l = 0; l < C->H.levels.size(); ++l) {
        const Level& lv = C->H.levels[l];
        std::fprintf(stderr, "[vasmg] level %zu: %lld vertices, %lld blocks, %d colours\n", l,
                     static_cast<long long>(lv.n), static_cast<long long>(lv.A.nnzb()), lv.ncolors);
      }
      for (const auto& ph : C->H.phase_ms)
        std::fprintf(stderr, "[vasmg] setup %-18s %9.1f ms\n", ph.first.c_str(), ph.second);
    }
    if (!C->host_only) {
      const auto t0 = std::chrono::steady_clock::now();
      C->gdev = gdev.get();
      upload_device(*C, nullptr);
      C->gdev = nullptr;
      if (gdev && o.smoother == VASMG_SMOOTHER_JACOBI) {
        galerkin_device_join(gdev.get());   // already started by the Jacobi set-up
        gdev.reset();
      } else if (gdev) {
        // the host copies of the level values arrive while the caller goes on;
        // each level's device copy is released once its values are home
        galerkin_device_start_downloads(gdev.get(), true);
        C->gdev_bg = gdev.release();
      }
      const double ms =
          std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
      // the upload's parts (host time until each returned; device work may run on)
      const double other = ms - C->upload_ms[0] - C->upload_ms[1] - C->upload_ms[2];
      C->H.phase_ms.emplace_back("upload: layouts", C->upload_ms[0] + std::max(other, 0.0));
      if (o.autotune) C->H.phase_ms.emplace_back("upload: autotune", C->upload_ms[1]);
      C->H.phase_ms.emplace_back("upload: graphs", C->upload_ms[2]);
      if (o.verbose)
        std::fprintf(stderr, "[vasmg] setup %-18s %9.1f ms (layouts %.1f, autotune %.1f, graphs %.1f)\n",
                     "upload", ms, C->upload_ms[0], C->upload_ms[1], C->upload_ms[2]);
    }
    *out = C.release();
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  } catch (const std::bad_alloc&) {
    g_last_error = "host allocation failed";
    return VASMG_ENOMEM;
  } catch (const std::exception& e) {
    g_last_error = e.what();
    return VASMG_EINVAL;
  }
}

void vasmg_free(vasmg_handle h) {
  if (!h) return;
  if (!h->host_only) (void)hipSetDevice(h->device);
  delete h;
}

vasmg_status vasmg_solve_device(vasmg_handle h, const double* d_rhs, const double* d_x0,
                                double* d_x, int32_t n_rhs, double rtol, void* stream,
                                vasmg_solve_info* info) {
  try {
    check_handle(h);
    if (!d_rhs || !d_x || n_rhs < 1) throw vasmg::Error{VASMG_EINVAL, "bad rhs/x/n_rhs"};
    if (!(rtol > 0.0)) throw vasmg::Error{VASMG_EINVAL, "rtol must be > 0"};
    if (h->nseg > 0) throw vasmg::Error{VASMG_EINVAL, "packed handle: use vasmg_solve_packed(_device)"};
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t stride = h->H.n_mesh_vertices * h->d;
    int worst = VASMG_OK;
    if (h->K > 0 && n_rhs > 1) {
      // block solve: K columns at a time share every matrix read
      for (int c0 = 0; c0 < n_rhs; c0 += h->K) {
        const int nc = std::min(h->K, n_rhs - c0);
        vasmg_solve_info* fi = info ? info + c0 : nullptr;
        int s = VASMG_OK;
        DISPATCH_K(h->K, {
          s = h->d == 2 ? solve_block<2, KK>(*h, d_rhs, d_x0, d_x, c0, nc, rtol, st, fi)
                        : solve_block<3, KK>(*h, d_rhs, d_x0, d_x, c0, nc, rtol, st, fi);
        });
        if (s != VASMG_OK && worst == VASMG_OK) worst = s;
      }
    } else {
      for (int c = 0; c < n_rhs; ++c) {
        const int s = h->d == 2 ? solve_one<2>(*h, d_rhs + c * stride, d_x0 ? d_x0 + c * stride : nullptr,
                                                d_x + c * stride, rtol, st, info ? info + c : nullptr)
                                : solve_one<3>(*h, d_rhs + c * stride, d_x0 ? d_x0 + c * stride : nullptr,
                                                d_x + c * stride, rtol, st, info ? info + c : nullptr);
        if (s != VASMG_OK && worst == VASMG_OK) worst = s;
      }
    }
    if (worst == VASMG_ENOTCONV) g_last_error = "PCG did not reach rtol within max_iters";
    if (worst == VASMG_EBREAKDOWN) g_last_error = "PCG breakdown (p^T A p <= 0 or not finite)";
    return static_cast<vasmg_status>(worst);
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_solve(vasmg_handle h, const double* rhs, const double* x0, double* x,
                         int32_t n_rhs, double rtol, vasmg_solve_info* info) {
  double *drhs = nullptr, *dx0 = nullptr, *dx = nullptr;
  try {
    check_handle(h);
    if (!rhs || !x || n_rhs < 1) throw vasmg::Error{VASMG_EINVAL, "bad rhs/x/n_rhs"};
    const size_t bytes = sizeof(double) * h->H.n_mesh_vertices * h->d * n_rhs;
    HIP_CHECK(hipMalloc(&drhs, bytes));
    HIP_CHECK(hipMalloc(&dx, bytes));
    HIP_CHECK(hipMemcpy(drhs, rhs, bytes, hipMemcpyHostToDevice));
    if (x0) {
      HIP_CHECK(hipMalloc(&dx0, bytes));
      HIP_CHECK(hipMemcpy(dx0, x0, bytes, hipMemcpyHostToDevice));
    }
    const vasmg_status s = vasmg_solve_device(h, drhs, dx0, dx, n_rhs, rtol, nullptr, info);
    const std::string msg = g_last_error;
    HIP_CHECK(hipMemcpy(x, dx, bytes, hipMemcpyDeviceToHost));
    (void)hipFree(drhs);
    (void)hipFree(dx);
    if (dx0) (void)hipFree(dx0);
    g_last_error = msg;
    return s;
  } catch (const vasmg::Error& e) {
    if (drhs) (void)hipFree(drhs);
    if (dx) (void)hipFree(dx);
    if (dx0) (void)hipFree(dx0);
    return fail_with(e);
  }
}

vasmg_status vasmg_solve_noalloc(vasmg_handle h, const double* rhs, const double* x0, double* x,
                                 int32_t n_rhs, double rtol, vasmg_solve_info* info) {
  try {
    check_handle(h);
    if (!rhs || !x || n_rhs < 1) throw vasmg::Error{VASMG_EINVAL, "bad rhs/x/n_rhs"};
    if (h->nseg > 0) throw vasmg::Error{VASMG_EINVAL, "packed handle: use vasmg_solve_packed(_device)"};
    const size_t vec = sizeof(double) * static_cast<size_t>(h->H.n_mesh_vertices) * h->d *
                       static_cast<size_t>(n_rhs);
    const size_t slot = (vec + 255) / 256 * 256;
    const size_t need = slot * (x0 ? 3 : 2);
    if (need > kScratchBytes)
      throw vasmg::Error{VASMG_EINVAL, "vasmg_solve_noalloc: " + std::to_string(need) +
                                           " bytes of staging needed, more than its fixed " +
                                           std::to_string(kScratchBytes) + "-byte array"};
    unsigned char* base = scratch_address(h->device);
    std::lock_guard<std::mutex> use(g_scratch_use[h->device]);
    double* drhs = reinterpret_cast<double*>(base);
    double* dx = reinterpret_cast<double*>(base + slot);
    double* dx0 = x0 ? reinterpret_cast<double*>(base + 2 * slot) : nullptr;
    HIP_CHECK(hipMemcpy(drhs, rhs, vec, hipMemcpyHostToDevice));
    if (x0) HIP_CHECK(hipMemcpy(dx0, x0, vec, hipMemcpyHostToDevice));
    const vasmg_status s = vasmg_solve_device(h, drhs, dx0, dx, n_rhs, rtol, nullptr, info);
    const std::string msg = g_last_error;
    HIP_CHECK(hipMemcpy(x, dx, vec, hipMemcpyDeviceToHost));
    g_last_error = msg;
    return s;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_pack(const vasmg_handle* parts, int32_t n_parts, vasmg_handle* out) {
  try {
    if (!out) throw vasmg::Error{VASMG_EINVAL, "null output"};
    *out = nullptr;
    if (!parts || n_parts < 1) throw vasmg::Error{VASMG_EINVAL, "no parts to pack"};
    const auto t0 = std::chrono::steady_clock::now();
    std::vector<const Hierarchy*> hs;
    const vasmg_options& o0 = parts[0] ? parts[0]->opt : vasmg_options{};
    int32_t max_iters = 0;
    for (int i = 0; i < n_parts; ++i) {
      vasmg_handle p = parts[i];
      if (!p) throw vasmg::Error{VASMG_EINVAL, "null part handle"};
      if (p->nseg > 0) throw vasmg::Error{VASMG_EINVAL, "a part is itself packed"};
      const vasmg_options& o = p->opt;
      if (o.preconditioner != VASMG_PRECOND_VASMG || o.cycle != VASMG_CYCLE_V ||
          o.smoother != VASMG_SMOOTHER_GS || o.block_rhs != 0 || o.color_blocks != 0)
        throw vasmg::Error{VASMG_EINVAL,
                           "packing needs the V-ASMG Gauss-Seidel V-cycle without block_rhs or colour blocks"};
      if (o.precision != o0.precision || o.n_pre != o0.n_pre || o.n_post != o0.n_post ||
          p->d != parts[0]->d)
        throw vasmg::Error{VASMG_EINVAL, "packed parts differ in dimension, precision or sweeps"};
      p->settle_host_values();
      hs.push_back(&p->H);
      max_iters = std::max(max_iters, o.max_iters);
    }
    auto C = std::make_unique<vasmg_ctx>();
    pack_hierarchies(hs, C->H);
    C->opt = o0;
    C->opt.host_only = 1;
    C->opt.max_iters = max_iters;
    C->d = parts[0]->d;
    C->DP = C->d == 3 ? 4 : 2;
    C->L = static_cast<int>(C->H.levels.size()) - 1;
    C->vc32 = o0.precision == VASMG_FP32_PRECOND;
    C->host_only = true;
    C->nseg = n_parts;
    C->seg_vertex_off.assign(1, 0);
    C->seg_free_off.assign(1, 0);
    for (int i = 0; i < n_parts; ++i) {
      C->seg_vertex_off.push_back(C->seg_vertex_off.back() + parts[i]->H.n_mesh_vertices);
      C->seg_free_off.push_back(C->seg_free_off.back() + parts[i]->H.levels[0].n);
      C->dense_off = C->dense_off || parts[i]->dense_off;
    }
    C->seg_level_off.resize(C->L + 1);
    for (int l = 0; l <= C->L; ++l) {   // a part shallower than l repeats its coarsest level
      std::vector<int64_t>& off = C->seg_level_off[l];
      off.assign(1, 0);
      for (const Hierarchy* p : hs)
        off.push_back(off.back() + p->levels[std::min<size_t>(l, p->levels.size() - 1)].n);
    }
    C->H.phase_ms.emplace_back(
        "pack", std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count());
    *out = C.release();
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  } catch (const std::bad_alloc&) {
    g_last_error = "host allocation failed";
    return VASMG_ENOMEM;
  }
}

vasmg_status vasmg_packed_info(vasmg_handle h, int32_t* n_parts, int64_t* vertex_offsets) {
  if (!h) {
    g_last_error = "null handle";
    return VASMG_EINVAL;
  }
  if (n_parts) *n_parts = h->nseg;
  if (vertex_offsets && h->nseg > 0)
    std::copy(h->seg_vertex_off.begin(), h->seg_vertex_off.end(), vertex_offsets);
  return VASMG_OK;
}

vasmg_status vasmg_solve_packed_device(vasmg_handle h, const double* d_rhs, double* d_x, double rtol,
                                       void* stream, vasmg_solve_info* info) {
  try {
    check_handle(h);
    if (h->nseg == 0) throw vasmg::Error{VASMG_EINVAL, "not a packed handle (vasmg_pack)"};
    if (!d_rhs || !d_x || !info) throw vasmg::Error{VASMG_EINVAL, "bad rhs/x/info"};
    if (!(rtol > 0.0)) throw vasmg::Error{VASMG_EINVAL, "rtol must be > 0"};
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int worst = h->d == 2 ? solve_packed<2>(*h, d_rhs, d_x, rtol, st, info)
                                : solve_packed<3>(*h, d_rhs, d_x, rtol, st, info);
    if (worst == VASMG_ENOTCONV) g_last_error = "PCG did not reach rtol within max_iters (some part)";
    if (worst == VASMG_EBREAKDOWN) g_last_error = "PCG breakdown in some part";
    return static_cast<vasmg_status>(worst);
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_solve_packed(vasmg_handle h, const double* rhs, double* x, double rtol,
                                vasmg_solve_info* info) {
  double *drhs = nullptr, *dx = nullptr;
  try {
    check_handle(h);
    if (h->nseg == 0) throw vasmg::Error{VASMG_EINVAL, "not a packed handle (vasmg_pack)"};
    if (!rhs || !x || !info) throw vasmg::Error{VASMG_EINVAL, "bad rhs/x/info"};
    const size_t bytes = sizeof(double) * h->H.n_mesh_vertices * h->d;
    HIP_CHECK(hipMalloc(&drhs, bytes));
    HIP_CHECK(hipMalloc(&dx, bytes));
    HIP_CHECK(hipMemcpy(drhs, rhs, bytes, hipMemcpyHostToDevice));
    const vasmg_status s = vasmg_solve_packed_device(h, drhs, dx, rtol, nullptr, info);
    const std::string msg = g_last_error;
    HIP_CHECK(hipMemcpy(x, dx, bytes, hipMemcpyDeviceToHost));
    (void)hipFree(drhs);
    (void)hipFree(dx);
    g_last_error = msg;
    return s;
  } catch (const vasmg::Error& e) {
    if (drhs) (void)hipFree(drhs);
    if (dx) (void)hipFree(dx);
    return fail_with(e);
  }
}

vasmg_status vasmg_upload(vasmg_handle h, void* stream) {
  try {
    if (!h) throw vasmg::Error{VASMG_EINVAL, "null handle"};
    if (!h->host_only || !h->allocs.empty())
      throw vasmg::Error{VASMG_EINVAL, "handle is already on the device"};
    upload_device(*h, static_cast<hipStream_t>(stream));
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  } catch (const std::bad_alloc&) {
    g_last_error = "host allocation failed";
    return VASMG_ENOMEM;
  }
}

vasmg_status vasmg_set_dense_tables(vasmg_handle h, int32_t on) {
  if (!h || !h->host_only || (on != 0 && on != 1)) {
    g_last_error = "vasmg_set_dense_tables: needs a host-only handle and 0 or 1";
    return VASMG_EINVAL;
  }
  h->dense_off = on == 0;
  return VASMG_OK;
}

vasmg_status vasmg_device_bytes(vasmg_handle h, int64_t* bytes) {
  if (!h || !bytes) {
    g_last_error = "null handle or output";
    return VASMG_EINVAL;
  }
  *bytes = h->host_only ? estimate_device_bytes(*h) : h->dev_bytes;
  return VASMG_OK;
}

vasmg_status vasmg_hierarchy_info(vasmg_handle h, int32_t* n_levels, int64_t* n_dofs, int32_t* dim) {
  if (!h) {
    g_last_error = "null handle";
    return VASMG_EINVAL;
  }
  if (n_levels) *n_levels = static_cast<int32_t>(h->H.levels.size());
  if (n_dofs) *n_dofs = h->H.levels[0].n * h->d;
  if (dim) *dim = h->d;
  return VASMG_OK;
}

vasmg_status vasmg_level_info(vasmg_handle h, int32_t level, int64_t* n_vertices, int64_t* n_blocks,
                              int32_t* n_colors, int64_t* p_nnz) {
  if (!h || level < 0 || level >= static_cast<int32_t>(h->H.levels.size())) {
    g_last_error = "null handle or level out of range";
    return VASMG_EINVAL;
  }
  const Level& lv = h->H.levels[level];
  if (n_vertices) *n_vertices = lv.n;
  if (n_blocks) *n_blocks = lv.A.nnzb();
  if (n_colors) *n_colors = lv.ncolors;
  if (p_nnz) *p_nnz = static_cast<int64_t>(lv.P.col.size());
  return VASMG_OK;
}

vasmg_status vasmg_export_level(vasmg_handle h, int32_t level, int64_t* keys, int32_t* cell,
                                int32_t* color, int64_t* rowptr, int32_t* cols, double* vals,
                                int64_t* p_rowptr, int32_t* p_cols, double* p_vals,
                                int32_t* block, uint8_t* fixed) {
  if (!h || level < 0 || level >= static_cast<int32_t>(h->H.levels.size())) {
    g_last_error = "null handle or level out of range";
    return VASMG_EINVAL;
  }
  try {
    h->settle_host_values();
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
  const Level& lv = h->H.levels[level];
  const int d = h->d;
  if (keys) {
    for (int64_t i = 0; i < lv.n; ++i)
      for (int a = 0; a < d; ++a)
        keys[i * d + a] = lv.keys.empty() ? -1 : static_cast<int64_t>(lv.keys[i][a]);
  }
  if (color) {
    for (int64_t i = 0; i < lv.n; ++i) color[i] = lv.color.empty() ? 0 : lv.color[i];
  }
  if (cell) {
    for (int64_t i = 0; i < lv.n; ++i) cell[i] = lv.cell.empty() ? 0 : lv.cell[i];
  }
  if (block) {
    for (int64_t i = 0; i < lv.n; ++i) block[i] = lv.block.empty() ? 0 : lv.block[i];
  }
  if (rowptr) std::copy(lv.A.rowptr.begin(), lv.A.rowptr.end(), rowptr);
  if (cols) std::copy(lv.A.col.begin(), lv.A.col.end(), cols);
  if (vals) {
    std::copy(lv.A.val.begin(), lv.A.val.end(), vals);
    if (!lv.fixed.empty())   // identity rows of the constrained components
      for (int64_t i = 0; i < lv.n; ++i)
        for (int64_t p = lv.A.rowptr[i]; p < lv.A.rowptr[i + 1]; ++p)
          if (lv.A.col[p] == i)
            for (int a = 0; a < d; ++a)
              if ((lv.fixed[i] >> a) & 1) vals[p * d * d + a * d + a] = 1.0;
  }
  if (fixed) {
    for (int64_t i = 0; i < lv.n; ++i) fixed[i] = lv.fixed.empty() ? 0 : lv.fixed[i];
  }
  if (p_rowptr) {
    if (lv.P.rowptr.empty())
      std::fill(p_rowptr, p_rowptr + lv.n + 1, 0);
    else
      std::copy(lv.P.rowptr.begin(), lv.P.rowptr.end(), p_rowptr);
  }
  if (p_cols) std::copy(lv.P.col.begin(), lv.P.col.end(), p_cols);
  if (p_vals) std::copy(lv.P.val.begin(), lv.P.val.end(), p_vals);
  return VASMG_OK;
}

vasmg_status vasmg_tree_info(vasmg_handle h, double* m, double* M, int32_t* max_depth) {
  if (!h) {
    g_last_error = "null handle";
    return VASMG_EINVAL;
  }
  if (m) *m = h->H.box_m;
  if (M) *M = h->H.box_M;
  if (max_depth) *max_depth = h->H.max_depth;
  return VASMG_OK;
}

vasmg_status vasmg_setup_phases(vasmg_handle h, vasmg_setup_phase* out, int32_t max_out,
                                int32_t* n_out) {
  if (!h || max_out < 0 || (max_out > 0 && !out)) {
    g_last_error = "null handle or output";
    return VASMG_EINVAL;
  }
  const auto& ph = h->H.phase_ms;
  for (int32_t i = 0; i < max_out && i < static_cast<int32_t>(ph.size()); ++i) {
    std::memset(out[i].name, 0, sizeof(out[i].name));
    std::strncpy(out[i].name, ph[i].first.c_str(), sizeof(out[i].name) - 1);
    out[i].ms = ph[i].second;
  }
  if (n_out) *n_out = static_cast<int32_t>(ph.size());
  return VASMG_OK;
}

#define DEBUG_PRELUDE(NEED_TRANSFER)          \
  check_handle(h);                            \
  check_level(h, level, NEED_TRANSFER);       \
  hipStream_t st = static_cast<hipStream_t>(stream);

vasmg_status vasmg_spmv_device(vasmg_handle h, int32_t level, int32_t precision, const double* d_x,
                               double* d_y, void* stream) {
  try {
    DEBUG_PRELUDE(false);
    DevLevel& lv = h->lev[level];
    auto run = [&](auto tag, auto dtag) {
      using T = decltype(tag);
      constexpr int D = decltype(dtag)::value;
      check_prec<T>(h, level);
      T* xin = static_cast<T*>(lv.x);
      T* yout = static_cast<T*>(lv.r);
      if (precision == VASMG_FP64 && h->vc32) {  // FP64 copy on the fine level of a mixed handle
        xin = reinterpret_cast<T*>(h->Z);
        yout = reinterpret_cast<T*>(h->Q);
      }
      debug_gather<T, D>(*h, level, d_x, xin, st);
      if (lv.cells)
        launch_cell_apply<T, D, 2>(lv, nullptr, xin, yout, st);
      else
        launch_spmv<T, D>(lv, xin, yout, nullptr, 0, st);
      debug_scatter<T, D>(*h, level, yout, d_y, st);
    };
    if (precision == VASMG_FP64) {
      if (h->d == 2) run(double(), std::integral_constant<int, 2>());
      else run(double(), std::integral_constant<int, 3>());
    } else {
      if (h->d == 2) run(float(), std::integral_constant<int, 2>());
      else run(float(), std::integral_constant<int, 3>());
    }
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_gs_sweep_device(vasmg_handle h, int32_t level, int32_t precision, int32_t backward,
                                   const double* d_b, double* d_x, void* stream) {
  try {
    DEBUG_PRELUDE(false);
    if (level == h->L) throw vasmg::Error{VASMG_EINVAL, "no smoother on the coarsest level"};
    DevLevel& lv = h->lev[level];
    if ((precision == VASMG_FP64) == h->vc32)
      throw vasmg::Error{VASMG_EINVAL, "GS precision must match the handle's V-cycle precision"};
    auto run = [&](auto tag, auto dtag) {
      using T = decltype(tag);
      constexpr int D = decltype(dtag)::value;
      check_prec<T>(h, level);
      T* b = static_cast<T*>(lv.b);
      T* x = static_cast<T*>(lv.x);
      debug_gather<T, D>(*h, level, d_b, b, st);
      debug_gather<T, D>(*h, level, d_x, x, st);
      launch_gs_sweep<T, D>(lv, backward != 0, false, b, x, static_cast<T*>(lv.s), st);
      debug_scatter<T, D>(*h, level, x, d_x, st);
    };
    if (precision == VASMG_FP64) {
      if (h->d == 2) run(double(), std::integral_constant<int, 2>());
      else run(double(), std::integral_constant<int, 3>());
    } else {
      if (h->d == 2) run(float(), std::integral_constant<int, 2>());
      else run(float(), std::integral_constant<int, 3>());
    }
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_restrict_device(vasmg_handle h, int32_t level, int32_t precision, const double* d_r,
                                   double* d_bc, void* stream) {
  try {
    DEBUG_PRELUDE(true);
    DevLevel& lv = h->lev[level];
    DevLevel& nx = h->lev[level + 1];
    if ((precision == VASMG_FP64) == h->vc32)
      throw vasmg::Error{VASMG_EINVAL, "transfer precision must match the handle's V-cycle precision"};
    auto run = [&](auto tag, auto dtag) {
      using T = decltype(tag);
      constexpr int D = decltype(dtag)::value;
      T* r = static_cast<T*>(lv.r);
      T* bc = static_cast<T*>(nx.b);
      debug_gather<T, D>(*h, level, d_r, r, st, true);
      launch_restrict<T, D>(lv, r, bc, st);
      debug_scatter<T, D>(*h, level + 1, bc, d_bc, st);
    };
    if (precision == VASMG_FP64) {
      if (h->d == 2) run(double(), std::integral_constant<int, 2>());
      else run(double(), std::integral_constant<int, 3>());
    } else {
      if (h->d == 2) run(float(), std::integral_constant<int, 2>());
      else run(float(), std::integral_constant<int, 3>());
    }
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_prolong_device(vasmg_handle h, int32_t level, int32_t precision, const double* d_e,
                                  double* d_x, void* stream) {
  try {
    DEBUG_PRELUDE(true);
    DevLevel& lv = h->lev[level];
    DevLevel& nx = h->lev[level + 1];
    if ((precision == VASMG_FP64) == h->vc32)
      throw vasmg::Error{VASMG_EINVAL, "transfer precision must match the handle's V-cycle precision"};
    auto run = [&](auto tag, auto dtag) {
      using T = decltype(tag);
      constexpr int D = decltype(dtag)::value;
      T* e = static_cast<T*>(nx.x);
      T* x = static_cast<T*>(lv.x);
      debug_gather<T, D>(*h, level + 1, d_e, e, st);
      debug_gather<T, D>(*h, level, d_x, x, st);
      launch_prolong<T, D>(lv, e, x, st);
      debug_scatter<T, D>(*h, level, x, d_x, st);
    };
    if (precision == VASMG_FP64) {
      if (h->d == 2) run(double(), std::integral_constant<int, 2>());
      else run(double(), std::integral_constant<int, 3>());
    } else {
      if (h->d == 2) run(float(), std::integral_constant<int, 2>());
      else run(float(), std::integral_constant<int, 3>());
    }
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_apply_precond_device(vasmg_handle h, const double* d_r, double* d_z, void* stream) {
  try {
    check_handle(h);
    if (h->opt.preconditioner != VASMG_PRECOND_VASMG)
      throw vasmg::Error{VASMG_EINVAL, "handle was not set up with the V-ASMG preconditioner"};
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto run = [&](auto tag, auto dtag) {
      using T = decltype(tag);
      constexpr int D = decltype(dtag)::value;
      T* b = static_cast<T*>(h->lev[0].b);
      T* x = static_cast<T*>(h->lev[0].x);
      debug_gather<T, D>(*h, 0, d_r, b, st);
      if (h->L == 0 && h->cinv) {
        hipLaunchKernelGGL((dev::k_coarse_apply<T, D>), dim3(1), dim3(dev::kBlock), 0, st,
                           static_cast<int>(h->n_coarse), h->cinv, b, x);
      } else if (h->L == 0) {
        hipLaunchKernelGGL((dev::k_coarse_solve<T, D>), dim3(1), dim3(dev::kBlock), 0, st,
                           static_cast<int>(h->n_coarse), h->chol, b, x);
      } else {
        enqueue_vcycle<T, D>(*h, st);
      }
      debug_scatter<T, D>(*h, 0, x, d_z, st);
    };
    if (h->vc32) {
      if (h->d == 2) run(float(), std::integral_constant<int, 2>());
      else run(float(), std::integral_constant<int, 3>());
    } else {
      if (h->d == 2) run(double(), std::integral_constant<int, 2>());
      else run(double(), std::integral_constant<int, 3>());
    }
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

vasmg_status vasmg_profile_iteration(vasmg_handle h, int32_t reps, void* stream,
                                     vasmg_phase_stat* out, int32_t max_out, int32_t* n_out) {
  try {
    check_handle(h);
    if (reps < 1 || !out || max_out < 1) throw vasmg::Error{VASMG_EINVAL, "bad reps/out"};
    if (h->opt.preconditioner != VASMG_PRECOND_VASMG)
      throw vasmg::Error{VASMG_EINVAL, "handle was not set up with the V-ASMG preconditioner"};
    hipStream_t st = static_cast<hipStream_t>(stream);
    vasmg_ctx& C = *h;
    // defined inputs: p = 1, V-cycle right-hand side = 1, flags cleared
    launch_fill<double>(C.P, C.n0p, 1.0, st);
    if (C.vc32)
      launch_fill<float>(static_cast<float*>(C.lev[0].b), C.n0p, 1.0f, st);
    else
      launch_fill<double>(static_cast<double*>(C.lev[0].b), C.n0p, 1.0, st);
    // running iterations that no step of these replays stops
    Scalars running{};
    running.rho = running.normF = 1.0;
    const std::vector<Scalars> state(std::max(C.nseg, 1), running);
    auto restart = [&] {
      HIP_CHECK(hipMemcpyAsync(C.sc, state.data(), sizeof(Scalars), hipMemcpyHostToDevice, st));
      if (C.nseg > 0)
        HIP_CHECK(hipMemcpyAsync(C.ssc, state.data(), sizeof(Scalars) * C.nseg, hipMemcpyHostToDevice, st));
      HIP_CHECK(hipStreamSynchronize(st));
    };
    Profiler prof{st, {}, {}, {}};
    const DevLevel& l0 = C.lev[0];
    const double n0 = l0.n, dd = C.d * C.d;
    const int tb = C.vc32 ? 4 : 8;
    const double spmv_bytes = (l0.nnz_lo + l0.nnz_up) * (dd * 8 + 4.0) + (n0 + 1) * 4 +
                              n0 * dd * 8 + 2 * C.n0p * 8.0 + n0 * 4;
    const double vec_bytes = C.n0p * (6 * 8.0 + tb) + C.n0p * (8.0 + tb) + C.n0p * (16.0 + tb);
    for (int r = 0; r < reps; ++r) {
      auto body = [&](auto dtag) {
        constexpr int D = decltype(dtag)::value;
        int np = 0;
        restart();
        run_phase(&prof, "spmv_f64", 0, 1, spmv_bytes, [&] {
          np = launch_spmv<double, D>(l0, C.P, C.Q, C.nseg > 0 ? nullptr : C.partial, C.n_partial, st);
        });
        const int launches = C.nseg > 0 || C.n0p <= dev::kSmallFlat ? 2 : 6;
        run_phase(&prof, "pcg_vectors", -1, launches, vec_bytes, [&] {
          if (C.nseg > 0) {
            enqueue_packed_update<D>(C, st);
            enqueue_packed_direction<D>(C, st);
          } else {
            enqueue_update(C, np, st);
            if (C.vc32)
              enqueue_direction(C, static_cast<const float*>(C.lev[0].x), st);
            else
              enqueue_direction(C, static_cast<const double*>(C.lev[0].x), st);
          }
        });
        if (C.vc32)
          enqueue_vcycle<float, D>(C, st, &prof);
        else
          enqueue_vcycle<double, D>(C, st, &prof);
      };
      if (C.d == 2)
        body(std::integral_constant<int, 2>());
      else
        body(std::integral_constant<int, 3>());
      HIP_CHECK(hipGetLastError());
      prof.finish();
    }
    const int n = static_cast<int>(std::min<size_t>(prof.stats.size(), max_out));
    for (int i = 0; i < n; ++i) {
      const PhaseStat& p = prof.stats[i];
      std::memset(&out[i], 0, sizeof(out[i]));
      std::snprintf(out[i].name, sizeof(out[i].name), "%s", p.name.c_str());
      out[i].level = p.level;
      out[i].launches = p.launches;
      out[i].ms = p.ms;
      out[i].bytes = p.bytes;
    }
    if (n_out) *n_out = n;
    return VASMG_OK;
  } catch (const vasmg::Error& e) {
    return fail_with(e);
  }
}

}  // extern "C"
