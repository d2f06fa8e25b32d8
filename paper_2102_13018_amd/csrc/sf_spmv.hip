// sf_spmv.hip -- the sparse matrix-vector products of Section 4.1 around the
// SF: a row-distributed matrix is split into a diagonal block A and an
// off-diagonal block B over the ghost vector lvec, and
//   y = M x:    SFBcast(x -> lvec) overlapped with y = A x, then y += B lvec;
//   y = M^T x:  y = A^T x, lvec = B^T x, then SFReduce SUM(lvec -> y).
// The CSR products are plain HIP kernels: a wavefront per 64 short rows whose
// entries it loads coalesced and sums out of the LDS (k_csr_rows, in column
// panels when x does not fit an L2), or, for small matrices and long or very
// uneven rows, G lanes
// of a wavefront per row (G a power of two near the mean row length), each
// lane striding over the row's entries, the lanes' partial sums combined by
// shuffles (k_csr_spmv).
#include <algorithm>
#include <new>
#include <vector>

#include "sf_device.h"

struct sf_csr_s {
  int64_t nrows = 0, ncols = 0, nnz = 0;
  std::vector<int64_t> h_rowptr;  // host copies (for the transpose)
  std::vector<int32_t> h_colidx;
  std::vector<double> h_values;
  int64_t *rowptr = nullptr;  // device
  int32_t *colidx = nullptr;
  double *values = nullptr;
  hipEvent_t ev = nullptr;  // the Bcast's completion, for the overlapped product
  int device = -1;
  int group = 1;  // lanes per row of k_csr_spmv
  // k_csr_rows: the entries by group of 64 rows, column panel, row
  // (panels 0: k_csr_spmv).  With several panels colidx / values hold that
  // order in place of the CSR order.
  int panels = 0;
  int chains = 0;  // running sums per row: 4, 8 or 16
  int64_t ngroups = 0;
  uint32_t *gbase = nullptr;   // [ngroups * panels + 1] first entry of each group's panel
  uint16_t *starts = nullptr;  // [ngroups * panels * 64] first entry of each row, relative to gbase
};

namespace sfi {

template <int G>
__global__ __launch_bounds__(kBlock) void k_csr_spmv(const int64_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ colidx,
                                                     const double *__restrict__ values, int64_t nrows,
                                                     const double *__restrict__ x, double *__restrict__ y,
                                                     int accumulate) {
  const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t row = gid / G;
  const int sub = (int)(gid % G);
  const bool ok = row < nrows;
  double s = 0.0;
  if (ok) {
    const int64_t k0 = rowptr[row], k1 = rowptr[row + 1];
    for (int64_t k = k0 + sub; k < k1; k += G) s += ld_stream(values + k) * x[ld_stream(colidx + k)];
  }
#pragma unroll
  for (int d = G / 2; d >= 1; d /= 2) s += __shfl_xor(s, d, G);
  if (ok && sub == 0) y[row] = accumulate ? y[row] + s : s;
}

// y = A x (or y += A x) over one column panel, a wavefront per group of 64
// rows: it loads the group's column indices and values coalesced, U * 64 at a
// time, gathers x for all of them, and leaves (value, x) in its own part of
// the LDS; each lane then sums its row's products there.  No load depends on a
// row's own offset, so a wavefront has U gathers per lane in flight whatever
// its rows' lengths.
//
// Bound by the gathers: a request per entry, served from the L2 at 235 G/s
// while x fits (190 beside the entry streams), at 115 G/s for an x of 8 MB and
// 78 G/s for 16 MB (random columns).  So an x beyond an L2 is cut into panels,
// one launch per panel (the launch boundary keeps every XCD on one panel),
// each adding to y.  Measured on 1M rows x 15 random entries, the matrix read
// from HBM (us): k_csr_spmv 158; here 160 with one panel, 124 with two, 114
// with three, 124 with four.  2M rows (x of 16 MB): 411 with one panel, 254
// with three, 248 with five.  250K rows x 16 entries: 51 -> 42; 1M rows x 4
// entries over an x of 2 MB: 33.3 -> 30.3; 300K rows x 15 over 2.4 MB, the
// matrix in the Infinity Cache: 30 -> 26; 1M rows of a 15-point stencil 69 ->
// 34.  Set aside: one launch whose resident wavefronts sweep the panels
// together (no faster than 111 on warm matrices against 92: they drift apart),
// panels bound to XCDs with partial results (103 + 9 for their sum), the next
// group's loads issued ahead (108 against 108 on a matrix from HBM; fewer,
// longer wavefronts 120).
//
// C fused running sums per row, the last four of their additions and the one
// to y with the roundings compensated: the error of a row is no larger than
// that of the lane tree of k_csr_spmv at every length taken (root mean square
// relative to the product, N(0,1) data, lane tree / here: 15 entries 1.11e-16 /
// 0.88e-16, in three panels 0.85e-16, 32 entries 1.17e-16 / 1.11e-16, all C = 4;
// 64 entries 1.28e-16 / 1.22e-16, C = 8; 128 entries 1.36e-16 / 1.33e-16, C =
// 16).  1M rows of a 15-entry band take 34.9 us with C = 4, 36.3 with 8.
// s += b, the rounding error added to c
__device__ __forceinline__ void comp_add(double b, double &s, double &c) {
#pragma clang fp contract(off)
  const double t = s + b;
  const double q = t - s;
  c += (s - (t - q)) + (b - q);
  s = t;
}
template <int U, int C>
__global__ __launch_bounds__(kBlock) void k_csr_rows(const uint32_t *__restrict__ gbase,
                                                     const uint16_t *__restrict__ starts,
                                                     const int32_t *__restrict__ colidx,
                                                     const double *__restrict__ values, int64_t nrows, int64_t ngroups,
                                                     int panels, int panel, const double *__restrict__ x,
                                                     double *__restrict__ y, int accumulate) {
  constexpr int kCap = U * 64;
  __shared__ double2 stage[kBlock / 64][kCap];
  const int lane = threadIdx.x & 63;
  double2 *lds = stage[threadIdx.x >> 6];
  const int64_t g = (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (g >= ngroups) return;
  const int64_t gp = g * panels + panel;
  const uint32_t b = gbase[gp];
  const int n = (int)(gbase[gp + 1] - b);
  const int s0 = starts[gp * 64 + lane];
  const int64_t row = g * 64 + lane;
  const double y0 = accumulate && row < nrows ? y[row] : 0.0;
  const int32_t *cb = colidx + b;
  const double *vb = values + b;
  int s1 = 0;
  double s = y0, comp = 0.0;         // the row's sum and its compensation
  double acc[C] = {};
  for (int c0 = 0; c0 < n; c0 += kCap) {
    // positions past n repeat the last entry; no row reads them
    int32_t col[U];
    double v[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; u++) col[u] = cb[min(c0 + u * 64 + lane, n - 1)];
#pragma unroll
    for (int u = 0; u < U; u++) v[u] = vb[min(c0 + u * 64 + lane, n - 1)];
    if (c0 == 0) {
      const int next = __shfl_down(s0, 1);
      s1 = lane == 63 ? n : next;
    }
#pragma unroll
    for (int u = 0; u < U; u++) xv[u] = x[col[u]];
#pragma unroll
    for (int u = 0; u < U; u++) lds[u * 64 + lane] = make_double2(v[u], xv[u]);
    // the stage is the wavefront's own and its LDS accesses complete in order:
    // only the compiler has to keep them so
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int z = min(s1 - c0, kCap);
    for (int j = max(s0 - c0, 0); j < z; j += C) {
#pragma unroll
      for (int h = 0; h < C; h += 4) {
        if (j + h >= z) break;
        double2 t[4];
#pragma unroll
        for (int k = 0; k < 4; k++) t[k] = lds[min(j + h + k, kCap - 1)];
#pragma unroll
        for (int k = 0; k < 4; k++) acc[h + k] = j + h + k < z ? fma(t[k].x, t[k].y, acc[h + k]) : acc[h + k];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
#pragma unroll
  for (int k = 0; k < 4; k++) {
    double a = acc[k];
    if constexpr (C == 8) a += acc[k + 4];
    if constexpr (C == 16) a = (a + acc[k + 4]) + (acc[k + 8] + acc[k + 12]);
    comp_add(a, s, comp);
  }
  // an infinite or NaN sum has no compensation
  if (row < nrows) y[row] = comp - comp == 0.0 ? s + comp : s;
}

// The tables of k_csr_rows from the CSR arrays and, for several panels of pw
// columns, the entries in (group, panel, row) order, a row's entries of a
// panel in their stored order (pcol, pval).  A wavefront per group, a lane per
// row; a group's entries stay in its range of the CSR arrays, so no scan over
// the groups is needed.  longest: the most entries of a row in a panel (set to
// 0 before).  Runs once per matrix.
__global__ __launch_bounds__(kBlock) void k_csr_panelize(const int64_t *__restrict__ rowptr,
                                                         const int32_t *__restrict__ colidx,
                                                         const double *__restrict__ values, int64_t nrows,
                                                         int64_t ngroups, int panels, int pw,
                                                         uint32_t *__restrict__ gbase, uint16_t *__restrict__ starts,
                                                         int32_t *__restrict__ pcol, double *__restrict__ pval,
                                                         int *__restrict__ longest) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (g >= ngroups) return;
  const int64_t row = g * 64 + lane;
  const int64_t k0 = rowptr[min(row, nrows)], k1 = rowptr[min(row + 1, nrows)];
  int64_t base = rowptr[g * 64];
  int most = 0;
  for (int p = 0; p < panels; p++) {
    const int32_t c0 = p * pw, c1 = p + 1 < panels ? c0 + pw : INT32_MAX;
    int cnt = 0;
    if (panels == 1)
      cnt = (int)(k1 - k0);
    else
      for (int64_t k = k0; k < k1; k++) cnt += colidx[k] >= c0 && colidx[k] < c1;
    most = max(most, cnt);
    int inc = cnt;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const int o = __shfl_up(inc, d);
      if (lane >= d) inc += o;
    }
    if (lane == 0) gbase[g * panels + p] = (uint32_t)base;
    starts[(g * panels + p) * 64 + lane] = (uint16_t)(inc - cnt);
    if (panels > 1) {
      int64_t at = base + inc - cnt;
      for (int64_t k = k0; k < k1; k++) {
        const int32_t c = colidx[k];
        if (c >= c0 && c < c1) {
          pcol[at] = c;
          pval[at] = values[k];
          at++;
        }
      }
    }
    base += __shfl(inc, 63);
  }
  if (g == ngroups - 1 && lane == 0) gbase[ngroups * panels] = (uint32_t)base;
#pragma unroll
  for (int d = 32; d > 0; d /= 2) most = max(most, __shfl_down(most, d));
  if (lane == 0) atomicMax(longest, most);
}

static int pick_group(int64_t nrows, int64_t nnz) {
  const double mean = nrows > 0 ? (double)nnz / (double)nrows : 1.0;
  int g = 1;
  while (g < 64 && g < mean) g *= 2;
  return g;
}

static unsigned group_blocks(int64_t ngroups) { return (unsigned)((ngroups + kBlock / 64 - 1) / (kBlock / 64)); }

static int csr_launch(const sf_csr_s *a, const double *x, double *y, int accumulate, hipStream_t st) {
  if (a->nrows == 0) return SF_OK;
  if (a->panels > 0) {
    // entries in flight: a whole group's panel where that is at most 384
    const bool four = a->nnz <= 256 * a->ngroups * a->panels;
    const auto kernel = a->chains == 4   ? (four ? k_csr_rows<4, 4> : k_csr_rows<6, 4>)
                        : a->chains == 8 ? (four ? k_csr_rows<4, 8> : k_csr_rows<6, 8>)
                                         : (four ? k_csr_rows<4, 16> : k_csr_rows<6, 16>);
    for (int p = 0; p < a->panels; p++)
      hipLaunchKernelGGL(kernel, dim3(group_blocks(a->ngroups)), dim3(kBlock), 0, st,
                         a->gbase, a->starts, a->colidx, a->values, a->nrows, a->ngroups, a->panels, p, x, y,
                         accumulate || p > 0 ? 1 : 0);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SF_OK : set_hip_error(e);
  }
  const int64_t threads = a->nrows * a->group;
  const unsigned g = (unsigned)((threads + kBlock - 1) / kBlock);
#define SF_CSR(G)                                                                                                 \
  case G:                                                                                                         \
    hipLaunchKernelGGL((k_csr_spmv<G>), dim3(g), dim3(kBlock), 0, st, a->rowptr, a->colidx, a->values, a->nrows, x, \
                       y, accumulate);                                                                            \
    break
  switch (a->group) {
    SF_CSR(1);
    SF_CSR(2);
    SF_CSR(4);
    SF_CSR(8);
    SF_CSR(16);
    SF_CSR(32);
    default: SF_CSR(64);
  }
#undef SF_CSR
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? SF_OK : set_hip_error(e);
}

static void csr_free(sf_csr_s *a) {
  if (a->rowptr) (void)hipFree(a->rowptr);
  if (a->colidx) (void)hipFree(a->colidx);
  if (a->values) (void)hipFree(a->values);
  if (a->gbase) (void)hipFree(a->gbase);
  if (a->starts) (void)hipFree(a->starts);
  if (a->ev) (void)hipEventDestroy(a->ev);
  delete a;
}

// Whether k_csr_rows takes the matrix, and with how many panels (us,
// k_csr_spmv / k_csr_rows):
//  * Enough groups of rows to give every SIMD one and a half (100K rows x 9
//    random entries 8.4 / 7.4, 70K rows 6.6 / 6.9, 10K rows x 24 5.4 / 7.2).
//  * Rows of at most kCsrRowMean entries a panel on average, none far above
//    that: a lane sums its row alone, so a long row holds up its wavefront,
//    the more the fewer wavefronts there are beside it (2% of rows of 98
//    entries among rows of 15: 150K rows 24.1 / 25, 300K 49.7 / 36.8, 1M 189 /
//    111), and its running sums grow beyond the lane tree's error.  Rows of
//    one entry are read coalesced by k_csr_spmv too (1M rows of a diagonal 5.8
//    / 8.2).
//  * One panel while x is at most kCsrOnePanel bytes (500K rows x 15 entries
//    over 4 MB: 46.9 us with one panel or two) or a group's columns lie within
//    a panel's width (a band); else panels of about kCsrPanelBytes that leave
//    a row kCsrPanelMin entries in each (every further panel reads and writes
//    y once more), given wavefronts for them (100K rows x 9 over 24 MB 17.7 /
//    18.8, 300K rows over 8 MB 32.6 / 27.1).  With one panel over a wider x
//    the gathers alone count, and k_csr_spmv has them all in flight where its
//    lanes take an entry each (1M rows x 7 random entries 75.3 / 79.3, of 7 on
//    average 86.3 / 80.7).
constexpr int64_t kCsrMinGroups = 1536;
constexpr int64_t kCsrEvenGroups = 4096;      // below: longest row 2 means + 16, from there 4 means + 32
constexpr int64_t kCsrPanelGroups = 2048;     // several panels only from here
constexpr double kCsrRowMean = 24.0;
constexpr int kCsrRowMost = 128;              // entries of a row in a panel
constexpr int64_t kCsrRowMax = 1000;          // of a row in all panels (a group's starts are 16 bits)
constexpr int64_t kCsrOnePanel = 9 << 19;     // 4.5 MiB; an XCD's L2 is 4 MiB
constexpr int64_t kCsrPanelBytes = 11 << 18;  // 2.75 MiB
constexpr double kCsrPanelMin = 4.0;
constexpr int kCsrPanelMax = 8;

static int csr_panels(const sf_csr_s *a) {
  if (a->nnz == 0 || a->nnz >= INT32_MAX) return 0;
  const int64_t groups = (a->nrows + 63) / 64;
  const double mean = (double)a->nnz / (double)a->nrows;
  int64_t longest = 0;
  for (int64_t i = 0; i < a->nrows; i++) longest = std::max(longest, a->h_rowptr[i + 1] - a->h_rowptr[i]);
  if (groups < kCsrMinGroups || longest <= 1 || longest > kCsrRowMax) return 0;
  if ((double)longest > (groups < kCsrEvenGroups ? 2.0 * mean + 16.0 : 4.0 * mean + 32.0)) return 0;
  int panels = 1;
  const int64_t xb = a->ncols * 8;
  if (xb > kCsrOnePanel) {
    const int64_t want = std::min<int64_t>((xb + kCsrPanelBytes - 1) / kCsrPanelBytes, kCsrPanelMax);
    panels = (int)std::max<int64_t>(1, std::min<int64_t>(want, (int64_t)(mean / kCsrPanelMin)));
    // mean column span of a sample of the groups
    const int64_t step = std::max<int64_t>(1, groups / 256);
    double span = 0.0;
    int64_t sampled = 0;
    for (int64_t g = 0; g < groups; g += step) {
      const int64_t k0 = a->h_rowptr[g * 64], k1 = a->h_rowptr[std::min(a->nrows, g * 64 + 64)];
      if (k0 == k1) continue;
      const auto mm = std::minmax_element(a->h_colidx.begin() + k0, a->h_colidx.begin() + k1);
      span += (double)(*mm.second - *mm.first);
      sampled++;
    }
    const bool band = span * std::max(panels, 2) <= (double)a->ncols * (double)sampled;
    if (band) panels = 1;
    if (!band && panels == 1 && longest <= a->group) return 0;
    if (panels > 1 && groups < kCsrPanelGroups) return 0;
  }
  if (panels == 1 && longest > kCsrRowMost) return 0;  // (several: csr_rows_plan looks at each panel)
  return mean > kCsrRowMean * panels ? 0 : panels;
}

static int csr_rows_plan(sf_csr_s *a) {
  const int panels = csr_panels(a);
  if (panels == 0) return SF_OK;
  const int64_t ngroups = (a->nrows + 63) / 64;
  const size_t gp = (size_t)ngroups * panels;
  uint32_t *gbase = nullptr;  // the word past its end: the most entries of a row in a panel
  uint16_t *starts = nullptr;
  int32_t *pcol = nullptr;
  double *pval = nullptr;
  int longest = 0;
  hipError_t e = hipMalloc(&gbase, (gp + 2) * sizeof(uint32_t));
  if (e == hipSuccess) e = hipMalloc(&starts, gp * 64 * sizeof(uint16_t));
  if (e == hipSuccess && panels > 1) e = hipMalloc(&pcol, (size_t)a->nnz * 4);
  if (e == hipSuccess && panels > 1) e = hipMalloc(&pval, (size_t)a->nnz * 8);
  if (e == hipSuccess) e = hipMemset(gbase + gp + 1, 0, sizeof(uint32_t));
  if (e == hipSuccess) {
    const int pw = (int)((a->ncols + panels - 1) / panels);
    hipLaunchKernelGGL(k_csr_panelize, dim3(group_blocks(ngroups)), dim3(kBlock), 0, nullptr, a->rowptr, a->colidx,
                       a->values, a->nrows, ngroups, panels, pw, gbase, starts, pcol, pval, (int *)(gbase + gp + 1));
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(&longest, gbase + gp + 1, sizeof(int), hipMemcpyDeviceToHost);
    if (e == hipSuccess && panels > 1 && longest <= kCsrRowMost) {
      std::swap(a->colidx, pcol);
      std::swap(a->values, pval);
    }
  }
  if (pcol) (void)hipFree(pcol);
  if (pval) (void)hipFree(pval);
  if (e != hipSuccess || longest > kCsrRowMost) {
    if (gbase) (void)hipFree(gbase);
    if (starts) (void)hipFree(starts);
    if (e == hipSuccess) return SF_OK;  // a row too long for a panel: k_csr_spmv serves the matrix
    if (e != hipErrorOutOfMemory) return set_hip_error(e);
    (void)hipGetLastError();  // no room for the tables: k_csr_spmv serves the matrix
    return SF_OK;
  }
  a->gbase = gbase;
  a->starts = starts;
  a->ngroups = ngroups;
  a->panels = panels;
  a->chains = longest <= 32 ? 4 : longest <= 64 ? 8 : 16;
  return SF_OK;
}

static int csr_upload(sf_csr_s *a) {
  hipError_t e = hipGetDevice(&a->device);
  if (e == hipSuccess) e = hipMalloc(&a->rowptr, (size_t)(a->nrows + 1) * 8);
  if (e == hipSuccess) e = hipMalloc(&a->colidx, (size_t)std::max<int64_t>(a->nnz, 1) * 4);
  if (e == hipSuccess) e = hipMalloc(&a->values, (size_t)std::max<int64_t>(a->nnz, 1) * 8);
  if (e == hipSuccess) e = hipMemcpy(a->rowptr, a->h_rowptr.data(), (size_t)(a->nrows + 1) * 8, hipMemcpyHostToDevice);
  if (e == hipSuccess && a->nnz)
    e = hipMemcpy(a->colidx, a->h_colidx.data(), (size_t)a->nnz * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess && a->nnz)
    e = hipMemcpy(a->values, a->h_values.data(), (size_t)a->nnz * 8, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&a->ev, hipEventDisableTiming);
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? SF_ERR_OOM : set_hip_error(e);
  a->group = pick_group(a->nrows, a->nnz);
  return csr_rows_plan(a);
}

}  // namespace sfi

using namespace sfi;

extern "C" int sf_csr_create(int64_t nrows, int64_t ncols, const int64_t *rowptr, const int32_t *colidx,
                             const double *values, sf_csr_t *out) {
  if (!out) return SF_ERR_ARG;
  *out = nullptr;
  if (nrows < 0 || ncols < 0 || nrows > INT32_MAX || ncols > INT32_MAX || !rowptr) return SF_ERR_ARG;
  if (rowptr[0] != 0) return SF_ERR_ARG;
  for (int64_t i = 0; i < nrows; i++)
    if (rowptr[i + 1] < rowptr[i]) return SF_ERR_ARG;
  const int64_t nnz = rowptr[nrows];
  if (nnz > 0 && (!colidx || !values)) return SF_ERR_ARG;
  for (int64_t k = 0; k < nnz; k++)
    if (colidx[k] < 0 || colidx[k] >= ncols) return SF_ERR_ARG;
  auto *a = new (std::nothrow) sf_csr_s();
  if (!a) return SF_ERR_OOM;
  try {
    a->nrows = nrows;
    a->ncols = ncols;
    a->nnz = nnz;
    a->h_rowptr.assign(rowptr, rowptr + nrows + 1);
    a->h_colidx.assign(colidx, colidx + nnz);
    a->h_values.assign(values, values + nnz);
  } catch (const std::bad_alloc &) {
    delete a;
    return SF_ERR_OOM;
  }
  int rc = csr_upload(a);
  if (rc) {
    csr_free(a);
    return rc;
  }
  *out = a;
  return SF_OK;
}

extern "C" int sf_csr_transpose(sf_csr_t a, sf_csr_t *out) {
  if (!a || !out) return SF_ERR_ARG;
  *out = nullptr;
  // counting sort of the entries by column; inside a column, by row
  std::vector<int64_t> rp((size_t)a->ncols + 1, 0);
  std::vector<int32_t> ci((size_t)a->nnz);
  std::vector<double> va((size_t)a->nnz);
  for (int64_t k = 0; k < a->nnz; k++) rp[(size_t)a->h_colidx[k] + 1]++;
  for (int64_t j = 0; j < a->ncols; j++) rp[j + 1] += rp[j];
  std::vector<int64_t> fill(rp.begin(), rp.end() - 1);
  for (int64_t i = 0; i < a->nrows; i++)
    for (int64_t k = a->h_rowptr[i]; k < a->h_rowptr[i + 1]; k++) {
      const int64_t at = fill[a->h_colidx[k]]++;
      ci[at] = (int32_t)i;
      va[at] = a->h_values[k];
    }
  return sf_csr_create(a->ncols, a->nrows, rp.data(), ci.data(), va.data(), out);
}

extern "C" int sf_csr_spmv(sf_csr_t a, const double *x, double *y, int32_t accumulate, hipStream_t stream) {
  if (!a || (a->nrows > 0 && (!y || (a->ncols > 0 && !x)))) return SF_ERR_ARG;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != a->device) return SF_ERR_ARG;
  return csr_launch(a, x, y, accumulate ? 1 : 0, stream);
}

extern "C" int sf_csr_get_choices(sf_csr_t a, int32_t *panels, int32_t *sums) {
  if (!a || !panels || !sums) return SF_ERR_ARG;
  *panels = a->panels;
  *sums = a->chains;
  return SF_OK;
}

extern "C" int sf_csr_destroy(sf_csr_t *a) {
  if (!a) return SF_ERR_ARG;
  if (*a) csr_free(*a);
  *a = nullptr;
  return SF_OK;
}

extern "C" int sf_spmv(sf_t sf, sf_csr_t A, sf_csr_t B, const double *x, double *lvec, double *y, hipStream_t stream,
                       hipStream_t comm_stream) {
  if (!sf || !A || !B) return SF_ERR_ARG;
  if (A->nrows != B->nrows || A->ncols != sf->nroots || B->ncols != sf->leafspace) return SF_ERR_ARG;
  const sf_unit u{SF_F64, 1};
  // the ghost values travel on comm_stream while the local product runs
  int rc = sf_bcast_begin(sf, u, x, lvec, SF_REPLACE, comm_stream);
  if (rc) return rc;
  hipError_t e = hipEventRecord(A->ev, comm_stream);
  if (e != hipSuccess) return set_hip_error(e);
  rc = sf_csr_spmv(A, x, y, 0, stream);
  if (rc) return rc;
  e = hipStreamWaitEvent(stream, A->ev, 0);
  if (e != hipSuccess) return set_hip_error(e);
  rc = sf_bcast_end(sf, u, x, lvec, SF_REPLACE, comm_stream);
  if (rc) return rc;
  return sf_csr_spmv(B, lvec, y, 1, stream);
}

extern "C" int sf_spmv_transpose(sf_t sf, sf_csr_t At, sf_csr_t Bt, const double *x, double *lvec, double *y,
                                 hipStream_t stream) {
  if (!sf || !At || !Bt) return SF_ERR_ARG;
  if (At->ncols != Bt->ncols || At->nrows != sf->nroots || Bt->nrows != sf->leafspace) return SF_ERR_ARG;
  const sf_unit u{SF_F64, 1};
  int rc = sf_csr_spmv(At, x, y, 0, stream);
  if (!rc) rc = sf_csr_spmv(Bt, x, lvec, 0, stream);
  if (!rc) rc = sf_reduce_begin(sf, u, lvec, y, SF_SUM, stream);
  if (!rc) rc = sf_reduce_end(sf, u, lvec, y, SF_SUM, stream);
  return rc;
}
