// Low-rank covariance: greedy pivoted Cholesky of the covariance on the
// quadrature nodes of a level ladder, and the right-hand sides Wgt_l L_l
// built from its rows.
#include "common.h"

namespace fosb {

struct LrCov {
  int kind;
  double s2, inv2l2, s3l;
};

__device__ __forceinline__ double lr_cov(const LrCov& c, double r2, double ndot) {
  switch (c.kind) {
    case FOSB_COV_GAUSSIAN: return c.s2 * exp(-r2 * c.inv2l2);
    case FOSB_COV_MATERN32: {
      const double a = sqrt(r2) * c.s3l;
      return c.s2 * (1.0 + a) * exp(-a);
    }
    case FOSB_COV_CONSTANT: return c.s2;
    default: return c.s2 * ndot;
  }
}

static LrCov lr_params(const fosb_cov& cov) {
  LrCov c;
  c.kind = cov.kind;
  c.s2 = cov.sigma * cov.sigma;
  c.inv2l2 = cov.ell > 0 ? 1.0 / (2.0 * cov.ell * cov.ell) : 0.0;
  c.s3l = cov.ell > 0 ? std::sqrt(3.0) / cov.ell : 0.0;
  return c;
}

// Candidate normals: Nc[c][off + q] = nrm[c][q / 6] for the Q = 6 nt nodes of one level.
__global__ void k_lr_node_normals(const double* __restrict__ nrm, int nt, int64_t off, int64_t nc,
                                  double* __restrict__ Nc) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= 6LL * nt) return;
  const int t = (int)(q / 6);
  for (int c = 0; c < 3; ++c) Nc[c * nc + off + q] = nrm[(int64_t)c * nt + t];
}

void lr_candidates(hipStream_t s, const Level& l, int64_t off, int64_t nc, double* Xc, double* Nc) {
  const int64_t Q = 6LL * l.mesh->h.nt;
  for (int c = 0; c < 3; ++c)
    FOSB_HIP(hipMemcpyAsync(Xc + c * nc + off, l.qx.as<double>() + c * Q, Q * sizeof(double),
                            hipMemcpyDeviceToDevice, s));
  hipLaunchKernelGGL(k_lr_node_normals, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, s, l.mesh->nrm.as<double>(),
                     (int)l.mesh->h.nt, off, nc, Nc);
  FOSB_LAUNCH_CHECK();
}

__global__ void k_lr_diag(const double* __restrict__ Nc, int64_t nc, LrCov cp, double* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nc) return;
  const double n0 = Nc[i], n1 = Nc[nc + i], n2 = Nc[2 * nc + i];
  d[i] = lr_cov(cp, 0.0, n0 * n0 + n1 * n1 + n2 * n2);
}

void lr_diag(hipStream_t s, const double* Nc, int64_t nc, const fosb_cov& cov, double* d) {
  hipLaunchKernelGGL(k_lr_diag, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s, Nc, nc, lr_params(cov), d);
  FOSB_LAUNCH_CHECK();
}

// The greedy factorisation runs on the device, two launches per column: the
// pivot kernel and the column kernel, ordered by the stream.  The host only
// reads the state once per batch of columns, so no column waits for it.
// pm[b] is the largest d of block b of LR_ROWS consecutive candidates.
constexpr int LR_ROWS = 64;    // candidates per workgroup of the column kernel: one per lane
constexpr int LR_SPLIT = 4;    // wavefronts of a workgroup, each summing a share of the previous columns

__device__ __forceinline__ double wave_max_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

__global__ __launch_bounds__(64) void k_lr_block_max(const double* __restrict__ d, int64_t nc, double* __restrict__ pm) {
  const int64_t i = (int64_t)blockIdx.x * LR_ROWS + threadIdx.x;
  const double m = wave_max_f64(i < nc ? d[i] : -1.0);
  if (threadIdx.x == 0) pm[blockIdx.x] = m;
}

// Pivot of column j: p, the lowest index with d[p] >= (1 - tie) max d.  The
// block maxima give max d and the first block that holds such an index, so one
// workgroup reads nblk + LR_ROWS values instead of scanning d twice (19.5 us a
// column over 40320 candidates before, 6 us now).  Row p of the previous
// columns is gathered into prow for the column kernel.  With j = max_rank, or
// once d[p] falls to tol times the first pivot's value, the state is done and
// the launches that follow it return at once.
__global__ __launch_bounds__(1024) void k_lr_pivot(const double* __restrict__ d, int64_t nc,
                                                   const double* __restrict__ pm, int nblk, double tie, double tol,
                                                   int j, int max_rank, const double* __restrict__ L,
                                                   double* __restrict__ prow, int64_t* __restrict__ piv,
                                                   LrState* __restrict__ st) {
  __shared__ double sm[1024];
  __shared__ int sb[1024];
  __shared__ long long sp;
  if (st->done) return;
  const int tid = threadIdx.x;
  double m = -1.0;
  for (int b = tid; b < nblk; b += 1024) m = fmax(m, pm[b]);
  sm[tid] = m;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (tid < o) sm[tid] = fmax(sm[tid], sm[tid + o]);
    __syncthreads();
  }
  const double thr = (1.0 - tie) * sm[0];
  int best = nblk;
  for (int b = tid; b < nblk; b += 1024)
    if (pm[b] >= thr) {
      best = b;
      break;
    }
  sb[tid] = best;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (tid < o) sb[tid] = min(sb[tid], sb[tid + o]);
    __syncthreads();
  }
  if (tid < 64) {
    const int64_t i = (int64_t)sb[0] * LR_ROWS + tid;
    const bool hit = sb[0] < nblk && i < nc && d[i] >= thr;
    const unsigned long long mask = __ballot(hit);
    const long long p = mask ? (long long)sb[0] * LR_ROWS + __ffsll(mask) - 1 : 0;
    if (tid == 0) {
      const double dp = d[p];
      if (j == 0) st->dmax0 = dp;
      st->last = dp;
      if (j >= max_rank || !(dp > tol * st->dmax0) || !(dp > 0.0)) {
        st->done = 1;
      } else {
        st->rank = j + 1;
        st->p = p;
        st->dp = dp;
        piv[j] = p;
      }
      sp = p;
    }
  }
  __syncthreads();
  const int64_t p = sp;
  for (int k = tid; k < j; k += 1024) prow[k] = L[(int64_t)k * nc + p];
}

// Column j of the factor (column-major, L[k * nc + i]) for the pivot of the state:
//   L[j][i] = (K(x_i, x_p) - sum_{k<j} L[k][i] L[k][p]) / sqrt(dp),  d[i] -= L[j][i]^2,  d[p] = 0.
// Bound by reading the previous columns (8 j nc bytes).  One lane per candidate
// and one serial sum per lane kept too few loads in flight: 104 us a column on
// average at nc = 40320, j up to 775 (1.2 TB/s).  The columns are dealt to four
// wavefronts, each with eight loads in flight, and row p comes from the gathered
// copy through scalar loads; the four partial sums are added in a fixed order.
__global__ __launch_bounds__(LR_ROWS * LR_SPLIT) void k_lr_column(const double* __restrict__ Xc,
                                                                  const double* __restrict__ Nc, int64_t nc, LrCov cp,
                                                                  double* __restrict__ L,
                                                                  const double* __restrict__ prow, int j,
                                                                  double* __restrict__ d, double* __restrict__ pm,
                                                                  const LrState* __restrict__ st) {
  __shared__ double part[LR_SPLIT][LR_ROWS];
  if (st->done) return;
  const int lane = threadIdx.x & 63;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * LR_ROWS + lane;
  const int64_t ir = i < nc ? i : nc - 1;   // lanes past the end read the last candidate and store nothing
  const int share = (j + LR_SPLIT - 1) / LR_SPLIT;
  const int k0 = g * share, k1 = min(j, k0 + share);
  double acc = 0.0;
  int k = k0;
  for (; k + 8 <= k1; k += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = L[(int64_t)(k + u) * nc + ir];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = fma(v[u], prow[k + u], acc);
  }
  for (; k < k1; ++k) acc = fma(L[(int64_t)k * nc + ir], prow[k], acc);
  part[g][lane] = acc;
  __syncthreads();
  if (threadIdx.x >= LR_ROWS) return;
  const int64_t p = st->p;
  const double e0 = Xc[ir] - Xc[p], e1 = Xc[nc + ir] - Xc[nc + p], e2 = Xc[2 * nc + ir] - Xc[2 * nc + p];
  const double nd = Nc[ir] * Nc[p] + Nc[nc + ir] * Nc[nc + p] + Nc[2 * nc + ir] * Nc[2 * nc + p];
  const double c = lr_cov(cp, e0 * e0 + e1 * e1 + e2 * e2, nd) -
                   ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
  const double v = c / sqrt(st->dp);
  double dn = -1.0;
  if (i < nc) {
    L[(int64_t)j * nc + i] = v;
    dn = (i == p) ? 0.0 : d[i] - v * v;
    d[i] = dn;
  }
  const double m = wave_max_f64(dn);
  if (lane == 0) pm[blockIdx.x] = m;
}

// Columns are enqueued in batches of this many between two reads of the state;
// launches past the last column return at once (a few microseconds each).
constexpr int LR_BATCH = 32;

void lr_factor(hipStream_t s, const double* Xc, const double* Nc, int64_t nc, const fosb_cov& cov, double tie,
               double tol, int max_rank, double* L, double* d, LrState& out, std::vector<int64_t>& pivots) {
  const int64_t nblk = (nc + LR_ROWS - 1) / LR_ROWS;
  if (nblk > INT32_MAX) fail(FOSB_E_UNSUPPORTED, "low-rank factor over %lld nodes", (long long)nc);
  DevBuf pm((size_t)nblk * sizeof(double)), prow((size_t)max_rank * sizeof(double));
  DevBuf piv((size_t)max_rank * sizeof(int64_t)), state(sizeof(LrState));
  LrState h{};
  FOSB_HIP(hipMemcpyAsync(state.p, &h, sizeof(h), hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(k_lr_block_max, dim3((unsigned)nblk), dim3(64), 0, s, d, nc, pm.as<double>());
  FOSB_LAUNCH_CHECK();
  for (int j = 0; j <= max_rank; ++j) {   // the pivot of column max_rank only measures the remainder
    hipLaunchKernelGGL(k_lr_pivot, dim3(1), dim3(1024), 0, s, d, nc, pm.as<double>(), (int)nblk, tie, tol, j, max_rank,
                       L, prow.as<double>(), piv.as<int64_t>(), state.as<LrState>());
    FOSB_LAUNCH_CHECK();
    if (j < max_rank) {
      hipLaunchKernelGGL(k_lr_column, dim3((unsigned)nblk), dim3(LR_ROWS * LR_SPLIT), 0, s, Xc, Nc, nc, lr_params(cov),
                         L, prow.as<double>(), j, d, pm.as<double>(), state.as<LrState>());
      FOSB_LAUNCH_CHECK();
    }
    if (j % LR_BATCH == LR_BATCH - 1 || j == max_rank) {
      FOSB_HIP(hipMemcpyAsync(&h, state.p, sizeof(h), hipMemcpyDeviceToHost, s));
      FOSB_HIP(hipStreamSynchronize(s));
      if (h.done) break;
    }
  }
  pivots.resize(h.rank);
  if (h.rank > 0)
    FOSB_HIP(hipMemcpyAsync(pivots.data(), piv.p, (size_t)h.rank * sizeof(int64_t), hipMemcpyDeviceToHost, s));
  FOSB_HIP(hipStreamSynchronize(s));
  out = h;
}

// Row-major copy of rows [off, off + n) of the column-major factor: Lr[i][k] = L[k][off + i].
__global__ __launch_bounds__(256) void k_lr_rows(const double* __restrict__ L, int64_t nc, int64_t off, int64_t n,
                                                 int rank, double* __restrict__ Lr) {
  __shared__ double tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  const int64_t i0 = (int64_t)blockIdx.x * 32, k0 = (int64_t)blockIdx.y * 32;
  for (int r = ty; r < 32; r += 8) {
    const int64_t k = k0 + r, i = i0 + tx;
    tile[r][tx] = (k < rank && i < n) ? L[k * nc + off + i] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = i0 + r, k = k0 + tx;
    if (i < n && k < rank) Lr[i * rank + k] = tile[tx][r];
  }
}

// M[m][k] = sum over the 12 nodes q of RWG m of Wgt[m][q] Lr[q][k] (M: N x rank,
// row-major; Wgt: [nt][3][6] weights of one incidence; Lr: the level's rows of the factor).
__global__ __launch_bounds__(256) void k_lr_rhs(const int32_t* __restrict__ edge_tri, const int32_t* __restrict__ edge_loc,
                                                int ne, const c128* __restrict__ W, const double* __restrict__ Lr,
                                                int rank, c128* __restrict__ M) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)ne * rank) return;
  const int64_t m = id / rank;
  const int k = (int)(id % rank);
  double ar = 0, ai = 0;
  for (int side = 0; side < 2; ++side) {
    const int t = edge_tri[side * ne + m];
    const int a = edge_loc[side * ne + m];
    for (int q = 0; q < 6; ++q) {
      const c128 w = W[((int64_t)t * 3 + a) * 6 + q];
      const double v = Lr[(6LL * t + q) * rank + k];
      ar += w.re * v;
      ai += w.im * v;
    }
  }
  M[m * rank + k] = c128{ar, ai};
}

// Lc (n x rank, complex128) = Lr (real)
__global__ void k_real_to_c128(const double* __restrict__ a, int64_t n, c128* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = c128{a[i], 0.0};
}

void lr_rows(hipStream_t s, const Level& l, const double* L, int64_t nc, int64_t off, int rank, double* Lr) {
  const int64_t Q = 6LL * l.mesh->h.nt;
  dim3 g((unsigned)((Q + 31) / 32), (unsigned)((rank + 31) / 32));
  hipLaunchKernelGGL(k_lr_rows, g, dim3(256), 0, s, L, nc, off, Q, rank, Lr);
  FOSB_LAUNCH_CHECK();
}

void real_to_c128(hipStream_t s, const double* a, int64_t n, c128* b) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_real_to_c128, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, n, b);
  FOSB_LAUNCH_CHECK();
}

void lr_rhs(hipStream_t s, const Level& l, int64_t dir, const double* L, int64_t nc, int64_t off, int rank,
            double* Lr, c128* M) {
  const Mesh& m = *l.mesh;
  const int64_t Q = 6LL * m.h.nt;
  dim3 g((unsigned)((Q + 31) / 32), (unsigned)((rank + 31) / 32));
  hipLaunchKernelGGL(k_lr_rows, g, dim3(256), 0, s, L, nc, off, Q, rank, Lr);
  FOSB_LAUNCH_CHECK();
  const int64_t total = (int64_t)m.h.ne * rank;
  hipLaunchKernelGGL(k_lr_rhs, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, m.edge_tri.as<int32_t>(),
                     m.edge_loc.as<int32_t>(), (int)m.h.ne, l.W.as<c128>() + dir * m.h.nt * 18, (const double*)Lr,
                     rank, M);
  FOSB_LAUNCH_CHECK();
}

}  // namespace fosb
