// The capacitance system J x = b (eq. SMW_linearsystemII; eq. innersystem_alpha
// for alpha < 1; eq. linearsystem_s for BDF-s) in the sine eigenbasis, for
// plans whose M and tau K are symmetric Toeplitz tridiagonals (uniform grids;
// 2D: in the DST-x domain of the line solves, along y).
//
// The sine vectors s_j diagonalise every P_k^{-1} M, hence J: with
// a_j = 1 + tau kappa_j / m_j,
//
//     J s_j = (1 + D_j) s_j,   D_j = alpha / (a_j^ell - alpha),
//
// and D_j falls below the rounding of 1 after a few modes (a_j^ell grows like
// exp(T kappa_j / m_j)).  So J = I + S diag(D) S^T with S the r modes whose
// D_j exceeds 2^-56, and GMRES started from b never leaves the space spanned
// by b's part outside span(S) and the r modes.  In the coordinates
// (c, rho), c = S^T b and rho = ||b - S c||, which are orthonormal, J is
// diag(1 + D_1, .., 1 + D_r, 1): GMRES on r + 1 numbers gives the iterates,
// residuals and iteration counts of GMRES on J itself.  BDF-s has s blocks
// of r coordinates and an s x s matrix per mode (I + C_j^ell (I - C_j^ell)^-1
// up to similarity, C_j the mode's companion matrix).
//
// D is not taken from the closed form but summed over the frequencies from the
// eigenvalues of the matrices P_k as the passes' tables round them, so that J
// stays consistent with pass B and C (sc_phi_kernel).
//
// Three launches, whatever the iteration count: project (sums pass B's
// partials into b and projects each 64-column block on the modes), norm
// (c, and each block's share of rho^2), solve (every block runs the small
// GMRES on its own copy in LDS -- cheaper than a launch and a round trip --
// and forms its columns of x = t b' + S x_c, b' = b - S c, t = x_rho / rho).
// What bounds them is latency: the tables are at most 192 rows of n doubles
// and b is read three times.  n = 8191, ell = 2048 (with the sum of pass B's
// partials, 5 us of it): 6.5 + 4.9 + 9.7 us, where J products, Arnoldi steps and
// the combination took 87; n = 4095, alpha = 0.01: 7.0 + 6.6 + 15.6, before 150;
// n <= 256 in one launch, n = 63 11.7 us.  Sums run in a fixed order and the batched
// launches use the same bodies, so results are the same alone and in a batch.
#include "pd_dd.h"
#include "pd_internal.h"
#include "pd_small.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int SC_DMAX = 192;     // s r: reduced coordinates without rho
constexpr int SC_S = 6;          // BDF orders
constexpr int SC_ONE = 4;        // column blocks of the one-launch form
// its dynamic LDS limit: 66.7 KiB of static LDS beside it, of 160 KiB
constexpr size_t SC_ONE_LDS = 80 * 1024;
constexpr double SC_CUT = 0x1p-56;

// ---- project: b (summed from pass B's partials, as reduce_fused_kernel) and
// cpart[blk][h r + j] = sum over the block's 64 columns of S[j][i] b_h[i] ----
constexpr int SCP_T = 1024, SCP_RS = 16, SCP_SLICES = 64;
constexpr int SCP_LDS = (SCP_SLICES + SC_S) * 64;   // doubles
__device__ __forceinline__ void sc_project_body(const ScJob &J, int blk, double *lds) {
  double (*sl)[64] = reinterpret_cast<double (*)[64]>(lds);
  double (*bs)[64] = sl + SCP_SLICES;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = J.n, i = blk * 64 + lane;
  const int ic = i < n ? i : n - 1;
  if (J.partials) {   // s = 1
    const int slices = (J.G + SCP_RS - 1) / SCP_RS;
    for (int q = w; q < slices; q += SCP_T / 64) {
      const int g0 = q * SCP_RS, g1 = g0 + SCP_RS < J.G ? g0 + SCP_RS : J.G;
      double v[SCP_RS];
#pragma unroll
      for (int u = 0; u < SCP_RS; ++u)
        v[u] = J.partials[(size_t)(g0 + u < g1 ? g0 + u : g1 - 1) * n + ic];
      double t = 0.0;
#pragma unroll
      for (int u = 0; u < SCP_RS; ++u)
        if (g0 + u < g1) t += v[u];
      sl[q][lane] = t;
    }
    __syncthreads();
    if (w == 0) {
      double t = 0.0;
      for (int q = 0; q < slices; ++q) t += sl[q][lane];
      if (i < n) J.b[i] = t;
      bs[0][lane] = i < n ? t : 0.0;
    }
  } else {
    for (int h = w; h < J.s; h += SCP_T / 64)
      bs[h][lane] = i < n ? J.bin[(size_t)h * n + ic] : 0.0;
  }
  __syncthreads();
  const int d = J.s * J.r;
  for (int e = w; e < d; e += SCP_T / 64) {
    const int h = e / J.r, j = e - h * J.r;
    const double v = pd_wave_sum(J.S[(size_t)j * J.ns + i] * bs[h][lane]);
    if (lane == 0) J.cpart[(size_t)blk * d + e] = v;
  }
}

// c[e] = sum over the blocks of cpart (fixed order), in LDS, by the block's
// first NT threads: dp (a power of two) >= d threads per group, the groups'
// sums added in order.
template <int NT>
__device__ __forceinline__ void sc_sum_c(const ScJob &J, const double *cpart, double *grp,
                                         double *c) {
  const int d = J.s * J.r;
  int dp = 1;
  while (dp < d) dp <<= 1;
  const int ng = NT / dp < 16 ? NT / dp : 16;   // the last sum is serial
  const int e = threadIdx.x & (dp - 1), g = threadIdx.x / dp;
  double t = 0.0;
  if (e < d && g < ng) {
#pragma unroll 8
    for (int b = g; b < J.nblk; b += ng) t += cpart[(size_t)b * d + e];
  }
  if (threadIdx.x < NT) grp[threadIdx.x] = t;
  __syncthreads();
  if (threadIdx.x < d) {
    double v = 0.0;
    for (int q = 0; q < ng; ++q) v += grp[q * dp + threadIdx.x];
    c[threadIdx.x] = v;
  }
  __syncthreads();
}

// (S y_h)[i] for the block's 64 columns, y in LDS [s][r]: the block's waves
// share the modes and wave h adds the parts in order (returned there; other
// waves return 0).  NW waves; part holds NW * s * 64 doubles.
template <int NW>
__device__ __forceinline__ double sc_expand(const ScJob &J, int blk, const double *y,
                                            double *part) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double *Sc = J.S + (size_t)blk * 64 + lane;
  double acc[SC_S] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int j = w; j < J.r; j += NW) {
    const double sv = Sc[(size_t)j * J.ns];
#pragma unroll
    for (int h = 0; h < SC_S; ++h)
      if (h < J.s) acc[h] += sv * y[h * J.r + j];
  }
#pragma unroll
  for (int h = 0; h < SC_S; ++h)
    if (h < J.s) part[(w * J.s + h) * 64 + lane] = acc[h];
  __syncthreads();
  double t = 0.0;
  if (w < J.s)
    for (int q = 0; q < NW; ++q) t += part[(q * J.s + w) * 64 + lane];
  return t;
}

// ---- norm: c, b' = b - S c (left in x), the block's share of rho^2 =
// ||b'||^2, and b' projected again.  b is up to max D times larger than x, so
// b' keeps a part in span(S) of rounding size relative to b; the second
// projection takes it out ("twice is enough") before x is formed from b' ----
constexpr int SCN_LDS = SCP_T + 256 + SCP_T * SC_S + 8;   // doubles
__device__ __forceinline__ void sc_norm_body(const ScJob &J, int blk, double *lds) {
  double *grp = lds, *c = grp + SCP_T, *part = c + 256, *rs = part + SCP_T * SC_S;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  sc_sum_c<SCP_T>(J, J.cpart, grp, c);
  if (blk == 0 && threadIdx.x < J.s * J.r) J.c[threadIdx.x] = c[threadIdx.x];
  const double t = sc_expand<SCP_T / 64>(J, blk, c, part);
  const int i = blk * 64 + lane;
  if (w < J.s) {
    const double *b = J.partials ? J.b : J.bin;
    double v = i < J.n ? b[(size_t)w * J.n + i] - t : 0.0;
    if (i < J.n) J.x[(size_t)w * J.n + i] = v;
    grp[w * 64 + lane] = v;
    v = pd_wave_sum(v * v);
    if (lane == 0) rs[w] = v;
  }
  __syncthreads();
  const int d = J.s * J.r;
  for (int e = w; e < d; e += SCP_T / 64) {
    const int h = e / J.r, j = e - h * J.r;
    const double v = pd_wave_sum(J.S[(size_t)j * J.ns + i] * grp[h * 64 + lane]);
    if (lane == 0) J.cpart2[(size_t)blk * d + e] = v;
  }
  if (threadIdx.x == 0) {
    double v = 0.0;
    for (int h = 0; h < J.s; ++h) v += rs[h];
    J.rpart[blk] = v;
  }
}

// ---- solve: GMRES on the d + 1 reduced coordinates, x = t b + S (x_c - t c) ----
constexpr int SCS_T = 256, SCS_W = SCS_T / 64;
__host__ __device__ inline size_t sc_solve_lds(int d, int MX) {   // doubles
  return (size_t)(MX + 1) * (d + 1) + (size_t)MX * (MX + 1) / 2 + MX;
}
// y = x_c - t c' (c' = S^T b') into ys[0 .. d), t into ys[d] (LDS), so that
// x = t b' + S y; the block's first SCS_W waves work, any further ones only keep the barriers.  record: write status.
__device__ __forceinline__ void sc_gmres(const ScJob &J, int MX, double rtol, double *ys,
                                         bool record, double *__restrict__ st_out,
                                         bool with_flag) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double c[256], ws[256], hs[64], yv[64];
  __shared__ double wsum[SCS_W];
  __shared__ double res_s, hn_s;
  __shared__ int done_s;
  const int d = J.s * J.r, dim = d + 1;
  double *V = reinterpret_cast<double *>(smem_raw);   // [MX + 1][dim]
  double *H = V + (size_t)(MX + 1) * dim;             // column j at j (j + 1) / 2
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int h0 = tid / J.r, m0 = tid - h0 * J.r;      // block and mode of coordinate tid < d
  // the coordinates of b
  double phi[SC_S];   // this coordinate's row of J - I
#pragma unroll
  for (int h = 0; h < SC_S; ++h)
    phi[h] = (h < J.s && tid < d) ? J.Phi[(size_t)(h0 * J.s + h) * J.r + m0] : 0.0;
  double v = 0.0;
  if (wv == 0) {
    double t = 0.0;
    for (int b = lane; b < J.nblk; b += 64) t += J.rpart[b];
    t = pd_wave_sum(t);
    if (lane == 0) c[d] = sqrt(t);
  }
  sc_sum_c<SCS_T>(J, J.cpart2, ws, ys);
  const double c2 = tid < d ? ys[tid] : 0.0;
  if (tid < d) c[tid] = J.c[tid] + c2;
  __syncthreads();
  if (tid < dim) v = c[tid];
  auto block_sum = [&](double x) {   // same order in every thread
    x = pd_wave_sum(x);
    if (lane == 0 && wv < SCS_W) wsum[wv] = x;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < SCS_W; ++q) t += wsum[q];
    __syncthreads();
    return t;
  };
  const double rho = c[d];
  const double beta = sqrt(block_sum(v * v));
  // wave 0's lanes: the rotations, the rotated right-hand side; g: its last entry
  double cs = 0.0, sn = 0.0, gl = 0.0, g = beta;
  if (tid == 0) {
    res_s = hn_s = beta;
    done_s = (beta == 0.0 || !isfinite(beta)) ? 1 : 0;
  }
  if (tid < dim) V[tid] = beta > 0.0 ? v * (1.0 / beta) : 0.0;
  __syncthreads();
  int m = 0;
  while (m < MX && !done_s) {
    const int j = m, nv = j + 1;
    const double *vj = V + (size_t)j * dim;
    double wr = 0.0;
    if (tid < dim) {
      wr = vj[tid];
      if (tid < d) {
#pragma unroll
        for (int h = 0; h < SC_S; ++h)
          if (h < J.s) wr += phi[h] * vj[h * J.r + m0];
      }
      ws[tid] = wr;
    }
    double hacc = 0.0;
    for (int pass = 0; pass < 2; ++pass) {   // classical Gram-Schmidt, twice
      __syncthreads();
      if (wv < SCS_W)
        for (int i = wv; i < nv; i += SCS_W) {
          double t = 0.0;
          for (int e = lane; e < dim; e += 64) t += V[(size_t)i * dim + e] * ws[e];
          t = pd_wave_sum(t);
          if (lane == 0) hs[i] = t;
        }
      __syncthreads();
      if (tid < nv) hacc += hs[tid];
      if (tid < dim) {
        for (int i = 0; i < nv; ++i) wr -= hs[i] * V[(size_t)i * dim + tid];
        ws[tid] = wr;
      }
    }
    const double hn = sqrt(block_sum(tid < dim ? wr * wr : 0.0));
    if (wv == 0) {
      double gr;
      pd_givens_column(hacc, hn, j, lane, cs, sn, gr, g);
      gl = lane == j ? gr : gl;
      if (lane < nv) H[(size_t)j * (j + 1) / 2 + lane] = hacc;
      if (lane == 0) {
        const double res = fabs(g);
        res_s = res;
        // dim vectors span the space: the solution is in it, and what is left of
        // hn is rounding that no further vector lowers
        hn_s = nv < dim ? hn : 0.0;
        done_s = (res <= rtol * beta || hn_s == 0.0 || !isfinite(res)) ? 1 : 0;
      }
    }
    if (tid < dim) V[(size_t)(j + 1) * dim + tid] = hn > 0.0 ? wr * (1.0 / hn) : 0.0;
    m = j + 1;
    __syncthreads();
  }
  // R y = g, then the reduced solution
  if (wv == 0) {
    const double yl = pd_back_substitute(gl, m, lane, [&](int k) {
      return lane <= k ? H[(size_t)k * (k + 1) / 2 + lane] : 0.0;
    });
    if (lane < m) yv[lane] = yl;
  }
  if (tid == 0) {
    if (record) {
      st_out[0] = res_s;
      st_out[1] = hn_s;
      st_out[2] = (double)m;
      st_out[3] = beta;
      if (with_flag) st_out[4] = done_s ? 1.0 : 0.0;
    }
  }
  __syncthreads();
  double xr = 0.0;
  if (tid < dim)
    for (int i = 0; i < m; ++i) xr += yv[i] * V[(size_t)i * dim + tid];
  if (tid == d) ys[d] = rho > 0.0 ? xr / rho : (m > 0 ? 1.0 : 0.0);
  __syncthreads();
  if (tid < d) ys[tid] = xr - ys[d] * c2;
  __syncthreads();
}

// The block's columns of x = t b' + S y (ys as sc_gmres leaves it, b' in x).
constexpr int SCC_LDS = SCS_T * SC_S;   // doubles
__device__ __forceinline__ void sc_columns(const ScJob &J, int blk, const double *ys,
                                           double *part) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, i = blk * 64 + lane;
  const double tb = ys[J.s * J.r];
  if (wv < SCS_W) {
    const double *Sc = J.S + i;
    double acc[SC_S] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int j = wv; j < J.r; j += SCS_W) {
      const double sv = Sc[(size_t)j * J.ns];
#pragma unroll
      for (int h = 0; h < SC_S; ++h)
        if (h < J.s) acc[h] += sv * ys[h * J.r + j];
    }
#pragma unroll
    for (int h = 0; h < SC_S; ++h)
      if (h < J.s) part[(wv * J.s + h) * 64 + lane] = acc[h];
  }
  __syncthreads();
  if (wv < SCS_W)
    for (int h = wv; h < J.s; h += SCS_W) {
      double t = 0.0;
      for (int q = 0; q < SCS_W; ++q) t += part[(q * J.s + h) * 64 + lane];
      if (i < J.n) J.x[(size_t)h * J.n + i] = tb * J.x[(size_t)h * J.n + i] + t;
    }
}

// ---- product J v = v + S (J - I) S^T v after a projection of v ----
__device__ __forceinline__ void sc_apply_body(const ScJob &J, int blk, double *lds) {
  double *grp = lds, *c = grp + SCP_T, *part = c + 256;
  __shared__ double y[256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  sc_sum_c<SCP_T>(J, J.cpart, grp, c);
  if (threadIdx.x < J.s * J.r) {
    const int k = threadIdx.x / J.r, j = threadIdx.x - k * J.r;
    double t = 0.0;
    for (int h = 0; h < J.s; ++h) t += J.Phi[(size_t)(k * J.s + h) * J.r + j] * c[h * J.r + j];
    y[threadIdx.x] = t;
  }
  __syncthreads();
  const double t = sc_expand<SCP_T / 64>(J, blk, y, part);
  const int i = blk * 64 + lane;
  if (w < J.s && i < J.n) J.x[(size_t)w * J.n + i] = J.bin[(size_t)w * J.n + i] + t;
}

__global__ void __launch_bounds__(SCP_T) sc_project_kernel(const ScJob J) {
  __shared__ double lds[SCP_LDS];
  sc_project_body(J, blockIdx.x, lds);
}
__global__ void __launch_bounds__(SCP_T) sc_norm_kernel(const ScJob J) {
  __shared__ double lds[SCN_LDS];
  sc_norm_body(J, blockIdx.x, lds);
}
__global__ void __launch_bounds__(SCS_T)
sc_solve_kernel(const ScJob J, int MX, double rtol, double *__restrict__ host) {
  __shared__ double ys[256], lds[SCC_LDS];
  sc_gmres(J, MX, rtol, ys, blockIdx.x == 0, host, true);
  sc_columns(J, blockIdx.x, ys, lds);
}
// n <= 256 (SC_ONE column blocks): all three steps in one block.  Every step
// works on the same column blocks in the same order, so results are those of
// the three launches.
__global__ void __launch_bounds__(SCP_T)
sc_one_kernel(const ScJob J, int MX, double rtol, double *__restrict__ host) {
  __shared__ double ys[256], lds[SCN_LDS];
  for (int b = 0; b < J.nblk; ++b) {
    sc_project_body(J, b, lds);
    __syncthreads();
  }
  for (int b = 0; b < J.nblk; ++b) {
    sc_norm_body(J, b, lds);
    __syncthreads();
  }
  sc_gmres(J, MX, rtol, ys, true, host, true);
  for (int b = 0; b < J.nblk; ++b) {
    sc_columns(J, b, ys, lds);
    __syncthreads();
  }
}
__global__ void __launch_bounds__(SCP_T) sc_apply_kernel(const ScJob J) {
  __shared__ double lds[SCN_LDS];
  sc_apply_body(J, blockIdx.x, lds);
}
__global__ void __launch_bounds__(SCP_T)
sc_project_batch_kernel(const ScJob *__restrict__ jobs, const int2 *__restrict__ map) {
  const int2 e = map[blockIdx.x];
  __shared__ double lds[SCP_LDS];
  sc_project_body(jobs[e.x], e.y, lds);
}
__global__ void __launch_bounds__(SCP_T)
sc_norm_batch_kernel(const ScJob *__restrict__ jobs, const int2 *__restrict__ map) {
  const int2 e = map[blockIdx.x];
  __shared__ double lds[SCN_LDS];
  sc_norm_body(jobs[e.x], e.y, lds);
}
__global__ void __launch_bounds__(SCS_T)
sc_gmres_batch_kernel(const ScJob *__restrict__ jobs, int MX, double rtol,
                      double *__restrict__ status) {
  __shared__ double ys[256];
  const ScJob &J = jobs[blockIdx.x];
  sc_gmres(J, MX, rtol, ys, true, status + 4 * blockIdx.x, false);
  if (threadIdx.x <= J.s * J.r) J.y[threadIdx.x] = ys[threadIdx.x];
}
__global__ void __launch_bounds__(SCS_T)
sc_columns_batch_kernel(const ScJob *__restrict__ jobs, const int2 *__restrict__ map) {
  __shared__ double ys[256], lds[SCC_LDS];
  const int2 e = map[blockIdx.x];
  const ScJob &J = jobs[e.x];
  if (threadIdx.x <= J.s * J.r) ys[threadIdx.x] = J.y[threadIdx.x];
  __syncthreads();
  sc_columns(J, e.y, ys, lds);
}

// ---- 2D: the lines along y of the DST-x domain, vectors [y][m] ----
//
// D(m, j) depends on kappa_m + kappa_j and is symmetric, so the modes are a
// q x q square (m, j < q; entries below the cut hold D = 0).  The coordinates
// c[j][m] = sum_y s_j(y) b[y][m], the norm of b - S c and x = t b + S y are
// contractions on the matrix cores (v_mfma_f64_16x16x4f64: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; D row l / 16 + 4 r, column l % 16
// sits in result r); GMRES on the q^2 + 1 coordinates is one block
// (pd_gmres_diag).  Before, every iteration was a parfor over all (k, m) lines
// and five vector launches.
typedef double v4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4d sc_mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One 16 x 16 tile of c per block, y split over the 4 waves.
// Grid: (ceil(q / 16), ceil(q / 16)).
__global__ void __launch_bounds__(256)
sc2_project_kernel(int n, int ns, int q, const double *__restrict__ S,
                   const double *__restrict__ b, double *__restrict__ c) {
  __shared__ v4d red[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m = blockIdx.x * 16 + (lane & 15), j0 = blockIdx.y * 16;
  const int mc = m < n ? m : n - 1;
  const double *Sr = S + (size_t)(j0 + (lane & 15)) * ns;   // rows past q are zero
  v4d acc = {0.0, 0.0, 0.0, 0.0};
  const int steps = ns / 4;
  constexpr int U = 8;
  for (int t0 = wv; t0 < steps; t0 += 4 * U) {
    double av[U], bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + 4 * u, y = 4 * (t < steps ? t : wv) + (lane >> 4);
      av[u] = t < steps ? Sr[y] : 0.0;                      // zero past n
      bv[u] = b[(size_t)(y < n ? y : n - 1) * n + mc];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc = sc_mfma(av[u], bv[u], acc);
  }
  red[wv][lane] = acc;
  __syncthreads();
  if (wv == 0 && m < q) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = j0 + (lane >> 4) + 4 * r;
      double t = red[0][lane][r];
      for (int w = 1; w < 4; ++w) t += red[w][lane][r];
      if (j < q) c[(size_t)j * q + m] = t;
    }
  }
}

// 16 rows y x 64 columns m per block, one 16 x 16 tile of S^T coef per wave.
// MODE 0: b' = b - S c into x and rpart[block] = sum of b'^2; MODE 1:
// x = t b' + S y (b = x = the b' of MODE 0, entry by entry), t = y[q^2].
// Grid: (ceil(n / 64), ceil(n / 16)).
template <int MODE>
__global__ void __launch_bounds__(256)
sc2_tile_kernel(int n, int ns, int q, const double *__restrict__ S,
                const double *b, const double *__restrict__ coef, double *x,
                double *__restrict__ rpart) {
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int y0 = blockIdx.y * 16, m = blockIdx.x * 64 + wv * 16 + (lane & 15);
  double bv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int y = y0 + (lane >> 4) + 4 * r;
    bv[r] = (y < n && m < n) ? b[(size_t)y * n + m] : 0.0;
  }
  v4d acc = {0.0, 0.0, 0.0, 0.0};
  if (blockIdx.x * 64 + wv * 16 < q) {
    const double *Sr = S + y0 + (lane & 15);
    const int steps = (q + 3) / 4;
    constexpr int U = 8;
    for (int t0 = 0; t0 < steps; t0 += U) {
      double av[U], cv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = 4 * (t0 + u) + (lane >> 4);
        const bool in = j < q && m < q;
        av[u] = Sr[(size_t)(j < q ? j : 0) * ns];
        cv[u] = in ? coef[(size_t)j * q + m] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) acc = sc_mfma(av[u], cv[u], acc);
    }
  }
  if constexpr (MODE == 0) {
    double t = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int y = y0 + (lane >> 4) + 4 * r;
      const double v = (y < n && m < n) ? bv[r] - acc[r] : 0.0;
      if (y < n && m < n) x[(size_t)y * n + m] = v;
      t += v * v;
    }
    t = pd_wave_sum(t);
    if (lane == 0) red[wv] = t;
    __syncthreads();
    if (threadIdx.x == 0)
      rpart[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
  } else {
    const double tb = coef[(size_t)q * q];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int y = y0 + (lane >> 4) + 4 * r;
      if (y < n && m < n) x[(size_t)y * n + m] = tb * bv[r] + acc[r];
    }
  }
}

// ---- tables, once per plan ----

// Orthonormal sine vectors j = 1..r in rows of ns entries, zero past n, and zero
// rows past r.  Grid: (ns / 64, ceil(rows / 4)).
__global__ void __launch_bounds__(256)
sc_rows_kernel(int n, int r, int rows, int ns, double *__restrict__ S) {
  const int i = blockIdx.x * 64 + (threadIdx.x & 63), j = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (j >= rows) return;
  const int N = n + 1, q = (int)((long)(j + 1) * (i + 1) % (2 * N));
  int a = q > N ? 2 * N - q : q;          // folded into [0, pi / 2]
  if (2 * a > N) a = N - a;
  const double v = sqrt(2.0 / N) * sinpi((double)a / (double)N);
  S[(size_t)j * ns + i] = (j < r && i < n) ? (q > N ? -v : v) : 0.0;
}

// Off-diagonal and diagonal entries of M and tau K, and their eigenvalues on the
// mode with sin^2(theta / 2) = s2: (d + 2 o) - 4 o s2.
struct SymmetricPair {
  double m[2], k[2];
};
__device__ __forceinline__ pd_dd sc_eigenvalue(const double (&o)[2], pd_dd s2) {
  return dd_add(dd_two_sum(o[1], 2.0 * o[0]), dd_mul(pd_dd{-4.0 * o[0], 0.0}, s2));
}
// The same of the symmetric complex matrix (o, d)
__device__ __forceinline__ pd_ddc sc_eigenvalue(cpx<double> o, cpx<double> d, pd_dd s2) {
  return pd_ddc{sc_eigenvalue({o.re, d.re}, s2), sc_eigenvalue({o.im, d.im}, s2)};
}

// Phi (J - I on the modes) sums terms of size up to D over the frequencies, and
// an error in it is one of x, which the solution multiplies by D again: in plain
// double, from the recurrence form's rounded constants, the error of U at D = 30
// was up to 7 times the J product's (n = 511, 64 steps, BDF3, nu = 0.003: 6.5e-14
// against 9.3e-15, now 1.5e-14; over 340 problems of D <= 1000 the two forms' errors
// now differ by 0.99 in the mean, 1.6 at most).  The sums are double-double, a block
// each; s2: sin^2(theta_j / 2), [r] high parts, then [r] low parts.
// P_k's entries are rounded as the passes' tables round them (pd_uniform_factors):
// near theta = 0 that rounding changes its eigenvalues most.
// BDF: weight gamma^(k) theta^(h), g [s][F2], theta from tw.  Grid: (r, s s).
__global__ void __launch_bounds__(256)
sc_phi_kernel(int F2, int r, int s, SymmetricPair u, const double *__restrict__ lam,
              const cpx<double> *__restrict__ g, const cpx<double> *__restrict__ tw, int ell,
              const double *__restrict__ s2s, double *__restrict__ Phi) {
  const int j = blockIdx.x, b = blockIdx.y / s, h = blockIdx.y - b * s;
  const pd_dd s2 = {s2s[j], s2s[r + j]};
  const pd_ddc m = {sc_eigenvalue(u.m, s2), pd_dd{0.0, 0.0}};
  pd_dd t = {0.0, 0.0};
  for (int k = threadIdx.x; k < F2; k += 256) {
    cpx<double> P[2];
    for (int i = 0; i < 2; ++i) {
      const double v = lam[2 * k] * u.m[i];   // rounded before the sum
      P[i] = cpx<double>{v + u.k[i], lam[2 * k + 1] * u.m[i]};
    }
    const pd_ddc z = dd_cdiv(m, sc_eigenvalue(P[0], P[1], s2));   // P_k^{-1} M on the mode
    pd_ddc w = dd_cplx(g[(size_t)b * F2 + k]);
    if (s > 1) w = dd_cmul(w, dd_cplx(tw[(k * h) & (ell - 1)]));
    t = dd_add(t, dd_cmul(w, z).re);
  }
  t = dd_block_sum(t);
  if (threadIdx.x == 0) Phi[(size_t)blockIdx.y * r + j] = t.h;
}

// The same in 2D (M = I): Phi[j][m] = D(m, j), th[m] the eigenvalue of line m as
// pd_line2d_factors rounds it.  Grid: (q, q).
__global__ void __launch_bounds__(64)
sc2_phi_kernel(int F2, int q, double off, double diag, const double *__restrict__ th,
               const double *__restrict__ lam, const cpx<double> *__restrict__ g,
               const double *__restrict__ s2s, double *__restrict__ Phi) {
  const int m = blockIdx.x, j = blockIdx.y;
  const pd_dd s2 = {s2s[j], s2s[q + j]};
  pd_dd t = {0.0, 0.0};
  for (int k = threadIdx.x; k < F2; k += 64) {
    const cpx<double> d = {lam[2 * k] + th[m] + diag, lam[2 * k + 1]};
    const pd_ddc z = dd_cdiv(dd_cplx({1.0, 0.0}), sc_eigenvalue({off, 0.0}, d, s2));
    t = dd_add(t, dd_cmul(dd_cplx(g[k]), z).re);
  }
  t = dd_block_sum(t);
  if (threadIdx.x == 0) Phi[(size_t)j * q + m] = t.h;
}

// ---- host: eigenvalues, the number of modes, tables ----

// sin^2(pi j / (2 (n + 1))) and the eigenvalues of M and tau K on mode j
// (1-based), without the cancellation of d + 2 o cos at smooth modes.
struct Mode {
  double s2, m, kap;
};
Mode mode_of(pd_plan p, int j) {
  const double *u = p->uni;
  const double s = std::sin(M_PI * (double)j / (2.0 * (p->n + 1)));
  Mode o;
  o.s2 = s * s;
  o.m = (u[1] + 2.0 * u[0]) - 4.0 * u[0] * o.s2;
  o.kap = (u[4] + 2.0 * u[3]) - 4.0 * u[3] * o.s2;
  return o;
}

// sin^2(theta_j / 2), j = 1..r: high parts, then low parts.
void mode_s2(int n, int r, std::vector<double> &out) {
  out.resize(2 * (size_t)r);
  const long double pi = 3.14159265358979323846264338327950288L;
  for (int j = 1; j <= r; ++j) {
    const long double s = std::sin(pi * j / (2.0L * (n + 1))), v = s * s;
    out[j - 1] = (double)v;
    out[r + j - 1] = (double)(v - (long double)out[j - 1]);
  }
}

// J - I on a mode with ratio z = tau kappa / m (BDF: tau beta kappa / m).
// decay falls with z and says which modes are kept; size is the largest entry
// of alpha C^ell (I - alpha C^ell)^-1, C the step's companion matrix (its powers
// by repeated squaring), infinite when the mode's block is (nearly) singular
// or not finite.
struct ModeSize {
  double decay = HUGE_VAL, size = HUGE_VAL;
};
ModeSize mode_size(pd_plan p, double z) {
  const int s = p->bdf_s;
  ModeSize o;
  if (!std::isfinite(z) || 1.0 + z == 0.0) return o;
  double C[SC_S][SC_S] = {}, T[SC_S][SC_S];
  for (int i = 0; i < s; ++i) C[0][i] = p->bdf_alpha[i] / (1.0 + z);
  for (int i = 1; i < s; ++i) C[i][i - 1] = 1.0;
  double big = 0.0;
  for (int l = 1; l < p->ell; l <<= 1) {
    big = 0.0;
    for (int i = 0; i < s; ++i)
      for (int k = 0; k < s; ++k) {
        double t = 0.0;
        for (int q = 0; q < s; ++q) t += C[i][q] * C[q][k];
        T[i][k] = t;
        big = std::max(big, std::fabs(t));
      }
    for (int i = 0; i < s; ++i)
      for (int k = 0; k < s; ++k) C[i][k] = T[i][k];
  }
  if (!std::isfinite(big)) return o;
  if (s == 1) {
    const double e = p->alpha * C[0][0];
    o.decay = o.size = e == 1.0 ? HUGE_VAL : std::fabs(e / (1.0 - e));
    return o;
  }
  o.decay = s * big;
  // X (I - C) = C: elimination on the columns, with pivoting (BDF has alpha 1)
  double A[SC_S][2 * SC_S];   // row k: column k of I - C, then column k of C
  for (int k = 0; k < s; ++k)
    for (int i = 0; i < s; ++i) {
      A[k][i] = (i == k ? 1.0 : 0.0) - C[i][k];
      A[k][s + i] = C[i][k];
    }
  for (int q = 0; q < s; ++q) {
    int b = q;
    for (int k = q + 1; k < s; ++k)
      if (std::fabs(A[k][q]) > std::fabs(A[b][q])) b = k;
    if (!(std::fabs(A[b][q]) > 0x1p-50 * (1.0 + big))) return o;
    for (int i = 0; i < 2 * s; ++i) std::swap(A[q][i], A[b][i]);
    for (int k = 0; k < s; ++k) {
      if (k == q) continue;
      const double f = A[k][q] / A[q][q];
      for (int i = q; i < 2 * s; ++i) A[k][i] -= f * A[q][i];
    }
  }
  o.size = 0.0;
  for (int k = 0; k < s; ++k)
    for (int i = 0; i < s; ++i) o.size = std::max(o.size, std::fabs(A[k][s + i] / A[k][k]));
  return o;
}

}  // namespace

// Columns of the mode table, padded to the 64-column blocks.
static int sc_stride(int n) { return (n + 63) / 64 * 64; }

// Doubles of the tables and workspace at r modes (1D).
static size_t sc_doubles(int n, int s, int r) {
  const size_t nblk = (size_t)sc_stride(n) / 64;
  return (size_t)r * sc_stride(n) + (size_t)s * s * r + 2 * nblk * s * r + nblk + 512;
}

size_t pd_sc_max_doubles(int n, int s) {
  return sc_doubles(n, s, std::min(n, SC_DMAX / s));
}

size_t pd_sc_size(pd_plan p) { return sc_doubles(p->n, p->bdf_s, p->sc_r); }

// Whether the plan's capacitance system is solved in the sine basis, and with
// how many modes (nothing changed if not: see below).
bool pd_sc_choose(pd_plan p) {
  const double *u = p->uni;
  const int n = p->n, s = p->bdf_s;
  // float64 GMRES plans on uniform 1D grids with symmetric M and K
  if (p->dims != 1 || p->prec != PD_FP64 || p->krylov != PD_KRYLOV_GMRES || p->sine ||
      p->autotune || !p->uniform || u[0] != u[2] || u[3] != u[5])
    return false;
  const bool scan = pd_use_scan(p);
  // m and kappa are linear in sin^2(theta / 2), so kappa / m is monotone where
  // m has one sign: for the usual signs it grows and D falls with j
  const Mode q1 = mode_of(p, 1), qn = mode_of(p, n);
  const double e1 = p->lam[0] * q1.m + q1.kap, en = p->lam[0] * qn.m + qn.kap;
  if (!(q1.m > 0.0 && qn.m > 0.0 && e1 > 0.0 && en > 0.0) || !(qn.kap / qn.m >= q1.kap / q1.m))
    return false;
  int r = 0;
  double worst = 0.0;
  for (int j = 1; j <= n; ++j) {
    const Mode q = mode_of(p, j);
    const ModeSize D = mode_size(p, q.kap / q.m);
    if (!(D.size < 1e15)) return false;
    if (D.decay <= SC_CUT) break;
    worst = std::max(worst, D.size);
    r = j;
    // more modes than the reduced system holds: the general product
    if (r * s > SC_DMAX) return false;
  }
  if (r < 1) r = 1;
  // The passes apply a rounded factorisation of every P_k, and J has to apply
  // the same.  The recurrence form's scans carry powers of the rounded matrix's
  // own root, so its eigenvalues are right over many rows.  The partition form's
  // elimination is off by cond(P_0) u, which must not show.  Backward Euler's b
  // comes from a pass of its own, whose rounding is that large anyway (errors at
  // n <= 256, limit 1e-12, as with the product).  BDF's b is taken from U_1, and a
  // consistent J corrects U_1's rounding with it: at a limit of 1e-12 errors were
  // up to 135 times the product's (n = 63, 32 steps, order 3, nu = 0.01: 4.8e-13,
  // 3.5e-15).
  const double cond0 = std::max(e1, en) / std::min(e1, en);
  if (!scan && !(worst * cond0 * 0x1p-53 <= (s == 1 ? 1e-12 : 1e-14))) return false;
  const int ns = sc_stride(n), nblk = ns / 64;
  p->sc_r = r;
  p->sc_ns = ns;
  p->sc_nblk = nblk;
  return true;
}

// S and Phi on the device, after the tables they are made from are in place;
// s2: host end of a copy, valid until the plan's stream is synchronised.
pd_status pd_sc_finish(pd_plan p, std::vector<double> &s2) {
  const int n = p->n, r = p->sc_r, s = p->bdf_s;
  mode_s2(n, r, s2);
  double *d = static_cast<double *>(p->spec);   // 2 r <= 2 n entries, not yet in use
  PD_HIP_CHECK(hipMemcpyAsync(d, s2.data(), s2.size() * sizeof(double), hipMemcpyHostToDevice,
                              p->stream));
  hipLaunchKernelGGL(sc_rows_kernel, dim3(p->sc_ns / 64, (r + 3) / 4), dim3(256), 0, p->stream, n,
                     r, r, p->sc_ns, p->sc_tab);
  SymmetricPair u;
  for (int i = 0; i < 2; ++i) {
    u.m[i] = p->uni[i];
    u.k[i] = p->uni[3 + i];
  }
  hipLaunchKernelGGL(sc_phi_kernel, dim3(r, s * s), dim3(256), 0, p->stream, p->F2, r, s, u,
                     p->lam64,
                     reinterpret_cast<const cpx<double> *>(s == 1 ? p->gJ64 : p->bdf_g),
                     reinterpret_cast<const cpx<double> *>(p->tw64), p->ell, d,
                     p->sc_tab + (size_t)r * p->sc_ns);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

// 2D: the sine modes along y of the lines m < q, q^2 + 1 coordinates for the
// one-block GMRES.
//
// The one-block iteration takes its^2 q^2 / (one CU's rate), the launches of the
// general one (J products over all lines and vectors of n^2) hardly less at n = 50
// than at 130.  Solves of 26 to 31 iterations, general / one-block, ms: n = q = 80
// 2.53 / 2.15, 90 2.67 / 2.47, 100 2.77 / 2.96, 120 3.01 / 4.14; n = 120, q = 97 2.98 /
// 2.78; n = 140, q = 103 3.69 / 3.23, q = 122 3.68 / 4.28; n = 160, q = 112 2.96 / 2.71.
// Where J - I is small the iterations are few (5 at 0.01, 14 at 5) and the one-block
// form wins at any q: n = q = 100, 4 steps, alpha = 0.01: 0.37 / 0.24.
constexpr int SC2_QMAX = 127;    // q^2 + 1 <= 16384 entries
static int sc2_limit(int n, double size) { return n < 200 && size > 8.0 ? 96 : SC2_QMAX; }
static int sc2_rows(int q) { return (q + 15) / 16 * 16; }
static int sc2_tiles(int n) { return ((n + 63) / 64) * ((n + 15) / 16); }
static size_t sc2_doubles(int n, int q) {
  const size_t q2 = (size_t)q * q;
  return (size_t)sc2_rows(q) * sc_stride(n) + 4 * (q2 + 2) + 3 * (size_t)q + sc2_tiles(n);
}
size_t pd_sc2_max_doubles(int n) { return sc2_doubles(n, std::min(n, SC2_QMAX)); }

bool pd_sc2_choose(pd_plan p) {
  const double *u = p->uni;
  const int n = p->n;
  // float64 GMRES plans of backward Euler with symmetric T
  if (p->dims != 2 || p->prec != PD_FP64 || p->krylov != PD_KRYLOV_GMRES || p->bdf_s > 1 ||
      !p->uniform || u[3] != u[5])
    return false;
  const Mode q1 = mode_of(p, 1), qn = mode_of(p, n);
  if (!(qn.kap >= q1.kap) || !(p->lam[0] + 2.0 * q1.kap > 0.0)) return false;
  int q = 0;
  double worst = 0.0;
  for (int j = 1; j <= n; ++j) {
    const double D = mode_size(p, q1.kap + mode_of(p, j).kap).size;
    if (!(D < 1e15)) return false;
    if (D <= SC_CUT) break;
    worst = std::max(worst, D);
    q = j;
    if (q > sc2_limit(n, worst)) return false;   // more modes: the general product
  }
  if (q < 1) q = 1;
  // partition-form lines (more than a wave each): as in 1D
  const double cond0 = (p->lam[0] + 2.0 * qn.kap) / (p->lam[0] + 2.0 * q1.kap);
  if (!pd_line2d_scan(p) && !(worst * cond0 * 0x1p-53 <= 1e-12)) return false;
  p->sc_r = q;
  p->sc_ns = sc_stride(n);
  return true;
}
size_t pd_sc2_size(pd_plan p) { return sc2_doubles(p->n, p->sc_r); }

namespace {
struct Sc2 {
  double *S, *s2, *th, *Phi, *c, *c2, *y, *rpart;
  explicit Sc2(pd_plan p) {
    const size_t q = p->sc_r, q2 = q * q + 2;
    S = p->sc_tab;
    s2 = S + (size_t)sc2_rows(p->sc_r) * p->sc_ns;
    th = s2 + 2 * q;
    Phi = th + q;
    c = Phi + q2;
    c2 = c + q2;
    y = c2 + q2;
    rpart = y + q2;
  }
};
}  // namespace

pd_status pd_sc2_finish(pd_plan p, std::vector<double> &tab) {
  const Sc2 t(p);
  const int n = p->n, q = p->sc_r, rows = sc2_rows(q);
  mode_s2(n, q, tab);
  for (int m = 0; m < q; ++m) tab.push_back(pd_line2d_theta(p, m));
  PD_HIP_CHECK(hipMemcpyAsync(t.s2, tab.data(), tab.size() * sizeof(double),
                              hipMemcpyHostToDevice, p->stream));
  hipLaunchKernelGGL(sc_rows_kernel, dim3(p->sc_ns / 64, rows / 4), dim3(256), 0, p->stream, n, q,
                     rows, p->sc_ns, t.S);
  hipLaunchKernelGGL(sc2_phi_kernel, dim3(q, q), dim3(64), 0, p->stream, p->F2, q, p->uni[3],
                     p->uni[4], t.th, p->lam64, reinterpret_cast<const cpx<double> *>(p->gJ64),
                     t.s2, t.Phi);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

static pd_status sc2_enqueue(pd_plan p, const double *b, double *x, double rtol) {
  const Sc2 t(p);
  const int n = p->n, ns = p->sc_ns, q = p->sc_r, qt = (q + 15) / 16;
  const dim3 tiles((n + 63) / 64, (n + 15) / 16);
  hipLaunchKernelGGL(sc2_project_kernel, dim3(qt, qt), dim3(256), 0, p->stream, n, ns, q, t.S, b,
                     t.c);
  hipLaunchKernelGGL((sc2_tile_kernel<0>), tiles, dim3(256), 0, p->stream, n, ns, q, t.S, b, t.c,
                     x, t.rpart);
  hipLaunchKernelGGL(sc2_project_kernel, dim3(qt, qt), dim3(256), 0, p->stream, n, ns, q, t.S, x,
                     t.c2);
  PD_HIP_CHECK(hipGetLastError());
  const pd_status st = pd_gmres_diag(p, q * q, t.c, t.c2, t.Phi, t.rpart, sc2_tiles(n), t.y, rtol);
  if (st != PD_OK) return st;
  hipLaunchKernelGGL((sc2_tile_kernel<1>), tiles, dim3(256), 0, p->stream, n, ns, q, t.S, x, t.y,
                     x, t.rpart);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

// The launches' job: b from pass B's partials (bin null) or from bin.
ScJob pd_sc_job(pd_plan p, const double *bin, double *x) {
  const int s = p->bdf_s, r = p->sc_r;
  ScJob J;
  J.n = p->n;
  J.ns = p->sc_ns;
  J.s = s;
  J.r = r;
  J.nblk = p->sc_nblk;
  const int nitems = pd_tri_nitems(p->tri, p->F2);
  J.G = nitems < p->tri_G ? nitems : p->tri_G;
  J.partials = bin ? nullptr : p->partials;
  J.bin = bin;
  J.b = p->bvec;
  J.x = x;
  double *t = p->sc_tab;
  J.S = t;
  t += (size_t)r * J.ns;
  J.Phi = t;
  t += (size_t)s * s * r;
  J.cpart = t;
  t += (size_t)J.nblk * s * r;
  J.cpart2 = t;
  t += (size_t)J.nblk * s * r;
  J.rpart = t;
  t += J.nblk;
  J.c = t;
  J.y = t + 256;
  return J;
}

size_t pd_sc_lds(const ScJob &J, int MX) { return sc_solve_lds(J.s * J.r, MX) * sizeof(double); }

// x = J^{-1} b to residual <= rtol ||b||, enqueued without synchronising;
// the status lands in the plan's pinned block (read with pd_gmres_read).
pd_status pd_sc_enqueue(pd_plan p, const double *bin, double *x, double rtol) {
  if (p->dims == 2) {
    if (!bin) {
      const pd_status st = pd_launch_reduce_partials(p, nullptr, p->bvec);
      if (st != PD_OK) return st;
    }
    return sc2_enqueue(p, bin ? bin : p->bvec, x, rtol);
  }
  const ScJob J = pd_sc_job(p, bin, x);
  if (J.nblk <= SC_ONE && pd_sc_lds(J, p->maxit) <= SC_ONE_LDS) {
    hipLaunchKernelGGL(sc_one_kernel, dim3(1), dim3(SCP_T), pd_sc_lds(J, p->maxit), p->stream, J,
                       p->maxit, rtol, p->host_dev);
    PD_HIP_CHECK(hipGetLastError());
    return PD_OK;
  }
  hipLaunchKernelGGL(sc_project_kernel, dim3(J.nblk), dim3(SCP_T), 0, p->stream, J);
  hipLaunchKernelGGL(sc_norm_kernel, dim3(J.nblk), dim3(SCP_T), 0, p->stream, J);
  hipLaunchKernelGGL(sc_solve_kernel, dim3(J.nblk), dim3(SCS_T), pd_sc_lds(J, p->maxit),
                     p->stream, J, p->maxit, rtol, p->host_dev);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

pd_status pd_sc_apply(pd_plan p, const double *v, double *Jv) {
  const ScJob J = pd_sc_job(p, v, Jv);
  hipLaunchKernelGGL(sc_project_kernel, dim3(J.nblk), dim3(SCP_T), 0, p->stream, J);
  hipLaunchKernelGGL(sc_apply_kernel, dim3(J.nblk), dim3(SCP_T), 0, p->stream, J);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

// One GMRES block per problem and a launch of its own for the columns of x:
// with many problems the redundant copies would fill the card (96 problems
// of up to 4095 columns: 222 us in the fused form; now 72 + 38 + 56 + 11, the
// lockstep GMRES before it 3400).
pd_status pd_sc_batch(const ScJob *jobs, int count, const int2 *map, int nblocks, size_t lds,
                      int MX, double rtol, double *status, hipStream_t s) {
  hipLaunchKernelGGL(sc_project_batch_kernel, dim3(nblocks), dim3(SCP_T), 0, s, jobs, map);
  hipLaunchKernelGGL(sc_norm_batch_kernel, dim3(nblocks), dim3(SCP_T), 0, s, jobs, map);
  hipLaunchKernelGGL(sc_gmres_batch_kernel, dim3(count), dim3(SCS_T), lds, s, jobs, MX, rtol,
                     status);
  hipLaunchKernelGGL(sc_columns_batch_kernel, dim3(nblocks), dim3(SCS_T), 0, s, jobs, map);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

void pd_sc_set_attributes(size_t max_lds) {
  pd_set_max_lds(reinterpret_cast<const void *>(&sc_solve_kernel), (int)max_lds);
  pd_set_max_lds(reinterpret_cast<const void *>(&sc_one_kernel), (int)max_lds);
  pd_set_max_lds(reinterpret_cast<const void *>(&sc_gmres_batch_kernel), (int)max_lds);
}
