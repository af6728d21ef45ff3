// Standalone float64 residual of the all-at-once system,
// ||G - A(U)||_F / ||G||_F (Algorithm 3, the residual test on U_1; here the
// accuracy report of a solve and the stopping test of refinement).
#include "pd_internal.h"
#include "pd_residual.h"
#include "pd_scan.h"

#include <cmath>
#include <mutex>

namespace {

constexpr int RB = 256;

// What bounds these kernels is memory, F and U once each (2D: U twice, its
// second reading at the next time step).  A wave owns 62 consecutive columns
// (two more lanes carry the neighbours) and walks down rows -- time rows in
// 1D, grid rows of one time step in 2D -- so that the stencil's other values
// are registers: the column's neighbours come by lane moves (DPP), the row
// above from the walk.  A point costs 2 (2D: 3) loads; with a thread per point
// it was 15 (14), and load instructions bounded the pass: n = 8191, ell =
// 2048 at 201 us, 255^2, ell = 512 at 270 us; now 51 to 64 us (303 MB, 4.7 TB/s at
// best) and 141 us, 65 and 204 us where the residual is written as float too.
constexpr int RCOLS = 62, RUN = 8;

// lane l's value from lane l - 1 / l + 1 (zero at the ends)
__device__ __forceinline__ double from_left(double v) { return pd_dpp<0x138, 0xF>(v, 0.0); }
__device__ __forceinline__ double from_right(double v) { return pd_dpp<0x130, 0xF>(v, 0.0); }

// Block sums of the three squared norms into red[3 * blockIdx.x ..].
__device__ __forceinline__ void put_norms(double rn, double gn, double un,
                                          double *__restrict__ red) {
  __shared__ double sr[RB / 64], sg[RB / 64], su[RB / 64];
  for (int off = 32; off > 0; off >>= 1) {
    rn += __shfl_down(rn, off, 64);
    gn += __shfl_down(gn, off, 64);
    un += __shfl_down(un, off, 64);
  }
  const int wid = threadIdx.x / 64, lane = threadIdx.x % 64;
  if (lane == 0) { sr[wid] = rn; sg[wid] = gn; su[wid] = un; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0, c = 0.0;
    for (int w = 0; w < RB / 64; ++w) { a += sr[w]; b += sg[w]; c += su[w]; }
    red[3 * blockIdx.x] = a;
    red[3 * blockIdx.x + 1] = b;
    red[3 * blockIdx.x + 2] = c;
  }
}

// 1D, rows [t0, t0 + rows) of a wave's columns; un: ||M U||^2 (Algorithm 3
// measures the residual against it).  STORE: the residual times dal (null: 1)
// as float, row t in the second half of the t/2-th complex128 row of a
// half spectrum (the complex64 spectrum it is transformed into fills the
// first halves).
template <bool STORE>
__global__ void __launch_bounds__(RB)
residual1d_kernel(int n, int ell, int groups, int rows, int items, double tau,
                  const double *__restrict__ u0, const double *__restrict__ F, const double *__restrict__ U,
                  const double *__restrict__ coef, const double *__restrict__ dal,
                  float *__restrict__ out, double *__restrict__ red) {
  const int lane = threadIdx.x & 63;
  double rn = 0.0, gn = 0.0, un = 0.0;
  for (int w = blockIdx.x * (RB / 64) + (threadIdx.x >> 6); w < items;
       w += gridDim.x * (RB / 64)) {
    const int chunk = w / groups, i = (w - chunk * groups) * RCOLS + lane - 1;
    const int t0 = chunk * rows, t1 = t0 + rows < ell ? t0 + rows : ell;
    const bool in = i >= 0 && i < n, mine = in && lane >= 1 && lane <= RCOLS;
    const int ic = i < 0 ? 0 : (i < n ? i : n - 1);
    const double ML = ic > 0 ? coef[ic] : 0.0, MD = coef[n + ic],
                 MU = ic < n - 1 ? coef[2 * n + ic] : 0.0;
    const double KL = ic > 0 ? coef[3 * n + ic] : 0.0, KD = coef[4 * n + ic],
                 KU = ic < n - 1 ? coef[5 * n + ic] : 0.0;
    double prev = t0 > 0 ? U[(size_t)(t0 - 1) * n + ic] : 0.0;
    for (int tb = t0; tb < t1; tb += RUN) {
      double f[RUN], u[RUN];
#pragma unroll
      for (int q = 0; q < RUN; ++q) {
        const size_t at = (size_t)(tb + q < t1 ? tb + q : t1 - 1) * n + ic;
        f[q] = F[at];
        u[q] = U[at];
      }
#pragma unroll
      for (int q = 0; q < RUN; ++q) {
        const int t = tb + q;
        if (t < t1) {
          double h = tau * f[q];
          if (t == 0) h += u0[ic];
          double z = h - u[q];
          if (t > 0) z += prev;
          prev = u[q];
          double g = MD * h;
          double r = MD * z - KD * u[q];
          double m = MD * u[q];
          const double hl = from_left(h), hr = from_right(h);
          const double zl = from_left(z), zr = from_right(z);
          const double ul = from_left(u[q]), ur = from_right(u[q]);
          g += ML * hl;
          r += ML * zl - KL * ul;
          m += ML * ul;
          g += MU * hr;
          r += MU * zr - KU * ur;
          m += MU * ur;
          if (mine) {
            rn += r * r;
            gn += g * g;
            un += m * m;
            if constexpr (STORE) {
              const double v = dal ? r * dal[t] : r;
              out[(size_t)(t >> 1) * 4 * n + 2 * n + (size_t)(t & 1) * n + i] = (float)v;
            }
          }
        }
      }
    }
  }
  put_norms(rn, gn, un, red);
}

// 2D (M = I), grid rows [y0, y0 + rows) of one time step; STORE: the residual
// as float64 [ell][n*n].
template <bool STORE>
__global__ void __launch_bounds__(RB)
residual2d_kernel(int n, int groups, int chunks, int rows, int items, double tau,
                  const double *__restrict__ u0, const double *__restrict__ F,
                  const double *__restrict__ U, const double *__restrict__ coef, Stencil2 sk,
                  double *__restrict__ out, double *__restrict__ red) {
  const int lane = threadIdx.x & 63;
  double rn = 0.0, gn = 0.0, un = 0.0;
  for (int w = blockIdx.x * (RB / 64) + (threadIdx.x >> 6); w < items;
       w += gridDim.x * (RB / 64)) {
    const int wy = w / groups, x = (w - wy * groups) * RCOLS + lane - 1;
    const int t = wy / chunks, y0 = (wy - t * chunks) * rows;
    const int y1 = y0 + rows < n ? y0 + rows : n;
    const bool in = x >= 0 && x < n, mine = in && lane >= 1 && lane <= RCOLS;
    const int xc = x < 0 ? 0 : (x < n ? x : n - 1);
    const size_t nbar = (size_t)n * n;
    const double *Ft = F + (size_t)t * nbar + xc, *Ut = U + (size_t)t * nbar + xc;
    const double *Up = t > 0 ? Ut - nbar : Ut;
    const double *KL = coef + 3 * (size_t)n, *KD = KL + n, *KU = KD + n;
    const double kdx = sk.uni ? sk.kd : KD[xc];
    const double klx = xc > 0 ? (sk.uni ? sk.kl : KL[xc]) : 0.0;
    const double kux = xc < n - 1 ? (sk.uni ? sk.ku : KU[xc]) : 0.0;
    double above = y0 > 0 ? Ut[(size_t)(y0 - 1) * n] : 0.0;
    double cur = Ut[(size_t)y0 * n];
    constexpr int RU2 = 4;
    for (int yb = y0; yb < y1; yb += RU2) {
      double f[RU2], un1[RU2], up[RU2];
#pragma unroll
      for (int q = 0; q < RU2; ++q) {
        const int y = yb + q < y1 ? yb + q : y1 - 1;
        f[q] = Ft[(size_t)y * n];
        un1[q] = Ut[(size_t)(y + 1 < n ? y + 1 : n - 1) * n];
        up[q] = Up[(size_t)y * n];
      }
#pragma unroll
      for (int q = 0; q < RU2; ++q) {
        const int y = yb + q;
        if (y < y1) {
          double h = tau * f[q];
          if (t == 0) h += u0[(size_t)y * n + xc];
          double z = h - cur;
          if (t > 0) z += up[q];
          const double kdy = sk.uni ? sk.kd : KD[y];
          double ku = (kdx + kdy) * cur;
          ku += klx * from_left(cur);
          ku += kux * from_right(cur);
          if (y > 0) ku += (sk.uni ? sk.kl : KL[y]) * above;
          if (y < n - 1) ku += (sk.uni ? sk.ku : KU[y]) * un1[q];
          const double r = z - ku;
          if (mine) {
            rn += r * r;
            gn += h * h;
            un += cur * cur;
            if constexpr (STORE) out[(size_t)t * nbar + (size_t)y * n + x] = r;
          }
          above = cur;
          cur = un1[q];
        }
      }
    }
  }
  put_norms(rn, gn, un, red);
}

// A wave's item is a walk over 32 rows (its first row above is read twice);
// past PD_RES_MAX_BLOCKS blocks of partial norms the waves take more items.
constexpr int PD_RES_MAX_BLOCKS = 8192;
struct ResLaunch {
  int groups, chunks, rows, items, blocks;
};
ResLaunch res_config(pd_plan p) {
  ResLaunch L;
  L.groups = (p->n + RCOLS - 1) / RCOLS;
  const int len = p->dims == 2 ? p->n : p->ell;
  L.rows = 32;
  L.chunks = (len + L.rows - 1) / L.rows;
  L.items = (p->dims == 2 ? p->ell : 1) * L.groups * L.chunks;
  const int want = (L.items + RB / 64 - 1) / (RB / 64);
  L.blocks = want < PD_RES_MAX_BLOCKS ? want : PD_RES_MAX_BLOCKS;
  return L;
}

// The residual pass into red (three partial norms per block) and, if asked
// for, the residual itself: 1D as float into a spectrum's second halves, 2D
// as float64 into the work array.
pd_status launch_residual(pd_plan p, const double *u0, const double *F, const double *U,
                          void *out, double *red) {
  const ResLaunch L = res_config(p);
  if (p->dims == 1) {
    const double *dal = p->alpha == 1.0 ? nullptr : p->dal;
    if (out)
      hipLaunchKernelGGL((residual1d_kernel<true>), dim3(L.blocks), dim3(RB), 0, p->stream, p->n,
                         p->ell, L.groups, L.rows, L.items, p->tau, u0, F, U, p->coef64, dal,
                         static_cast<float *>(out), red);
    else
      hipLaunchKernelGGL((residual1d_kernel<false>), dim3(L.blocks), dim3(RB), 0, p->stream, p->n,
                         p->ell, L.groups, L.rows, L.items, p->tau, u0, F, U, p->coef64, dal,
                         static_cast<float *>(nullptr), red);
  } else {
    const Stencil2 sk{p->uniform ? 1 : 0, p->uni[3], p->uni[4], p->uni[5]};
    if (out)
      hipLaunchKernelGGL((residual2d_kernel<true>), dim3(L.blocks), dim3(RB), 0, p->stream, p->n,
                         L.groups, L.chunks, L.rows, L.items, p->tau, u0, F, U, p->coef64, sk,
                         static_cast<double *>(out), red);
    else
      hipLaunchKernelGGL((residual2d_kernel<false>), dim3(L.blocks), dim3(RB), 0, p->stream, p->n,
                         L.groups, L.chunks, L.rows, L.items, p->tau, u0, F, U, p->coef64, sk,
                         static_cast<double *>(nullptr), red);
  }
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

// Sum the 3 * nb partial norms in a fixed order (each thread a strided run,
// then a fixed tree in LDS) into tot[0..2].
__global__ void __launch_bounds__(RB) sum_partials_kernel(int nb, const double *__restrict__ red,
                                                          double *__restrict__ tot) {
  __shared__ double s[3][RB];
  double a = 0.0, b = 0.0, c = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < nb; i += RB) {
    a += red[3 * i];
    b += red[3 * i + 1];
    c += red[3 * i + 2];
  }
  s[0][threadIdx.x] = a;
  s[1][threadIdx.x] = b;
  s[2][threadIdx.x] = c;
  __syncthreads();
  for (int w = RB / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int q = 0; q < 3; ++q) s[q][threadIdx.x] += s[q][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 3) tot[threadIdx.x] = s[threadIdx.x][0];
}

constexpr int PD_NORM_SLOT = 5;   // of the plan's pinned status block (8 doubles)

}  // namespace

int pd_residual_blocks(pd_plan p) { return res_config(p).blocks; }

// Enqueues the residual pass and its norms' totals (into the pinned status
// block; read with pd_residual_read after a synchronisation).
pd_status pd_residual_enqueue(pd_plan p, const double *u0, const double *F, const double *U,
                              void *out) {
  const pd_status st = launch_residual(p, u0, F, U, out, p->red);
  if (st != PD_OK) return st;
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(RB), 0, p->stream, pd_residual_blocks(p),
                     p->red, p->host_dev + PD_NORM_SLOT);
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

pd_status pd_residual_read(pd_plan p, double *rn2, double *gn2, double *un2) {
  const volatile double *h = p->host_pin + PD_NORM_SLOT;
  const double a = h[0], b = h[1], c = h[2];
  if (!std::isfinite(a) || !std::isfinite(b) || !std::isfinite(c)) {
    pd_set_error("non-finite residual norm");
    return PD_ENONFINITE;
  }
  *rn2 = a;
  *gn2 = b;
  *un2 = c;
  return PD_OK;
}

// Sum the 2*nblk partial norms left in p->red by a residual pass.
pd_status pd_sum_norms(pd_plan p, int nblk, double *rn2, double *gn2) {
  std::vector<double> h(2 * (size_t)nblk);
  PD_HIP_CHECK(hipMemcpyAsync(h.data(), p->red, h.size() * sizeof(double),
                              hipMemcpyDeviceToHost, p->stream));
  PD_HIP_CHECK(hipStreamSynchronize(p->stream));
  double a = 0.0, b = 0.0;
  for (int i = 0; i < nblk; ++i) { a += h[2 * i]; b += h[2 * i + 1]; }
  *rn2 = a;
  *gn2 = b;
  return PD_OK;
}

pd_status pd_residual_norms(pd_plan p, const double *u0, const double *F, const double *U,
                            double *rn2, double *gn2, double *un2) {
  const pd_status st = pd_residual_enqueue(p, u0, F, U, nullptr);
  if (st != PD_OK) return st;
  PD_HIP_CHECK(hipStreamSynchronize(p->stream));
  return pd_residual_read(p, rn2, gn2, un2);
}

// ---------------------------------------------------------------------------
// The allocation-free residual (paradiag_residual_noalloc): the per-block
// partial norms live in a file-scope device array instead of the plan's
// reduction buffer, and the totals are summed on the device into the plan's
// pinned status block (a copy of them took 8 us more: n = 63, 2D, 36 -> 27 us a
// call), so the call allocates nothing on the device or the host.  Every call on a
// GPU shares that GPU's copy of the array; calls that overlap on one GPU race.
// ---------------------------------------------------------------------------
constexpr int PD_NOALLOC_MAX_BLOCKS = 8192;
constexpr size_t PD_NOALLOC_SCRATCH_DOUBLES = 3 * (size_t)PD_NOALLOC_MAX_BLOCKS;
static __device__ __align__(256) double scratch[PD_NOALLOC_SCRATCH_DOUBLES];

namespace {

std::mutex g_scratch_mu;
constexpr int PD_MAX_DEVICES = 64;
double *g_scratch_ptr[PD_MAX_DEVICES] = {};

// Device address of this GPU's copy of `scratch`, looked up once per device
// with that device current (in host code the array's name is not a device
// address).
pd_status scratch_address(int device, double **out) {
  if (device < 0 || device >= PD_MAX_DEVICES) {
    pd_set_error("device index out of range for the scratch table");
    return PD_EINVAL;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    int cur = 0;
    PD_HIP_CHECK(hipGetDevice(&cur));
    if (cur != device) PD_HIP_CHECK(hipSetDevice(device));
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !ptr) {
      pd_set_error(std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
      return PD_EHIP;
    }
    g_scratch_ptr[device] = static_cast<double *>(ptr);
  }
  *out = g_scratch_ptr[device];
  return PD_OK;
}

}  // namespace

extern "C" pd_status paradiag_residual_noalloc(pd_plan p, const double *u0, const double *F,
                                               const double *U, double *rel) {
  if (!p || !rel || !u0 || !F || !U) {
    pd_set_error("invalid residual arguments");
    return PD_EINVAL;
  }
  if (p->bdf_s > 1) {
    pd_set_error("paradiag_residual_noalloc: backward-Euler plans only (bdf_order 1)");
    return PD_ENOTSUP;
  }
  const int nb = pd_residual_blocks(p);
  if (nb > PD_NOALLOC_MAX_BLOCKS) {
    pd_set_error("paradiag_residual_noalloc: the residual pass needs " + std::to_string(nb) +
                 " partial-norm blocks, above the static scratch's " +
                 std::to_string(PD_NOALLOC_MAX_BLOCKS));
    return PD_ENOTSUP;
  }
  double *red = nullptr;
  pd_status st = scratch_address(p->device, &red);
  if (st != PD_OK) return st;
  // every block writes its three partial norms, so nothing needs clearing
  st = launch_residual(p, u0, F, U, nullptr, red);
  if (st != PD_OK) return st;
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(RB), 0, p->stream, nb, red,
                     p->host_dev + PD_NORM_SLOT);
  PD_HIP_CHECK(hipGetLastError());
  PD_HIP_CHECK(hipStreamSynchronize(p->stream));
  const volatile double *h = p->host_pin + PD_NORM_SLOT;
  const double a = h[0], b = h[1];
  if (!std::isfinite(a) || !std::isfinite(b)) {
    pd_set_error("non-finite residual norm");
    return PD_ENONFINITE;
  }
  *rel = (b > 0.0) ? std::sqrt(a / b) : std::sqrt(a);
  return PD_OK;
}

pd_status pd_residual_impl(pd_plan p, const double *u0, const double *F, const double *U,
                           double *rel, double *est) {
  double a, b, c;
  pd_status st = pd_residual_norms(p, u0, F, U, &a, &b, &c);
  if (st != PD_OK) return st;
  *rel = (b > 0.0) ? std::sqrt(a / b) : std::sqrt(a);
  if (est) *est = (p->err_factor > 0.0 && c > 0.0) ? p->err_factor * std::sqrt(a / c) : -1.0;
  return PD_OK;
}
