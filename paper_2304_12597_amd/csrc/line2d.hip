// 2D shifted solves by separation (Section 6.1, 2D heat equation with
// K = I (x) T + T (x) I): after an orthonormal DST-I along x, the shifted
// block P_k = lambda_k I + tau K splits, for every x-sine-mode m with
// T s_m = theta_m s_m, into one tridiagonal system along y,
//
//     ((lambda_k + tau theta_m) I + tau T) y = d,
//
// so the parfor over k becomes a parfor over (k, m) of n-row line solves.
// Spectra here are [ell/2+1][n*n] in the DST-x domain, index y*n + m.  A block
// owns S consecutive m for a range of frequencies (partition form, mode 1: for
// one frequency); its tile [y][m0..m0+S) is
// staged through LDS with coalesced row segments, and each line is solved by
// P threads from constants precomputed per (k, m): float64 lines of at most
// one wave by the recurrence form of pd_scan.h (the lines are symmetric
// Toeplitz), the others by the chunked solver of pd_partition.h.
#include "pd_partition.h"
#include "pd_scan.h"

#include <algorithm>
#include <type_traits>

namespace {

template <typename R, int MR, int MODE, bool SCAN>
__global__ void __launch_bounds__(512, 4)
line2d_kernel(int n, int F2, int P, int S, int mgroups, int kchunk,
              const cpx<R> *__restrict__ fac, R toff, const double *__restrict__ gw,
              const cpx<R> *__restrict__ in, const double *__restrict__ vin,
              const double *__restrict__ xv, double wscale, cpx<R> *__restrict__ out,
              double *__restrict__ partials) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // constants per line, in global memory and in LDS
  constexpr int NF = SCAN ? pd_scan_entries<MR>() : 6 * (MR - 1);
  const int tid = threadIdx.x;
  const int g = tid / P;
  const int lt = tid - g * P;
  const int rows = P * MR;
  const int sstride = rows + 2;
  const size_t nbar = (size_t)n * n;
  cpx<R> *stage = reinterpret_cast<cpx<R> *>(smem_raw) + (size_t)g * sstride;
  Row3<R> *xch = reinterpret_cast<Row3<R> *>(smem_raw) + (size_t)g * P;
  size_t region = (size_t)S * sstride * sizeof(cpx<R>);
  const size_t accb = (size_t)S * rows * sizeof(double);
  if (accb > region) region = accb;
  region = (region + 15) & ~(size_t)15;
  cpx<R> *lfac_all = reinterpret_cast<cpx<R> *>(smem_raw + region);
  cpx<R> *lfac = lfac_all + (size_t)g * NF;

  const int mg = blockIdx.x % mgroups;
  const int m0 = mg * S;
  const int m = m0 + g;
  const bool mact = m < n;
  const int s0 = lt * MR;
  int len = n - s0;
  len = len < 0 ? 0 : (len > MR ? MR : len);
  int kbeg, kend;
  if (MODE == 1) {
    kbeg = blockIdx.x / mgroups;
    kend = kbeg + 1;
  } else {
    const int kc = blockIdx.x / mgroups;
    kbeg = kc * kchunk;
    kend = kbeg + kchunk < F2 ? kbeg + kchunk : F2;
  }
  const cpx<R> zero = {R(0), R(0)};
  const cpx<R> cc = {toff, R(0)};
  // tile entry idx = y S + gg (S a power of two): shifts, no division
  const int lgS = __builtin_ctz(S);
  const int tile = n * S;
  constexpr int U = 8;   // loads in flight per thread

  double acc[(MODE == 1) ? 1 : MR];
  R xr[(MODE == 2) ? 1 : MR];   // mode 1: -w x on this line; mode 2: v on this line
  R vr[(MODE == 2) ? MR : 1];
#pragma unroll
  for (int q = 0; q < MR; ++q) {
    if constexpr (MODE != 1) acc[q] = 0.0;
    const size_t i = (size_t)(s0 + q) * n + m;
    if constexpr (MODE == 1) xr[q] = (xv && mact && q < len) ? (R)(-wscale * xv[i]) : R(0);
    if constexpr (MODE == 2) vr[q] = (mact && q < len) ? (R)vin[i] : R(0);
  }

  for (int k = kbeg; k < kend; ++k) {
    __syncthreads();
    for (int idx = tid; idx < S * NF; idx += blockDim.x) {
      const int gg = idx / NF, j = idx - gg * NF;
      const int mm = m0 + gg < n ? m0 + gg : n - 1;
      lfac_all[gg * NF + j] = fac[((size_t)k * n + mm) * NF + j];
    }
    if constexpr (MODE != 2) {
      // U loads in flight per thread (at clamped, valid addresses), then the
      // LDS stores; columns past n stage zeros
      const cpx<R> *src = in + (size_t)k * nbar;
      for (int b = tid; b < tile; b += U * (int)blockDim.x) {
        cpx<R> v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b + u * (int)blockDim.x;
          const int ic = idx < tile ? idx : tile - 1;
          const int y = ic >> lgS, mm = m0 + (ic & (S - 1));
          const cpx<R> t = src[(size_t)y * n + (mm < n ? mm : n - 1)];
          v[u] = pd_sel(mm < n, t, zero);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b + u * (int)blockDim.x;
          if (idx < tile)
            reinterpret_cast<cpx<R> *>(smem_raw)[(size_t)(idx & (S - 1)) * sstride + (idx >> lgS) + 1] = v[u];
        }
      }
    }
    __syncthreads();
    cpx<R> d[MR];
#pragma unroll
    for (int q = 0; q < MR; ++q) {
      cpx<R> v = zero;
      if (q < len) {
        if constexpr (MODE == 2) {
          v.re = vr[q];
        } else {
          v = stage[s0 + q + 1];
          if constexpr (MODE == 1) v.re += xr[q];
        }
      }
      d[q] = v;
    }
    if constexpr (SCAN)
      scan_solve_group<R, MR, CplxOps<R>, MODE == 1>(d, len, lt, P, lfac);
    else
      partition_solve<R, MR>(d, len, lt, P, lfac, xch, cc, cc);
    if constexpr (MODE == 1) {
      __syncthreads();
#pragma unroll
      for (int q = 0; q < MR; ++q)
        if (q < len) stage[s0 + q + 1] = d[q];
      __syncthreads();
      cpx<R> *dst = out + (size_t)k * nbar;
      for (int idx = tid; idx < tile; idx += blockDim.x) {
        const int y = idx >> lgS, gg = idx & (S - 1);
        const int mm = m0 + gg;
        if (mm < n)
          dst[(size_t)y * n + mm] =
              reinterpret_cast<cpx<R> *>(smem_raw)[(size_t)gg * sstride + y + 1];
      }
    } else {
      double gr = gw[2 * k], gi = gw[2 * k + 1];
      if constexpr (SCAN) {
        // the recurrence form returns kappa y: fold 1/kappa into the weight
        const cpx<R> ik = lfac[4];
        const double t = gr * (double)ik.re - gi * (double)ik.im;
        gi = gr * (double)ik.im + gi * (double)ik.re;
        gr = t;
      }
#pragma unroll
      for (int q = 0; q < MR; ++q)
        if (q < len) acc[q] += gr * (double)d[q].re - gi * (double)d[q].im;
    }
  }

  if constexpr (MODE != 1) {
    __syncthreads();
    double *sd = reinterpret_cast<double *>(smem_raw);
#pragma unroll
    for (int q = 0; q < MR; ++q) sd[(size_t)g * rows + s0 + q] = acc[q];
    __syncthreads();
    const int kc = blockIdx.x / mgroups;
    double *dst = partials + (size_t)kc * nbar;
    for (int idx = tid; idx < tile; idx += blockDim.x) {
      const int y = idx >> lgS, gg = idx & (S - 1);
      const int mm = m0 + gg;
      if (mm < n) dst[(size_t)y * n + mm] = sd[(size_t)gg * rows + y];
    }
  }
}

// Modes 0 and 1 in the recurrence form (float64, a line within a wave).  A
// block keeps its S columns and walks over a chunk of the frequencies; the
// blocks that walk over the same frequencies side by side are on one XCD, where
// they share the lines at the columns' edges.  (The next rows in registers while
// this item's lines are solved spilled: two blocks share a CU at 128 VGPRs.)
// Before, staged rows fell on two banks, a scan took 136 lane moves through LDS
// per wave, and an item five barriers.  n = 511, 129 frequencies: mode 1 407 -> 235 us
// (1.07 GB, 4.6 TB/s), mode 0 285 -> 160 us (0.54 GB); n = 256: 89 -> 53, 70 -> 41 us;
// n = 255, complex64, 257 frequencies: 163 -> 95, 127 -> 67 us.  Bound: mode 1 by
// the bytes, mode 0 by the solves' arithmetic and the barriers.
template <int MR, int MODE, bool IN32>
__global__ void __launch_bounds__(512, 4)
line2d_scan_kernel(int n, int F2, int P, int S, int mgroups, int kchunk,
                   const cpx<double> *__restrict__ fac, const double *__restrict__ gw,
                   const void *in, const double *__restrict__ xv, double wscale,
                   cpx<double> *out, double *__restrict__ partials) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  using Cx = cpx<double>;
  using In = typename std::conditional<IN32, cpx<float>, Cx>::type;
  constexpr int NF = pd_scan_entries<MR>();
  constexpr int FU = MR == 8 ? 2 : NF;   // constants per thread: NF / P, P >= 16 with 8 rows
  const int tid = threadIdx.x, g = tid / P, lt = tid - g * P;
  const int stride = pd_line_stride(n, S);
  const size_t nbar = (size_t)n * n;
  Cx *tile = reinterpret_cast<Cx *>(smem_raw);
  Cx *tabs = tile + (size_t)S * stride;
  Cx *line = tile + (size_t)g * stride;
  const Cx *tb = tabs + g * NF;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int kc = b / mgroups, m0 = (b - kc * mgroups) * S, m = m0 + g;
  const int kbeg = kc * kchunk, kend = kbeg + kchunk < F2 ? kbeg + kchunk : F2;
  const int s0 = lt * MR;
  int len = n - s0;
  len = len < 0 ? 0 : (len > MR ? MR : len);
  const Cx zero = {0.0, 0.0};
  double acc[MODE == 1 ? 1 : MR];
  double xr[MODE == 1 ? MR : 1];   // -w x on this thread's rows
#pragma unroll
  for (int q = 0; q < MR; ++q) {
    if constexpr (MODE == 0) acc[q] = 0.0;
    if constexpr (MODE == 1)
      xr[q] = (xv && m < n && q < len) ? -wscale * xv[(size_t)(s0 + q) * n + m] : 0.0;
  }
  // this thread's share of a tile: rows y0 + u P of column mm, and of its
  // constants.  Offsets are formed where they are used (32 bits, from a
  // register the compiler cannot keep them for): two blocks share a CU
  const int lgS = __builtin_ctz(S), cl = tid & (S - 1);
  const bool mact = m0 + cl < n;
  const int mm = mact ? m0 + cl : n - 1;
  int y0 = tid >> lgS;
  auto at = [&](int u) {   // entry of row y0 + u P
    if constexpr (MR == 8)
      return cl * stride + pd_line_entry(y0) + u * (P + (P >> 3));   // P a multiple of 8
    else
      return cl * stride + pd_line_entry(y0 + u * P);
  };
  In v[MR];
  Cx fv[FU];
  auto load = [&](int k) {
    const In *src = static_cast<const In *>(in) + (size_t)k * nbar;
#pragma unroll
    for (int u = 0; u < MR; ++u) {
      const int y = y0 + u * P;
      v[u] = src[(unsigned)((y < n ? y : n - 1) * n + mm)];
    }
    const Cx *fs = fac + ((size_t)k * n + m0) * NF;
    const int last = (n - m0 < S ? n - m0 : S) * NF - 1;
#pragma unroll
    for (int u = 0; u < FU; ++u) {
      const int e = tid + u * (int)blockDim.x;
      const Cx t = fs[(unsigned)(e < last ? e : last)];
      fv[u] = Cx{t.re, t.im};
    }
  };
  for (int k = kbeg; k < kend; ++k) {
    asm volatile("" : "+v"(y0));
    load(k);
    if (k != kbeg) __syncthreads();   // the item before has been stored
#pragma unroll
    for (int u = 0; u < MR; ++u) {
      const int y = y0 + u * P;
      if (y < n) tile[at(u)] = pd_sel(mact, Cx{(double)v[u].re, (double)v[u].im}, zero);
    }
#pragma unroll
    for (int u = 0; u < FU; ++u) {
      const int e = tid + u * (int)blockDim.x;
      if (e < S * NF) tabs[e] = Cx{fv[u].re, fv[u].im};
    }
    __syncthreads();
    Cx d[MR];
#pragma unroll
    for (int q = 0; q < MR; ++q) {
      Cx t = zero;
      if (q < len) {
        t = line[pd_line_entry(s0 + q)];
        if constexpr (MODE == 1) t.re += xr[q];
      }
      d[q] = t;
    }
    if (MR == 8 || P >= 16)   // 8 rows: n > 64, P >= 16
      scan_solve_lanes<double, MR, CplxOps<double>, MODE == 1>(d, len, lt, P, tb);
    else
      scan_solve_group<double, MR, CplxOps<double>, MODE == 1>(d, len, lt, P, tb);
    if constexpr (MODE == 1) {
      // every thread reads and writes its own rows of the tile only
#pragma unroll
      for (int q = 0; q < MR; ++q)
        if (q < len) line[pd_line_entry(s0 + q)] = d[q];
      __syncthreads();
      Cx *dst = out + (size_t)k * nbar;
#pragma unroll
      for (int u = 0; u < MR; ++u) {
        const int y = y0 + u * P;
        if (y < n && mact) dst[(unsigned)(y * n + mm)] = tile[at(u)];
      }
    } else {
      // the recurrence form returns kappa y: fold 1/kappa into the weight
      const Cx ik = tb[4];
      const double gr = gw[2 * k] * ik.re - gw[2 * k + 1] * ik.im;
      const double gi = gw[2 * k] * ik.im + gw[2 * k + 1] * ik.re;
#pragma unroll
      for (int q = 0; q < MR; ++q)
        if (q < len) acc[q] += gr * d[q].re - gi * d[q].im;
    }
  }
  if constexpr (MODE == 0) {
    __syncthreads();
    double *sd = reinterpret_cast<double *>(smem_raw);
#pragma unroll
    for (int q = 0; q < MR; ++q)
      if (q < len) sd[2 * ((size_t)g * stride + pd_line_entry(s0 + q))] = acc[q];
    __syncthreads();
    double *dst = partials + (size_t)kc * nbar;
#pragma unroll
    for (int u = 0; u < MR; ++u) {
      const int y = y0 + u * P;
      if (y < n && mact) dst[(unsigned)(y * n + mm)] = sd[2 * at(u)];
    }
  }
}

template <int MR, int MODE, bool IN32>
void launch2d_scan(pd_plan p, const void *in, const double *xv, void *out) {
  const Line2DConfig &L = p->l2d;
  hipLaunchKernelGGL((line2d_scan_kernel<MR, MODE, IN32>), dim3(L.nkc * L.mgroups), dim3(L.block),
                     pd_line_lds(p->n, LineShape{MR, L.P, L.S}), p->stream, p->n, p->F2, L.P, L.S, L.mgroups,
                     L.kchunk, reinterpret_cast<const cpx<double> *>(p->fac64), p->gB64, in, xv,
                     p->w, static_cast<cpx<double> *>(out), p->partials);
}

template <typename R, int MR, bool SCAN>
pd_status launch2d_form(pd_plan p, int mode, const void *in, const double *xv, void *out) {
  const Line2DConfig &L = p->l2d;
  const cpx<R> *fac = (sizeof(R) == 8) ? reinterpret_cast<const cpx<R> *>(p->fac64)
                                       : reinterpret_cast<const cpx<R> *>(p->fac32);
  const R toff = (R)p->uni[3];
  mode &= 0xff;
  if constexpr (SCAN) {
    if (mode != 2) {
      // in32: complex64 right-hand sides, mode 1 writes complex128 elsewhere
      if (mode == 1 && p->in32) launch2d_scan<MR, 1, true>(p, in, xv, out);
      else if (mode == 1) launch2d_scan<MR, 1, false>(p, in, xv, out);
      else if (p->in32) launch2d_scan<MR, 0, true>(p, in, xv, out);
      else launch2d_scan<MR, 0, false>(p, in, xv, out);
      PD_HIP_CHECK(hipGetLastError());
      return PD_OK;
    }
  }
  auto launch = [&](auto m, int blocks, const double *gw, const cpx<R> *src, const double *v) {
    hipLaunchKernelGGL((line2d_kernel<R, MR, decltype(m)::value, SCAN>), dim3(blocks), dim3(L.block),
                       L.lds, p->stream, p->n, p->F2, L.P, L.S, L.mgroups, L.kchunk, fac, toff, gw,
                       src, v, xv, p->w, reinterpret_cast<cpx<R> *>(out), p->partials);
  };
  if (mode == 2) {
    launch(std::integral_constant<int, 2>{}, L.nkc * L.mgroups, p->gJ64, nullptr,
           static_cast<const double *>(in));
  } else if constexpr (!SCAN) {
    const cpx<R> *src = reinterpret_cast<const cpx<R> *>(in);
    if (mode == 1)
      launch(std::integral_constant<int, 1>{}, p->F2 * L.mgroups, p->gB64, src, nullptr);
    else
      launch(std::integral_constant<int, 0>{}, L.nkc * L.mgroups, p->gB64, src, nullptr);
  }
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

template <typename R, int MR>
pd_status launch2d(pd_plan p, int mode, const void *in, const double *xv, void *out) {
  if constexpr (sizeof(R) == 8) {
    // always so with complex64 spectra (pd_mixed64_ok)
    if (pd_line2d_scan(p)) return launch2d_form<R, MR, true>(p, mode, in, xv, out);
  }
  return launch2d_form<R, MR, false>(p, mode, in, xv, out);
}

}  // namespace

Line2DConfig pd_choose_line2d(int n, int F2, int prec, int cus) {
  Line2DConfig L;
  const size_t cb = (prec == PD_FP64) ? 16 : 8;
  const LineShape shape = pd_line_shape(n);
  L.MR = shape.MR;
  L.P = shape.P;
  L.S = shape.S;
  L.block = L.P * L.S;
  L.mgroups = (n + L.S - 1) / L.S;
  // enough blocks for the frequency sums: split k into chunks
  L.nkc = 1;
  while (L.nkc * L.mgroups < 2 * cus && L.nkc < F2) L.nkc *= 2;
  L.kchunk = (F2 + L.nkc - 1) / L.nkc;
  L.nkc = (F2 + L.kchunk - 1) / L.kchunk;
  const size_t rows = (size_t)L.P * L.MR;
  size_t region = (size_t)L.S * (rows + 2) * cb;
  const size_t accb = (size_t)L.S * rows * sizeof(double);
  if (accb > region) region = accb;
  region = (region + 15) & ~(size_t)15;
  L.lds = region + (size_t)L.S * 6 * (L.MR - 1) * cb;
  return L;
}

double pd_line2d_theta(const pd_plan p, int m) {
  return p->uni[4] + 2.0 * p->uni[3] * std::cos((m + 1) * M_PI / (p->n + 1));
}

// Factors for every (k, m): b = lambda_k + tau theta_m + tau T_d, a = c = tau T_off.
// float64 plans into fac, the others rounded to float into fac32.
void pd_line2d_factors(const pd_plan p, std::vector<double> &fac, std::vector<float> &fac32) {
  const int n = p->n, F2 = p->F2, MR = p->l2d.MR;
  const size_t NF = pd_line2d_entries(p);
  const bool f32 = p->prec != PD_FP64;
  if (f32)
    fac32.assign((size_t)F2 * n * NF * 2, 0.0f);
  else
    fac.assign((size_t)F2 * n * NF * 2, 0.0);
  const double tl = p->uni[3], td = p->uni[4];
  const bool scan = pd_line2d_scan(p);
  std::vector<double> th(n);
  for (int m = 0; m < n; ++m) th[m] = pd_line2d_theta(p, m);
  const int mblk = (n + 63) / 64;   // units of 64 lines of a frequency
  pd_parallel_rows(F2 * mblk, 4, [&](int unit) {
    const int k = unit / mblk, ma = (unit - k * mblk) * 64, mb = ma + 64 < n ? ma + 64 : n;
    double row[2 * 6 * 7];   // rounded to float below (8 rows per thread at most)
    for (int m = ma; m < mb; ++m) {
      const double theta = th[m];
      if (scan) {
        pd_scan_table({tl, 0.0}, {p->lam[2 * k] + theta + td, p->lam[2 * k + 1]}, {tl, 0.0},
                      p->lam[2 * k + 1] == 0.0, n, MR,
                      reinterpret_cast<std::complex<double> *>(&fac[((size_t)k * n + m) * NF * 2]));
        continue;
      }
      double *dst = f32 ? row : &fac[((size_t)k * n + m) * NF * 2];
      pd_partition_factors(tl, 0.0, p->lam[2 * k] + theta + td, p->lam[2 * k + 1], tl, 0.0, MR,
                           dst);
      if (f32) std::copy(row, row + NF * 2, fac32.begin() + ((size_t)k * n + m) * NF * 2);
    }
  });
}

pd_status pd_launch_line2d(pd_plan p, int mode, const void *in, const double *xv, void *out) {
  const int MR = p->l2d.MR;
  if (p->prec == PD_FP64) {
    if (MR == 4) return launch2d<double, 4>(p, mode, in, xv, out);
    if (MR == 8) return launch2d<double, 8>(p, mode, in, xv, out);
  } else {
    if (MR == 4) return launch2d<float, 4>(p, mode, in, xv, out);
    if (MR == 8) return launch2d<float, 8>(p, mode, in, xv, out);
  }
  pd_set_error("unsupported 2D line configuration");
  return PD_ENOTSUP;
}

void pd_line2d_set_attributes(size_t max_lds) {
  const int v = (int)max_lds;
  const void *fns[] = {
      reinterpret_cast<const void *>(&line2d_scan_kernel<4, 0, true>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<4, 1, true>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<4, 0, false>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<4, 1, false>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<8, 0, true>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<8, 1, true>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<8, 0, false>),
      reinterpret_cast<const void *>(&line2d_scan_kernel<8, 1, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 4, 0, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 4, 1, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 4, 2, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 4, 2, true>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 8, 0, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 8, 1, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 8, 2, false>),
      reinterpret_cast<const void *>(&line2d_kernel<double, 8, 2, true>),
      reinterpret_cast<const void *>(&line2d_kernel<float, 4, 0, false>),
      reinterpret_cast<const void *>(&line2d_kernel<float, 4, 1, false>),
      reinterpret_cast<const void *>(&line2d_kernel<float, 4, 2, false>),
      reinterpret_cast<const void *>(&line2d_kernel<float, 8, 0, false>),
      reinterpret_cast<const void *>(&line2d_kernel<float, 8, 1, false>),
      reinterpret_cast<const void *>(&line2d_kernel<float, 8, 2, false>)};
  for (const void *f : fns)
    pd_set_max_lds(f, v);
}
