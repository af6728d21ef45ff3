// Shifted solves of general (non-constant) tridiagonal M and K in float64:
// the parfor of Algorithm 1 on graded meshes, 64 < n <= 4096.
//
// P_k = L U without pivoting, l_i = a_i / d_{i-1}, d_i = b_i - l_i c_{i-1}, so a
// solve is two first-order recurrences,
//
//     v_i = y_i - l_i v_{i-1},       x_i = v_i / d_i - (c_i / d_i) x_{i+1}.
//
// A group of P threads (whole waves) solves one system, 8 rows to a thread:
// each thread runs its rows from a zero start together with the product of the
// multipliers, a scan over the chunk maps x -> m x + c (DPP inside a wave, the
// waves' maps through LDS) gives the value that enters each chunk, and the
// rows take it times their products; backwards the same.  The pivots are a
// serial recurrence, but only the one before each chunk is needed from
// outside: a plan keeps P of them per frequency (formed once on the device, a
// wave per frequency: 180 us at n = 3001, beside the host's work on the other
// tables), and the thread's own 8 are 8 reciprocals.  That is 2 F2 P doubles instead of
// a table of every row's factors.
//
// What bounds it is latency -- 129 systems of 3001 rows leave half the CUs
// idle -- so the point is the length of the chain: one sweep of 8 reciprocals and
// two scans of 6 steps, three barriers, against two such sweeps, 9 reduction
// steps of a reciprocal and two barriers each in the partition form
// (tridiag_kernel).  n = 3001, ell = 256: pass B 68 -> 18 us, pass C 68 -> 22 us,
// J product 55 -> 15 us, the solve 375 -> 155 us.  Coefficients are kept a second
// time in the threads' order (row q of every thread side by side), so that their
// loads coalesce.
//
// There is no pivoting.  A plan uses this form only if every pivot is at least 1/16
// of its diagonal entry (checked when the pivots are formed); otherwise, and for
// float32 plans, the partition form runs, which does not pivot either.  The check
// does not bound growth: a diagonal entry far below its row's others passes and
// makes the next pivot large (b_i = d_i + l_i c_{i-1}, two large terms), and the
// backward error then grows with the largest pivot against its row.  The partition
// form is worse there: transport by central differences on a graded mesh, n = 200,
// pivots up to 6.3e3 times their rows: backward error 8.5e-15, partition form 1.1e-11.
// n <= 512 takes a wave per system whatever n is (identity rows past it): n = 200,
// ell = 256, pass B 57 -> 15 us, pass C 55 -> 18 us, J product 44 -> 13 us,
// the solve 315 -> 130 us of kernels.
#include "pd_scan.h"

#include <algorithm>
#include <vector>

namespace {

using Cx = cpx<double>;
constexpr int MR = PD_LU_ROWS;

// 1 / |a|^2: the hardware reciprocal and one step of third order.
__device__ __forceinline__ double lu_rsq(Cx a) {
  const double d = a.re * a.re + a.im * a.im;
  const double r = __builtin_amdgcn_rcp(d), e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ Cx lu_recip(Cx a) {
  const double r = lu_rsq(a);
  return Cx{a.re * r, -a.im * r};
}
__device__ __forceinline__ Cx nmul(Cx a, Cx b) {   // -a b
  return Cx{a.im * b.im - a.re * b.re, -a.re * b.im - a.im * b.re};
}
__device__ __forceinline__ Cx fma_c(Cx s, Cx b, Cx c) {   // s + b c
  return Cx{s.re + b.re * c.re - b.im * c.im, s.im + b.re * c.im + b.im * c.re};
}

// Coefficient row d of thread lt's row q: cT[(d MR + q) P + lt], d = ML MD MU
// KL KD KU (tau K); rows past n hold the identity (MD = 0, KD = 1).
struct LuRow {
  double ml, md, mu, kl, kd, ku;
};

__global__ void __launch_bounds__(64)
lu_rows_kernel(int n, int P, const double *__restrict__ coef, double *__restrict__ cT) {
  const int i = blockIdx.x * 64 + threadIdx.x, d = blockIdx.y;
  cT[((size_t)d * MR + i % MR) * P + i / MR] = i < n ? coef[(size_t)d * n + i] : (d == 4 ? 1.0 : 0.0);
}

// One wave per frequency: the pivots before every chunk, piv[k P + lt] =
// d_{lt MR - 1} (1 for lt = 0), by the serial recurrence, which every lane
// runs (64 rows' b_i and a_i c_{i-1} at a time from LDS); bad[k] is 1 where a
// pivot is too small against its diagonal entry or that entry beyond 1e-93 and
// 1e93, else 0.
__global__ void __launch_bounds__(64)
lu_pivots_kernel(int n, int P, const double *__restrict__ coef, const double *__restrict__ lam,
                 Cx *__restrict__ piv, double *__restrict__ bad) {
  __shared__ Cx row[64][2], piv64[64];
  const int k = blockIdx.x, lane = threadIdx.x;
  const double lr = lam[2 * k], li = lam[2 * k + 1];
  const double *ML = coef, *MD = coef + n, *MU = coef + 2 * (size_t)n;
  const double *KL = coef + 3 * (size_t)n, *KD = coef + 4 * (size_t)n, *KU = coef + 5 * (size_t)n;
  Cx d = {1.0, 0.0};
  bool small = false;
  for (int i0 = 0; i0 < P * MR; i0 += 64) {
    if (i0 >= n) {   // identity rows
      if (lane < 64 / MR) piv[(size_t)k * P + i0 / MR + lane] = Cx{1.0, 0.0};
      continue;
    }
    const int i = i0 + lane;
    Cx b = {1.0, 0.0}, ac = {0.0, 0.0};
    if (i < n) {
      b = Cx{lr * MD[i] + KD[i], li * MD[i]};
      if (i > 0)
        ac = nmul(Cx{lr * ML[i] + KL[i], li * ML[i]}, Cx{lr * MU[i - 1] + KU[i - 1], li * MU[i - 1]});
    }
    __syncthreads();
    row[lane][0] = b;
    row[lane][1] = ac;
    __syncthreads();
    if (lane == 0) piv[(size_t)k * P + i0 / MR] = d;
#pragma unroll 8
    for (int r = 0; r < 64; ++r) {
      const Cx br = row[r][0];
      // -a c / d as (-a c conj(d)) / |d|^2: the product beside the reciprocal
      const Cx ac = row[r][1], t = {ac.re * d.re + ac.im * d.im, ac.im * d.re - ac.re * d.im};
      const double q = lu_rsq(d);
      d = Cx{fma(t.re, q, br.re), fma(t.im, q, br.im)};
      piv64[r] = d;   // every lane the same value
    }
    __syncthreads();
    const Cx dl = piv64[lane];
    const double dd = dl.re * dl.re + dl.im * dl.im, bb = b.re * b.re + b.im * b.im;
    // the numerator above is of the entries' third power: entries beyond 1e-93 and
    // 1e93 leave the form to the partition method
    small = small || !(dd * 256.0 >= bb) || !(bb > 1e-186 && bb < 1e186) || !(dd < 1e300);
    if (lane % MR == MR - 1 && lane < 63) piv[(size_t)k * P + (i + 1) / MR] = dl;
  }
  small = __any(small);
  if (lane == 0) bad[k] = small ? 1.0 : 0.0;
}

// MODE as for tridiag_kernel: 0 accumulates Re(gw_k y_k) into partial rows, 1
// writes y_k, 2 accumulates with the right-hand side M v.
template <int MODE>
__global__ void __launch_bounds__(512)
lu_solve_kernel(int n, int F2, int P, int spb, int nitems, const double *__restrict__ cT,
                const double *__restrict__ lam, const Cx *__restrict__ piv,
                const double *__restrict__ gw, const Cx *__restrict__ in,
                const double *__restrict__ vin, const double *__restrict__ xv, double wscale,
                int rhs_has_mass, Cx *__restrict__ out, double *__restrict__ partials,
                const double *__restrict__ skip) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ Cx xw[2][8][2];   // per wave: (value, multiplier), forward and backward
  if (skip && *skip != 0.0) return;
  const int tid = threadIdx.x, g = tid / P, lt = tid - g * P;
  const int lane = lt & 63, wv = lt >> 6, NW = P >> 6, w0 = (tid - lt) >> 6;
  const int gs = pd_lu_group(P);
  Cx *stage = reinterpret_cast<Cx *>(smem_raw) + (size_t)g * gs;
  const int s0 = lt * MR;
  const Cx zero = {0.0, 0.0}, one = {1.0, 0.0};
  unsigned lq = lt;   // lt for addresses
  auto coef = [&](int d, int q) { return (cT + (size_t)(d * MR + q) * P)[lq]; };

  double acc[MODE == 1 ? 1 : MR];
  double base[MODE == 0 ? 1 : MR];   // mode 1: -w M x, mode 2: M v, on this thread's rows
  if constexpr (MODE != 1) {
#pragma unroll
    for (int q = 0; q < MR; ++q) acc[q] = 0.0;
  }
  if constexpr (MODE != 0) {
    const double *v = MODE == 2 ? vin : xv;
    double *sv = reinterpret_cast<double *>(stage);
    for (int i = lt; i < P * MR + 2; i += P) {      // entry i: v_{i-1}
      const int r = i - 1, rc = r < 0 ? 0 : (r < n ? r : n - 1);
      const double t = v ? v[rc] : 0.0;
      sv[pd_lu_entry(i)] = (r >= 0 && r < n) ? t : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MR; ++q) {
      const int i = s0 + q + 1;
      double t = coef(1, q) * sv[pd_lu_entry(i)];
      t += coef(0, q) * sv[pd_lu_entry(i - 1)];
      t += coef(2, q) * sv[pd_lu_entry(i + 1)];
      base[q] = MODE == 2 ? t : -wscale * t;
    }
  }

  for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
    const int k0 = item * spb + g;
    const bool active = k0 < F2;
    const int k = active ? k0 : F2 - 1;
    const double lr = lam[2 * k], li = lam[2 * k + 1];
    // the coefficients are loaded, and the addresses formed, per item: kept
    // over the items they would take more than 96 registers
    asm volatile("" : "+v"(lq));
    const int s0 = (int)lq * MR;
    Cx d[MR];
    if constexpr (MODE != 2) {
      __syncthreads();   // the staging area is free
      const Cx *src = in + (size_t)k * n;
#pragma unroll
      for (int u = 0; u < MR; ++u) {
        const int r = (int)lq + u * P;
        const Cx t = src[r < n ? r : n - 1];
        stage[pd_lu_entry(r + 1)] = r < n ? t : zero;
      }
      if (lt == 0) stage[pd_lu_entry(0)] = zero;
      if (lt == 1) stage[pd_lu_entry(P * MR + 1)] = zero;
    }
    // this system's rows and the pivot before them, while the loads land
    Cx e = lu_recip(piv[(size_t)k * P + lq]), cp = zero;   // 1 / d_{q-1}, c_{q-1}
    if (lt > 0) {
      const double mu = (cT + (size_t)(2 * MR + MR - 1) * P)[lq - 1];
      const double ku = (cT + (size_t)(5 * MR + MR - 1) * P)[lq - 1];
      cp = Cx{lr * mu + ku, li * mu};
    }
    if constexpr (MODE != 2) {
      __syncthreads();
#pragma unroll
      for (int q = 0; q < MR; ++q) {
        const int i = s0 + q + 1;
        Cx t = stage[pd_lu_entry(i)];
        if (!rhs_has_mass) {
          const double md = coef(1, q), ml = coef(0, q), mu = coef(2, q);
          const Cx l = stage[pd_lu_entry(i - 1)], r = stage[pd_lu_entry(i + 1)];
          t = Cx{md * t.re + ml * l.re + mu * r.re, md * t.im + ml * l.im + mu * r.im};
        }
        if constexpr (MODE == 1) t.re += base[q];
        d[q] = t;
      }
    } else {
#pragma unroll
      for (int q = 0; q < MR; ++q) d[q] = Cx{base[q], 0.0};
    }
    // forward: d[q] = v_q from a zero start, f[q] = the product that carries
    // the value before the chunk; then both times 1 / d_q, u[q] = -c_q / d_q
    Cx f[MR], u[MR];
    Cx v = zero, p = one;
#pragma unroll
    for (int q = 0; q < MR; ++q) {
      if (q == MR / 2) asm volatile("" : "+v"(lq), "+v"(v.re));   // the second half's later
      const double ml = coef(0, q), md = coef(1, q), mu = coef(2, q);
      const Cx a = {lr * ml + coef(3, q), li * ml}, b = {lr * md + coef(4, q), li * md};
      const Cx nl = nmul(a, e);              // -l_q
      e = lu_recip(fma_c(b, nl, cp));
      cp = Cx{lr * mu + coef(5, q), li * mu};
      v = fma_c(d[q], nl, v);
      p = cmul(nl, p);
      d[q] = cmul(e, v);
      f[q] = cmul(e, p);
      u[q] = nmul(cp, e);
    }
    // the value entering the chunk
    Cx c = v, m = p;
    using A = CplxOps<double>;
    pd_scan_step<0x111, 0xF, A>(c, m);   // row_shr:1, 2, 4, 8
    pd_scan_step<0x112, 0xF, A>(c, m);
    pd_scan_step<0x114, 0xF, A>(c, m);
    pd_scan_step<0x118, 0xF, A>(c, m);
    pd_scan_step<0x142, 0xA, A>(c, m);   // row_bcast:15 into rows 1 and 3
    pd_scan_step<0x143, 0xC, A>(c, m);   // row_bcast:31 into rows 2 and 3
    if (lane == 63) {
      xw[0][w0 + wv][0] = c;
      xw[0][w0 + wv][1] = m;
    }
    const Cx ec = pd_dpp<0x138, 0xF>(c, zero), em = pd_dpp<0x138, 0xF>(m, one);   // wave_shr:1
    __syncthreads();
    {
      Cx C = zero;
      for (int w = 0; w < wv; ++w) C = fma_c(xw[0][w0 + w][0], xw[0][w0 + w][1], C);
      const Cx V = fma_c(ec, em, C);
#pragma unroll
      for (int q = 0; q < MR; ++q) d[q] = fma_c(d[q], f[q], V);
    }
    // backward: d[q] = x_q from a zero end, u[q] = the product to the value after
#pragma unroll
    for (int q = MR - 2; q >= 0; --q) {
      d[q] = fma_c(d[q], u[q], d[q + 1]);
      u[q] = cmul(u[q], u[q + 1]);
    }
    c = d[0];
    m = u[0];
    pd_scan_step<0x101, 0xF, A>(c, m);   // row_shl:1, 2, 4, 8
    pd_scan_step<0x102, 0xF, A>(c, m);
    pd_scan_step<0x104, 0xF, A>(c, m);
    pd_scan_step<0x108, 0xF, A>(c, m);
    {
      auto from = [](Cx x, int l) { return Cx{__shfl(x.re, l, 64), __shfl(x.im, l, 64)}; };
      const int srcA = ((lane | 15) + 1) & 63;
      const Cx oc = from(c, srcA), om = from(m, srcA);
      const bool in1 = ((lane >> 4) & 1) == 0;
      c = pd_sel(in1, fma_c(c, m, oc), c);
      m = pd_sel(in1, cmul(m, om), m);
      const Cx oc2 = from(c, 32), om2 = from(m, 32);
      const bool in2 = lane < 32;
      c = pd_sel(in2, fma_c(c, m, oc2), c);
      m = pd_sel(in2, cmul(m, om2), m);
    }
    if (lane == 0) {
      xw[1][w0 + wv][0] = c;
      xw[1][w0 + wv][1] = m;
    }
    const Cx bc = pd_dpp<0x130, 0xF>(c, zero), bm = pd_dpp<0x130, 0xF>(m, one);   // wave_shl:1
    __syncthreads();
    {
      Cx C = zero;
      for (int w = NW - 1; w > wv; --w) C = fma_c(xw[1][w0 + w][0], xw[1][w0 + w][1], C);
      const Cx W = fma_c(bc, bm, C);
#pragma unroll
      for (int q = 0; q < MR; ++q) d[q] = fma_c(d[q], u[q], W);
    }
    if constexpr (MODE == 1) {
      // the staging area was last read before the two barriers above
#pragma unroll
      for (int q = 0; q < MR; ++q) stage[pd_lu_entry(s0 + q + 1)] = d[q];
      __syncthreads();
      if (active) {
        Cx *dst = out + (size_t)k * n;
#pragma unroll
        for (int j = 0; j < MR; ++j) {
          const int r = (int)lq + j * P;
          if (r < n) dst[r] = stage[pd_lu_entry(r + 1)];
        }
      }
    } else if (active) {
      const double gr = gw[2 * k], gi = gw[2 * k + 1];
#pragma unroll
      for (int q = 0; q < MR; ++q) acc[q] += gr * d[q].re - gi * d[q].im;
    }
  }

  if constexpr (MODE != 1) {
    __syncthreads();
    double *sd = reinterpret_cast<double *>(stage);
#pragma unroll
    for (int q = 0; q < MR; ++q) sd[pd_lu_entry(s0 + q)] = acc[q];
    __syncthreads();
    const Cx *all = reinterpret_cast<const Cx *>(smem_raw);
    for (int i = tid; i < n; i += blockDim.x) {
      double s = 0.0;
      for (int h = 0; h < spb; ++h)
        s += reinterpret_cast<const double *>(all + (size_t)h * gs)[pd_lu_entry(i)];
      partials[(size_t)blockIdx.x * n + i] = s;
    }
  }
}

constexpr int LU_T = PD_LU_BLOCK;
int lu_items(const pd_plan p) {
  const int spb = LU_T / pd_lu_threads(p->n);
  return (p->F2 + spb - 1) / spb;
}

}  // namespace

// Doubles of the coefficients in the threads' order, the pivots and their
// flags; 0 when the plan is not of this form.  n <= 64 is one round of the
// partition form, too: a solve takes 198 against 200 us at n = 63, 178 against 431
// at n = 65, and the plan's creation 45 us more than the partition form's.
size_t pd_lu_doubles(const pd_plan p) {
  if (p->dims != 1 || p->prec != PD_FP64 || p->uniform || p->autotune || p->n <= 64 || p->n > 4096)
    return 0;
  const int P = pd_lu_threads(p->n);
  return 6 * (size_t)P * MR + 2 * (size_t)p->F2 * P + p->F2;
}

// Blocks of a launch that sums over the frequencies.
int pd_lu_blocks(const pd_plan p, int cus) { return std::min(lu_items(p), cus); }

static double *lu_flags(pd_plan p) {
  const int P = pd_lu_threads(p->n);
  return p->lu_tab + 6 * (size_t)P * MR + 2 * (size_t)p->F2 * P;
}

// Fills p->lu_tab on the plan's stream from coef64 and lam64, the first tables
// of a creation: the pivots are formed while the host makes the others.
pd_status pd_lu_setup(pd_plan p) {
  const int n = p->n, P = pd_lu_threads(n);
  double *piv = p->lu_tab + 6 * (size_t)P * MR;
  hipLaunchKernelGGL(lu_rows_kernel, dim3(P * MR / 64, 6), dim3(64), 0, p->stream, n, P, p->coef64,
                     p->lu_tab);
  hipLaunchKernelGGL(lu_pivots_kernel, dim3(p->F2), dim3(64), 0, p->stream, n, P, p->coef64,
                     p->lam64, reinterpret_cast<Cx *>(piv), lu_flags(p));
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

// bad, the host's end of a copy, is valid once the stream is synchronised.  The
// form may be used if no entry of bad (one per frequency) is then set.
pd_status pd_lu_flags(pd_plan p, std::vector<double> &bad) {
  bad.assign(p->F2, 1.0);
  PD_HIP_CHECK(hipMemcpyAsync(bad.data(), lu_flags(p), p->F2 * sizeof(double),
                              hipMemcpyDeviceToHost, p->stream));
  return PD_OK;
}

pd_status pd_launch_lu(pd_plan p, int mode, const void *in, const double *xv, void *out) {
  const int has_mass = (mode & 0x100) ? 1 : 0;
  mode &= 0xff;
  const int P = pd_lu_threads(p->n), spb = LU_T / P, nitems = lu_items(p);
  const int G = mode == 1 ? nitems : p->lu_G;
  const Cx *piv = reinterpret_cast<const Cx *>(p->lu_tab + 6 * (size_t)P * MR);
#define PD_LU(M, GW, IN, VIN, XV, O, PART)                                                     \
  hipLaunchKernelGGL((lu_solve_kernel<M>), dim3(G), dim3(LU_T), pd_lu_lds(P, spb), p->stream,     \
                     p->n, p->F2, P, spb, nitems, p->lu_tab, p->lam64, piv, GW, IN, VIN, XV,     \
                     p->w, has_mass, O, PART, p->gm_skip)
  if (mode == 1)
    PD_LU(1, nullptr, static_cast<const Cx *>(in), nullptr, xv, static_cast<Cx *>(out), nullptr);
  else if (mode == 0)
    PD_LU(0, p->gB64, static_cast<const Cx *>(in), nullptr, nullptr, nullptr, p->partials);
  else
    PD_LU(2, p->gJ64, nullptr, static_cast<const double *>(in), nullptr, nullptr, p->partials);
#undef PD_LU
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

void pd_lu_set_attributes(size_t max_lds) {
  pd_set_max_lds(reinterpret_cast<const void *>(&lu_solve_kernel<0>), (int)max_lds);
  pd_set_max_lds(reinterpret_cast<const void *>(&lu_solve_kernel<1>), (int)max_lds);
  pd_set_max_lds(reinterpret_cast<const void *>(&lu_solve_kernel<2>), (int)max_lds);
}
