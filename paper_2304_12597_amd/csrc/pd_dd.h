// Double-double arithmetic (pairs h + l, l below the rounding of h) for tables
// that are formed once per plan: error-free sums (Knuth's two-sum) and
// products (by fused multiply-add), about 2^-100 relative each.
#pragma once
#include "pd_internal.h"

struct pd_dd {
  double h, l;
};
struct pd_ddc {
  pd_dd re, im;
};

__device__ __forceinline__ pd_dd dd_two_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return pd_dd{s, (a - (s - t)) + (b - t)};
}
__device__ __forceinline__ pd_dd dd_norm(double h, double l) {   // |h| >= |l|
  const double s = h + l;
  return pd_dd{s, l - (s - h)};
}
__device__ __forceinline__ pd_dd dd_add(pd_dd a, pd_dd b) {
  pd_dd s = dd_two_sum(a.h, b.h);
  const pd_dd t = dd_two_sum(a.l, b.l);
  s = dd_norm(s.h, s.l + t.h);
  return dd_norm(s.h, s.l + t.l);
}
__device__ __forceinline__ pd_dd dd_neg(pd_dd a) { return pd_dd{-a.h, -a.l}; }
__device__ __forceinline__ pd_dd dd_mul(pd_dd a, pd_dd b) {
  const double p = a.h * b.h;
  double e = fma(a.h, b.h, -p);
  e = fma(a.h, b.l, fma(a.l, b.h, e));
  return dd_norm(p, e);
}
__device__ __forceinline__ pd_dd dd_recip(pd_dd a) {
  const double q = 1.0 / a.h;
  const double e = fma(-a.l, q, fma(-a.h, q, 1.0));
  return dd_norm(q, q * e);
}
__device__ __forceinline__ pd_ddc dd_cplx(cpx<double> a) {
  return pd_ddc{pd_dd{a.re, 0.0}, pd_dd{a.im, 0.0}};
}
__device__ __forceinline__ pd_ddc dd_cadd(pd_ddc a, pd_ddc b) {
  return pd_ddc{dd_add(a.re, b.re), dd_add(a.im, b.im)};
}
__device__ __forceinline__ pd_ddc dd_cmul(pd_ddc a, pd_ddc b) {
  return pd_ddc{dd_add(dd_mul(a.re, b.re), dd_neg(dd_mul(a.im, b.im))),
                dd_add(dd_mul(a.re, b.im), dd_mul(a.im, b.re))};
}
__device__ __forceinline__ pd_ddc dd_scale(pd_ddc a, pd_dd s) {
  return pd_ddc{dd_mul(a.re, s), dd_mul(a.im, s)};
}
__device__ __forceinline__ pd_ddc dd_ldexp(pd_ddc a, int e) {
  return pd_ddc{pd_dd{ldexp(a.re.h, e), ldexp(a.re.l, e)}, pd_dd{ldexp(a.im.h, e), ldexp(a.im.l, e)}};
}
// num / den, both scaled by a power of two first: matrices may be of any scale,
// and |den|^2 of entries of 1e-150 or 1e150 leaves the range.
__device__ __forceinline__ pd_ddc dd_cdiv(pd_ddc num, pd_ddc den) {
  int e;
  (void)frexp(fmax(fabs(den.re.h), fabs(den.im.h)), &e);
  num = dd_ldexp(num, -e);
  den = dd_ldexp(den, -e);
  const pd_dd d = dd_add(dd_mul(den.re, den.re), dd_mul(den.im, den.im));
  return dd_scale(dd_cmul(num, pd_ddc{den.re, dd_neg(den.im)}), dd_recip(d));
}

// Sum over a block of whole waves (at most 16), in thread 0.
__device__ __forceinline__ pd_dd dd_block_sum(pd_dd v) {
  __shared__ pd_dd part[16];
  for (int off = 32; off > 0; off >>= 1)
    v = dd_add(v, pd_dd{__shfl_down(v.h, off, 64), __shfl_down(v.l, off, 64)});
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) v = dd_add(v, part[w]);
  return v;
}
