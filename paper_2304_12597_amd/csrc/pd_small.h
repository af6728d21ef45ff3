// Steps of a small GMRES that one wave can do without LDS: lane i holds entry
// i of a column, and the serial chains (Givens rotations, back substitution)
// pass their scalars by lane reads.  A chain through LDS or memory costs a load's
// latency per link: 40 to 500 cycles against a few.  255^2 mixed
// 82 -> 51 us a system; 5001 points 21.3 -> 17.1 us; an Arnoldi step of 3001
// unknowns 8.7 -> 6.9 us.  What is left is barriers between the dot products.
#pragma once
#include "pd_scan.h"

__device__ __forceinline__ double pd_readlane(double v, int l) {
  return pd_readlane(cpx<double>{v, 0.0}, l).re;
}

// Sum over the wave, in every lane: prefix sums inside the rows of 16 lanes,
// then across them.
__device__ __forceinline__ double pd_wave_sum(double v) {
  v += pd_dpp<0x111, 0xF>(v, 0.0);   // row_shr:1, 2, 4, 8
  v += pd_dpp<0x112, 0xF>(v, 0.0);
  v += pd_dpp<0x114, 0xF>(v, 0.0);
  v += pd_dpp<0x118, 0xF>(v, 0.0);
  v += pd_dpp<0x142, 0xA>(v, 0.0);   // row_bcast:15, row_bcast:31
  v += pd_dpp<0x143, 0xC>(v, 0.0);
  return pd_readlane(v, 63);
}

// Column j of H, entries 0..j in h's lanes and hn below: the rotations before it
// (cs, sn: lane i holds rotation i), then its own, which lane j keeps.  g is
// g_j on entry; on return h's lanes hold column j of R, gj the rotated g_j and
// g is g_{j+1} (whose modulus is the residual).  j < 64.
__device__ __forceinline__ void pd_givens_column(double &h, double hn, int j, int lane, double &cs,
                                                 double &sn, double &gj, double &g) {
  double a = pd_readlane(h, 0);
  for (int i = 0; i < j; ++i) {
    const double b = pd_readlane(h, i + 1), c = pd_readlane(cs, i), s = pd_readlane(sn, i);
    const double t = c * a + s * b;
    a = -s * a + c * b;
    h = lane == i ? t : h;
  }
  const double rr = hypot(a, hn);
  const double c = (rr == 0.0) ? 1.0 : a / rr, s = (rr == 0.0) ? 0.0 : hn / rr;
  h = lane == j ? rr : h;
  cs = lane == j ? c : cs;
  sn = lane == j ? s : sn;
  gj = c * g;
  g = -s * g;
}

// R y = g for m <= 64 unknowns: lane i holds g_i and gets y_i; col(k) is this
// lane's entry of column k of R (any value in lanes > k).
template <typename Col>
__device__ __forceinline__ double pd_back_substitute(double g, int m, int lane, Col col) {
  double y = 0.0, next = m > 0 ? col(m - 1) : 0.0;
  for (int k = m - 1; k >= 0; --k) {
    const double r = next;
    if (k > 0) next = col(k - 1);   // in flight during this step
    const double d = pd_readlane(r, k), gk = pd_readlane(g, k);
    const double yk = (d != 0.0) ? gk / d : 0.0;
    y = lane == k ? yk : y;
    g -= r * yk;
  }
  return y;
}
