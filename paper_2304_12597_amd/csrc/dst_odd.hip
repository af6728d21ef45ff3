// Orthonormal DST-I of rows of n = N - 1 values, N = 2^m >= 32, two rows a
// transform: with z = ext(a) + i ext(b) the odd extensions of length 2N,
// Z[k] = 2 S_b[k] - 2i S_a[k].
//
// The first radix-8 stage splits z into eight sequences of length M = N / 4,
// w_p[j] = W^{jp} sum_r z[j + r M] e^{-2 pi i r p / 8}, W = e^{-pi i / N}, whose
// transforms are Z[8q + p].  z is odd, so Z[8q + p] = -Z[8(M - 1 - q) + 8 - p]:
// the sequences p = 5, 6, 7 need not be formed.  The butterflies of j and M - j
// take the same eight row values (z negated and reversed gives X'_p =
// -e^{-2 pi i p / 8} X_{8-p}), so one butterfly straight from the rows, with no
// staging of the extension, writes both entries of the five sequences:
//     w_p[j] = X_p W^{jp},   w_p[M - j] = -X_{8-p} conj(W^{jp}).
// The remaining stages run on 5/8 of the points of the FFT of length 2N, and
// nothing is written for the extension: LDS traffic is half of what it was.
// What bounds it now: the rows' bytes.  n = 511, 130816 rows, 1.07 GB: the full
// FFT took 452 us (MODE 0) and 376 us (MODE 2), this 268 and 265 us (4.0 TB/s);
// n = 255, 130560 rows, 0.53 GB: 161 and 180 us before, 116 and 113 us now (4.7 TB/s).
#include "pd_fft.h"
#include "pd_internal.h"

#include <cmath>

namespace {

using namespace pdfft;
using Cx = cpx<double>;

// C row pairs per block; column 5 c + p of LDS holds w_p of pair c.
// MODE 0: rows tau F (+ u0 on the first nu0 elements); 2: rows of in.
// ACC: out += the transform.  out may be in.
template <int MODE, int ACC>
__global__ void __launch_bounds__(320)
dst_odd_kernel(int n, int rows, int C, int stride, double tau, const double *__restrict__ u0,
               long nu0, const double *__restrict__ F, const double *in,
               const Cx *__restrict__ tw, double *out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Cx *lds = reinterpret_cast<Cx *>(smem_raw);
  const int N = n + 1, M = N / 4, lgM = __builtin_ctz(M), tid = threadIdx.x, T = blockDim.x;
  const int r0 = blockIdx.x * 2 * C;
  Cx *twl = lds + 5 * C * stride;
  {
    const int LO = pd_tw_lo(M), E = pd_tw_entries(M);   // of length M: every 8th of tw
    for (int m = tid; m < E; m += T) twl[m] = tw[8 * (m < LO ? m : (m - LO) * 64)];
  }
  const double *src = MODE == 0 ? F : in;
  const int half = C << (lgM - 1);
  if (tid < half + C) {
    const bool mid = tid >= half;   // the butterfly of j = M / 2, its own mirror
    const int c = mid ? tid - half : tid >> (lgM - 1), j = mid ? M / 2 : tid & (M / 2 - 1);
    const int ra = r0 + 2 * c;
    double x[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const long row = ra + h < rows ? ra + h : rows - 1;
      const double *p = src + row * n - 1;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ia = j + r * M, ib = N - ia;
        const bool end = r == 0 && j == 0;   // x_0 = x_N = 0
        const double a = p[end ? 1 : ia], b = p[end ? 1 : ib];
        x[h][r] = end ? 0.0 : a;
        x[h][4 + r] = end ? 0.0 : b;
      }
    }
    if constexpr (MODE == 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const long row = ra + h < rows ? ra + h : rows - 1;
        const double *p = u0 + row * n - 1;
        const bool first = row * n < nu0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ia = j + r * M, ib = N - ia;
          const bool add = first && !(r == 0 && j == 0);
          x[h][r] = tau * x[h][r] + (add ? p[ia] : 0.0);
          x[h][4 + r] = tau * x[h][4 + r] + (add ? p[ib] : 0.0);
        }
      }
    }
    Cx v[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = Cx{x[0][r], x[1][r]};
      v[4 + r] = Cx{-x[0][4 + r], -x[1][4 + r]};
    }
    small_dft<double, false, 8>(v);
    const Cx w1 = tw[j], w2 = cmul(w1, w1), w3 = cmul(w2, w1), w4 = cmul(w2, w2);
    const Cx w[5] = {Cx{1.0, 0.0}, w1, w2, w3, w4};
    Cx *col = lds + (size_t)5 * c * stride + pd_fpad(j);
    Cx *mir = lds + (size_t)5 * c * stride + pd_fpad(M - j);
    const bool both = j != 0 && !mid;
#pragma unroll
    for (int p = 0; p < 5; ++p) {
      col[p * stride] = p ? cmul(v[p], w[p]) : v[0];
      if (both) {
        const Cx y = v[(8 - p) & 7];
        const Cx t = p ? Cx{y.re * w[p].re + y.im * w[p].im, y.im * w[p].re - y.re * w[p].im} : y;
        mir[p * stride] = Cx{-t.re, -t.im};
      }
    }
  }
  __syncthreads();
  fft_lds<double, false>(lds, M, 5 * C, stride, twl);
  const double scale = 0.5 * sqrt(2.0 / (double)N);
  const int lgN = lgM + 2, total = C << lgN;
  constexpr int U = 4;
  for (int base = tid; base < total; base += U * T) {
    Cx s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = base + u * T < total ? base + u * T : 0;
      const int c = idx >> lgN, k = (idx & n) + 1, p = k & 7, q = k >> 3;
      const bool flip = p > 4;
      const int e = flip ? M - 1 - q : (q < M ? q : 0);   // idx & n = n: the padding, not stored
      const Cx z = lds[(size_t)(5 * c + (flip ? 8 - p : p)) * stride + pd_fpad(e)];
      const double g = flip ? -scale : scale;
      s[u] = Cx{-z.im * g, z.re * g};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = base + u * T, c = idx >> lgN, i = idx & n, ra = r0 + 2 * c;
      if (idx >= total || i == n || ra >= rows) continue;
      double *o = out + (size_t)ra * n + i;
      if (ACC) s[u].re += o[0];
      o[0] = s[u].re;
      if (ra + 1 < rows) {
        if (ACC) s[u].im += o[n];
        o[n] = s[u].im;
      }
    }
  }
}

}  // namespace

// tw[m] = exp(-pi i m / (n + 1))
pd_status pd_launch_dst_odd(int n, int rows, int mode, double tau, const double *u0, long nu0,
                            const double *F, const double *in, const double *tw, double *out,
                            int accumulate, hipStream_t stream) {
  const int M = (n + 1) / 4, C = pd_odd_pairs(n), stride = pd_fft_col_stride(M);
  const int T = pd_odd_threads(n);
  if (!pd_odd_ok(n) || T > 320 || T < C * M / 2 + C) return PD_ENOTSUP;
  const Cx *w = reinterpret_cast<const Cx *>(tw);
#define PD_DO(MO, A)                                                                             \
  hipLaunchKernelGGL((dst_odd_kernel<MO, A>), dim3((rows + 2 * C - 1) / (2 * C)), dim3(T),       \
                     pd_odd_lds(n), stream, n, rows, C, stride, tau, u0, nu0, F, in, w, out)
  if (mode == 0) PD_DO(0, 0);
  else if (accumulate) PD_DO(2, 1);
  else PD_DO(2, 0);
#undef PD_DO
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

void pd_dst_odd_set_attributes(size_t max_lds) {
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_odd_kernel<0, 0>), (int)max_lds);
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_odd_kernel<2, 0>), (int)max_lds);
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_odd_kernel<2, 1>), (int)max_lds);
}
