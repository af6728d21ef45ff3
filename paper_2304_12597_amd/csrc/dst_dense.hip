// Orthonormal DST-I of many short rows as a product on the matrix cores.
//
// With u_j = x_j - x_{N-j} and v_j = x_j + x_{N-j} (N = n + 1; v_{N/2} = x_{N/2}
// for even N) the transform splits into two real products of half the size,
//
//     S_{2m} = sum_j u_j sin(2 pi j m / N),   S_{2m-1} = sum_j v_j sin(pi j (2m-1) / N),
//
// n^2 multiply-adds a row (v_mfma_f64_16x16x4: 72 TFLOP/s here), against two
// FFTs of length 2^ceil(log2(2n-1)) with four LDS passes each in chirp-z form.
// A block folds 32 rows into LDS; a wave takes 16 outputs of each parity for
// all 32 rows, so that a lane holds pairs S_{2m-1}, S_{2m} of adjacent addresses
// and stores them straight from its accumulators.  The sines come from L2 in the
// order of the lanes (16 bytes a lane for two steps).  Blocks walk over the
// rows, two to a CU, and load the next 32 while the products run.
// What bounds it: the products (n = 256, 65536 rows: 55 us at the peak rate) and
// the rows' bytes (56 us) about equally.  Measured there: chirp-z 310 us (MODE
// 0) and 282 us (MODE 2), this 115 and 106 us (matrix cores busy 62% of it).
// With few rows or many points the chirp-z form wins (pd_dst_dense_pays).
#include "pd_internal.h"

#include <cmath>

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double pair8 __attribute__((ext_vector_type(2), aligned(8)));   // rows start on 8 bytes
constexpr int RB = PD_DENSE_ROWS;

// Fragments: [tile][chunk of 8 inputs][part: v, u][lane][2 steps]; lane l holds
// output 16 tile + l % 16 + 1 and input 8 chunk + 2 (l / 16) + step + 1.
// q[m] = sin(pi m / N), m = 0..2N-1.
__global__ void __launch_bounds__(256)
dense_table_kernel(int n, double scale, const double *__restrict__ q, double *__restrict__ tab) {
  const DenseShape s = pd_dense_shape(n);
  const int chunks = s.ki / 8, N = n + 1;
  const long total = (long)s.tiles * chunks * 256;
  for (long e = blockIdx.x * 256L + threadIdx.x; e < total; e += 256L * gridDim.x) {
    const int step = e & 1, l = (int)(e >> 1) & 63, part = (int)(e >> 7) & 1;
    const long tc = e >> 8;
    const int c = (int)(tc % chunks), t = (int)(tc / chunks);
    const int m = 16 * t + (l & 15) + 1, j = 8 * c + 2 * (l >> 4) + step + 1;
    const int k = part == 0 ? 2 * m - 1 : 2 * m;
    const bool in = k <= n && (part == 0 ? 2 * j <= N : 2 * j < N);
    tab[e] = in ? scale * q[(int)((long)j * k % (2 * N))] : 0.0;
  }
}

// MODE 0: rows h = tau F (+ u0 on the first nu0 elements); 2: rows of in.
// ACC: out += the transform.  out may be in.  JI: loads per row and lane,
// ceil(ki / 64).  NF: groups of 16 rows per wave (1: so few tiles that two
// waves share one).  The next 32 rows are loaded while the products run.
template <int MODE, int ACC, int JI, int NF>
__global__ void __launch_bounds__(640, JI <= 2 ? 4 : 1)
dst_dense_kernel(int n, int rows, double tau, const double *__restrict__ u0, long nu0,
                 const double *__restrict__ F, const double *in, const double *__restrict__ tab,
                 double *out) {
  extern __shared__ __align__(16) double fold[];   // [part][RB][stride]
  const DenseShape s = pd_dense_shape(n);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int N = n + 1, nblk = (rows + RB - 1) / RB;
  const double *src = MODE == 0 ? F : in;
  constexpr int RW = RB / 8;
  double xa[RW][JI], xb[RW][JI];
  auto load = [&](int blk) {
#pragma unroll
    for (int u = 0; u < RW; ++u) {
      const int r = blk * RB + wv + u * s.waves;
      const double *p = src + (long)(r < rows ? r : rows - 1) * n - 1;
#pragma unroll
      for (int i = 0; i < JI; ++i) {
        const int j = lane + 1 + 64 * i, ja = 2 * j <= N ? j : 1;
        xa[u][i] = p[ja];
        xb[u][i] = p[N - ja];
      }
    }
  };
  load(blockIdx.x);
  const int chunks = s.ki / 8;
  const int f0 = NF == 1 ? wv & 1 : 0;
  const double *lv = fold + ((lane & 15) + 16 * f0) * s.stride + 2 * (lane >> 4);
  const int fr = 16 * s.stride, up = RB * s.stride;
  for (int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int r0 = blk * RB;
    if (blk != (int)blockIdx.x) __syncthreads();   // the rows before have been used
#pragma unroll
    for (int u = 0; u < RW; ++u) {
      const int r = wv + u * s.waves;
      const long base = (long)(r0 + r) * n - 1;
#pragma unroll
      for (int i = 0; i < JI; ++i) {
        const int j = lane + 1 + 64 * i;
        const bool pair = 2 * j < N, mid = 2 * j == N;
        double a = xa[u][i], b = xb[u][i];
        if constexpr (MODE == 0) {
          a *= tau;
          b *= tau;
          if (r0 + r < rows && base + 1 < nu0 && 2 * j <= N) {
            a += u0[base + j];
            b += u0[base + N - j];
          }
        }
        if (r < RB && j <= s.ki) {
          fold[r * s.stride + j - 1] = pair ? a + b : (mid ? a : 0.0);
          fold[(RB + r) * s.stride + j - 1] = pair ? a - b : 0.0;
        }
      }
    }
    __syncthreads();
    const int next = blk + gridDim.x;
    load(next < nblk ? next : blk);
    for (int t = NF == 1 ? wv >> 1 : wv; t < s.tiles; t += NF == 1 ? s.waves / 2 : s.waves) {
      const double2 *tb = reinterpret_cast<const double2 *>(tab) + (size_t)t * chunks * 128 + lane;
      v4d ov[NF] = {}, ev[NF] = {};   // odd and even outputs of the groups
#pragma unroll 4
      for (int c = 0; c < chunks; ++c) {
        const double2 bv = tb[c * 128], bu = tb[c * 128 + 64];
        const double *a = lv + 8 * c;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const double2 av = *reinterpret_cast<const double2 *>(a + f * fr);
          const double2 au = *reinterpret_cast<const double2 *>(a + f * fr + up);
          ov[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.x, ov[f], 0, 0, 0);
          ev[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(au.x, bu.x, ev[f], 0, 0, 0);
          ov[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, bv.y, ov[f], 0, 0, 0);
          ev[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(au.y, bu.y, ev[f], 0, 0, 0);
        }
      }
      const int i = 2 * (16 * t + (lane & 15));   // S_{i+1}, S_{i+2} at i, i + 1
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = r0 + 16 * (f + f0) + (lane >> 4) + 4 * q;
          if (row >= rows || i >= n) continue;
          double *o = out + (size_t)row * n + i;
          if (i + 1 < n) {
            pair8 v = {ov[f][q], ev[f][q]};
            if constexpr (ACC) v += *reinterpret_cast<const pair8 *>(o);
            *reinterpret_cast<pair8 *>(o) = v;
          } else {
            *o = ACC ? *o + ov[f][q] : ov[f][q];
          }
        }
    }
  }
}

template <int MODE, int ACC, int JI>
void dense_launch(const DenseShape &s, int n, int rows, double tau, const double *u0, long nu0,
                  const double *F, const double *in, const double *frag, double *out,
                  hipStream_t stream) {
  const size_t lds = pd_dense_lds(s);
  const int nblk = (rows + RB - 1) / RB, fit = lds <= 80 * 1024 ? 512 : 256;
  const dim3 grid(nblk < fit ? nblk : fit), block(64 * s.waves);
  if (JI == 1 && s.tiles <= 4)
    hipLaunchKernelGGL((dst_dense_kernel<MODE, ACC, 1, 1>), grid, block, lds, stream, n, rows, tau,
                       u0, nu0, F, in, frag, out);
  else
    hipLaunchKernelGGL((dst_dense_kernel<MODE, ACC, JI, 2>), grid, block, lds, stream, n, rows, tau,
                       u0, nu0, F, in, frag, out);
}

}  // namespace

// Doubles of the sine table and its fragments; 0: the FFT forms.  The products
// take n^2 / 72 TFLOP/s a row, the chirp-z form grows with its FFT length:
// per row 1.4 against 3.4 ns at n = 100, 3.0 / 5.1 at 200, 5.4 / 10.9 at 300,
// 9.3 / 11.2 at 400, 12.7 / 11.3 at 500 (4096 rows).  Where n + 1 is a power of
// two the FFT of half the length wins: n = 255, 130560 rows: 161 us, product 218.
size_t pd_dst_dense_doubles(int n) {
  if (n < 16 || n > PD_DENSE_MAX || ((n + 1) & n) == 0) return 0;
  const DenseShape s = pd_dense_shape(n);
  return 2 * (size_t)(n + 1) + (size_t)s.tiles * (s.ki / 8) * 256;
}

// Whether the product is the faster form for this many rows.  Its time hardly
// depends on them until every CU has its blocks of 32 (one a CU for n > 316, else
// two), and is that of one block, which grows with n^2; the chirp-z form takes one
// or two rows a block and grows from some 1000 rows on.  Chirp-z / product, us:
// n = 100: 9.1 / 4.5 at 2 rows, 13.4 / 5.4 at 4096; n = 160: 8.7 / 8.8 and 20.2 /
// 10.1; n = 200: 9.6 / 10.9 at 512, 13.3 / 11.3 at 2048; n = 300: 16.5 / 20.3 at 1024,
// 25.1 / 20.8 at 2048; n = 400: 25.5 / 34.6 at 2048, 44.8 / 37.0 at 4096; n = 440:
// 11.3 / 35.5 at 2, 45.1 / 41.1 at 4096.
bool pd_dst_dense_pays(int n, long rows) {
  return n <= 144 || rows >= (n <= 316 ? 6L : 10L) * n;
}

// q (2N doubles at the start of the table) is in place on the stream.
pd_status pd_dst_dense_build(int n, double *tab, hipStream_t stream) {
  hipLaunchKernelGGL(dense_table_kernel, dim3(64), dim3(256), 0, stream, n, sqrt(2.0 / (n + 1)),
                     tab, tab + 2 * (size_t)(n + 1));
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

pd_status pd_launch_dst_dense(int n, int rows, int mode, double tau, const double *u0, long nu0,
                              const double *F, const double *in, const double *tab, double *out,
                              int accumulate, hipStream_t stream) {
  const DenseShape s = pd_dense_shape(n);
  const double *frag = tab + 2 * (size_t)(n + 1);
#define PD_DD(J)                                                                                \
  do {                                                                                          \
    if (mode == 0)                                                                              \
      dense_launch<0, 0, J>(s, n, rows, tau, u0, nu0, F, in, frag, out, stream);                \
    else if (accumulate)                                                                        \
      dense_launch<2, 1, J>(s, n, rows, tau, u0, nu0, F, in, frag, out, stream);                \
    else                                                                                        \
      dense_launch<2, 0, J>(s, n, rows, tau, u0, nu0, F, in, frag, out, stream);                \
  } while (0)
  switch (pd_dense_loads(s)) {
    case 1: PD_DD(1); break;
    case 2: PD_DD(2); break;
    case 3: PD_DD(3); break;
    case 4: PD_DD(4); break;
    default: return PD_ENOTSUP;   // n <= 440: ki <= 224
  }
#undef PD_DD
  PD_HIP_CHECK(hipGetLastError());
  return PD_OK;
}

namespace {
template <int MODE, int ACC>
void dense_attributes(int v) {
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_dense_kernel<MODE, ACC, 1, 1>), v);
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_dense_kernel<MODE, ACC, 1, 2>), v);
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_dense_kernel<MODE, ACC, 2, 2>), v);
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_dense_kernel<MODE, ACC, 3, 2>), v);
  pd_set_max_lds(reinterpret_cast<const void *>(&dst_dense_kernel<MODE, ACC, 4, 2>), v);
}
}  // namespace

void pd_dst_dense_set_attributes(size_t max_lds) {
  dense_attributes<0, 0>((int)max_lds);
  dense_attributes<2, 0>((int)max_lds);
  dense_attributes<2, 1>((int)max_lds);
}
