// Launch shapes and LDS layouts of kernels whose index arithmetic depends on
// them: plain functions of the sizes, for the kernels, their launches and host
// checks over every admitted size alike (no HIP needed).
#pragma once
#include <cstddef>

#ifdef __HIPCC__
#define PD_SHAPE __host__ __device__ __forceinline__
#else
#define PD_SHAPE inline
#endif

// LDS column layout of the time and DST transforms: entry i of a column sits
// at pd_fpad(i) = i + i/8, which spreads the power-of-two strides of the
// Stockham stages over all LDS banks; columns are pd_fft_col_stride(N)
// entries apart (odd, so that columns start on different banks).
PD_SHAPE int pd_fpad(int i) { return i + (i >> 3); }
PD_SHAPE int pd_fft_col_stride(int N) {
  const int s = pd_fpad(N - 1) + 1;
  return s | 1;
}
// Twiddles of a length-N transform in LDS: lo[m] = w^m for m < min(N, 64) and
// hi[h] = w^(64 h) for h < max(N / 64, 1); w^m = hi[m / 64] lo[m % 64].
PD_SHAPE int pd_tw_lo(int N) { return N < 64 ? N : 64; }
PD_SHAPE int pd_tw_entries(int N) { return pd_tw_lo(N) + (N < 64 ? 1 : N / 64); }

// ---- the DST as a product (dst_dense.hip) ----
constexpr int PD_DENSE_ROWS = 32;   // rows per block
constexpr int PD_DENSE_MAX = 440;
struct DenseShape {
  int kv, ki, ko, stride, tiles, waves;
};
PD_SHAPE DenseShape pd_dense_shape(int n) {
  DenseShape s;
  s.kv = (n + 1) / 2;                  // inputs and outputs of the odd part
  s.ki = (s.kv + 7) / 8 * 8;           // inputs: two steps of 4 at a time
  s.ko = (s.kv + 15) / 16 * 16;        // outputs: tiles of 16
  s.stride = s.ki + 2;                 // 2 x odd: 16 rows' pairs of inputs on distinct banks
  s.tiles = s.ko / 16;
  const int rounds = (s.tiles + 9) / 10;
  s.waves = (s.tiles + rounds - 1) / rounds;
  if (s.waves < 8) s.waves = 8;        // 4 rows a wave in the load
  return s;
}
PD_SHAPE size_t pd_dense_lds(const DenseShape &s) {
  return 2 * (size_t)PD_DENSE_ROWS * s.stride * sizeof(double);
}
PD_SHAPE int pd_dense_loads(const DenseShape &s) { return (s.ki + 63) / 64; }   // per row and lane

// ---- the DST of 2^m - 1 by the odd extension (dst_odd.hip) ----
// n + 1 a power of two, at least 32 (a thread per butterfly and the M / 2
// ones); 2D plans end at n = 1024.
PD_SHAPE bool pd_odd_ok(int n) { return ((n + 1) & n) == 0 && n >= 31 && n <= 1023; }
PD_SHAPE int pd_odd_pairs(int n) { return 512 / ((n + 1) / 4); }   // 5 waves, three blocks to a CU
PD_SHAPE int pd_odd_threads(int n) {
  return (5 * pd_odd_pairs(n) * ((n + 1) / 4) / 8 + 63) / 64 * 64;
}
PD_SHAPE size_t pd_odd_lds(int n) {
  const int M = (n + 1) / 4;
  return ((size_t)5 * pd_odd_pairs(n) * pd_fft_col_stride(M) + pd_tw_entries(M)) * 16;
}

// ---- 2D line solves in the recurrence form (line2d.hip) ----
// Rows and threads of a line, lines of a block.
struct LineShape {
  int MR, P, S;
};
PD_SHAPE LineShape pd_line_shape(int n) {
  LineShape L;
  L.MR = (n <= 64) ? 4 : 8;
  L.P = 1;
  while (L.P * L.MR < n) L.P *= 2;
  L.S = 1;
  while (L.P * L.S * 2 <= 512) L.S *= 2;
  if (L.S > n) {
    L.S = 1;
    while (L.S * 2 <= n) L.S *= 2;
  }
  return L;
}
// Entry i of a line at i + i/8 (a thread's 8 rows 9 apart), lines apart so that
// the 16 lanes of a staging access, 16 / S rows of S lines, fall on different
// banks.
PD_SHAPE int pd_line_entry(int i) { return i + (i >> 3); }
PD_SHAPE int pd_line_stride(int n, int S) {
  const int e = pd_line_entry(n - 1);
  return S < 16 ? (e + 16) / 16 * 16 + 16 / S : (e + 1) | 1;
}
constexpr int pd_line_constants(int MR) { return 9 + MR; }
PD_SHAPE size_t pd_line_lds(int n, const LineShape &L) {
  return (size_t)L.S * (pd_line_stride(n, L.S) + pd_line_constants(L.MR)) * 16;
}

// ---- general matrices by two recurrences (tridiag_lu.hip) ----
constexpr int PD_LU_ROWS = 8;      // rows per thread
constexpr int PD_LU_BLOCK = 512;   // threads of a block
PD_SHAPE int pd_lu_threads(int n) {   // of a group: a power of two, whole waves
  int P = 64;
  while (P * PD_LU_ROWS < n) P *= 2;
  return P;
}
// entry of row i of a group's staging area: 8 rows of a thread 9 apart
PD_SHAPE int pd_lu_entry(int i) { return i + (i >> 3); }
// entries of a group: one halo row each side
PD_SHAPE int pd_lu_group(int P) { return pd_lu_entry(P * PD_LU_ROWS + 1) + 1; }
PD_SHAPE size_t pd_lu_lds(int P, int spb) { return (size_t)spb * pd_lu_group(P) * 16; }
