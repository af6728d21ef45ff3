// The launch shapes and LDS layouts that the kernels use (pd_shapes.h), over
// every size that they admit: each row or pair has its own place inside the
// launch's LDS, and the threads cover their work.
#include "../../paper_2304_12597_amd/csrc/pd_shapes.h"

#include <cstdio>
#include <set>
#include <vector>

static int failures = 0;
#define CHECK(x)                                          \
  do {                                                    \
    if (!(x)) {                                           \
      std::printf("size %d: %s\n", size, #x);             \
      ++failures;                                         \
    }                                                     \
  } while (0)
constexpr size_t LDS = 160 * 1024;

int main() {
  for (int size = 16; size <= PD_DENSE_MAX; ++size) {
    const DenseShape s = pd_dense_shape(size);
    CHECK(s.kv == (size + 1) / 2 && s.ki >= s.kv && s.ki % 8 == 0 && s.ko >= s.kv && s.ko % 16 == 0);
    CHECK(s.tiles * 16 == s.ko && 2 * s.ko >= size);
    // a wave takes every s.waves-th tile; 4 rows a wave in the load
    CHECK(s.waves <= 10 && 4 * s.waves >= PD_DENSE_ROWS);
    CHECK(pd_dense_loads(s) <= 4 && 64 * pd_dense_loads(s) >= s.ki);
    // inputs 1..ki of a row below the next row's; both parts inside the LDS
    CHECK(s.ki <= s.stride && pd_dense_lds(s) <= LDS);
    std::set<int> banks;
    for (int r = 0; r < 16; ++r) banks.insert(2 * r * s.stride % 64);
    CHECK(banks.size() == 16);
  }
  for (int size = 1; size <= 2047; ++size) {
    if (!pd_odd_ok(size)) continue;
    const int M = (size + 1) / 4, C = pd_odd_pairs(size), T = pd_odd_threads(size);
    const int stride = pd_fft_col_stride(M);
    CHECK(C >= 1 && T <= 320 && T % 64 == 0);
    CHECK(C * M / 2 + C <= T);                     // a thread per butterfly and middle one
    CHECK(5 * C * M <= 8 * T);                     // the FFT stages' eight points a thread
    CHECK(pd_fpad(M - 1) < stride);
    CHECK(((size_t)5 * C * stride + pd_tw_entries(M)) * 16 <= pd_odd_lds(size));
    CHECK(pd_odd_lds(size) <= LDS);
  }
  for (int size = 2; size <= 512; ++size) {
    const LineShape L = pd_line_shape(size);
    const int stride = pd_line_stride(size, L.S), NF = pd_line_constants(L.MR);
    CHECK(L.P <= 64 && L.P * L.MR >= size && L.P * L.S <= 512 && L.S <= size);
    std::vector<char> used((size_t)L.S * stride, 0);
    for (int g = 0; g < L.S; ++g)
      for (int i = 0; i < size; ++i) {
        const int e = g * stride + pd_line_entry(i);
        CHECK(e < L.S * stride && !used[e]);
        if (e < L.S * stride) used[e] = 1;
      }
    // the staging step y0 + u P of 8 rows a thread
    if (L.MR == 8) {
      CHECK(L.P % 8 == 0 && L.P >= 16);
      for (int y = 0; y < L.P; ++y)
        for (int u = 0; u < 8; ++u)
          CHECK(pd_line_entry(y + u * L.P) == pd_line_entry(y) + u * (L.P + (L.P >> 3)));
    }
    // a thread's share of the constants: 2 with 8 rows, else all of a line
    CHECK(L.S * NF <= L.P * L.S * (L.MR == 8 ? 2 : NF));
    CHECK(((size_t)L.S * stride + (size_t)L.S * NF) * 16 <= pd_line_lds(size, L));
    CHECK(pd_line_lds(size, L) <= 82 * 1024);      // two blocks to a CU
  }
  for (int size = 2; size <= 4096; ++size) {
    const int P = pd_lu_threads(size), spb = PD_LU_BLOCK / P, gs = pd_lu_group(P);
    CHECK(P % 64 == 0 && P <= PD_LU_BLOCK && P * PD_LU_ROWS >= size && spb * P == PD_LU_BLOCK);
    // rows -1..P MR of a group, the halo rows among them, apart and in order
    int last = -1;
    for (int i = 0; i <= P * PD_LU_ROWS + 1; ++i) {
      CHECK(pd_lu_entry(i) > last);
      last = pd_lu_entry(i);
    }
    CHECK(last < gs && (size_t)spb * gs * 16 <= pd_lu_lds(P, spb) && pd_lu_lds(P, spb) <= LDS);
  }
  if (failures) return 1;
  std::printf("ok\n");
  return 0;
}
