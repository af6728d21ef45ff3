// A plan moved to another stream takes its inner plan (mixed precision) along.
#include "../../paper_2304_12597_amd/csrc/pd_internal.h"

#include <cstdio>

int main() {
  int x = 0, y = 0;
  const hipStream_t a = reinterpret_cast<hipStream_t>(&x), b = reinterpret_cast<hipStream_t>(&y);
  pd_plan_s plain, mixed, inner;
  plain.stream = mixed.stream = inner.stream = a;
  mixed.inner = &inner;
  pd_bind_stream(&plain, b);
  pd_bind_stream(&mixed, b);
  if (plain.stream != b || mixed.stream != b || inner.stream != b) {
    std::printf("a stream was left behind\n");
    return 1;
  }
  std::printf("ok\n");
  return 0;
}
