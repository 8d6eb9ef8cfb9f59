// Host check of quot_rn, compiled from the library's header: equal to the division
// rounded once, bit for bit, for divisors a caller may ask for (finite, positive).
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <random>

#include "smki_internal.h"

static long bad = 0, small = 0, cases = 0;

static void check(float a, float b) {
  const float got = quot_rn(a, 1.0 / (double)b, b), want = a / b;
  ++cases;
  if (std::fabs((double)a / (double)b) < 0x1p-120) ++small;   // the branch that divides
  uint32_t g, w;
  memcpy(&g, &got, 4);
  memcpy(&w, &want, 4);
  const bool same = std::isnan(want) ? std::isnan(got) : g == w;
  if (!same && ++bad < 20) printf("wrong: %a / %a = %a, not %a\n", a, b, want, got);
}

int main() {
  std::mt19937 rng(7);
  auto positive = [&]() {   // any finite positive float, subnormals included
    const uint32_t u = rng() % 0x7F7FFFFFu + 1;
    float f;
    memcpy(&f, &u, 4);
    return f;
  };
  const float special[] = {0.0f, -0.0f, 0x1p-149f, 0x1p-126f, 0x1.fffffep-127f, 1.0f, 0x1p-120f,
                           0x1.fffffep127f, INFINITY, NAN};
  for (long i = 0; i < 3'000'000; ++i) {
    const float a = positive(), b = positive();
    check(a, b);
    check(-a, b);
  }
  for (int i = 0; i < 20'000; ++i) {
    const float b = positive();
    for (float a : special) {
      check(a, b);
      check(-a, b);
    }
  }
  // numerators whose quotients lie around 2^-120 and in the subnormal range
  for (int i = 0; i < 1'000'000; ++i) {
    const float b = std::ldexp(1.0f + (float)(rng() >> 9) * 0x1p-23f, (int)(rng() % 60) - 30);
    const float m = 1.0f + (float)(rng() >> 9) * 0x1p-23f;
    check((float)std::ldexp((double)m * b, -120 + (int)(rng() % 3) - 1), b);
    check((float)std::ldexp((double)m * b, -126 - (int)(rng() % 24)), b);
  }
  // quotients that are midpoints of subnormals: an inexact product would turn them
  for (int i = 0; i < 1'000'000; ++i) {
    const float b = std::ldexp((float)((rng() & 0x7FFu) | 1u), (int)(rng() % 80) + 20);
    const double q = std::ldexp((double)((rng() & 0xFFFu) | 1u), -150);
    check((float)(q * b), b);
  }
  // numerators next to (a midpoint of binary32) x (the divisor)
  for (float b : {0.05f, 0.1f, 0.2f, 0.25f, 0.3f, 1.0f / 3.0f, 0.3002929985523224f, 7.0f})
    for (int i = 0; i < 200'000; ++i) {
      const double m = std::ldexp((double)((rng() >> 8) | (1u << 24) | 1u), -(int)(rng() % 40));
      const float a = (float)(m * b);
      for (float v : {a, std::nextafter(a, 0.0f), std::nextafter(a, INFINITY)}) check(v, b);
    }
  printf("%ld quotients, %ld below 2^-120\n", cases, small);
  if (bad || small < 100'000) return printf("%ld wrong\n", bad), 1;
  printf("ok\n");
  return 0;
}
