// Host-side check of the HiF4 quantizers' element arithmetic (device_fp4.h, compiled for the host):
//  - hif4_round against the comparison with every midpoint in float64 (exact there), for every
//    level-1 fraction m and shift b: all float32 within 2^15 places of each midpoint and of the
//    saturation, strided float32 in between and far outside, at several exponents of the scale;
//  - zeros, subnormals, infinities (saturate) and NaN (code 0, no other element touched);
//  - hif4_code_bytes: magnitude and sign of x for every element position;
//  - hif4_c1 at each threshold 1.75 s1(c) and one place around it, and for strided float32.
//
// Usage: hif4_round_check [plant]; plant = 1 rounds the reference's ties up, plant = 2 expects the
// threshold itself in the next code: each must be reported.
#include <cstdio>
#include <cstdlib>
#include <limits>

#include "device_fp4.h"

using namespace resq;

static int g_errors = 0;

static void fail(const char* what, int c1, int b, float x, double got, double want) {
  if (g_errors < 20) std::printf("  FAIL %s: c1 %d b %d x %a: %g, expected %g\n", what, c1, b, (double)x, got, want);
  ++g_errors;
}

int main(int argc, char** argv) {
  const int plant = argc > 1 ? std::atoi(argv[1]) : 0;
  const float inf = std::numeric_limits<float>::infinity(), nan = std::numeric_limits<float>::quiet_NaN();
  long long n = 0;
  for (int e : {0, 1, 17, 31, 46, 62, 63})
    for (int m = 0; m < 4; ++m)
      for (int b = 0; b < 3; ++b) {
        const int c1 = 4 * e + m;
        const Hif4Grid g = hif4_grid(c1, hif4_inv_q(c1), b);
        const double step = std::ldexp(4.0 + m, e - 35 - b);
        if ((double)g.step != step) fail("step", c1, b, 0.f, g.step, step);
        auto want = [&](float x) {  // midpoints passed: a tie goes to the even neighbour
          int k = 0;
          for (int j = 0; j < 7; ++j) {
            const double mid = (j + 0.5) * step, ax = std::fabs((double)x);
            if (ax > mid || (ax == mid && (j % 2 == 1 || plant == 1))) k = j + 1;
          }
          return k;
        };
        auto check = [&](float x) {
          ++n;
          const float k = hif4_round(x, g);
          if (std::fabs(k) != (float)want(x)) fail("round", c1, b, x, k, want(x));
        };
        for (int j = 0; j < 8; ++j) {
          const float mid = (float)((j + 0.5) * step);
          const uint32_t u = __float_as_uint(mid);
          for (int d = -(1 << 15); d <= (1 << 15); ++d) {
            check(__uint_as_float(u + d));
            if ((d & 63) == 0) check(-__uint_as_float(u + d));
          }
        }
        for (uint32_t u = 0; u < 0x7F800000u; u += 1009u + 977u * (u % 3)) check(__uint_as_float(u));
        for (float x : {0.f, -0.f, 1e-45f, -1e-45f, std::numeric_limits<float>::min(), 3.4028234e38f, -3.4028234e38f}) check(x);
        for (float x : {inf, -inf})
          if (std::fabs(hif4_round(x, g)) != 7.f) fail("infinity", c1, b, x, hif4_round(x, g), 7);
        for (float x : {nan, -nan})
          if (std::fabs(hif4_round(x, g)) != 0.f) fail("NaN", c1, b, x, hif4_round(x, g), 0);
        const float xs[10] = {0.f, -0.f, (float)step, (float)(-3 * step), (float)(6 * step), inf, -inf, nan, -nan, (float)(-0.2 * step)};
        const uint32_t codes[10] = {0, 8, 1, 11, 6, 7, 15, 0, 8, 8};
        for (int i = 0; i < 10; ++i)
          for (int at = 0; at < 4; ++at) {
            float x[4] = {(float)step, (float)(2 * step), (float)(-3 * step), (float)(4 * step)}, k[4];
            uint32_t w[4] = {1, 2, 11, 4};
            x[at] = xs[i];
            w[at] = codes[i];
            for (int q = 0; q < 4; ++q) k[q] = hif4_round(x[q], g);
            const uint32_t got = hif4_code_bytes(k, x), exp = w[0] | w[1] << 8 | w[2] << 16 | w[3] << 24;
            if (got != exp) fail("code bytes", c1, b, xs[i], got, exp);
          }
      }
  // level-1 codes
  for (int c = 0; c < 256; ++c) {
    const float t = (float)(1.75 * std::ldexp(1 + (c & 3) / 4.0, (c >> 2) - 31));
    const int at = plant == 2 && c < 255 ? c + 1 : c;
    if (hif4_c1(t) != at) fail("c1 at its threshold", c, 0, t, hif4_c1(t), at);
    const float above = std::nextafter(t, inf), below = std::nextafter(t, 0.f);
    if (hif4_c1(above) != std::min(c + 1, 255)) fail("c1 above", c, 0, above, hif4_c1(above), c + 1);
    if (hif4_c1(below) != c) fail("c1 below", c, 0, below, hif4_c1(below), c);
  }
  int last = 0;
  for (uint32_t u = 0; u <= 0x7F800000u; u += 127u) {
    const int c = hif4_c1(__uint_as_float(u));
    if (c < last || c > 255) fail("c1 order", c, 0, __uint_as_float(u), c, last);
    last = c;
  }
  if (hif4_c1(0.f) != 0 || hif4_c1(inf) != 255) fail("c1 ends", 0, 0, 0.f, hif4_c1(0.f), 0);
  std::printf("%lld values, %d errors\n", n, g_errors);
  return g_errors == 0 ? 0 : 1;
}
