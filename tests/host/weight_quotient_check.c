// Host-side check of the quotient the weight quantiser kernel computes (csrc/fq_wquant.hip): for every E4M3 number
// s > 0 up to a power of two (significands 8 .. 15 and 1 .. 7; scaling both operands by a power of two moves nothing) and
// every STRIDE-th FP32 x with s / 8 <= x <= 16 s, rint of
//     fma(fma(-q, s, x), r, q),  q = x * r,  r = 1 / s        (all FP32, IEEE)
// must equal rint of the IEEE quotient x / s.  (Below s / 8 both round to 0: the correction is at most |q|.  The sign
// of x changes nothing.)  Exit status 0 = no difference.
// usage: weight_quotient_check [STRIDE]
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
static inline uint32_t bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
static inline float from(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
int main(int argc, char** argv) {
  const uint32_t stride = argc > 1 ? (uint32_t)atoi(argv[1]) : 1u;
  long long bad = 0, total = 0;
  for (int m = 1; m < 16; ++m) {
    const float s = (float)m * 0.015625f;                  // (any power of two)
    const float r = 1.0f / s;
    const uint32_t lo = bits(0.125f * s), hi = bits(16.0f * s);
    #pragma omp parallel for schedule(static) reduction(+ : bad, total)
    for (uint32_t b = lo; b <= hi; b += stride) {
      const float x = from(b);
      const float q = x * r;
      const float got = fmaf(fmaf(-q, s, x), r, q);
      ++total;
      if (rintf(got) != rintf(x / s)) ++bad;
    }
  }
  printf("total %lld  code differences %lld\n", total, bad);
  return bad != 0;
}
