// Host-side check of two short divisions in the weight quantiser kernel (csrc/fq_wquant.hip), all FP32, IEEE:
//   sigma = x / 7 as  q = x * c, fma(fma(-7, q, x), c, q)  with c = fp32(1 / 7): every significand of x (scaling by a power of
//           two moves nothing while the residual is normal: x from 2^-100 on; below, sigma is far under the smallest E4M3 number)
//   r = 1 / s as  fma(fma(-s, r0, 1), r0, r0)  from any r0 within one unit of the quotient: every E4M3 significand s
// Exit status 0 = no difference from the IEEE quotients.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
static inline uint32_t bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
static inline float from(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
int main(void) {
  long long bad = 0;
  const float c = 1.0f / 7.0f, scales[3] = {0x1p-100f, 1.0f, 0x1p100f};
  for (int k = 0; k < 3; ++k)
    for (uint32_t f = 0; f < (1u << 23); ++f) {
      const float x = from(0x3F800000u | f) * scales[k], q = x * c;
      if (bits(fmaf(fmaf(-7.0f, q, x), c, q)) != bits(x / 7.0f)) ++bad;
    }
  for (int e = -9; e <= 8; ++e)
    for (int m = 8; m < 16; ++m) {
      const float s = ldexpf((float)m, e - 3), r = 1.0f / s;
      for (int d = -1; d <= 1; ++d) {
        const float r0 = from(bits(r) + (uint32_t)d);
        if (bits(fmaf(fmaf(-s, r0, 1.0f), r0, r0)) != bits(r)) ++bad;
      }
    }
  printf("differences %lld\n", bad);
  return bad != 0;
}
