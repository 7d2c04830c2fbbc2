// Host-side check of the arithmetic of the activation quantiser (csrc/fq_common.h), all FP32, IEEE.  For every finite bf16
// absmax > 0 with s = absmax / 448 in [2^-60, 2^60] (every STRIDE-th one; STRIDE = 1 is the exhaustive run):
//   scale       fma(fma(-448, q, absmax), c, q) with c = fp32(1 / 448), q = absmax * c, is the IEEE quotient s
//   reciprocal  fma(fma(-s, r0, 1), r0, r0) is the IEEE quotient r = 1 / s for every r0 within one unit of it
//   quotient    for every bf16 x, |x| <= absmax, both signs (zeros too), the E4M3 code, sign included, of
//               fma(fma(q, s, -x), -r, q) with q = x * r is that of the IEEE quotient x / s
// Exit status 0 = no difference.  usage: activation_quotient_check [STRIDE]
#include <math.h>
#include <omp.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
static inline float from(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static inline uint32_t bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
// E4M3 code of a float with |f| < 464, nearest even: the code whose value plus half a step is reached first
static uint8_t e4m3(float f) {
  const uint32_t u = bits(f);
  const uint8_t sign = (uint8_t)((u >> 24) & 0x80);
  const float a = fabsf(f);
  if (a < 0x1p-6f) return (uint8_t)(sign | (int)nearbyintf(a * 512.0f));       // subnormals, units of 2^-9 (8 of them: the first binade)
  const uint32_t m = u & 0x7FFFFFFFu, r = m + 0x7FFFFu + ((m >> 20) & 1u);      // three fraction bits are left
  return (uint8_t)(sign | ((r >> 20) - (120u << 3)));
}
int main(int argc, char** argv) {
  const int stride = argc > 1 ? atoi(argv[1]) : 1;
  const float c = 1.0f / 448.0f;
  long long bad = 0, total = 0;
  #pragma omp parallel for schedule(dynamic, 16) reduction(+ : bad, total)
  for (int ab = 1; ab < 0x7F80; ab += stride) {
    const float amax = from((uint32_t)ab << 16), s = amax / 448.0f;
    if (!(s >= 0x1p-60f && s <= 0x1p60f)) continue;
    const float sq = amax * c, r = 1.0f / s;
    if (bits(fmaf(fmaf(-448.0f, sq, amax), c, sq)) != bits(s)) ++bad;
    for (int d = -1; d <= 1; ++d) {
      const float r0 = from(bits(r) + (uint32_t)d);
      if (bits(fmaf(fmaf(-s, r0, 1.0f), r0, r0)) != bits(r)) ++bad;
    }
    for (int xb = 0; xb <= ab; ++xb)
      for (uint32_t sg = 0; sg < 2; ++sg) {
        const float x = from(((uint32_t)xb << 16) | (sg << 31)), q = x * r, got = fmaf(fmaf(q, s, -x), -r, q);
        const float want = fminf(fmaxf(x / s, -448.0f), 448.0f);
        ++total;
        if (!(fabsf(got) < 449.0f) || e4m3(got) != e4m3(want)) ++bad;
      }
  }
  printf("total %lld  differences %lld\n", total, bad);
  return bad != 0;
}
