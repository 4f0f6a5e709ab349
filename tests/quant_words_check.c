/* Checks the kernels' short form of the fp16 quantizer over every input it
 * takes: for every width b = 1..8, every largest magnitude A of a row (positive
 * finite fp16 bits) whose scale s = fp16(A / (2^b - 1)) is normal, and every
 * fp16 x with |x| <= A (both zeros), the word from one fma,
 *   u = bits 16..22 of fma(x', 1 / (2 s), 128 + 2^(b-1)) for b <= 7,
 *   u = bits 15..22 of fma(x', 1 / (2 s), 256 + 128) for b = 8,
 *   x' = x, with values in [-s, 0) replaced by -s and -0 by +0,
 * must equal 2^(b-1) + floor(x / (2 s)), the quotient taken in float64.
 * Prints "tested <count>" and exits 0, or prints the first failure and exits 1.
 * With the argument "plant" the values in [-s, 0) are left as they are, which
 * must fail. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

static float half_value(uint32_t h) {
  const int e = (h >> 10) & 31;
  const int m = h & 1023;
  const float v = e ? ldexpf((float)(1024 + m), e - 25) : ldexpf((float)m, -24);
  return h & 0x8000u ? -v : v;
}

/* fp16 bits of v >= 0, nearest even */
static uint32_t half_bits(float v) {
  int e;
  if (v < 0x1p-14f) return (uint32_t)lrintf(v * 0x1p24f);
  frexpf(v, &e); /* v = f 2^e, 1/2 <= f < 1 */
  const uint32_t m = (uint32_t)lrintf(ldexpf(v, 11 - e)); /* 1024..2048 */
  return ((uint32_t)(e + 13) << 10) + m; /* m = 1024: implicit one adds to the exponent field */
}

int main(int argc, char** argv) {
  static float value[32768];
  const int plant = argc > 1 && strcmp(argv[1], "plant") == 0;
  for (uint32_t h = 0; h < 0x7C00u; ++h) value[h] = half_value(h);
  long long tested = 0;
  int failed = 0;
  for (int b = 1; b <= 8; ++b) {
    static uint32_t top[32768]; /* largest A of each scale */
    memset(top, 0, sizeof top);
    for (uint32_t A = 1; A < 0x7C00u; ++A) top[half_bits(value[A] / (float)((1 << b) - 1))] = A;
    const float base = (b == 8 ? 256.0f : 128.0f) + (float)(1 << (b - 1));
#pragma omp parallel for schedule(dynamic, 64) reduction(+ : tested) reduction(| : failed)
    for (uint32_t sb = 0x0400u; sb < 0x7C00u; ++sb) {
      if (top[sb] == 0) continue;
      const float s = value[sb], rh = (1.0f / s) * 0.5f;
      const double inv = 1.0 / (2.0 * (double)s); /* only to bracket: the floor is corrected below */
      int bad = 0;
      for (uint32_t h = 0; h <= top[sb]; ++h) {
        for (int neg = 0; neg < 2; ++neg) {
          const float x = neg ? -value[h] : value[h];
          float xp = neg && h == 0 ? 0.0f : x;
          if (neg && h > 0 && h < sb && !plant) xp = -s;
          const float f = fmaf(xp, rh, base);
          uint32_t bits;
          memcpy(&bits, &f, 4);
          int want = (int)floor((double)x * inv);
          while ((double)want * 2.0 * (double)s > (double)x) --want;
          while ((double)(want + 1) * 2.0 * (double)s <= (double)x) ++want;
          bad |= (int)((bits >> (b == 8 ? 15 : 16)) & 0xFFu) != want + (1 << (b - 1));
        }
      }
      tested += 2ll * (top[sb] + 1);
      failed |= bad;
    }
  }
  if (failed) {
    printf("the short form differs\n");
    return 1;
  }
  printf("tested %lld\n", tested);
  return 0;
}
