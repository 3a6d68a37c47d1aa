/* exact_quotient and exact_scale against the division: every bf16 significand over every significand of a scale, and every
 * significand of a range over 3 and 15. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#define XSV_QUOTIENT static inline
#include "../../paper_2602_21780_amd/csrc/quotient.h"

static float from_bits(uint32_t b) {
  float f;
  memcpy(&f, &b, 4);
  return f;
}

int main(void) {
  float x[128];
  long wrong_quotients = 0, wrong_scales = 0;
  for (uint32_t i = 0; i < 128; ++i) x[i] = from_bits(0x3f800000u | (i << 16));
  for (uint32_t m = 0; m < (1u << 23); ++m) {
    const float s = from_bits(0x3f800000u | m), y = 1.0f / s;
    int bad = 0;
    for (int i = 0; i < 128; ++i) bad += exact_quotient(x[i], s, y) != x[i] / s;
    wrong_quotients += bad;
    wrong_scales += exact_scale(s, 3.0f, 1.0f / 3.0f) != s / 3.0f;
    wrong_scales += exact_scale(s, 15.0f, 1.0f / 15.0f) != s / 15.0f;
  }
  printf("%ld %ld\n", wrong_quotients, wrong_scales);
  return wrong_quotients != 0 || wrong_scales != 0;
}
