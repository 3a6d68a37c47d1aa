// The two divisions of the quantizers without a division instruction.  Plain C, so that the exhaustive check of their exactness
// (tests/c/quotient_check.c) runs on the very code that the kernels inline.  XSV_QUOTIENT: the function qualifiers.
// To be compiled without contraction of products and sums (every rounding below is meant).
#ifndef XSV_QUOTIENT_H_
#define XSV_QUOTIENT_H_

// x / s rounded to nearest, bit for bit the IEEE quotient, for x a bf16 number, from y = RN(1 / s): a product and one
// correction with its remainder.  That one correction is enough holds for every pair of an 8-bit significand x and a 24-bit
// significand s (2^30 quotients; the exponents do not matter while nothing over- or underflows); a second one would be needed
// only for x of full precision.  For |x / s| < 1/2 the intermediates may lose bits to underflow, which cannot move rint() of
// the result off zero.
XSV_QUOTIENT float exact_quotient(float x, float s, float y) {
  const float q = x * y;
  return __builtin_fmaf(__builtin_fmaf(-q, s, x), y, q);
}

// RN(d / levels), levels = 3 or 15, by the same one correction; inv = RN(1 / levels).  Holds for every significand of d.
XSV_QUOTIENT float exact_scale(float d, float levels, float inv) {
  const float s = d * inv;
  return __builtin_fmaf(__builtin_fmaf(-s, levels, d), inv, s);
}

#endif
