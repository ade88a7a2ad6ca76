// fp64 exponential for non-positive arguments, shared by the sampling acceptance kernels: internal
// to the library. gfx950 (CDNA4) only.
#ifndef FSPAD_EXP_NONPOS_H
#define FSPAD_EXP_NONPOS_H

#include <hip/hip_runtime.h>

namespace fspad_detail {

// exp(x) for x <= 0 in fp64: x = n ln2 + r, |r| <= ln2/2, degree-11 Taylor polynomial
// (truncation below 1e-14 relative), scaled by 2^n. n is rounded with the 1.5*2^52 shift (its
// integer value then sits in the low word of the shifted number) and 2^n is assembled from its
// exponent bits, which keeps the whole routine on full-rate multiply-adds. Returns 0 below
// -708 (where the true value is under 1e-307: its absence moves no sum by a representable amount).
__device__ __forceinline__ double exp_nonpos(double x) {
  // Branch-free on purpose: with an early return every call becomes a block of its own and the
  // compiler rebuilds the 64-bit constants in each (more moves than arithmetic).
  const bool vanishes = !(x >= -708.0);  // also catches NaN
  x = fmax(x, -708.0);                   // NaN -> -708: the arithmetic below stays in range
  const double shift = 6755399441055744.0;  // 1.5 * 2^52
  const double t = fma(x, 1.4426950408889634074, shift);
  const double n = t - shift;
  const int ni = (int)__double2loint(t);   // low word of the shifted value: n as a 32-bit integer (n in [-1022, 0])
  double r = fma(-n, 6.93147180369123816490e-01, x);
  r = fma(-n, 1.90821492927058770002e-10, r);
  double p = 1.0 / 39916800.0;
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  const double scale = __hiloint2double((ni + 1023) << 20, 0);   // 2^n
  return vanishes ? 0.0 : p * scale;
}

// The same for a loop over many arguments, with a table of 2^(j/32) in LDS (table-driven exponential after Tang, the argument
// reduced with ln2 in two parts after Cody and Waite, as above): x = (32 n + j) ln2/32 + r,
// |r| <= ln2/64, degree-5 Taylor polynomial (truncation below 2.3e-15 relative): 20 fp64 instructions per
// weight of a sum instead of 25. 32 entries of 8 bytes fill the 64 banks: lanes that read different entries
// meet no conflict. x is finite or -infinity; below -708 the result is that of -708 (3e-308, which moves no sum
// that holds a 1) instead of 0.
static __device__ const double kExp2Table[32] = {
    0x1.0000000000000p+0, 0x1.059b0d3158574p+0, 0x1.0b5586cf9890fp+0, 0x1.11301d0125b51p+0,
    0x1.172b83c7d517bp+0, 0x1.1d4873168b9aap+0, 0x1.2387a6e756238p+0, 0x1.29e9df51fdee1p+0,
    0x1.306fe0a31b715p+0, 0x1.371a7373aa9cbp+0, 0x1.3dea64c123422p+0, 0x1.44e086061892dp+0,
    0x1.4bfdad5362a27p+0, 0x1.5342b569d4f82p+0, 0x1.5ab07dd485429p+0, 0x1.6247eb03a5585p+0,
    0x1.6a09e667f3bcdp+0, 0x1.71f75e8ec5f74p+0, 0x1.7a11473eb0187p+0, 0x1.82589994cce13p+0,
    0x1.8ace5422aa0dbp+0, 0x1.93737b0cdc5e5p+0, 0x1.9c49182a3f090p+0, 0x1.a5503b23e255dp+0,
    0x1.ae89f995ad3adp+0, 0x1.b7f76f2fb5e47p+0, 0x1.c199bdd85529cp+0, 0x1.cb720dcef9069p+0,
    0x1.d5818dcfba487p+0, 0x1.dfc97337b9b5fp+0, 0x1.ea4afa2a490dap+0, 0x1.f50765b6e4540p+0};
__device__ __forceinline__ double exp_nonpos_table(double x, const double* table) {
  x = fmax(x, -708.0);
  const double shift = 6755399441055744.0;  // 1.5 * 2^52
  const double t = fma(x, 46.166241308446828384, shift);   // 32 / ln2
  const double k = t - shift;
  const int ki = (int)__double2loint(t);    // 32 n + j in [-32686, 0]: n >= -1022, root * 2^n is a normal number
  double r = fma(-k, 6.93147180369123816490e-01 / 32.0, x);   // (ln2's leading 32 bits: the product is exact)
  r = fma(-k, 1.90821492927058770002e-10 / 32.0, r);
  double p = 1.0 / 120.0;
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  const double root = table[ki & 31];
  return p * __hiloint2double(__double2hiint(root) + ((ki << 15) & (int)0xfff00000), __double2loint(root));   // root * 2^n
}

}  // namespace fspad_detail
#endif
