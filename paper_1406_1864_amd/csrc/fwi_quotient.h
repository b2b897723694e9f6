// x / plus with inv = 1 / plus at hand (plus finite and at least 1, |x| infinite
// or far below 2^1000): the product with inv and one correction from its exact
// remainder, which rounds like the division.  The remainder's sign is chosen so
// that a zero keeps its own, and the bound under it, which no finite remainder
// reaches, takes the place of the NaN that an infinite x leaves: the quotient
// then is infinite too.  Host and device code.
//   The bound costs 1 to 2 % of a small grid's forward sweep (16 shots of
// 288 x 128 cells, 1500 steps: 5.34 -> 5.45 ms; 2 shots of 40 x 32, gradient:
// 0.996 -> 1.005 ms); a comparison and a choice of the result cost 2.5 to
// 4.5 %, a branch to the division for rows with a NaN as much as the bound.
#pragma once
#if defined(__HIPCC__)
#define FWI_HOST_DEVICE __host__ __device__
#else
#define FWI_HOST_DEVICE
#endif

namespace fwi {

FWI_HOST_DEVICE inline double quotient(double x, double plus, double inv) {
  const double q = x * inv;
  const double r = __builtin_fmax(__builtin_fma(q, plus, -x), -0x1p1000);
  return __builtin_fma(-r, inv, q);
}

}  // namespace fwi
