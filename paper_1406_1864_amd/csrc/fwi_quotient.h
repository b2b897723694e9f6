// Quotients by one divisor, finite and at least 1: the product with its
// reciprocal, kept as a sum hi + lo of two doubles (about 105 bits), rounded
// once: x hi + x lo is within 2^-104 of x / divisor, so that it rounds like the
// division.  hi is the reciprocal rounded down and lo positive, so that an
// infinite x has the infinite quotient (and no infinity is subtracted from
// another); zeros keep their sign.  Two operations a quotient: the product
// with a plain reciprocal and a correction from its remainder take three and
// make a NaN of infinities (16 shots of 288 x 128 cells, 1500 steps: misfit
// 5.33 ms, gradient 17.95; with one more to bound that remainder 5.44, 17.90;
// as here 5.25, 17.53).  Host and device code.
#pragma once
#include <stdint.h>
#include <string.h>
#if defined(__HIPCC__)
#define FWI_HOST_DEVICE __host__ __device__
#else
#define FWI_HOST_DEVICE
#endif

namespace fwi {

struct Reciprocal {
  double hi, lo;
};

FWI_HOST_DEVICE inline Reciprocal reciprocal(double divisor) {
  double hi = 1.0 / divisor;
  if (__builtin_fma(-hi, divisor, 1.0) < 0.0) {  // rounded up: the double below
    uint64_t b;
    memcpy(&b, &hi, sizeof(b));
    --b;
    memcpy(&hi, &b, sizeof(b));
  }
  // (an exact hi leaves nothing to lo, whose product with infinity must be infinite)
  return Reciprocal{hi, __builtin_fmax(__builtin_fma(-hi, divisor, 1.0) * hi, 0x1p-1000)};
}

FWI_HOST_DEVICE inline double quotient(double x, Reciprocal r) { return __builtin_fma(x, r.hi, x * r.lo); }

}  // namespace fwi
