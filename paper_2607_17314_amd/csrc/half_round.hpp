// FP64 to FP16 with one rounding, as the split kernels need it for their (hi, lo) pairs. The
// card converts FP64 to FP32 and FP32 to FP16 only, and the compiler's own direct conversion is
// about 35 integer instructions. Here the value is first cut to the 20 fraction bits of its
// high word, with a one in the last of them if anything was cut off: that is exact in FP32,
// and rounding it to FP16's 10 bits gives what rounding the value itself would, since the cut
// bits only matter as "something is left" (round to odd).
#pragma once
#include "mfma_f64.hpp"

namespace xtc {

__device__ __forceinline__ _Float16 half_of(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32) | (lo < 1u ? lo : 1u);
  float f = (float)__builtin_bit_cast(double, (unsigned long long)hi << 32);
  keep_vector(f);   // else the two conversions are taken for one from FP64
  return (_Float16)f;
}

}  // namespace xtc
