// Least sum and its source in one number (used by the forward kernels).
#pragma once

#include <hip/hip_runtime.h>

namespace gs {

// The fp32 bits of a sum in the upper word, the index of its source in the lower.  Sums lie
// between +0 and +inf (tables with other entries, NaN among them, are reported in the data status and
// their results mean nothing), so the pair read as a double is finite and not negative (its exponent
// is 0x7f8 at most), and doubles order the pairs by sum, then by index: ONE V_MIN_F64 keeps the least sum together with the lowest source that
// attains it, where compare and two selects are three.
typedef unsigned pair_t __attribute__((ext_vector_type(2)));

static __device__ __forceinline__ pair_t pair_min(pair_t a, pair_t b) {
  double x = __builtin_bit_cast(double, a);
  // (inline assembly: fmin() would be preceded by instructions that quieten NaN)
  asm("v_min_f64 %0, %1, %2" : "=v"(x) : "v"(x), "v"(__builtin_bit_cast(double, b)));
  return __builtin_bit_cast(pair_t, x);
}

static __device__ __forceinline__ float pair_sum(pair_t p) {
  const unsigned bits = p.y; // (a copy: bit_cast of a vector's element reads element 0)
  return __builtin_bit_cast(float, bits);
}

// Lower words of eight pairs.  The compiler keeps each in the register below the one that takes
// the sums, so that forming a pair is the addition alone.
struct PairIndex {
  unsigned k[8];
  __device__ __forceinline__ PairIndex() {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      k[i] = i;
      asm("" : "+v"(k[i])); // (goes away where no pair is formed)
    }
  }
};

} // namespace gs
