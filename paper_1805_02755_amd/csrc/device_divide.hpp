// Division by numbers that the host knows before the launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ce {

// Division of 32-bit numbers by one the host knows: the estimate from the
// reciprocal rounded down is at most two too small.
struct Divisor {
  uint32_t d, reciprocal;
  __host__ __device__ explicit Divisor(uint32_t v) : d(v), reciprocal(0xFFFFFFFFu / v) {}
  __host__ __device__ Divisor(uint32_t v, uint32_t r) : d(v), reciprocal(r) {}
  __host__ __device__ uint32_t split(uint32_t x, uint32_t* rest) const {
    uint32_t q = (uint32_t)(((uint64_t)x * reciprocal) >> 32), r = x - q * d;
    for (int k = 0; k < 2; ++k)
      if (r >= d) {
        r -= d;
        ++q;
      }
    *rest = r;
    return q;
  }
};

}  // namespace ce
