// Which sums over a theta row hold no rounding at all.  (No device code of its own: also compiled for the host.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlda {

// Weights are fp32 numbers, counts whole ones.  With `least` the bits of the smallest weight, of binary exponent e,
// every product is a whole multiple of 2^(e - 23), and so is every sum of products; fp64 holds all such numbers
// below 2^(e + 30) exactly.  Sums below that (weights and counts are not negative, so all their parts are) are
// the same in whatever order they are added up, and with whatever is added first and taken off again later.
// Returned: the upper dword that the sum, as a double that carries 2^log2_scale as a factor, has to be less than.
// (Denormal weights, and 0, are multiples of 2^-149: taken as exponent -126.  A sum that is infinite or no number has a larger
// upper dword.)
__host__ __device__ inline uint32_t exact_sums_below(uint32_t least, int log2_scale) {
    const uint32_t biased = least >> 23;
    return (uint32_t)((int)(biased > 1u ? biased : 1u) - 127 + 30 + log2_scale + 1023) << 20;
}

}  // namespace mlda
