// remainder.hpp -- the draw's remainder, in a file of its own without HIP's headers, so that a CPU program can compile it too
// (with a __device__, __forceinline__, __builtin_amdgcn_rcpf and __mul24 of its own).
#pragma once
#include <stdint.h>

namespace pgxwave {

// n mod d for 1 <= d <= 1024, any n.  The quotient in floats is off by at most 2^10 / d + 1, so what is left of n lies within 2^10 + d of [0, d) and its own
// quotient, taken half a unit up, cannot round to the wrong side.  (The tests run this function for every d and some 100000 n each, most of them around multiples
// of d over all 32 bits: on the CPU with reciprocals one unit in the last place off either way, as the instruction may give them, and on the GPU.)  The general
// division takes four of the slow 32-bit products where this takes one, in a chain that nothing else fills.
__device__ __forceinline__ uint32_t remainder_of(uint32_t n, uint32_t d) {
  const float f = __builtin_amdgcn_rcpf((float)d);
  const uint32_t left = n - (uint32_t)__builtin_fminf((float)n * f, 4294967040.0f) * d;
  return left - (uint32_t)__mul24((int)__builtin_floorf(__builtin_fmaf((float)(int32_t)left, f, 0.5f * f)), (int)d);
}

}  // namespace pgxwave
