// Residues of integer-valued doubles modulo small odd moduli, as elements of the matrix cores.
#pragma once

#include <hip/hip_runtime.h>

namespace hsb {

// v - m * round(v / m), in [-(m-1)/2, (m-1)/2], for an integer-valued double |v| < 2^48 and an
// odd modulus 113 <= m < 256.  The computed v * fl(1/m) is within |v/m| 2^-52 < 2^-10 of v/m,
// while v/m, with m odd, is never closer than 1/(2m) > 2^-9 to a half-integer: the rounded
// quotient is exact, and so are q m and the difference (fma).
__device__ __forceinline__ double smod_d(double v, double m, double inv_m) {
  return fma(-rint(v * inv_m), m, v);
}

// Residue r (an integer in [-(m-1)/2, (m-1)/2], as a double) as the element of kind EK: a signed
// byte (0), or the bits of a bfloat16 (1) or an IEEE half (2), both exact for |r| <= 256.
template <int EK>
__device__ __forceinline__ unsigned residue_bits(double r) {
  if constexpr (EK == 0) return (unsigned)(int)r & 0xffu;
  else if constexpr (EK == 1) return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)(float)r);
  // through int and float (both exact here): a direct double -> half cast is rounded in software
  else return (unsigned)__builtin_bit_cast(unsigned short, (_Float16)(float)(int)r);
}

}  // namespace hsb
