// Counter-based random numbers for the sampling kernel: Philox-4x32 with 10 rounds
// (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy as 1, 2, 3", SC'11),
// written from the published round function, and the Gumbel transform used with it.
#pragma once

#include "common.hip.h"

namespace oapl {

// a ^ b ^ c in one instruction (0x96 is the truth table of the three-way exclusive or).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
  return a ^ b ^ c;
#endif
}

// One round on the counter words, with the round's key.  The high and low halves of a product come from one 32 x 32 -> 64
// bit multiplication.
__device__ __forceinline__ void philox_round(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
  const uint64_t p0 = (uint64_t)0xD2511F53u * c[0], p1 = (uint64_t)0xCD9E8D57u * c[2];
  c[0] = xor3((uint32_t)(p1 >> 32), c[1], k0);
  c[2] = xor3((uint32_t)(p0 >> 32), c[3], k1);
  c[1] = (uint32_t)p1;
  c[3] = (uint32_t)p0;
}
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t (&out)[4]) {
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
#pragma unroll
  for (int round = 0; round < 10; ++round) philox_round(out, k0 + round * 0x9E3779B9u, k1 + round * 0xBB67AE85u);
}

// Standard Gumbel variate from one 32-bit word: u = ((x >> 9) + 1/2) * 2^-23 lies strictly inside
// (0, 1) and is exact in binary32 (it is 1.(x >> 9) - (1 - 2^-24), which is exact too); g = -ln(-ln u), each logarithm the
// hardware's base-2 one times ln 2, the outer with ln 2 in two parts.  Both arguments are normal numbers (2^-24 .. 17), so
// nothing of logf's care for others is needed.  Over all 2^23 words the error against 64 bits is 8.3e-8 (root mean
// square), 1.55e-6 (largest); with logf it was 9.6e-8 and 1.88e-6.
__device__ __forceinline__ float gumbel_from_bits(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr float kLn2Hi = 0.693147182464599609375f, kLn2Lo = -1.90465429995776804525e-9f;
  const uint32_t one_to_two = __builtin_amdgcn_alignbit(0x7Fu, x, 9);   // 0x3F800000 | x >> 9
  const float u = __builtin_bit_cast(float, one_to_two) - 0.999999940395355224609375f;
  const float e = __builtin_amdgcn_logf(u) * -kLn2Hi;
  const float l = __builtin_amdgcn_logf(e);
  return __builtin_fmaf(l, -kLn2Hi, l * -kLn2Lo);
#else
  return 0.f;   // the host pass needs the signature only
#endif
}

// (score, index) pairs compare by score, ties to the smaller index.
__device__ __forceinline__ bool better(float sa, int ia, float sb, int ib) { return sa > sb || (sa == sb && ia < ib); }

}  // namespace oapl
