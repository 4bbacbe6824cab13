// Sums of products of residues on the int8 matrix cores.
//
// A residue below 2^30 is four signed bytes, v = sum_b v_b 256^b with
// v_b in [-128, 127].  A contraction over residue pairs runs as one int8
// matrix product per pair of bytes (x, y), accumulated by x + y in seven
// exact int32 sums; fold_bytes brings them back to one residue.
#pragma once
#include <hip/hip_runtime.h>

#include "modp.hpp"

namespace snc {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// v < 2^31 as four signed bytes
__device__ __forceinline__ uint32_t balance4(uint32_t v) { return (v + 0x00808080u) ^ 0x00808080u; }

// 2^56 mod p, canonical
__device__ __forceinline__ uint32_t fold_const(const PrimeC& c) {
  return canon2(redc((uint64_t)c.r2 << 24, c.p, c.pinv), c.p);
}

// sum_d acc[d] 256^d 2^-32 mod p, canonical.  A contraction of n residue
// pairs leaves |acc[d]| <= 4 n 2^14; n <= 5056 (one parity of the largest degree
// bound in whole blocks; the remaindering sums at most 1536) keeps them below
// 2^28.4.  The sum is split at 2^24: the lower part is
// below 2^44.5 in magnitude, the upper below 2^52.5, and with p > 2^29.9 both
// turn positive by p 2^17 and p 2^24; the upper one comes back by k56 =
// fold_const.
__device__ __forceinline__ uint32_t fold_bytes(int a0, int a1, int a2, int a3, int a4, int a5, int a6, uint32_t k56,
                                               const PrimeC& c) {
  const int64_t lo = (int64_t)a0 + (int64_t)a1 * 256 + (int64_t)a2 * 65536;
  const int64_t hi = (int64_t)a3 + (int64_t)a4 * 256 + (int64_t)a5 * 65536 + (int64_t)a6 * 16777216;
  const uint32_t h = redc((uint64_t)(hi + ((int64_t)c.p << 24)), c.p, c.pinv);  // < 2^23 + p
  const uint64_t t = (uint64_t)(lo + ((int64_t)c.p << 17)) + (uint64_t)h * k56;  // < 2^61 + 2^48
  return canon2(redc(t, c.p, c.pinv), c.p);
}

}  // namespace snc
