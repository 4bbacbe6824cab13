// Sums of products of residues on the vector unit: sixteen 64-bit
// multiply-adds per reduction, one operand uniform across the wavefront.
#pragma once
#include <hip/hip_runtime.h>

#include "modp.hpp"

namespace snc {

// s + a 2^-32 mod p for a sum a of sixteen canonical products: a stays below
// 16 p^2 < 2^64, and a 2^-32 = hi + REDC(lo) mod p splits it without REDC's
// own sum (which could pass 2^64): hi = a >> 32 < 4p is taken below 2p,
// REDC(lo) = mulhi(lo pinv, p) + (lo != 0) <= p (lo plus the low word of m p
// is 0 mod 2^32), so hi + REDC(lo) < 3p and s + it < 4p.
__device__ __forceinline__ uint32_t fold16(uint32_t s, uint64_t a, const PrimeC& c) {
  uint32_t hi = (uint32_t)(a >> 32);
  const uint32_t h2 = hi - 2 * c.p;
  hi = h2 < hi ? h2 : hi;
  const uint32_t lo = (uint32_t)a;
  const uint32_t r = __umulhi(lo * c.pinv, c.p) + (lo != 0u ? 1u : 0u);
  return canon(s + hi + r, c.p);
}

// s + sum_{q<64} U[q] S[-q] with U in LDS (16-byte aligned), uniform across the
// wavefront, and S per lane; s canonical in, out.  U is read four words at a time at one
// address for the whole wavefront (no vector-unit instruction per word), and
// sixteen products per reduction (fold16).  len: products needed, uniform.
__device__ __forceinline__ uint32_t toeplitz64(uint32_t s, const uint32_t* U, const uint32_t* S, const PrimeC& c,
                                               int len = 64) {
#pragma unroll
  for (int g = 0; g < 64 && g < len; g += 16) {
    const uint4* U4 = reinterpret_cast<const uint4*>(U + g);
    const uint4 ua = U4[0], ub = U4[1], uc = U4[2], ud = U4[3];
    const uint32_t w16[16] = {ua.x, ua.y, ua.z, ua.w, ub.x, ub.y, ub.z, ub.w,
                              uc.x, uc.y, uc.z, uc.w, ud.x, ud.y, ud.z, ud.w};
    uint64_t acc = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc += (uint64_t)w16[q] * S[-(g + q)];
    s = fold16(s, acc, c);
  }
  return s;
}

}  // namespace snc
