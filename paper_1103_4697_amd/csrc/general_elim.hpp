// General elimination of one (prime, point) instance, any degree pattern.
#pragma once
#include <hip/hip_runtime.h>

#include "eval_elim.hpp"

namespace snc {

// ---------------------------------------------------------------------------
// General elimination for one instance, any degree pattern: formal-degree
// corrections (res_{m,n} = (-1)^{n(m-m')} g_n^{m-m'} res_{m',n} when f's
// leading coefficients vanish, = f_m^{n-n'} res_{m,n'} when g's do, 0 when
// both do), then Euclid with true remainders.  Arrays are bottom-aligned
// (index = y-degree); runs for the rare abnormal lanes, or for every
// instance when a y-degree exceeds the register classes.
// ---------------------------------------------------------------------------
static __device__ uint32_t res_general(uint32_t* F, int m, uint32_t* G, int n, const PrimeC& c) {
  if (m == 0 && n == 0) return c.r1;
  if (n == 0) return mpow(G[0], (uint32_t)m, c);
  if (m == 0) return mpow(F[0], (uint32_t)n, c);
  int mm = m;
  while (mm >= 0 && F[mm] == 0) --mm;
  int nn = n;
  while (nn >= 0 && G[nn] == 0) --nn;
  if (mm < 0 || nn < 0) return 0;
  if (mm < m && nn < n) return 0;
  uint32_t acc = c.r1;
  if (mm < m) {
    acc = mmulc(acc, mpow(G[n], (uint32_t)(m - mm), c), c.p, c.pinv);
    if ((n * (m - mm)) & 1) acc = mneg(acc, c.p);
  }
  if (nn < n) acc = mmulc(acc, mpow(F[m], (uint32_t)(n - nn), c), c.p, c.pinv);
  uint32_t* Ap = F;
  uint32_t* Bp = G;
  int a = mm, b = nn;
  while (true) {
    if (a == 0) return mmulc(acc, mpow(Ap[0], (uint32_t)b, c), c.p, c.pinv);
    if (b == 0) return mmulc(acc, mpow(Bp[0], (uint32_t)a, c), c.p, c.pinv);
    if (a < b) {
      uint32_t* t = Ap; Ap = Bp; Bp = t;
      int ti = a; a = b; b = ti;
      if ((a * b) & 1) acc = mneg(acc, c.p);
      continue;
    }
    const uint32_t inv = minv(Bp[b], c);
    int r = a;
    while (r >= b) {
      const uint32_t q = mmulc(Ap[r], inv, c.p, c.pinv);
      if (q) {
        uint32_t* A = Ap + (r - b);
        int i = 0;
        for (; i + 8 <= b; i += 8) {  // the two arrays never overlap: all loads of a step are in flight together
          uint32_t x[8], y[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) { x[u] = A[i + u]; y[u] = Bp[i + u]; }
#pragma unroll
          for (int u = 0; u < 8; ++u) A[i + u] = msub(x[u], mmulc(q, y[u], c.p, c.pinv), c.p);
        }
        for (; i < b; ++i) A[i] = msub(A[i], mmulc(q, Bp[i], c.p, c.pinv), c.p);
      }
      Ap[r] = 0;
      --r;
      while (r >= 0 && Ap[r] == 0) --r;
    }
    if (r < 0) return 0;
    acc = mmulc(acc, mpow(Bp[b], (uint32_t)(a - r), c), c.p, c.pinv);
    if ((a * b) & 1) acc = mneg(acc, c.p);
    uint32_t* t = Ap; Ap = Bp; Bp = t;  // (A, B) <- (B, R)
    a = b; b = r;
  }
}

// z, z^2, z^3, z^4 = x, x^2, x^3, x^4: hstep4 on consecutive powers
__device__ __forceinline__ XPow point_powers(uint32_t x, const PrimeC& c) {
  XPow P;
  P.z1 = x;
  P.z2 = mmulc(x, x, c.p, c.pinv);
  P.z3 = mmulc(P.z2, x, c.p, c.pinv);
  P.z4 = mmulc(P.z2, P.z2, c.p, c.pinv);
  return P;
}

// Row q of a group at the point (canonical): the eight coefficients of a pair
// of chunks are requested together and take two steps of Horner's rule in x^4.
__device__ __forceinline__ uint32_t eval_row(const uint32_t* g, int len, int q, const XPow& X, const PrimeC& c) {
  uint32_t a = 0;
  int k = len & ~7;
  g += q;
  if (len & HCHUNK) {
    const uint32_t* v = g + 4 * k;  // x^k, x^(k+2), x^(k+1), x^(k+3)
    a = hstep4(0u, v[0], v[8], v[4], v[12], X, c);
  }
#pragma unroll 2
  for (k -= 8; k >= 0; k -= 8) {
    const uint32_t* e = g + 4 * k;  // four even powers, then four odd ones
    const uint32_t v0 = e[0], v2 = e[4], v4 = e[8], v6 = e[12], v1 = e[16], v3 = e[20], v5 = e[24], v7 = e[28];
    a = hstep4(a, v4, v5, v6, v7, X, c);
    a = hstep4(a, v0, v1, v2, v3, X, c);
  }
  return canon4(a, c.p);
}

// The deg + 1 rows of an operand at the lane's point, F[i] the coefficient of
// y^i, by the pair of lanes of +-x as in the evaluation kernel.
__device__ __forceinline__ void eval_operand(uint32_t* F, const uint32_t* r, const RowDesc* rd, int deg, int odd,
                                             const XPow& X, const PrimeC& c) {
  for (int t0 = 0; t0 <= deg; t0 += ROWGRP) {
    const RowDesc d = rd[t0 / ROWGRP];
    uint32_t a[4] = {0u, 0u, 0u, 0u};
    if (d.len > 0) {
      if (deg - t0 >= 2) eval_group<4>(a, r + d.off, d.len, odd, X, c);
      else eval_group<2>(a, r + d.off, d.len, odd, X, c);
    }
#pragma unroll
    for (int q = 0; q < ROWGRP; ++q)
      if (t0 + q <= deg) F[deg - t0 - q] = canon4(a[q], c.p);
  }
}

// One instance per lane; lanes 2i and 2i + 1 of a wavefront call together, for
// points j = 2i and 2i + 1 of one prime (both or neither).  MAXY: the largest
// y-degree of the instances this variant runs (the size of the per-lane value
// arrays).  Bound by the issue of the 64-bit multiply-adds of a lone wavefront
// per SIMD: a prime's abnormal instances share the workgroup that interpolates
// it.  Whole calls, with the pair's evaluation and the loads of eight update
// steps in flight, against one row after the other with a load and a dependent
// step per coefficient: even in y of y-degree 4 and x-degree 700 (5,602 points
// of 5 primes) 17.3 -> 1.8 ms, y- and x-degree 62 (3,700 points) 14.6 -> 5.0 ms;
// y-degree 70, above the register classes, 1.06 -> 0.57 ms.
template <int MAXY>
__device__ __attribute__((noinline)) uint32_t general_instance(const ResJob* job, const PrimeC* primes,
                                                               const RowDesc* rows, const uint32_t* ws,
                                                               const uint32_t* points, int pi, int j) {
  const ResJob& J = *job;
  const PrimeC c = primes[pi];
  const uint32_t* r = ws + J.res_off + (int64_t)pi * J.T;
  const XPow X = pair_powers(points, pi, j, j & 1, c);
  const RowDesc* ra = rows + J.rows_off;
  const RowDesc* rb = ra + J.rstride;
  uint32_t F[MAXY + 1], G[MAXY + 1];
  eval_operand(F, r, ra, J.m, j & 1, X, c);
  eval_operand(G, r, rb, J.n, j & 1, X, c);
  uint32_t res = res_general(F, J.m, G, J.n, c);
  if (J.sign) res = mneg(res, c.p);
  return res;
}

// LDS written by some lanes of a wavefront, read by others
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same value by one wavefront, y-degrees up to MAXY_FAST: a row of each
// operand per lane in the evaluation, a coefficient per lane in the
// elimination, which is division-free (an elementary step replaces A by
// lc(B) A - lc(A) x^s B; its scale goes to one denominator, inverted at the
// end).  F, G: MAXY_FAST + 1 words of LDS of the wavefront's own.  A lone
// abnormal instance of degree 40 takes a wavefront 60 us and a lane 250 us; of
// degree 16, 25 and 88 us; of degree 4, 5 and 14 us.
__device__ __attribute__((noinline)) uint32_t general_instance_wave(const ResJob* job, const PrimeC* primes,
                                                                    const RowDesc* rows, const uint32_t* ws,
                                                                    const uint32_t* points, int pi, int j,
                                                                    uint32_t* F, uint32_t* G, int lane) {
  const int m = job->m, n = job->n;
  const PrimeC c = primes[pi];
  const uint32_t* r = ws + job->res_off + (int64_t)pi * job->T;
  const XPow X = point_powers(point_mont(points, pi, j, c), c);
  const RowDesc* ra = rows + job->rows_off;
  const RowDesc* rb = ra + job->rstride;
  for (int x = lane; x < m + n + 2; x += 64) {
    const bool first = x <= m;
    const int t = first ? x : x - m - 1;
    const RowDesc d = (first ? ra : rb)[t / ROWGRP];
    const uint32_t v = eval_row(r + d.off, d.len, t % ROWGRP, X, c);
    if (first) F[m - t] = v;
    else G[n - t] = v;
  }
  wave_sync();
  uint32_t acc = c.r1, den = c.r1;
  if (job->sign) acc = mneg(acc, c.p);
  if (m == 0 && n == 0) return acc;
  if (n == 0) return mmulc(acc, mpow(G[0], (uint32_t)m, c), c.p, c.pinv);
  int a = m, b = n;
  while (a >= 0 && F[a] == 0) --a;
  while (b >= 0 && G[b] == 0) --b;
  if (a < 0 || b < 0 || (a < m && b < n)) return 0;
  if (a < m) {
    acc = mmulc(acc, mpow(G[n], (uint32_t)(m - a), c), c.p, c.pinv);
    if ((n * (m - a)) & 1) acc = mneg(acc, c.p);
  }
  if (b < n) acc = mmulc(acc, mpow(F[m], (uint32_t)(n - b), c), c.p, c.pinv);
  uint32_t* A = F;
  uint32_t* B = G;
  for (;;) {
    if (a < b) {
      uint32_t* t = A; A = B; B = t;
      const int ti = a; a = b; b = ti;
      if ((a * b) & 1) acc = mneg(acc, c.p);
    }
    if (b == 0) {
      acc = mmulc(acc, mpow(B[0], (uint32_t)a, c), c.p, c.pinv);
      break;
    }
    // A <- lc(B)^e (A mod B); zero leading entries cost no step
    const uint32_t lb = B[b];
    int rd = a, e = 0;
    while (rd >= b) {
      const uint32_t nla = c.p - A[rd];
      const int sh = rd - b;
      if (lane < rd) {
        const uint32_t y = lane >= sh ? B[lane - sh] : 0u;
        A[lane] = canon(mmul2(lb, A[lane], nla, y, c.p, c.pinv), c.p);
      }
      wave_sync();
      ++e;
      --rd;
      while (rd >= 0 && A[rd] == 0) --rd;
    }
    if (rd < 0) return 0;
    const int ex = e * b - (a - rd);
    if (ex >= 0) den = mmulc(den, mpow(lb, (uint32_t)ex, c), c.p, c.pinv);
    else acc = mmulc(acc, mpow(lb, (uint32_t)(-ex), c), c.p, c.pinv);
    if ((a * b) & 1) acc = mneg(acc, c.p);
    uint32_t* t = A; A = B; B = t;  // (A, B) <- (B, R)
    a = b;
    b = rd;
  }
  return mmulc(acc, minv(den, c), c.p, c.pinv);
}

}  // namespace snc

