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
        for (int i = 0; i < b; ++i)
          Ap[r - b + i] = msub(Ap[r - b + i], mmulc(q, Bp[i], c.p, c.pinv), c.p);
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

// MAXY: the largest y-degree of the instances this variant runs (the size
// of the per-lane value arrays)
template <int MAXY>
__device__ __attribute__((noinline)) uint32_t general_instance(const ResJob* job, const PrimeC* primes,
                                                               const RowDesc* rows, const uint32_t* ws,
                                                               const uint32_t* points, int pi, int j) {
  const ResJob& J = *job;
  const PrimeC c = primes[pi];
  const uint32_t* r = ws + J.res_off + (int64_t)pi * J.T;
  const uint32_t X = point_mont(points, pi, j, c);
  const RowDesc* ra = rows + J.rows_off;
  const RowDesc* rb = ra + J.rstride;
  uint32_t F[MAXY + 1], G[MAXY + 1];
  for (int t = 0; t <= J.m; ++t) F[J.m - t] = canon(horner_grouped(r, ra[t / ROWGRP], t % ROWGRP, X, c), c.p);
  for (int t = 0; t <= J.n; ++t) G[J.n - t] = canon(horner_grouped(r, rb[t / ROWGRP], t % ROWGRP, X, c), c.p);
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
// abnormal instance costs a lane about 220 us of serial loads and updates
// (degree 40), a wavefront about a tenth.
__device__ __attribute__((noinline)) uint32_t general_instance_wave(const ResJob* job, const PrimeC* primes,
                                                                    const RowDesc* rows, const uint32_t* ws,
                                                                    const uint32_t* points, int pi, int j,
                                                                    uint32_t* F, uint32_t* G, int lane) {
  const int m = job->m, n = job->n;
  const PrimeC c = primes[pi];
  const uint32_t* r = ws + job->res_off + (int64_t)pi * job->T;
  const uint32_t X = point_mont(points, pi, j, c);
  const RowDesc* ra = rows + job->rows_off;
  const RowDesc* rb = ra + job->rstride;
  for (int x = lane; x < m + n + 2; x += 64) {
    const bool first = x <= m;
    const int t = first ? x : x - m - 1;
    const uint32_t v = canon(horner_grouped(r, (first ? ra : rb)[t / ROWGRP], t % ROWGRP, X, c), c.p);
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

