// HIP kernels of the multi-modular resultant res_y(f, g) (Section 4,
// "Symbolic Speedups"): reduction of the inputs, elimination above the register
// classes and Chinese remaindering up to 64 primes, written for gfx950: 64-wide
// wavefronts, full-rate 32-bit multiplies, LDS staging.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "eval_elim.hpp"
#include "general_elim.hpp"

namespace snc {

// ---------------------------------------------------------------------------
// Constant tables (filled once per device by upload_tables)
// ---------------------------------------------------------------------------
__device__ PrimeC g_primes[KMAX];
__device__ uint32_t g_garner[KMAX];            // Montgomery form of (P_i mod p_i)^-1
__device__ uint32_t g_wtab[KMAX * KMAX];       // [j*KMAX + i] = Montgomery form of P_j mod p_i (j < i)
__device__ uint32_t g_ptab[(KMAX + 1) * LPS];  // row j: P_j = prod_{l<j} p_l, little-endian limbs

// per-device kernel attributes (called once per device before any launch)
__global__ void k_crt_combine(CrtTables tb, const ResJob* jobs, const int32_t* job_list, const int64_t* prefix,
                              int njobs, int lx_max, uint32_t* ws);

hipError_t configure_kernels() {
  return hipFuncSetAttribute((const void*)k_crt_combine, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)(CRT_COMB_PER_BLOCK * 3 * lx_of(KMAX) * sizeof(uint32_t)));
}

void upload_tables(const PrimeC* primes, const uint32_t* garner_c, const uint32_t* wtab,
                   const uint32_t* ptab, hipStream_t s) {
  (void)hipMemcpyToSymbolAsync(HIP_SYMBOL(g_primes), primes, sizeof(PrimeC) * KMAX, 0,
                               hipMemcpyHostToDevice, s);
  (void)hipMemcpyToSymbolAsync(HIP_SYMBOL(g_garner), garner_c, sizeof(uint32_t) * KMAX, 0,
                               hipMemcpyHostToDevice, s);
  (void)hipMemcpyToSymbolAsync(HIP_SYMBOL(g_wtab), wtab, sizeof(uint32_t) * KMAX * KMAX, 0,
                               hipMemcpyHostToDevice, s);
  (void)hipMemcpyToSymbolAsync(HIP_SYMBOL(g_ptab), ptab, sizeof(uint32_t) * (KMAX + 1) * LPS, 0,
                               hipMemcpyHostToDevice, s);
}

__global__ void k_zero_u32(uint32_t* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

void launch_zero_u32(uint32_t* p, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
}

// ---------------------------------------------------------------------------
// (1) Modular reduction of the input coefficients (moved on-device; the
//     paper notes the host-side reduction as a bottleneck).
//     residue[prime][t] = Montgomery form of c_t mod p, c_t signed, nl limbs.
// ---------------------------------------------------------------------------
//     A lane takes one coefficient through RED_PRIMES primes, so a limb is read
//     once for eight multiply-adds.  15 resultants of degree-15 curves with
//     2048-bit coefficients (2052 primes): 77 us here, against 545 us of the
//     evaluation's 1,075 when each of its 64-point blocks reduced its prime's
//     limbs again, a Horner step per limb.  Bound by the multiply-adds.
__device__ uint32_t g_pow32[(int64_t)KMAX * POW32_ROW];

__global__ __launch_bounds__(64) void k_pow32_init() {
  const int pi = blockIdx.x * 64 + threadIdx.x;
  const PrimeC c = g_primes[pi];
  uint32_t* row = g_pow32 + (int64_t)pi * POW32_ROW;
  uint32_t v = c.r2;  // 2^64
  for (int l = 0; l <= 64; ++l) {
    row[l] = v;
    if (l == 64) row[POW32_STEP] = canon2(redc((uint64_t)v, c.p, c.pinv), c.p);  // 2^2048 2^64 2^-32
    v = mmulc(v, c.r2, c.p, c.pinv);
  }
}

void launch_pow32_init(hipStream_t s) { hipLaunchKernelGGL(k_pow32_init, dim3(KMAX / 64), dim3(64), 0, s); }

const uint32_t* pow32_table() {
  static const uint32_t* cache[64] = {nullptr};
  int dev = 0;
  (void)hipGetDevice(&dev);
  if (dev >= 0 && dev < 64 && cache[dev]) return cache[dev];
  void* p = nullptr;
  (void)hipGetSymbolAddress(&p, HIP_SYMBOL(g_pow32));
  if (dev >= 0 && dev < 64) cache[dev] = (const uint32_t*)p;
  return (const uint32_t*)p;
}

__global__ __launch_bounds__(64) void k_reduce(const ResJob* jobs, const int64_t* prefix, int njobs,
                                               const uint32_t* ws, uint32_t* wsw) {
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[jj];
  const int nb = (J.T + 63) / 64;
  const int64_t lb = b - prefix[jj];
  const int p0 = (int)(lb / nb) * RED_PRIMES;
  const int t = (int)(lb % nb) * 64 + threadIdx.x;
  if (t >= J.T) return;
  PrimeC c[RED_PRIMES];
#pragma unroll
  for (int r = 0; r < RED_PRIMES; ++r) c[r] = g_primes[p0 + r];  // KMAX is a multiple of RED_PRIMES
  uint32_t v[RED_PRIMES];
  reduce_limbs<RED_PRIMES>(v, ws + J.coef_off + t, J.nl, J.T, c, g_pow32 + (int64_t)p0 * POW32_ROW);
#pragma unroll
  for (int r = 0; r < RED_PRIMES; ++r)
    if (p0 + r < J.k) wsw[J.res_off + (int64_t)(p0 + r) * J.T + t] = v[r];
}
static_assert(KMAX % RED_PRIMES == 0, "whole groups of primes");

void launch_reduce(const ResJob* jobs_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks,
                   const uint32_t* ws, uint32_t* res_base, hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_reduce, dim3((unsigned)nblocks), dim3(64), 0, s, jobs_d,
                     blk_prefix_d, njobs, ws, res_base);
}

__global__ void k_elim_general_all(const ResJob* jobs, const int32_t* job_list,
                                   const int64_t* prefix, int njobs, int64_t ninst,
                                   const RowDesc* rows, uint32_t* ws, const uint32_t* points) {
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < ninst;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int jj = find_job(prefix, njobs, idx);
    const ResJob J = jobs[job_list[jj]];
    const int64_t li = idx - prefix[jj];
    const int np = npts_of(J.D);
    const int pi = (int)(li / np), j = (int)(li % np);
    ws[J.pts_off + (int64_t)pi * np + j] =
        general_instance<MAXY_GEN>(jobs + job_list[jj], g_primes, rows, ws, points, pi, j);
  }
}

void launch_elim_general_all(const ResJob* jobs_d, const int32_t* job_list_d,
                             const int64_t* inst_prefix_d, int njobs, int64_t ninst,
                             const RowDesc* rows_d, uint32_t* ws, hipStream_t s) {
  if (ninst <= 0) return;
  int64_t blocks = (ninst + 63) / 64;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_elim_general_all, dim3((unsigned)blocks), dim3(64), 0, s, jobs_d, job_list_d,
                     inst_prefix_d, njobs, ninst, rows_d, ws, points_table());
}

// ---------------------------------------------------------------------------
// (5) Chinese remaindering per coefficient.
//   digits: Garner's mixed-radix digits y_j, X = sum_j y_j P_j, with
//     y_i = (r_i - S_i) (P_i)^-1 mod p_i,  S_i = sum_{j<i} y_j P_j mod p_i.
//     One wavefront per coefficient, primes in blocks of 64 (lane l holds
//     prime 64 s + l of block s).  In block s the digits come one after
//     another: digit q is broadcast from lane q and folded into the later
//     primes of the block.  The finished block then goes to every later
//     block s2 at once, S_i += sum_q y_{64s+q} (P_{64s+q} mod p_i), sixteen
//     products per reduction.  S_i waits in digit slot i until digit i is
//     written there.  The 64 x 64 tiles of W = (P_j mod p_i) are staged in
//     LDS, double-buffered and shared by the block's wavefronts.
//   combine: X in binary by Horner over the digits; the balanced value is
//     X - M when X > (M-1)/2, decided on the digits ((M-1)/2 has digits
//     (p_j - 1)/2), written as L two's-complement limbs.
// ---------------------------------------------------------------------------
constexpr int CRT_TILE = 64 * 64;                          // words of one W tile
constexpr int CRT_PRE = CRT_TILE / (64 * CRT_COEF_PER_BLOCK);  // tile words fetched per thread

__global__ __launch_bounds__(64 * CRT_COEF_PER_BLOCK) void k_crt_digits(CrtTables tb, const ResJob* jobs,
                                                                        const int32_t* job_list,
                                                                        const int64_t* prefix,
                                                                        int njobs, uint32_t* ws) {
  __shared__ uint32_t wt[2][CRT_TILE];  // tile (s, s2): [q][l] = W[64 s + q][64 s2 + l]
  const int64_t b = xcd_block(blockIdx.x, gridDim.x);
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[job_list ? job_list[jj] : jj];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = (int)(b - prefix[jj]) * CRT_COEF_PER_BLOCK + wave;
  const bool active = t <= J.D;  // the block's waves share one job; idle ones still meet the barriers
  const int k = J.k;
  const int nsl = (k + 63) >> 6;
  const int n1 = J.D + 1;
  const uint32_t* V = ws + J.val_off;
  uint32_t* dig = ws + J.dig_off + (int64_t)(active ? t : 0) * k;
  if (active)
    for (int i = lane; i < k; i += 64) dig[i] = 0;  // the partial sums S_i start at zero
  uint32_t pre[CRT_PRE];
  auto fetch = [&](int s, int s2) {
#pragma unroll
    for (int e = 0; e < CRT_PRE; ++e) {
      const int x = threadIdx.x + e * 64 * CRT_COEF_PER_BLOCK;
      const int row = 64 * s + (x >> 6), col = 64 * s2 + (x & 63);
      pre[e] = (row < k && col < k) ? tb.wtab[(int64_t)row * tb.wstride + col] : 0u;
    }
  };
  fetch(0, 0);
  uint32_t ymine = 0;  // digit 64 s + lane of the current block
  const int ntiles = nsl * (nsl + 1) / 2;
  int s = 0, s2 = 0;
  for (int tau = 0; tau < ntiles; ++tau) {
    uint32_t* w = wt[tau & 1];
#pragma unroll
    for (int e = 0; e < CRT_PRE; ++e) w[threadIdx.x + e * 64 * CRT_COEF_PER_BLOCK] = pre[e];
    __syncthreads();
    int ns = s, ns2 = s2 + 1;  // the next tile, fetched while this one is worked on
    if (ns2 == nsl) { ++ns; ns2 = ns; }
    if (tau + 1 < ntiles) fetch(ns, ns2);
    const int i = 64 * s2 + lane;
    const bool ok = active && i < k;
    const PrimeC c = tb.primes[i < k ? i : 0];
    if (s2 == s) {  // digits of block s
      const int nq = min(64, k - 64 * s);
      const uint32_t g = tb.garner[i < k ? i : 0];
      const uint32_t r = ok ? V[(int64_t)i * n1 + t] : 0u;
      uint32_t S = ok ? dig[i] : 0u;
      for (int q = 0; q < nq; ++q) {
        const uint32_t cand = canon(redc((uint64_t)msub(r, S, c.p) * g, c.p, c.pinv), c.p);
        const uint32_t y = __builtin_amdgcn_readlane(cand, q);
        if (lane == q) ymine = cand;
        if (lane > q) S = madd(S, canon(redc((uint64_t)y * w[q * 64 + lane], c.p, c.pinv), c.p), c.p);
      }
      if (ok) dig[i] = ymine;
    } else {  // block s into block s2 > s (s is not the last block: 64 digits)
      uint32_t acc = ok ? dig[i] : 0u;  // < 2p from here on
#pragma unroll
      for (int q = 0; q < 64; q += 16) {
        // sixteen products y < 2^30 times W < p stay below 2^34 p < 2^64 (four
        // partial sums); with sum = hi 2^32 + lo, sum 2^-32 = hi + lo 2^-32,
        // where hi < 4p and the REDC of lo alone is at most p
        uint64_t part[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          part[u] = 0;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int qq = q + 4 * u + v;
            part[u] += (uint64_t)__builtin_amdgcn_readlane(ymine, qq) * w[qq * 64 + lane];
          }
        }
        const uint64_t sum = (part[0] + part[1]) + (part[2] + part[3]);
        uint32_t hi = (uint32_t)(sum >> 32);
        const uint32_t h2 = hi - 2 * c.p;
        hi = h2 < hi ? h2 : hi;  // [0, 4p) -> [0, 2p)
        uint32_t t = hi + redc((uint64_t)(uint32_t)sum, c.p, c.pinv);  // < 3p + 1
        const uint32_t t2 = t - 2 * c.p;
        t = t2 < t ? t2 : t;  // -> [0, 2p)
        acc += t;
        const uint32_t a2 = acc - 2 * c.p;
        acc = a2 < acc ? a2 : acc;  // [0, 4p) -> [0, 2p)
      }
      if (ok) dig[i] = canon(acc, c.p);
    }
    s = ns;
    s2 = ns2;
  }
}

// X = sum_j y_j P_j for the workgroup's CRT_COMB_PER_BLOCK coefficients,
// lanes over limbs: wavefront w of the CRT_COEF_PER_BLOCK takes limbs
// 64 w + 64 CRT_COEF_PER_BLOCK i + lane of every coefficient of the workgroup,
// so each limb of P_j is read once per workgroup.
// Limb l accumulates sum_j y_j P_j[l] (< 2^72) as lo (64 bits) + hi; its low
// word stays at limb l and the rest, a carry below 2^41, goes to limb l+1.
// Lane 0 of wavefront c then propagates the carries of coefficient c,
// subtracts M = P_k when X > (M-1)/2 (decided on the digits: (M-1)/2 has
// digits (p_j - 1)/2) and writes L two's-complement limbs.
__global__ __launch_bounds__(64 * CRT_COEF_PER_BLOCK) void k_crt_combine(CrtTables tb, const ResJob* jobs,
                                                                         const int32_t* job_list,
                                                                         const int64_t* prefix, int njobs,
                                                                         int lx_max, uint32_t* ws) {
  constexpr int C = CRT_COMB_PER_BLOCK;
  extern __shared__ uint32_t csm[];
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[job_list ? job_list[jj] : jj];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t0 = (int)(b - prefix[jj]) * C;
  const int nc = min(C, J.D + 1 - t0);  // coefficients of this block (>= 1)
  const int k = J.k;
  const int lx = lx_of(k);
  const uint32_t* d0 = ws + J.dig_off + (int64_t)t0 * k;  // digits of coefficient t0 + c at d0[c k + j]
  for (int l0 = 64 * wave; l0 < lx; l0 += 64 * CRT_COEF_PER_BLOCK) {
    const int l = l0 + lane;
    uint64_t lo[C];
    uint32_t hi[C];
#pragma unroll
    for (int c = 0; c < C; ++c) { lo[c] = 0; hi[c] = 0; }
    // P_j has at most 30 j / 32 + 1 limbs, so limbs >= l0 need j >= 32 l0 / 30 - 1
    int j0 = (32 * l0) / 30 - 1;
    if (j0 < 0) j0 = 0;
#pragma unroll 16
    for (int j = j0; j < k; ++j) {  // sixteen limb loads in flight per wavefront
      const uint32_t pl = l < tb.pstride ? tb.ptab[(int64_t)j * tb.pstride + l] : 0u;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const uint64_t pr = (uint64_t)(c < nc ? d0[c * k + j] : 0u) * pl;
        lo[c] += pr;
        hi[c] += lo[c] < pr ? 1u : 0u;
      }
    }
    if (l < lx) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        uint32_t* Xl = csm + c * 3 * lx_max;  // [lx] low words, then [2 lx] 64-bit carries as word pairs
        Xl[l] = (uint32_t)lo[c];
        const uint64_t cl = (lo[c] >> 32) | ((uint64_t)hi[c] << 32);
        Xl[lx_max + 2 * l] = (uint32_t)cl;
        Xl[lx_max + 2 * l + 1] = (uint32_t)(cl >> 32);
      }
    }
  }
  __syncthreads();
  if (wave >= nc) return;
  const int t = t0 + wave;
  const uint32_t* d = d0 + (int64_t)wave * k;
  const uint32_t* Xlo = csm + wave * 3 * lx_max;
  const uint32_t* Xc = Xlo + lx_max;
  if (lane != 0) return;
  const uint32_t* dt = d;
  int cmp = 0;
  for (int j = k - 1; j >= 0; --j) {
    const uint32_t h = (tb.primes[j].p - 1) >> 1;
    if (dt[j] != h) { cmp = dt[j] > h ? 1 : -1; break; }
  }
  const bool sub = cmp > 0;
  const uint32_t* M = tb.ptab + (int64_t)k * tb.pstride;
  uint32_t* out = ws + J.out_off + (int64_t)t * J.L;
  uint64_t carry = 0;
  int64_t borrow = 0;
  for (int l = 0; l < lx; ++l) {
    const uint64_t sv = (uint64_t)Xlo[l] + carry;
    uint32_t v = (uint32_t)sv;
    carry = (sv >> 32) + ((uint64_t)Xc[2 * l] | ((uint64_t)Xc[2 * l + 1] << 32));
    if (sub) {
      const int64_t dv = (int64_t)v - (int64_t)(l < tb.pstride ? M[l] : 0u) - borrow;
      borrow = dv < 0 ? 1 : 0;
      v = (uint32_t)(dv + (borrow << 32));
    }
    if (l < J.L) out[l] = v;
  }
  for (int l = lx; l < J.L; ++l) out[l] = sub ? 0xffffffffu : 0u;
}

// Chinese remaindering with few primes (k <= KC <= CRT_KS), the usual case of
// batched resultants: one lane per coefficient, so that every table constant
// is uniform across the wavefront (scalar loads) and no lane idles on a
// short prime list.
//   digits (Garner): y_i = (r_i - S_i) (P_i mod p_i)^-1 mod p_i with
//     S_i = sum_{j<i} y_j (P_j mod p_i), summed sixteen products per
//     reduction; the lane's digits wait in LDS (digit j at yl[64 j + lane]).
//   binary value: Horner's rule X <- X p_j + y_j from the top digit down in
//     LC registers, the multiply-add chain touching only the limbs X can
//     occupy so far (after digit j, X < P_k / P_j < 2^(30 (k - j))).
//   balanced result: X - M when X > (M-1)/2, decided on the digits on the
//     way down ((M-1)/2 has digits (p_j - 1)/2); L two's-complement limbs.
constexpr int CRT_KS = 128;                 // largest prime count of this path
__device__ __align__(64) uint32_t g_wts[CRT_KS * CRT_KS];  // [i][j] = Montgomery form of P_j mod p_i for j < i, else 0

__global__ void k_crt_small_init() {
  const int i = blockIdx.x;
  for (int j = threadIdx.x; j < CRT_KS; j += blockDim.x)
    g_wts[i * CRT_KS + j] = j < i ? g_wtab[(int64_t)j * KMAX + i] : 0u;
}

void launch_crt_small_init(hipStream_t s) {
  static_assert(CRT_KS <= KMAX, "small-path primes come from the table");
  hipLaunchKernelGGL(k_crt_small_init, dim3(CRT_KS), dim3(64), 0, s);
}

template <int KC>
__global__ __launch_bounds__(64) void k_crt_small(const ResJob* jobs, const int32_t* job_list, const int64_t* prefix,
                                                  int njobs, uint32_t* ws) {
  static_assert(KC <= CRT_KS && KC % 16 == 0, "prime capacity of the small path, whole groups of 16 digits");
  constexpr int LC = (30 * KC + 31) / 32 + 2;  // limbs of X (as lx_of)
  __shared__ uint32_t yl[KC * 64];
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[job_list[jj]];
  const int lane = threadIdx.x;
  const int t0 = (int)(b - prefix[jj]) * 64 + lane;
  const bool live = t0 <= J.D;
  const int t = live ? t0 : J.D;  // lanes past the last coefficient repeat it and store nothing
  const int k = J.k, n1 = J.D + 1;
  const uint32_t* V = ws + J.val_off + t;
  // Digits four at a time: the sums of rows i0..i0+3 over the digits before
  // i0 share each digit read (groups of sixteen: y_j < p_j and W < p_i, so
  // sixteen products stay below 2^64), then the block's own digits follow in
  // order with their products inside the block.  The digit slots start at
  // zero, so a group that reaches past i0 reads zeros for the digits not
  // computed yet (each lane reads only its own slots: no barrier).
  for (int j = 0; j < KC; ++j) yl[64 * j + lane] = 0u;
  // S < 2p, a sum below 2^64: S + a 2^-32 = S + hi + REDC(lo) with hi < 4p
  // taken below 2p and REDC(lo) <= p, back below 2p
  auto fold = [](uint32_t S, uint64_t a, const PrimeC& c) {
    uint32_t hi = (uint32_t)(a >> 32);
    const uint32_t h2 = hi - 2 * c.p;
    hi = h2 < hi ? h2 : hi;                                       // [0, 2p)
    uint32_t v = hi + redc((uint64_t)(uint32_t)a, c.p, c.pinv);  // < 3p + 1
    const uint32_t v2 = v - 2 * c.p;
    v = v2 < v ? v2 : v;  // [0, 2p)
    S += v;
    const uint32_t s2 = S - 2 * c.p;
    return s2 < S ? s2 : S;  // [0, 2p)
  };
  for (int i0 = 0; i0 < k; i0 += 4) {
    PrimeC cr[4];
    uint32_t S[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int r = 0; r < 4; ++r) cr[r] = g_primes[i0 + r];  // i0 + 3 < KC: rows of the table exist
    for (int j0 = 0; j0 < i0; j0 += 16) {
      uint32_t wv[4][16];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint4* w4 = reinterpret_cast<const uint4*>(g_wts + (i0 + r) * CRT_KS + j0);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const uint4 x = w4[h];
          wv[r][4 * h] = x.x; wv[r][4 * h + 1] = x.y; wv[r][4 * h + 2] = x.z; wv[r][4 * h + 3] = x.w;
        }
      }
      uint64_t acc[4] = {0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const uint64_t y = yl[64 * (j0 + u) + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] += y * wv[r][u];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) S[r] = fold(S[r], acc[r], cr[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + r;
      if (i >= k) break;  // uniform
      uint64_t a = 0;
#pragma unroll
      for (int q = 0; q < r; ++q) a += (uint64_t)yl[64 * (i0 + q) + lane] * g_wts[i * CRT_KS + i0 + q];
      const uint32_t Sf = fold(S[r], a, cr[r]);
      const uint32_t rv = V[(int64_t)i * n1];
      yl[64 * i + lane] =
          canon(redc((uint64_t)msub(rv, canon2(Sf, cr[r].p), cr[r].p) * g_garner[i], cr[r].p, cr[r].pinv), cr[r].p);
    }
  }
  uint32_t X[LC];
#pragma unroll
  for (int l = 0; l < LC; ++l) X[l] = 0;
  int cmp = 0;  // sign of X - (M-1)/2, from the top digit down
  for (int j = k - 1; j >= 0; --j) {
    const uint32_t p = g_primes[j].p;
    const uint32_t y = yl[64 * j + lane];
    const uint32_t h = (p - 1) >> 1;
    if (cmp == 0 && y != h) cmp = y > h ? 1 : -1;
    const int len = (30 * (k - j) + 31) / 32 + 1;  // limbs X can occupy after this step (uniform)
    uint64_t carry = y;
#pragma unroll
    for (int l0 = 0; l0 < LC; l0 += 8) {
      if (l0 < len) {  // uniform: chunks above X's length are skipped (they hold zeros)
#pragma unroll
        for (int l = l0; l < l0 + 8 && l < LC; ++l) {
          const uint64_t v = (uint64_t)X[l] * p + carry;
          X[l] = (uint32_t)v;
          carry = v >> 32;
        }
      }
    }
  }
  const bool sub = cmp > 0;
  if (sub) {  // X - M, M = P_k (uniform limbs), two's complement over LC limbs
    const uint32_t* M = g_ptab + (int64_t)k * LPS;
    uint32_t borrow = 0;
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      const uint64_t d = (uint64_t)X[l] - M[l] - borrow;
      X[l] = (uint32_t)d;
      borrow = (uint32_t)(d >> 63);
    }
  }
  if (!live) return;
  uint32_t* out = ws + J.out_off + (int64_t)t * J.L;
  const int L = J.L;
#pragma unroll
  for (int l = 0; l < LC; ++l)
    if (l < L) out[l] = X[l];
  for (int l = LC; l < L; ++l) out[l] = sub ? 0xffffffffu : 0u;
}

void launch_crt_small(int cls, const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d, int njobs,
                      int64_t nblocks, uint32_t* ws, hipStream_t s) {
  if (nblocks <= 0) return;
  const dim3 g((unsigned)nblocks), blk(64);
  switch (CRT_SMALL_K[cls]) {
    case 32: hipLaunchKernelGGL(k_crt_small<32>, g, blk, 0, s, jobs_d, job_list_d, prefix_d, njobs, ws); break;
    case 64: hipLaunchKernelGGL(k_crt_small<64>, g, blk, 0, s, jobs_d, job_list_d, prefix_d, njobs, ws); break;
    default: hipLaunchKernelGGL(k_crt_small<128>, g, blk, 0, s, jobs_d, job_list_d, prefix_d, njobs, ws); break;
  }
}

void launch_crt_digits(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d,
                       int njobs, int64_t nblocks, uint32_t* ws, hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_crt_digits, dim3((unsigned)nblocks), dim3(64 * CRT_COEF_PER_BLOCK), 0, s, tb,
                     jobs_d, job_list_d, prefix_d, njobs, ws);
}

void launch_crt_combine(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d,
                        int njobs, int64_t nblocks, int kmax, uint32_t* ws, hipStream_t s) {
  if (nblocks <= 0) return;
  const int lxm = lx_of(kmax);
  const size_t shmem = (size_t)CRT_COMB_PER_BLOCK * 3 * lxm * sizeof(uint32_t);
  static_assert((size_t)CRT_COMB_PER_BLOCK * 3 * ((30 * KMAX + 31) / 32 + 2) * 4 <= 160 * 1024,
                "combination buffers for the whole table fit the LDS of a CU");
  hipLaunchKernelGGL(k_crt_combine, dim3((unsigned)nblocks), dim3(64 * CRT_COEF_PER_BLOCK), shmem, s, tb, jobs_d,
                     job_list_d, prefix_d, njobs, lxm, ws);
}

CrtTables global_crt_tables() {
  static CrtTables cache[64];
  static bool have[64] = {false};
  int dev = 0;
  (void)hipGetDevice(&dev);
  if (dev >= 0 && dev < 64 && have[dev]) return cache[dev];
  CrtTables t{};
  void* p = nullptr;
  (void)hipGetSymbolAddress(&p, HIP_SYMBOL(g_primes)); t.primes = (const PrimeC*)p;
  (void)hipGetSymbolAddress(&p, HIP_SYMBOL(g_garner)); t.garner = (const uint32_t*)p;
  (void)hipGetSymbolAddress(&p, HIP_SYMBOL(g_wtab)); t.wtab = (const uint32_t*)p;
  (void)hipGetSymbolAddress(&p, HIP_SYMBOL(g_ptab)); t.ptab = (const uint32_t*)p;
  t.wstride = KMAX;
  t.pstride = LPS;
  if (dev >= 0 && dev < 64) { cache[dev] = t; have[dev] = true; }
  return t;
}

}  // namespace snc
