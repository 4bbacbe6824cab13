// Interpolation mod p from the values at x = 0..D: the images of the bivariate
// gcd (Section 2.1, "Lifting Phase": FastLift's Q), one workgroup per
// (coefficient, prime).
//   Newton coefficients of equispaced data, a_k = (Delta^k v_0) / k!, are the
//   convolution a_k = sum_{i<=k} (v_i / i!) ((-1)^{k-i} / (k-i)!).  The Newton
//   form P = sum_k a_k N_k, N_k = x (x-1) ... (x-k+1), is expanded blockwise:
//   with blocks of 64 terms starting at b = 64j,
//     Q_j = sum_{t<64} a_{b+t} prod_{i=b}^{b+t-1} (x - i),   F_j = prod_{i=b}^{b+63} (x - i),
//   and P = Q_0 + F_0 (Q_1 + F_1 (Q_2 + ...)).
//   Both the convolution and the products P F_j are Toeplitz sums; a
//   wavefront owns 64 consecutive outputs (one per lane), takes the uniform
//   operand from a register by readlane and the sliding one from LDS (one
//   coalesced read per product), and reduces every 8 products.  Q_j and F_j
//   are built by the wavefront that computed a_{64j..64j+63}, by 64 steps of
//   a one-lane shift (DPP) and a multiply-add, without barriers.
//
// The tables (180 MB) are this file's own: its code object is loaded and they
// are filled when a bivariate gcd first interpolates on a device, not with the
// context.  Loading takes 0.4 ms a megabyte, whether or not a kernel reads it.
#include <hip/hip_runtime.h>

#include <mutex>
#include <set>

#include "eval_elim.hpp"
#include "runtime_internal.hpp"
#include "toeplitz.hpp"

namespace snc {

constexpr int IB = 64;    // Newton terms per block (one per lane)
constexpr int IPAD = 64;  // zero words below index 0 of the sliding operands
static_assert((4 * ((MAX_D + IB) / IB * IB) + 2 * IPAD) * 4 <= 160 * 1024,
              "interpolation buffers for the largest degree bound exceed the LDS of a CU");

// Montgomery form of 1/t! for every prime of the table and t <= MAX_D
__device__ uint32_t g_ifact[(int64_t)KMAX * (MAX_D + 1)];

__global__ void k_ifact_init(const PrimeC* primes) {
  const int pi = blockIdx.x * blockDim.x + threadIdx.x;
  if (pi >= KMAX) return;
  const PrimeC c = primes[pi];
  uint32_t f = c.r1;
  for (int t = 2; t <= MAX_D; ++t) f = mmulc(f, to_mont((uint32_t)t, c), c.p, c.pinv);
  uint32_t inv = minv(f, c);  // 1/MAX_D!
  uint32_t* row = g_ifact + (int64_t)pi * (MAX_D + 1);
  for (int t = MAX_D; t >= 1; --t) {
    row[t] = inv;
    inv = mmulc(inv, to_mont((uint32_t)t, c), c.p, c.pinv);
  }
  row[0] = inv;
}

// lane L receives lane L-1 of v, lane 0 receives 0
__device__ __forceinline__ uint32_t lane_shr1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138 /* wave_shr:1 */, 0xf, 0xf, true);
}

// Montgomery coefficients of x^0 .. x^63 of F_j = (x - 64j)(x - 64j - 1) ... (x - 64j - 63)
// (x^64 implied) for every prime and the blocks j < FB_NBLK
constexpr int FB_NBLK = 64;
__device__ uint32_t g_fblk[(int64_t)KMAX * FB_NBLK * 64];

// one wavefront per (prime, block): F <- F (x - (64 j + t)) for t = 0..63,
// coefficient of x^lane in lane (the x^64 term leaves lane 63 and is implied)
__global__ __launch_bounds__(64) void k_fblk_init(const PrimeC* primes) {
  const int pi = blockIdx.x / FB_NBLK, j = blockIdx.x % FB_NBLK, lane = threadIdx.x;
  const PrimeC c = primes[pi];
  uint32_t f = lane == 0 ? c.r1 : 0u;
  for (int t = 0; t < 64; ++t) {
    const uint32_t nk = to_mont(c.p - (uint32_t)(64 * j + t), c);  // -(64 j + t)
    const uint32_t fprev = lane_shr1(f);
    f = canon(redc((uint64_t)nk * f + ((uint64_t)fprev << 32), c.p, c.pinv), c.p);
  }
  g_fblk[((int64_t)pi * FB_NBLK + j) * 64 + lane] = f;
}

__device__ __forceinline__ uint32_t bcast(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// s + sum_{q<64} u_q S[-q] with u_q = lane q of u (broadcast by readlane) and
// S per lane; s canonical in, out
__device__ __forceinline__ uint32_t toeplitz64_bc(uint32_t s, uint32_t u, const uint32_t* S, const PrimeC& c) {
#pragma unroll
  for (int g = 0; g < IB; g += 8) {
    uint64_t acc = 0;
#pragma unroll
    for (int q = g; q < g + 8; ++q) acc += (uint64_t)bcast(u, q) * S[-q];  // 8 p^2 < 2^63
    s = canon(s + redc(acc, c.p, c.pinv), c.p);
  }
  return s;
}

__global__ __launch_bounds__(INTERP_THREADS) void k_interp(const PrimeC* primes, const ResJob* jobs,
                                                           const int64_t* prefix, int njobs, uint32_t* ws) {
  extern __shared__ uint4 sm4[];  // sections 16-byte aligned: IPAD and Dp are multiples of 64 words
  uint32_t* sm = reinterpret_cast<uint32_t*>(sm4);
  constexpr int NW = INTERP_THREADS / 64;
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[jj];
  const int pi = (int)(b - prefix[jj]);
  const PrimeC c = primes[pi];
  const int n1 = J.D + 1;
  const int nblk = (n1 + IB - 1) / IB;
  const int Dp = nblk * IB;
  const uint32_t* V = ws + J.pts_off + (int64_t)pi * n1;  // values at the points
  uint32_t* C = ws + J.val_off + (int64_t)pi * n1;        // coefficients
  const uint32_t* IF = g_ifact + (int64_t)pi * (MAX_D + 1);
  uint32_t* Wp = sm;             // [IPAD + Dp]: zeros, then w_j = (-1)^j / j!; later a P buffer
  uint32_t* Qb = Wp + IPAD + Dp; // [Dp]: Q_j at 64j
  uint32_t* Fb = Qb + Dp;        // [Dp]: coefficients 0..63 of F_j at 64j (x^64 implied)
  uint32_t* P1 = Fb + Dp;        // [IPAD + Dp]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // w_j = (-1)^j / j! behind IPAD zeros; u_i = v_i / i! staged in P1 (free until the expansion)
  uint32_t* U = P1;
  for (int t = tid; t < IPAD + Dp; t += INTERP_THREADS) {
    const int j = t - IPAD;
    uint32_t w = 0;
    if (j >= 0 && j < n1) {
      const uint32_t f = IF[j];
      w = (j & 1) ? mneg(f, c.p) : f;
    }
    Wp[t] = w;
    if (t < Dp) U[t] = t < n1 ? mmulc(canon(V[t], c.p), IF[t], c.p, c.pinv) : 0u;
  }
  __syncthreads();

  for (int ob = wave; ob < nblk; ob += NW) {
    const int b0 = ob * IB;
    // a_k for k = b0 + lane
    const uint32_t* wk = Wp + IPAD + b0 + lane;
    uint32_t a = 0;
    for (int ib = 0; ib <= ob; ++ib) a = toeplitz64(a, U + ib * IB, wk - ib * IB, c);
    // Q_ob and F_ob, coefficient of x^lane in lane (F_ob from its table when
    // the block has one)
    const int len = min(IB, n1 - b0);
    const uint32_t nk = to_mont(c.p - (uint32_t)(b0 + lane), c);  // -(b0 + lane)
    uint32_t q = lane == 0 ? bcast(a, len - 1) : 0u;
    const bool ftab = ob < FB_NBLK;  // uniform
    uint32_t f = ftab ? g_fblk[((int64_t)pi * FB_NBLK + ob) * 64 + lane] : (lane == 0 ? c.r1 : 0u);
    for (int s = 0; s < IB; ++s) {
      if (!ftab) {
        const uint32_t fprev = lane_shr1(f);  // F <- F (x - (b0 + s))
        f = canon(redc((uint64_t)bcast(nk, s) * f + ((uint64_t)fprev << 32), c.p, c.pinv), c.p);
      }
      const int kq = len - 2 - s;           // Q <- Q (x - (b0 + kq)) + a_{b0 + kq}
      if (kq >= 0) {
        const uint32_t add = bcast(a, kq);
        const uint32_t qprev = lane_shr1(q) + (lane == 0 ? add : 0u);
        q = canon(redc((uint64_t)bcast(nk, kq) * q + ((uint64_t)qprev << 32), c.p, c.pinv), c.p);
      }
    }
    Qb[b0 + lane] = q;
    Fb[b0 + lane] = f;
  }
  __syncthreads();

  // P = Q_{nblk-1}; P <- P F_j + Q_j for j = nblk-2 .. 0.  Entries above the
  // current degree stay zero, so whole 64-blocks are computed and stored.
  uint32_t* Pa = Wp;
  uint32_t* Pb = P1;
  const int lastb = (nblk - 1) * IB;
  const int lastlen = n1 - lastb;
  for (int t = tid; t < IPAD + Dp; t += INTERP_THREADS) {
    const int x = t - IPAD;
    Pa[t] = (x >= 0 && x < lastlen) ? Qb[lastb + x] : 0u;
    Pb[t] = 0u;
  }
  __syncthreads();
  int dP = lastlen - 1;
  for (int j = nblk - 2; j >= 0; --j) {
    const int dN = dP + IB;
    const int nob = dN / IB + 1;
    for (int ob = wave; ob < nob; ob += NW) {
      const int t = ob * IB + lane;
      const uint32_t* pt = Pa + IPAD + t;  // P[t - i] = pt[-i]
      uint32_t s = pt[-IB];                // x^64 term of F_j
      if (t < IB) s = madd(s, Qb[j * IB + t], c.p);
      Pb[IPAD + t] = toeplitz64(s, Fb + j * IB, pt, c);
    }
    __syncthreads();
    uint32_t* tmp = Pa; Pa = Pb; Pb = tmp;
    dP = dN;
  }
  for (int t = tid; t < n1; t += INTERP_THREADS) C[t] = from_mont(Pa[IPAD + t], c);
}

// ---------------------------------------------------------------------------
// Block-parallel interpolation (degree bounds below 64 IFF_J).
//   With G_j = x (x-1) ... (x - 64j + 1) the Newton form is P = sum_j G_j Q_j
//   (Q_j as above), so the blocks of 64 coefficients of P are independent
//   sums of Toeplitz products.  Two launches, each with one workgroup per
//   (resultant, prime, block):
//   k_interp_q:   Newton coefficients a_{64j..64j+63} (the convolution units
//                 over input blocks spread over the wavefronts, summed in LDS)
//                 and Q_j, stored in the workspace;
//   k_interp_out: coefficients 64 ob .. 64 ob + 63 of P as sum_{j >= ob} of
//                 G_j Q_j (one wavefront per j).
//   The G_j come from a table filled once per device.
// ---------------------------------------------------------------------------
constexpr int IFF_W = 32 * IFF_J * (IFF_J - 1) + IFF_J;  // words per prime: rows j < IFF_J of degree 64 j
__host__ __device__ constexpr int iff_off(int j) { return 32 * j * (j - 1) + j; }
constexpr int IBT = IFF_J;  // wavefronts per workgroup (one per input block or Newton block)

// Montgomery form of the coefficients of G_j for the first IFF_K primes
__device__ uint32_t g_ffact[(int64_t)IFF_K * IFF_W];

__global__ __launch_bounds__(256) void k_ffact_init(const PrimeC* primes) {
  __shared__ uint32_t buf[2][64 * IFF_J + 1];
  const int pi = blockIdx.x;
  const PrimeC c = primes[pi];
  uint32_t* out = g_ffact + (int64_t)pi * IFF_W;
  for (int m = threadIdx.x; m <= 64 * IFF_J; m += 256) buf[0][m] = m == 0 ? c.r1 : 0u;
  if (threadIdx.x == 0) out[iff_off(0)] = c.r1;
  __syncthreads();
  int cur = 0;
  for (int t = 0; t < 64 * (IFF_J - 1); ++t) {  // multiply by (x - t): degree t -> t + 1
    const uint32_t nt = to_mont(t == 0 ? 0u : c.p - (uint32_t)t, c);
    for (int m = threadIdx.x; m <= t + 1; m += 256) {
      const uint32_t lo = m >= 1 ? buf[cur][m - 1] : 0u;
      const uint32_t hi = m <= t ? buf[cur][m] : 0u;
      buf[cur ^ 1][m] = madd(lo, mmulc(nt, hi, c.p, c.pinv), c.p);
    }
    __syncthreads();
    cur ^= 1;
    if ((t + 1) % 64 == 0) {  // G_j complete, j = (t + 1) / 64
      const int j = (t + 1) / 64;
      for (int m = threadIdx.x; m <= t + 1; m += 256) out[iff_off(j) + m] = buf[cur][m];
    }
  }
}

__global__ __launch_bounds__(64 * IBT) void k_interp_q(const PrimeC* primes, const ResJob* jobs,
                                                       const int64_t* prefix, int njobs, uint32_t* ws) {
  __shared__ __align__(16) uint32_t U[64 * IFF_J];  // v_i / i!
  __shared__ uint32_t Wp[IPAD + 64 * IFF_J];  // zeros, then (-1)^j / j!
  __shared__ uint32_t part[IFF_J][64];        // convolution units of this Newton block
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[jj];
  const int n1 = J.D + 1;
  const int nblk = (n1 + 63) / 64;
  const int64_t lb = b - prefix[jj];
  const int pi = (int)(lb / nblk);
  const int j = (int)(lb % nblk);             // Newton block
  const PrimeC c = primes[pi];
  const uint32_t* V = ws + J.pts_off + (int64_t)pi * n1;
  const uint32_t* IF = g_ifact + (int64_t)pi * (MAX_D + 1);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int top = 64 * (j + 1);               // inputs and weights below 64 (j + 1) are read
  for (int t = tid; t < IPAD + top; t += 64 * IBT) {
    const int i = t - IPAD;
    uint32_t w = 0;
    if (i >= 0 && i < n1) {
      const uint32_t f = IF[i];
      w = (i & 1) ? mneg(f, c.p) : f;
    }
    Wp[t] = w;
    if (t < top) U[t] = t < n1 ? mmulc(canon(V[t], c.p), IF[t], c.p, c.pinv) : 0u;
  }
  __syncthreads();
  // a_k, k = 64 j + lane: input block ib on wavefront ib
  if (wave <= j) part[wave][lane] = toeplitz64(0u, U + wave * 64, Wp + IPAD + 64 * (j - wave) + lane, c);
  __syncthreads();
  if (wave != 0) return;
  uint32_t a = 0;
  for (int ib = 0; ib <= j; ++ib) a = madd(a, part[ib][lane], c.p);
  // Q_j, coefficient of x^lane in lane
  const int b0 = 64 * j;
  const int len = min(64, n1 - b0);
  const uint32_t nk = to_mont(c.p - (uint32_t)(b0 + lane), c);  // -(b0 + lane)
  uint32_t q = lane == 0 ? bcast(a, len - 1) : 0u;
  for (int s = 0; s + 2 <= len; ++s) {  // Q <- Q (x - (b0 + kq)) + a_{b0 + kq}, kq = len - 2 - s
    const int kq = len - 2 - s;
    const uint32_t add = bcast(a, kq);
    const uint32_t qprev = lane_shr1(q) + (lane == 0 ? add : 0u);
    q = canon(redc((uint64_t)bcast(nk, kq) * q + ((uint64_t)qprev << 32), c.p, c.pinv), c.p);
  }
  ws[J.nq_off + (int64_t)pi * nblk * 64 + b0 + lane] = q;
}

__global__ __launch_bounds__(64 * IBT) void k_interp_out(const PrimeC* primes, const ResJob* jobs,
                                                         const int64_t* prefix, int njobs, uint32_t* ws) {
  __shared__ uint32_t Gs[IFF_J][128];   // coefficients 64 ob - 64 .. 64 ob + 63 of G_j
  __shared__ uint32_t outp[IFF_J][64];  // G_j Q_j on this block
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[jj];
  const int n1 = J.D + 1;
  const int nblk = (n1 + 63) / 64;
  const int64_t lb = b - prefix[jj];
  const int pi = (int)(lb / nblk);
  const int ob = (int)(lb % nblk);      // output block
  const PrimeC c = primes[pi];
  const uint32_t* GF = g_ffact + (int64_t)pi * IFF_W;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = ob + wave;              // Newton block of this wavefront
  if (j < nblk) {
    for (int m = lane; m < 128; m += 64) {
      const int g = 64 * ob - 64 + m;
      Gs[wave][m] = (g >= 0 && g <= 64 * j) ? GF[iff_off(j) + g] : 0u;
    }
    const uint32_t q = ws[J.nq_off + (int64_t)pi * nblk * 64 + 64 * j + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    outp[wave][lane] = toeplitz64_bc(0u, q, &Gs[wave][64 + lane], c);
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t s = 0;
    for (int w = 0; w < nblk - ob; ++w) s = madd(s, outp[w][lane], c.p);
    const int t = 64 * ob + lane;
    if (t < n1) ws[J.val_off + (int64_t)pi * n1 + t] = from_mont(s, c);
  }
}

void launch_interp_blk(const ResJob* jobs_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks, uint32_t* ws,
                       hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_interp_q, dim3((unsigned)nblocks), dim3(64 * IBT), 0, s, global_crt_tables().primes,
                     jobs_d, blk_prefix_d, njobs, ws);
  hipLaunchKernelGGL(k_interp_out, dim3((unsigned)nblocks), dim3(64 * IBT), 0, s, global_crt_tables().primes,
                     jobs_d, blk_prefix_d, njobs, ws);
}

size_t interp_lds_bytes(int max_D) {
  const size_t Dp = (size_t)((max_D + 1 + IB - 1) / IB) * IB;
  return (4 * Dp + 2 * IPAD) * sizeof(uint32_t);
}

void launch_interp(const ResJob* jobs_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks,
                   int max_D, uint32_t* ws, hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_interp, dim3((unsigned)nblocks), dim3(INTERP_THREADS), interp_lds_bytes(max_D), s,
                     global_crt_tables().primes, jobs_d, blk_prefix_d, njobs, ws);
}

// on the call's stream; other contexts wait for it under the lock
int ensure_int_interp(int device, hipStream_t s, std::string& err) {
  static std::mutex mu;
  static std::set<int> done;
  std::lock_guard<std::mutex> lk(mu);
  if (done.count(device)) return SNC_OK;
  static_assert(IFF_K <= KMAX, "falling-factorial table covers table primes only");
  const PrimeC* primes = global_crt_tables().primes;
  hipError_t e = hipFuncSetAttribute((const void*)k_interp, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_ifact_init, dim3(KMAX / 64), dim3(64), 0, s, primes);
    hipLaunchKernelGGL(k_fblk_init, dim3(KMAX * FB_NBLK), dim3(64), 0, s, primes);
    hipLaunchKernelGGL(k_ffact_init, dim3(IFF_K), dim3(256), 0, s, primes);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) { err = std::string("interpolation tables: ") + hipGetErrorString(e); return SNC_EDEVICE; }
  done.insert(device);
  return SNC_OK;
}

}  // namespace snc
