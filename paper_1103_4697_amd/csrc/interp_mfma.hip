// Interpolation mod p on the matrix cores (Section 4, "Symbolic Speedups":
// the images over Z_p at points are combined into coefficients over Z_p).
//
// Points.  +-q^i mod p, i = 0..D/2, with Q = q^2 of order above MAX_D / 2 mod
// p.  P(x) = E(x^2) + x O(x^2), so the pair of values at +-q^i gives E and O
// at Q^i: two interpolations of half the size at powers of Q.  With
// phi_m = (Q - 1)(Q^2 - 1) ... (Q^m - 1) the Newton polynomials at those points
// satisfy
//   N_k(Q^i) = Q^C(k,2) phi_i / phi_{i-k},
//   N_k(z)   = sum_i (-1)^{k-i} Q^C(k-i,2) phi_k / (phi_i phi_{k-i}) z^i
// (the q-binomial theorem), and 1 / sum_m z^m / phi_m = sum_m t_m z^m,
// t_m = (-1)^m Q^C(m,2) / phi_m.  So values v_i become coefficients c_i by two
// products with the same sequence t, lower and upper triangular Toeplitz, and
// scalings by tables:
//   u_i = v_i / phi_i,   b_k = sum_{i <= k} t_{k-i} u_i,
//   e_k = b_k psi_k,     psi_k = phi_k Q^-C(k,2) / 2,
//   c_i = (1 / phi_i) sum_{k >= i} t_{k-i} e_k,
// v_i the sum of the pair's values for E and their difference over q^i for O
// (psi holds the factor 1/2 of both).  At points 0..D the expansion of the
// Newton form needs falling factorials that differ from block to block.
//
// Mapping.  A workgroup takes one prime and a group of jobs.  Outputs go in
// blocks of 64; a row of the matrix product is one (job, parity, block), and step d
// multiplies the rows' input blocks at distance d by the 64 x 64 Toeplitz
// block T_d, the same for every row.  T_d is never stored: column n of a tile
// is output 4 n + kappa (kappa = 0..3), so a lane's 16 contraction entries
// are consecutive bytes of t that start at a multiple of four plus a shift
// common to the wavefront.  Five words read from LDS give the operands of all
// four kappa by byte alignment.
//
// Bounds and figures (MI355X).  The sums over the whole degree were 64-bit
// multiply-adds on the vector unit (one wavefront per (resultant, prime) at
// 77% of its issue slots, or a workgroup with barriers per block), with the
// expansion of each Newton block a further sixth.  512 pairs of degrees 8..40
// (25,000 (resultant, prime) pairs, degree bounds up to 1,600): 1,100 -> 240
// us.  No unit is at its limit there: counters show 47% of the vector unit's
// issue slots, 32% of LDS cycles (almost half of them bank conflicts) and the
// matrix cores busy 24% of theirs; the rest is the latency of the phases
// between the barriers.  One pair of degree bound 3,072 with 262 primes: 523
// -> 51 us.  Degree bound 225, 15 pairs, 2,052 primes: 248 -> 94 us (52%, 28%
// and 11%: staging and folding weigh more in short sums); degree bound 552, 35
// primes: 13 (two launches) -> 10.3 us; degree bound 36, 5 primes: 8.4 (two
// launches) -> 7.1 us, both latency.
#include <hip/hip_runtime.h>

#include "eval_elim.hpp"
#include "general_elim.hpp"
#include "mfma_modp.hpp"

namespace snc {

constexpr int IM_N = MAX_D / 2 + 1;                    // coefficients of one parity, at most
constexpr int IM_DP = (IM_N + 63) / 64 * 64;           // whole blocks
constexpr int IM_TROW = IM_DP + 64;                    // bytes of a plane of t per prime (zeros past IM_N)

__device__ uint32_t g_iphi[(size_t)KMAX * IM_N];   // Montgomery form of 1 / phi_m
__device__ uint32_t g_psi[(size_t)KMAX * IM_N];    // Montgomery form of psi_m
__device__ __align__(16) int8_t g_tq[(size_t)KMAX * 4 * IM_TROW];  // bytes of t_m (Montgomery form), four planes
__device__ uint32_t g_points[(size_t)KMAX * POINT_ROW];
__device__ uint32_t g_ipoints[(size_t)KMAX * POINT_ROW];  // the same powers of 1/q

// inclusive product over the lanes up to this one (DOWN: from this one up)
template <bool DOWN>
__device__ __forceinline__ uint32_t wave_product(uint32_t v, int lane, const PrimeC& c) {
  for (int d = 1; d < 64; d *= 2) {
    const uint32_t o = (uint32_t)(DOWN ? __shfl_down((int)v, d) : __shfl_up((int)v, d));
    if (DOWN ? lane + d < 64 : lane >= d) v = mmulc(v, o, c.p, c.pinv);
  }
  return v;
}

// One prime per wavefront, 64 entries at a time: running products by a scan
// over the lanes, powers by a step of 64 (0.14 ms for the whole table;
// a thread per prime, one entry after the other with scattered stores, 3.8).
__global__ __launch_bounds__(64) void k_points_init(const PrimeC* primes) {
  const int pi = blockIdx.x, lane = threadIdx.x;
  const PrimeC c = primes[pi];
  uint32_t* ip = g_iphi + (size_t)pi * IM_N;
  uint32_t* ps = g_psi + (size_t)pi * IM_N;
  int8_t* tq = g_tq + (size_t)pi * 4 * IM_TROW;
  auto mul = [&](uint32_t a, uint32_t b) { return mmulc(a, b, c.p, c.pinv); };
  constexpr int NB = (IM_N + 63) / 64;
  // the least q >= 2 with Q = q^2 of order above IM_N - 1
  uint32_t q = 0, Q = 0;
  for (uint32_t g = 2; q == 0; ++g) {
    const uint32_t gm = to_mont(g, c);
    Q = mul(gm, gm);
    const uint32_t step = mpow(Q, 64, c);
    uint32_t v = mpow(Q, (uint32_t)lane, c);
    bool one = false;
    for (int b = 0; b < NB; ++b) {
      const int m = 64 * b + lane;
      one |= m >= 1 && m < IM_N && v == c.r1;
      v = mul(v, step);
    }
    if (!__any(one)) q = gm;
  }
  const uint32_t qi = minv(q, c), Qi = mul(qi, qi);
  // factors Q^m - 1 (1 at m = 0 and past the end) and phi_m, their products, into psi's row
  auto factor = [&](int m, uint32_t Qm) { return m >= 1 && m < IM_N ? msub(Qm, c.r1, c.p) : c.r1; };
  const uint32_t Q64 = mpow(Q, 64, c), Qi64 = mpow(Qi, 64, c);
  uint32_t Qm = mpow(Q, (uint32_t)lane, c), carry = c.r1;
  for (int b = 0; b < NB; ++b) {
    const int m = 64 * b + lane;
    const uint32_t f = mul(carry, wave_product<false>(factor(m, Qm), lane, c));
    if (m < IM_N) ps[m] = f;
    carry = (uint32_t)__shfl((int)f, 63);
    Qm = mul(Qm, Q64);
  }
  // 1 / phi_m from the top down
  carry = minv(carry, c);
  for (int b = NB - 1; b >= 0; --b) {
    const int m = 64 * b + lane;
    Qm = mul(Qm, Qi64);
    const uint32_t f = wave_product<true>(factor(m, Qm), lane, c);
    const uint32_t above = (uint32_t)__shfl_down((int)f, 1);
    if (m < IM_N) ip[m] = lane < 63 ? mul(carry, above) : carry;
    carry = mul(carry, (uint32_t)__shfl((int)f, 0));
  }
  // t_m and psi_m: Q^C(m,2) and its inverse by C(m + 64, 2) = C(m, 2) + 64 m + C(64, 2)
  const uint32_t c0 = (uint32_t)(lane * (lane - 1) / 2);
  uint32_t Qc = mpow(Q, c0, c), Qr = mul(mpow(Q64, (uint32_t)lane, c), mpow(Q, 2016, c));
  uint32_t hc = mul(mpow(Qi, c0, c), to_mont((c.p + 1) / 2, c));
  uint32_t Hr = mul(mpow(Qi64, (uint32_t)lane, c), mpow(Qi, 2016, c));
  const uint32_t Q4096 = mpow(Q64, 64, c), Qi4096 = mpow(Qi64, 64, c);
  for (int m = lane; m < IM_N; m += 64) {
    uint32_t t = mul(Qc, ip[m]);
    if (m & 1) t = mneg(t, c.p);
    const uint32_t w = balance4(t);
    for (int b = 0; b < 4; ++b) tq[(size_t)b * IM_TROW + m] = (int8_t)(w >> (8 * b));
    ps[m] = mul(ps[m], hc);
    Qc = mul(Qc, Qr);
    hc = mul(hc, Hr);
    Qr = mul(Qr, Q4096);
    Hr = mul(Hr, Qi4096);
  }
  for (int x = lane; x < POINT_ROW; x += 64) {
    const uint32_t e = x < 32 ? (uint32_t)x : 32u * (uint32_t)(x - 32);
    g_points[(size_t)pi * POINT_ROW + x] = mpow(q, e, c);
    g_ipoints[(size_t)pi * POINT_ROW + x] = mpow(qi, e, c);
  }
}

constexpr int IM_THREADS = 256;
constexpr int IM_WAVES = IM_THREADS / 64;
constexpr int IM_MAXROWS = 192;
constexpr int IM_LOADS = 4;   // pairs of values a thread has in flight
constexpr int IM_MARKS = 16;  // abnormal instances of a workgroup that take a wavefront each
static_assert(2 * (IM_DP / 64) <= IM_MAXROWS, "the rows of one job of the largest degree bound");
constexpr int IM_SEQ = 2 * IM_JOBS;  // sequences of a group: the even and the odd coefficients of each job

// LDS of a group: the planes of t (reversed and ascending, or one after the
// other where both do not fit; zeros below index 0), then for each sequence
// the planes of u and of e
__host__ __device__ constexpr int im_tplane(int Dp) { return Dp + 144; }
__host__ __device__ constexpr bool im_both(int Dp) { return Dp <= 4096; }
static_assert(4 * im_tplane(IM_DP) + 16 * IM_DP + 8 * 1024 <= 160 * 1024,
              "the buffers of the largest degree bound fit the LDS of a CU");

// bytes sh .. sh + 15 of five words
template <int SH>
__device__ __forceinline__ v4i align16(const uint32_t (&d)[5]) {
  v4i r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = SH == 0 ? (int)d[i] : SH == 4 ? (int)d[i + 1] : (int)__builtin_amdgcn_alignbyte(d[i + 1], d[i], SH & 3);
  return r;
}

// One unit: 16 rows, the NK columns kappa = NK H + 0 .. NK - 1 of each n.
// STAGE 1 reads t reversed (step d goes down in memory), STAGE 2 ascending.
// a0 / astep: LDS byte offset of the lane's row operand at d = 0 and its
// change per step; valid for d <= K, zeros from zoff otherwise.  A step's
// operands are read while the step before multiplies.
struct ToeplitzOps {
  v4i a[4];
  uint32_t t[4][5];
};

template <int STAGE, int NK, int H>
__device__ __forceinline__ void toeplitz_unit(v4i (&acc)[NK][7], const uint8_t* sm, int len, int K, int a0, int astep,
                                              int aplane, int zoff, int b0, int bplane) {
#pragma unroll
  for (int x = 0; x < NK; ++x)
#pragma unroll
    for (int d = 0; d < 7; ++d) acc[x][d] = v4i{0, 0, 0, 0};
  constexpr int bstep = STAGE == 1 ? -64 : 64;
  constexpr int SH0 = (STAGE == 1 ? 3 : 4) - NK * H, SH1 = NK == 2 ? SH0 - 1 : SH0;
  auto load = [&](ToeplitzOps& o, int d) {
    const bool ok = d <= K;
    const int ad = ok ? a0 + d * astep : zoff, ap = ok ? aplane : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) o.a[q] = *reinterpret_cast<const v4i*>(sm + ad + q * ap);
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const uint32_t* tw = reinterpret_cast<const uint32_t*>(sm + b0 + d * bstep + y * bplane);
#pragma unroll
      for (int i = 0; i < 5; ++i) o.t[y][i] = tw[i];
    }
  };
  auto mul = [&](const ToeplitzOps& o) {
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const v4i f0 = align16<SH0>(o.t[y]), f1 = align16<SH1>(o.t[y]);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        acc[0][x + y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(o.a[x], f0, acc[0][x + y], 0, 0, 0);
        if constexpr (NK == 2)
          acc[1][x + y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(o.a[x], f1, acc[1][x + y], 0, 0, 0);
      }
    }
  };
  ToeplitzOps p, q;
  load(p, 0);
  for (int d = 0; d < len; d += 2) {
    load(q, min(d + 1, len - 1));
    mul(p);
    if (d + 1 < len) {
      load(p, min(d + 2, len - 1));
      mul(q);
    }
  }
}

// LDS of a workgroup and its rows, as the stages see them
struct InterpLds {
  uint8_t* sm;
  const int32_t *row, *n1, *blk, *u;
  const int64_t* val;
  int TP, Dp, zoff, t0;  // t0: byte offset of the stage's planes of t
};

// One stage on one unit: the products, then e = b psi into the job's planes
// (stage 1) or the coefficients c = b / phi to memory (stage 2).
template <int STAGE, int NK, int H>
__device__ __forceinline__ void interp_unit(const InterpLds& S, int tile, int lane, const uint32_t* scale, uint32_t* ws,
                                            uint32_t k56, const PrimeC& c) {
  const int n = lane & 15, kg = lane >> 4;
  const int row = S.row[16 * tile + n];
  const int jj = row < 0 ? 0 : row >> 16, K = row < 0 ? -1 : row & 0xffff;
  const int len = __builtin_amdgcn_readfirstlane((S.row[16 * tile] & 0xffff) + 1);
  const int dp = 64 * S.blk[jj];
  v4i acc[NK][7];
  // input blocks K, K - 1, .. of u, or dp / 64 - 1 - K and up of e
  const int a0 = S.u[jj] + (STAGE == 1 ? 64 * K : 4 * dp + dp - 64 - 64 * K) + 16 * kg;
  const int b0 = S.t0 + (STAGE == 1 ? S.Dp + 64 : 60) - 4 * n + 16 * kg;
  toeplitz_unit<STAGE, NK, H>(acc, S.sm, len, K, a0, STAGE == 1 ? -64 : 64, dp, S.zoff, b0, S.TP);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int orow = S.row[16 * tile + 4 * kg + r];
    if (orow < 0) continue;
    const int oj = orow >> 16, oK = orow & 0xffff, n1 = S.n1[oj], ob = S.blk[oj];
    const int k0 = 64 * (STAGE == 1 ? oK : ob - 1 - oK) + 4 * n + NK * H;
    uint32_t w[NK];
#pragma unroll
    for (int e = 0; e < NK; ++e) {
      const uint32_t b = fold_bytes(acc[e][0][r], acc[e][1][r], acc[e][2][r], acc[e][3][r], acc[e][4][r],
                                    acc[e][5][r], acc[e][6][r], k56, c);
      w[e] = k0 + e < n1 ? mmulc(b, scale[k0 + e], c.p, c.pinv) : 0u;
    }
    if constexpr (STAGE == 1) {
      uint8_t* E = S.sm + S.u[oj] + 256 * ob + k0;
#pragma unroll
      for (int e = 0; e < NK; ++e) w[e] = balance4(w[e]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (NK == 2)
          *reinterpret_cast<uint16_t*>(E + q * 64 * ob) =
              (uint16_t)(((w[0] >> (8 * q)) & 0xffu) | (((w[1] >> (8 * q)) & 0xffu) << 8));
        else
          E[q * 64 * ob] = (uint8_t)(w[0] >> (8 * q));
      }
    } else {
      uint32_t* C = ws + S.val[oj];  // coefficients of x^(2 k) or x^(2 k + 1)
#pragma unroll
      for (int e = 0; e < NK; ++e)
        if (k0 + e < n1) C[2 * (k0 + e)] = from_mont(w[e], c);
    }
  }
}

template <int STAGE>
__device__ __forceinline__ void interp_stage(const InterpLds& S, int ntile, int wave, int lane, const uint32_t* scale,
                                             uint32_t* ws, uint32_t k56, const PrimeC& c) {
  if (ntile == 1) {  // one tile: a column class per wavefront
    switch (wave) {
      case 0: interp_unit<STAGE, 1, 0>(S, 0, lane, scale, ws, k56, c); break;
      case 1: interp_unit<STAGE, 1, 1>(S, 0, lane, scale, ws, k56, c); break;
      case 2: interp_unit<STAGE, 1, 2>(S, 0, lane, scale, ws, k56, c); break;
      default: interp_unit<STAGE, 1, 3>(S, 0, lane, scale, ws, k56, c); break;
    }
    return;
  }
  // units (tile, column pair) longest first, dealt to the wavefronts forth and back
  for (int x = wave, turn = 0; x < 2 * ntile;
       ++turn, x = turn * IM_WAVES + ((turn & 1) ? IM_WAVES - 1 - wave : wave)) {
    if (x & 1) interp_unit<STAGE, 2, 1>(S, x >> 1, lane, scale, ws, k56, c);
    else interp_unit<STAGE, 2, 0>(S, x >> 1, lane, scale, ws, k56, c);
  }
}

__global__ __launch_bounds__(IM_THREADS) void k_interp_mfma(const PrimeC* primes, const ResJob* jobs,
                                                            const int32_t* job_list, const int32_t* gstart,
                                                            const int64_t* gprefix, int ngroups, const RowDesc* rows,
                                                            uint32_t* ws) {
  extern __shared__ uint4 im_sm[];
  __shared__ int64_t sPts[IM_JOBS], sVal[IM_SEQ];
  __shared__ int32_t sN1[IM_SEQ], sBlk[IM_SEQ], sU[IM_SEQ];  // sequence 2 j + parity of job j
  __shared__ int32_t sRow[IM_MAXROWS + 16];  // sequence << 16 | block distance K; -1 past the last row
  __shared__ int32_t sPair[IM_JOBS + 1];     // pairs of points (whole blocks) before each job
  __shared__ int32_t nmark, mark[IM_MARKS];
  __shared__ uint32_t gen[IM_WAVES][2 * (MAXY_FAST + 1)];
  uint8_t* sm = reinterpret_cast<uint8_t*>(im_sm);
  const int g = find_job(gprefix, ngroups, blockIdx.x);
  const int pi = (int)(blockIdx.x - gprefix[g]);
  const int s0 = gstart[g], nj = gstart[g + 1] - s0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const PrimeC c = primes[pi];
  const int ns = 2 * nj;
  if (tid < ns) {
    const ResJob& J = jobs[job_list[s0 + (tid >> 1)]];
    const bool on = J.k > pi;  // jobs of the group with fewer primes sit this one out
    const int odd = tid & 1;
    const int n = !on ? 0 : odd ? (J.D + 1) / 2 : J.D / 2 + 1;
    sN1[tid] = n;
    sBlk[tid] = (n + 63) / 64;
    sVal[tid] = J.val_off + (int64_t)pi * (J.D + 1) + odd;
    if (!odd) sPts[tid >> 1] = J.pts_off + (int64_t)pi * npts_of(J.D);
  }
  for (int r = tid; r < IM_MAXROWS + 16; r += IM_THREADS) sRow[r] = -1;
  if (tid == 0) nmark = 0;
  __syncthreads();
  int nrows = 0, mxb = 0;
  for (int j = 0; j < ns; ++j) { nrows += sBlk[j]; mxb = max(mxb, sBlk[j]); }
  const int Dp = 64 * mxb, TP = im_tplane(Dp);
  const bool both = im_both(Dp);  // room for t in both orders
  const int zoff = (both ? 8 : 4) * TP, ubase = zoff + 16;
  // rows by K (the number of input blocks before the last one that an output
  // block reads) from the top, so that a tile's rows need about the same steps
  for (int x = tid; x < ns * mxb; x += IM_THREADS) {
    const int j = x / mxb, K = x % mxb;
    if (K >= sBlk[j]) continue;
    int pos = 0;
    for (int i = 0; i < ns; ++i) pos += max(0, sBlk[i] - (K + 1)) + (i < j && sBlk[i] > K ? 1 : 0);
    sRow[pos] = j << 16 | K;
  }
  if (tid < ns) {
    int off = ubase;
    for (int i = 0; i < tid; ++i) off += 512 * sBlk[i];
    sU[tid] = off;
  }
  if (tid < 4) reinterpret_cast<uint32_t*>(sm + zoff)[tid] = 0u;
  if (tid <= nj) {
    int off = 0;
    for (int i = 0; i < tid; ++i) off += 64 * sBlk[2 * i];
    sPair[tid] = off;
  }
  __syncthreads();
  const uint32_t* ip = g_iphi + (size_t)pi * IM_N;
  const uint32_t* iq = g_ipoints + (size_t)pi * POINT_ROW;  // q^-i = iq[32 + i / 32] iq[i mod 32]
  // The pairs of values of all jobs and their factors, IM_LOADS at a time per
  // thread; the first are requested before t is staged.
  uint2 vv[IM_LOADS];
  uint32_t vp[IM_LOADS], va[IM_LOADS], vb[IM_LOADS];
  int vj[IM_LOADS], vi[IM_LOADS];
  auto load_pairs = [&](int x0) {
    int j = 0;
#pragma unroll
    for (int u = 0; u < IM_LOADS; ++u) {
      const int x = x0 + u * IM_THREADS;
      vj[u] = -1;
      if (x < sPair[nj]) {
        while (x >= sPair[j + 1]) ++j;
        vj[u] = j;
        vi[u] = x - sPair[j];
        vv[u] = make_uint2(0u, 0u);
        if (vi[u] < sN1[2 * j]) vv[u] = *reinterpret_cast<const uint2*>(ws + sPts[j] + 2 * vi[u]);
        vp[u] = ip[min(vi[u], IM_N - 1)];
        va[u] = iq[32 + (vi[u] >> 5)];
        vb[u] = iq[vi[u] & 31];
      }
    }
  };
  load_pairs(tid);
  const uint32_t* ps = g_psi + (size_t)pi * IM_N;
  const int8_t* tq = g_tq + (size_t)pi * 4 * IM_TROW;
  // t reversed: the word at byte y holds t at Dp + 67 - y and the three below
  for (int y = 4 * tid; y < TP; y += 4 * IM_THREADS) {
    const int x0 = Dp + 64 - y;
    const bool in = x0 >= 0 && x0 < IM_TROW;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w = in ? *reinterpret_cast<const uint32_t*>(tq + (size_t)q * IM_TROW + x0) : 0u;
      *reinterpret_cast<uint32_t*>(sm + q * TP + y) = __builtin_amdgcn_perm(0u, w, 0x00010203u);
    }
  }
  // t ascending: the word at byte y holds t at y - 64 and the three above
  auto load_ascending = [&](int at) {
    for (int y = 4 * tid; y < TP; y += 4 * IM_THREADS) {
      const int x0 = y - 64;
      const bool in = x0 >= 0 && x0 < IM_TROW;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint32_t*>(sm + at + q * TP + y) =
            in ? *reinterpret_cast<const uint32_t*>(tq + (size_t)q * IM_TROW + x0) : 0u;
    }
  };
  if (both) load_ascending(4 * TP);
  __syncthreads();
  // u of both parities from the pairs of values.  Instances the evaluation
  // marked abnormal are computed here: a wavefront each while there are few (a
  // lane alone takes three to four times as long), else a lane each (a pair whose
  // remainders skip degrees at every point marks all of them).
  // p = 1 / phi_i, r = q^-i below 2p
  auto put_u = [&](int j, int i, uint32_t v0, uint32_t v1, uint32_t p, uint32_t r) {
    v0 = canon(v0, c.p);
    v1 = canon(v1, c.p);
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) {
      const int s = 2 * j + odd;
      if (i >= 64 * sBlk[s]) continue;
      uint32_t v = odd ? v0 + c.p - v1 : v0 + v1;  // < 2p
      if (odd) v = mmul(v, r, c.p, c.pinv);
      const uint32_t w = i < sN1[s] ? balance4(mmulc(v, p, c.p, c.pinv)) : 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) sm[sU[s] + q * 64 * sBlk[s] + i] = (uint8_t)(w >> (8 * q));
    }
  };
  auto each_pair = [&](auto&& f) {
    for (int x0 = tid; x0 < sPair[nj]; x0 += IM_LOADS * IM_THREADS) {
      if (x0 != tid) load_pairs(x0);
#pragma unroll
      for (int u = 0; u < IM_LOADS; ++u)
        if (vj[u] >= 0) f(vj[u], vi[u], vv[u].x, vv[u].y, vp[u], mmul(va[u], vb[u], c.p, c.pinv));
    }
  };
  each_pair([&](int j, int i, uint32_t v0, uint32_t v1, uint32_t p, uint32_t r) {
    if (__builtin_expect(v0 == ABN_MARK || v1 == ABN_MARK, 0)) {
      for (int e = 0; e < 2; ++e)
        if ((e ? v1 : v0) == ABN_MARK) {
          const int x = atomicAdd(&nmark, 1);
          if (x < IM_MARKS) mark[x] = j << 16 | (2 * i + e);
        }
    }
    put_u(j, i, v0, v1, p, r);
  });
  __syncthreads();
  if (__builtin_expect(nmark != 0, 0)) {
    // the group decides, not the first mark to arrive.  From y-degree 16 up to four rounds of wavefronts
    // (degree 40, 16 marks: 315 us a call against 348 of a lane each; 32: 554 against 374), below two (degree 8,
    // 8 marks: 71 against 88, a round of wavefronts 14)
    int mm = 0;
    for (int j = 0; j < nj; ++j) mm = max(mm, (int)jobs[job_list[s0 + j]].m);
    const int most = mm >= 16 ? IM_MARKS : 2 * IM_WAVES;
    if (nmark <= most) {
      for (int x = wave; x < nmark; x += IM_WAVES) {
        const int j = mark[x] >> 16, i = mark[x] & 0xffff;
        const uint32_t v = general_instance_wave(jobs + job_list[s0 + j], primes, rows, ws, g_points, pi, i,
                                                 gen[wave], gen[wave] + MAXY_FAST + 1, lane);
        if (lane == 0) ws[sPts[j] + i] = v;
      }
      __syncthreads();
      if (tid < nmark) {
        const int j = mark[tid] >> 16, i = (mark[tid] & 0xffff) >> 1;
        put_u(j, i, ws[sPts[j] + 2 * i], ws[sPts[j] + 2 * i + 1], ip[i],
              mmul(iq[32 + (i >> 5)], iq[i & 31], c.p, c.pinv));
      }
    } else {
      // pairs of lanes take the pairs of points of which at least one is marked
      for (int x = tid; x < 2 * sPair[nj]; x += IM_THREADS) {
        int j = 0;
        while (x >= 2 * sPair[j + 1]) ++j;
        const int i = x - 2 * sPair[j];
        uint32_t* V = ws + sPts[j];
        if (i >= 2 * sN1[2 * j]) continue;
        const uint32_t v = V[i];
        if (v == ABN_MARK || V[i ^ 1] == ABN_MARK) {
          const uint32_t w = general_instance<MAXY_FAST>(jobs + job_list[s0 + j], primes, rows, ws, g_points, pi, i);
          if (v == ABN_MARK) V[i] = w;
        }
      }
      __syncthreads();
      load_pairs(tid);
      each_pair([&](int j, int i, uint32_t v0, uint32_t v1, uint32_t p, uint32_t r) { put_u(j, i, v0, v1, p, r); });
    }
    __syncthreads();
  }
  const uint32_t k56 = fold_const(c);
  const int ntile = (nrows + 15) / 16;
  InterpLds S{sm, sRow, sN1, sBlk, sU, sVal, TP, Dp, zoff, 0};
  interp_stage<1>(S, ntile, wave, lane, ps, ws, k56, c);
  __syncthreads();
  if (!both) {
    load_ascending(0);
    __syncthreads();
  }
  S.t0 = both ? 4 * TP : 0;
  interp_stage<2>(S, ntile, wave, lane, ip, ws, k56, c);
}

int interp_mfma_blocks(int D) { return (D / 2 + 64) / 64 + ((D + 1) / 2 + 63) / 64; }

size_t interp_mfma_lds(int max_D, int blocks) {
  const int Dp = (max_D / 2 + 64) / 64 * 64;
  return (im_both(Dp) ? 8 : 4) * (size_t)im_tplane(Dp) + 16 + 512 * (size_t)blocks;
}

hipError_t configure_interp_mfma() {
  return hipFuncSetAttribute((const void*)k_interp_mfma, hipFuncAttributeMaxDynamicSharedMemorySize, 152 * 1024);
}

void launch_points_init(hipStream_t s) {
  hipLaunchKernelGGL(k_points_init, dim3(KMAX), dim3(64), 0, s, global_crt_tables().primes);
}

const uint32_t* points_table() {
  static const uint32_t* cache[64] = {nullptr};
  int dev = 0;
  (void)hipGetDevice(&dev);
  if (dev >= 0 && dev < 64 && cache[dev]) return cache[dev];
  void* p = nullptr;
  (void)hipGetSymbolAddress(&p, HIP_SYMBOL(g_points));
  if (dev >= 0 && dev < 64) cache[dev] = (const uint32_t*)p;
  return (const uint32_t*)p;
}

void launch_interp_mfma(const ResJob* jobs_d, const int32_t* job_list_d, const int32_t* gstart_d,
                        const int64_t* gprefix_d, int ngroups, int64_t nblocks, size_t lds, const RowDesc* rows_d,
                        uint32_t* ws, hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_interp_mfma, dim3((unsigned)nblocks), dim3(IM_THREADS), lds, s, global_crt_tables().primes,
                     jobs_d, job_list_d, gstart_d, gprefix_d, ngroups, rows_d, ws);
}

}  // namespace snc
