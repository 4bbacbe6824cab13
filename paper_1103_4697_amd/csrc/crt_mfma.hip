// Chinese remaindering with more than 64 primes on the matrix cores (Section
// 4, "Symbolic Speedups": combining the images over Z_p into integers).
//
// Both halves of the reconstruction are contractions with constant matrices
// shared by every coefficient, and residues below 2^30 are four signed bytes,
// so they run as int8 matrix products with exact int32 accumulators.
//
// Representation.  The primes are taken in blocks of 64.  With Q_s the
// product of the primes before block s, N_s the product of block s, every
// block but the last contributes sum_j z_j V_j, V_j = Q_s N_s / p_j (Lagrange
// form inside the block, no serial chain), and the last block, of 1..64
// primes, sum_j z_j P_j with Garner's mixed-radix digits.  z_j < p_j; a
// block's sum lies in [0, 64 Q_s N_s) instead of [0, Q_s N_s), which the next
// blocks absorb, so the total X' is the least residue X mod M or X + M
// (M the product of all k primes): the last block's digit block has at least
// one prime p > 2^29, hence 0 <= X' < M (1 + 2^-22).
//
//   digits   z_i = (r_i - S_i) c_i mod p_i, S_i = sum_j z_j (V_j mod p_i)
//            over the earlier blocks, c_i = V_i^-1 mod p_i: matrix products
//            of the z bytes (LDS) with a resident table of the bytes of
//            V_j mod p_i in operand order (read once, straight to registers).
//   product  limb sums of X' = sum_j z_j V_j: matrix product of the z bytes
//            with the bytes of V_j, the four bytes of a z_j and of each
//            window of V_j side by side on the contraction index.
//   carry    64-bit limb sums to limbs, and the balanced value.
//
// Bounds and figures (MI355X; 15 resultants of degree-15 curves with
// 2048-bit coefficients: 2052 primes, 3,300 coefficients of 1,923 limbs, about
// 1.1e11 byte products in each half).  The lanes-over-primes kernels issued a
// 64-bit multiply-add per (digit, prime) and per (digit, limb) and were bound
// by them: digits 2610 us, binary value 3113 us.  Here: digits 171 us, a chain
// of 33 blocks with a barrier pair each in 220 workgroups, fewer than CUs
// (counters: matrix cores busy 28%, vector unit 23% of its issue slots, LDS
// 9%); product 354 us (0.3 P byte products/s), a barrier and a round trip to
// L2 for every 16 primes with four workgroups a CU (matrix cores 15%, LDS 19%,
// vector unit 18%, 2.7 TB/s of HBM); carry 42 us, the 51 MB of limb sums, of
// which a workgroup reads 64 bytes of each line (143 MB fetched, 3.4 TB/s).
// With 412 primes (degree 12, 512 bits): 150 + 204 us before, 24 + 34 + 11 us
// now; with 262 primes and 3,073 coefficients: 99 + 134 us before, 15 + 19 + 9
// us now; with 79 primes: 17 + 24 us before, 8 + 8 + 8 us now.  Up to 64 primes there is no earlier block to contract with
// and the lanes-over-primes pair serves (33..64 primes here: 26 us a call
// against 21).  In a large batch with 65..128 primes (30,000 coefficients): 48
// + 27 + 24 us against 158 of one lane per coefficient.
#include <hip/hip_runtime.h>

#include "eval_elim.hpp"
#include "mfma_modp.hpp"

namespace snc {

constexpr int CM_NB = KMAX / 64;   // blocks of primes in the table
static_assert(KMAX % 64 == 0, "whole blocks");
constexpr int CM_WAVES = 8;        // wavefronts of a digits workgroup: 4 column tiles x 2 halves of the contraction
constexpr int CM_THREADS = 64 * CM_WAVES;

// bytes of V_j mod p_i (Montgomery form, balanced), matrix operand order:
// [block of i][16 columns of it][block of j, below i's][byte][lane][16 rows]
__host__ __device__ constexpr int cm_tile(int ib, int it, int jb) { return 2 * ib * (ib - 1) + it * ib + jb; }
__device__ __align__(16) int8_t g_vfrag[(size_t)cm_tile(CM_NB, 0, 0) * 4 * 64 * 16];
__device__ uint32_t g_vinv[KMAX];                       // Montgomery form of V_i^-1 mod p_i
// Balanced bytes (each word four signed bytes, sum b_s 256^s) of V_j and P_j:
// both are below 2^(1920 (s + 1) - 29) for j in block s, so 60 (s + 1) words
// hold them, the top one without a carry out.
__host__ __device__ constexpr int cm_words(int s) { return 60 * (s + 1); }
__host__ __device__ constexpr int64_t cm_row(int j) {
  const int64_t s = j >> 6;
  return 64 * 30 * s * (s + 1) + (int64_t)(j & 63) * cm_words((int)s);
}
static_assert(cm_words(CM_NB - 1) <= LPS, "the rows of the product table are as long");
__device__ uint32_t g_vbal[(size_t)cm_row(KMAX)];
__device__ uint32_t g_pbal[(size_t)cm_row(KMAX)];

__global__ __launch_bounds__(64) void k_crtm_vinv(CrtTables tb) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  const PrimeC c = tb.primes[i];
  uint32_t v = c.r1;
  for (int l = 0; l < 64 * (i / 64 + 1); ++l)
    if (l != i) v = mmulc(v, to_mont(tb.primes[l].p, c), c.p, c.pinv);
  g_vinv[i] = minv(v, c);
}

// one lane's 16 rows of the four byte planes; V_j = P_{64 (s + 1)} / p_j
__global__ __launch_bounds__(64) void k_crtm_frag(CrtTables tb) {
  const int tile = blockIdx.x, lane = threadIdx.x;
  const int jb = tile % CM_NB, it = tile / CM_NB % 4, ib = tile / (4 * CM_NB);
  if (jb >= ib) return;
  const int i = 64 * ib + 16 * it + (lane & 15);
  const PrimeC c = tb.primes[i];
  const int top = 64 * (jb + 1);
  const uint32_t P = top < i ? tb.wtab[(size_t)top * tb.wstride + i] : minv(tb.garner[i], c);
  int8_t* out = g_vfrag + (size_t)cm_tile(ib, it, jb) * 4096 + lane * 16;
  for (int e = 0; e < 16; ++e) {
    const int j = 64 * jb + 16 * (lane >> 4) + e;
    const uint32_t inv = minv(to_mont(tb.primes[j].p, c), c);
    const uint32_t w = balance4(mmulc(P, inv, c.p, c.pinv));
    for (int b = 0; b < 4; ++b) out[b * 1024 + e] = (int8_t)(w >> (8 * b));
  }
}

// exact quotient V_j = P_{64 (s + 1)} / p_j limb by limb (the quotient's limb
// is the running limb times p^-1 mod 2^32), and P_j, both in balanced bytes
__global__ __launch_bounds__(64) void k_crtm_balance(CrtTables tb) {
  const int j = blockIdx.x * 64 + threadIdx.x;
  const uint32_t p = tb.primes[j].p, inv = 0u - tb.primes[j].pinv;
  const uint32_t* A = tb.ptab + (size_t)(64 * (j / 64 + 1)) * tb.pstride;
  const uint32_t* B = tb.ptab + (size_t)j * tb.pstride;
  uint32_t* V = g_vbal + cm_row(j);
  uint32_t* P = g_pbal + cm_row(j);
  uint32_t borrow = 0, cv = 0, cp = 0;
  for (int l = 0; l < cm_words(j / 64); ++l) {
    const uint32_t a = A[l];
    const uint32_t q = (a - borrow) * inv;
    borrow = __umulhi(q, p) + (a < borrow ? 1u : 0u);
    const uint64_t yv = (uint64_t)q + 0x80808080u + cv;
    V[l] = (uint32_t)yv ^ 0x80808080u;
    cv = (uint32_t)(yv >> 32);
    const uint64_t yp = (uint64_t)B[l] + 0x80808080u + cp;
    P[l] = (uint32_t)yp ^ 0x80808080u;
    cp = (uint32_t)(yp >> 32);
  }
}

// ---------------------------------------------------------------------------
// Digits.  A workgroup takes ROWS coefficients of one job through the blocks
// of primes in order; wavefront w works on the 16 columns w mod 4 of a block
// and on half of the earlier blocks' contraction.
// ---------------------------------------------------------------------------

template <int ROWS>
__global__ __launch_bounds__(CM_THREADS) void k_crtm_digits(CrtTables tb, const ResJob* jobs, const int32_t* job_list,
                                                            const int64_t* prefix, int njobs, uint32_t* ws) {
  extern __shared__ uint4 cm_sm[];
  __shared__ uint32_t wt[64 * 64];       // the last block's W = P_j mod p_i, [j][i]
  __shared__ uint32_t Sp[2][ROWS][64];   // the two halves' sums S
  int8_t* Z = reinterpret_cast<int8_t*>(cm_sm);  // z bytes [block][byte][16 digits of it][row][16]
  const int64_t bb = blockIdx.x;
  const int64_t b = ROWS == 16 ? bb : bb >> 1;   // the prefix counts groups of 16 coefficients
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[job_list[jj]];
  const int k = J.k, n1 = J.D + 1, nf = (k - 1) >> 6;
  const int t0 = (int)(b - prefix[jj]) * 16 + (ROWS == 16 ? 0 : 8 * (int)(bb & 1));
  if (t0 >= n1) return;  // the second half of a group of 16 may be empty (whole workgroup)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int it = wave & 3, half = wave >> 2;
  const int col = 16 * it + (lane & 15);
  const int row0 = 4 * (lane >> 4);
  const uint32_t* V = ws + J.val_off;
  uint32_t* dig = ws + J.dig_off;
  // the last block's table and residues of the primes past k are never used
  for (int x = threadIdx.x; x < 64 * 64; x += CM_THREADS) {
    const int j = 64 * nf + (x >> 6), i = 64 * nf + (x & 63);
    wt[x] = (j < k && i < k) ? tb.wtab[(size_t)j * tb.wstride + i] : 0u;
  }
  for (int s = 0; s <= nf; ++s) {
    const int i = 64 * s + col;
    const int ic = i < k ? i : k - 1;
    const PrimeC c = tb.primes[ic];
    uint32_t rv[4] = {0u, 0u, 0u, 0u};
    const bool owner = half == 0 && s < nf && row0 < ROWS;
    if (owner) {
#pragma unroll
      for (int r = 0; r < 4; ++r) rv[r] = V[(size_t)i * n1 + min(t0 + row0 + r, n1 - 1)];
    }
    v4i acc[7];
#pragma unroll
    for (int d = 0; d < 7; ++d) acc[d] = v4i{0, 0, 0, 0};
    const v4i* F = reinterpret_cast<const v4i*>(g_vfrag) + (size_t)cm_tile(s, it, 0) * 256 + lane;
    const v4i* Zr = reinterpret_cast<const v4i*>(Z) + (lane >> 4) * ROWS + (lane & (ROWS - 1));
#pragma unroll 2
    for (int jb = half; jb < s; jb += 2) {
      v4i bv[4], av[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) bv[q] = F[(size_t)jb * 256 + q * 64];
#pragma unroll
      for (int q = 0; q < 4; ++q) av[q] = Zr[(jb * 4 + q) * 4 * ROWS];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          acc[x + y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[x], bv[y], acc[x + y], 0, 0, 0);
    }
    const uint32_t k56 = fold_const(c);
    uint32_t S[4];
    if (row0 < ROWS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) S[r] = fold_bytes(acc[0][r], acc[1][r], acc[2][r], acc[3][r], acc[4][r], acc[5][r], acc[6][r], k56, c);
      if (half == 1 || s == nf) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Sp[half][row0 + r][col] = S[r];
      }
    }
    __syncthreads();
    if (owner) {
      const uint32_t vi = g_vinv[i];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t St = madd(S[r], Sp[1][row0 + r][col], c.p);
        const uint32_t z = canon2(redc((uint64_t)msub(rv[r], St, c.p) * vi, c.p, c.pinv), c.p);
        const uint32_t w = balance4(z);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          Z[(((s * 4 + q) * 4 + it) * ROWS + row0 + r) * 16 + (lane & 15)] = (int8_t)(w >> (8 * q));
        if (t0 + row0 + r < n1) dig[(size_t)(t0 + row0 + r) * k + i] = w;
      }
    }
    __syncthreads();
  }
  // the last block: Garner's digits one after another, lanes over its primes,
  // ROWS / CM_WAVES coefficients per wavefront side by side
  constexpr int RPW = ROWS / CM_WAVES;
  const int i = 64 * nf + lane;
  const int nq = k - 64 * nf;
  const PrimeC c = tb.primes[i < k ? i : k - 1];
  const uint32_t g = tb.garner[i < k ? i : k - 1];
  uint32_t R[RPW], S[RPW], y[RPW];
#pragma unroll
  for (int u = 0; u < RPW; ++u) {
    const int row = wave * RPW + u;
    R[u] = i < k ? V[(size_t)i * n1 + min(t0 + row, n1 - 1)] : 0u;
    S[u] = madd(Sp[0][row][lane], Sp[1][row][lane], c.p);
    y[u] = 0;
  }
  for (int q = 0; q < nq; ++q) {
    const uint32_t w = wt[q * 64 + lane];
#pragma unroll
    for (int u = 0; u < RPW; ++u) {
      const uint32_t cand = canon2(redc((uint64_t)msub(R[u], S[u], c.p) * g, c.p, c.pinv), c.p);
      const uint32_t yq = __builtin_amdgcn_readlane(cand, q);
      y[u] = lane == q ? cand : y[u];
      // lanes up to q hold finished digits: their S is not read again
      S[u] = madd(S[u], canon2(redc((uint64_t)yq * w, c.p, c.pinv), c.p), c.p);
    }
  }
#pragma unroll
  for (int u = 0; u < RPW; ++u) {
    const int t = t0 + wave * RPW + u;
    if (i < k && t < n1) dig[(size_t)t * k + i] = balance4(y[u]);
  }
}

// ---------------------------------------------------------------------------
// Product.  Limb sums of X' for 64 limbs x 64 coefficients of a job.  The
// contraction index runs over (prime, byte of z): row (limb q, byte r) of the
// first operand holds, for prime j, the window of bytes 4q + r, .., 4q + r - 3
// of V_j, built from two words by a byte permutation on the way into LDS.
// Tile r of a wavefront is byte r of 32 limbs, so a lane ends with the four
// byte sums of its limbs in its own registers.
// ---------------------------------------------------------------------------
constexpr int CP_L = 64, CP_T = 64;  // limbs and coefficients of a workgroup
constexpr int CP_J = 16;             // primes per step (64 bytes of the contraction)

__device__ __forceinline__ uint4 load_words4(const uint32_t* p) {  // 4-byte aligned
  uint4 v;
  __builtin_memcpy(&v, p, sizeof v);
  return v;
}

__global__ __launch_bounds__(256) void k_crtm_product(const ResJob* jobs, const int32_t* job_list,
                                                      const int64_t* prefix, int njobs, uint32_t* ws) {
  __shared__ uint4 As[2][4][4 * CP_L];  // [16-byte group][byte r][limb]
  __shared__ uint4 Bs[2][4][CP_T];      // [16-byte group][coefficient]
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b);
  const ResJob J = jobs[job_list[jj]];
  const int k = J.k, n1 = J.D + 1, nf = (k - 1) >> 6, lx = lx_of(k);
  const int nlt = (lx + CP_L - 1) / CP_L;
  const int lb = (int)(b - prefix[jj]);
  const int l0 = (nlt - 1 - lb % nlt) * CP_L, t0 = lb / nlt * CP_T;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t* dig = ws + J.dig_off;
  // block s has fewer than 60 (s + 1) limbs (and one more balanced byte): the
  // earlier ones do not reach limb l0
  int s0 = (l0 - 2) / 60 - 1;
  s0 = s0 < 0 ? 0 : s0 > nf ? nf : s0;
  // staging: thread = (16-byte group g, limb q) of the first operand, and
  // (g, coefficient q) of the second
  const int g = tid >> 6, q = tid & 63;
  const int wq = l0 + q;
  const bool tok = t0 + q < n1;
  const uint32_t* dg = dig + (size_t)(tok ? t0 + q : 0) * k;
  uint32_t cur[4], prv[4];
  uint4 zw;
  auto fetch = [&](int j0) {
    const int j = j0 + 4 * g;
    const int s = j0 >> 6, words = cm_words(s);  // a step's primes are of one block
    const uint32_t* row = (s < nf ? g_vbal : g_pbal) + cm_row(64 * s) + (size_t)(j - 64 * s) * words;
    const bool lok = wq < words, lokp = wq > 0 && wq <= words;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool jok = j + e < k;
      cur[e] = jok && lok ? row[e * words + wq] : 0u;
      prv[e] = jok && lokp ? row[e * words + wq - 1] : 0u;
    }
    if (j + 4 <= k) {
      zw = load_words4(dg + j);
    } else {
      zw.x = j < k ? dg[j] : 0u;
      zw.y = j + 1 < k ? dg[j + 1] : 0u;
      zw.z = j + 2 < k ? dg[j + 2] : 0u;
      zw.w = 0u;
    }
    if (!tok) zw = make_uint4(0u, 0u, 0u, 0u);
  };
  v16i acc[4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[r][e] = 0;
  const int lw = 32 * (wave & 1), tw = 32 * (wave >> 1);
  fetch(64 * s0);
  int buf = 0;
  for (int j0 = 64 * s0; j0 < k; j0 += CP_J, buf ^= 1) {
    constexpr uint32_t sel0 = 0x01020304u;  // bytes 4 + r, 3 + r, 2 + r, 1 + r of (prv, cur)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t sel = sel0 + 0x01010101u * r;
      As[buf][g][r * CP_L + q] =
          make_uint4(__builtin_amdgcn_perm(cur[0], prv[0], sel), __builtin_amdgcn_perm(cur[1], prv[1], sel),
                     __builtin_amdgcn_perm(cur[2], prv[2], sel), __builtin_amdgcn_perm(cur[3], prv[3], sel));
    }
    Bs[buf][g][q] = zw;
    __syncthreads();
    if (j0 + CP_J < k) fetch(j0 + CP_J);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int gg = 2 * h + (lane >> 5);
      const v4i bv = *reinterpret_cast<const v4i*>(&Bs[buf][gg][tw + (lane & 31)]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const v4i av = *reinterpret_cast<const v4i*>(&As[buf][gg][r * CP_L + lw + (lane & 31)]);
        acc[r] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, acc[r], 0, 0, 0);
      }
    }
    // the other buffer is written next; its readers passed this step's barrier
  }
  const int t = t0 + tw + (lane & 31);
  if (t >= n1) return;
  int64_t* part = reinterpret_cast<int64_t*>(ws + J.pts_off);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int l = l0 + lw + (e & 3) + 8 * (e >> 2) + 4 * (lane >> 5);
    const int64_t v = (int64_t)acc[0][e] + (int64_t)acc[1][e] * 256 + (int64_t)acc[2][e] * 65536 +
                      (int64_t)acc[3][e] * 16777216;
    if (l < lx) part[(size_t)l * n1 + t] = v;
  }
}

// ---------------------------------------------------------------------------
// Carry.  Eight coefficients per workgroup, a thread per 32 limbs.  A
// segment's carry-out goes to the next segment until none is left (after the
// first round a carry is -1, 0 or 1 and almost always stops at once).  The
// balanced value is X' - M when X' > (M - 1) / 2 = M >> 1.
// ---------------------------------------------------------------------------
constexpr int CC_T = 8, CC_S = 32;
constexpr int CC_MAXSEG = ((30 * KMAX + 31) / 32 + 2 + CC_S - 1) / CC_S;
static_assert(CC_T * ((CC_MAXSEG + 7) / 8 * 8) <= 1024, "a workgroup holds every segment");

__global__ __launch_bounds__(1024) void k_crtm_carry(CrtTables tb, const ResJob* jobs, const int32_t* job_list,
                                                     const int64_t* prefix, int njobs, uint32_t* ws) {
  __shared__ int32_t cr[CC_MAXSEG + 8][CC_T];
  const int64_t b = blockIdx.x;
  const int jj = find_job(prefix, njobs, b >> 1);  // the prefix counts groups of 16 coefficients
  const ResJob J = jobs[job_list[jj]];
  const int k = J.k, n1 = J.D + 1, lx = lx_of(k);
  const int t0 = (int)((b >> 1) - prefix[jj]) * 16 + CC_T * (int)(b & 1);
  if (t0 >= n1) return;  // uniform
  const int tl = threadIdx.x & (CC_T - 1), seg = threadIdx.x / CC_T;
  const int t = t0 + tl, nseg = (lx + CC_S - 1) / CC_S;
  const bool on = seg < nseg && t < n1;
  const int64_t* part = reinterpret_cast<const int64_t*>(ws + J.pts_off);
  uint32_t v[CC_S];
  int64_t c = 0;
#pragma unroll
  for (int e = 0; e < CC_S; ++e) {
    const int l = seg * CC_S + e;
    const int64_t x = (on && l < lx ? part[(size_t)l * n1 + t] : 0) + c;
    v[e] = (uint32_t)x;
    c = x >> 32;
  }
  // carries between segments, until every one is absorbed
  auto settle = [&]() {
    for (;;) {
      if (seg < nseg) cr[seg][tl] = (int32_t)c;
      __syncthreads();
      const int32_t in = seg > 0 && seg < nseg ? cr[seg - 1][tl] : 0;
      c = in;
      if (in != 0) {
#pragma unroll
        for (int e = 0; e < CC_S; ++e) {
          const int64_t x = (int64_t)v[e] + c;
          v[e] = (uint32_t)x;
          c = x >> 32;
        }
      }
      if (!__syncthreads_or(c != 0)) break;
    }
  };
  settle();
  const uint32_t* M = tb.ptab + (size_t)k * tb.pstride;
  uint32_t m[CC_S + 1];
#pragma unroll
  for (int e = 0; e <= CC_S; ++e) {
    const int l = seg * CC_S + e;
    m[e] = seg < nseg && l < LPS ? M[l] : 0u;
  }
  int cmp = 0;
#pragma unroll
  for (int e = CC_S - 1; e >= 0; --e) {
    const uint32_t h = (m[e] >> 1) | (m[e + 1] << 31);
    if (cmp == 0 && v[e] != h) cmp = v[e] > h ? 1 : -1;
  }
  if (seg < nseg) cr[seg][tl] = cmp;
  __syncthreads();
  int top = 0;
  for (int s = nseg - 1; s >= 0 && top == 0; --s) top = cr[s][tl];
  __syncthreads();
  c = 0;
  if (top > 0) {
#pragma unroll
    for (int e = 0; e < CC_S; ++e) {
      const int64_t x = (int64_t)v[e] - (int64_t)m[e] + c;
      v[e] = (uint32_t)x;
      c = x >> 32;
    }
  }
  settle();
  if (!on) return;
  uint32_t* out = ws + J.out_off + (size_t)t * J.L + seg * CC_S;
  const int nl = J.L - seg * CC_S;
#pragma unroll
  for (int e = 0; e < CC_S; e += 4) {
    if (e + 4 <= nl) {
      const uint4 w = make_uint4(v[e], v[e + 1], v[e + 2], v[e + 3]);
      __builtin_memcpy(out + e, &w, sizeof w);
    } else {
#pragma unroll
      for (int f = 0; f < 4; ++f)
        if (e + f < nl) out[e + f] = v[e + f];
    }
  }
}

// rows of a digits workgroup: 16 (a whole operand tile) while their z bytes
// fit the LDS beside the static arrays, else 8
constexpr size_t CM_LDS = (size_t)34 * 4096;
static_assert(CM_LDS + 64 * 64 * 4 + 2 * 16 * 64 * 4 <= 160 * 1024, "a digits workgroup fits the LDS of a CU");
static_assert((size_t)(CM_NB - 1) * 2048 <= CM_LDS, "eight rows fit for the whole table");

hipError_t configure_crt_mfma() {
  hipError_t e = hipFuncSetAttribute((const void*)k_crtm_digits<16>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CM_LDS);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_crtm_digits<8>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CM_LDS);
}

void launch_crt_mfma_init(const CrtTables& tb, hipStream_t s) {
  hipLaunchKernelGGL(k_crtm_vinv, dim3(CM_NB), dim3(64), 0, s, tb);
  hipLaunchKernelGGL(k_crtm_frag, dim3(CM_NB * 4 * CM_NB), dim3(64), 0, s, tb);
  hipLaunchKernelGGL(k_crtm_balance, dim3(CM_NB), dim3(64), 0, s, tb);
}

void launch_crt_mfma_digits(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d,
                            const int64_t* prefix_d, int njobs, int64_t ngroups, int kmax, uint32_t* ws,
                            hipStream_t s) {
  if (ngroups <= 0) return;
  const int nf = (kmax - 1) / 64;
  if ((size_t)nf * 4096 <= CM_LDS)
    hipLaunchKernelGGL(k_crtm_digits<16>, dim3((unsigned)ngroups), dim3(CM_THREADS), (size_t)nf * 4096, s, tb, jobs_d,
                       job_list_d, prefix_d, njobs, ws);
  else
    hipLaunchKernelGGL(k_crtm_digits<8>, dim3((unsigned)(2 * ngroups)), dim3(CM_THREADS), (size_t)nf * 2048, s, tb,
                       jobs_d, job_list_d, prefix_d, njobs, ws);
}

void launch_crt_mfma_product(const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d, int njobs,
                             int64_t ntiles, uint32_t* ws, hipStream_t s) {
  if (ntiles <= 0) return;
  hipLaunchKernelGGL(k_crtm_product, dim3((unsigned)ntiles), dim3(256), 0, s, jobs_d, job_list_d, prefix_d, njobs, ws);
}

void launch_crt_mfma_carry(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d,
                           const int64_t* prefix_d, int njobs, int64_t ngroups, int kmax, uint32_t* ws,
                           hipStream_t s) {
  if (ngroups <= 0) return;
  const int nseg = (lx_of(kmax) + CC_S - 1) / CC_S;
  hipLaunchKernelGGL(k_crtm_carry, dim3((unsigned)(2 * ngroups)), dim3((unsigned)(CC_T * ((nseg + 7) / 8 * 8))), 0, s,
                     tb, jobs_d, job_list_d, prefix_d, njobs, ws);
}

int64_t crt_mfma_groups(int n1) { return (n1 + 15) / 16; }
int64_t crt_mfma_tiles(int n1, int k) {
  return (int64_t)((lx_of(k) + CP_L - 1) / CP_L) * ((n1 + CP_T - 1) / CP_T);
}

}  // namespace snc
