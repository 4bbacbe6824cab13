// Internal declarations shared by the host runtime and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "modp.hpp"

namespace snc {

constexpr int KMAX = 3072;        // primes in the modulus table (log2 of their product ~ 92100)
constexpr int LPS = 2884;         // limb stride of the prime-product table (30*3072/32 + 4)
constexpr int MAXY_FAST = 64;     // largest y-degree handled by the register-resident elimination
constexpr int MAXY_GEN = 255;     // largest y-degree handled at all
constexpr int EE_WAVES = 1;       // wavefronts per eval_elim workgroup
constexpr int EE_BLOCK = 64 * EE_WAVES;
constexpr int INTERP_THREADS = 1024;
constexpr int MAX_D = 10000;     // largest degree bound: the interpolations keep a prime's values and tables in LDS
constexpr int CRT_COEF_PER_BLOCK = 4;   // one wavefront per coefficient (digits)
constexpr int CRT_COMB_PER_BLOCK = 2;   // coefficients per combination workgroup (four wavefronts over limbs)
constexpr int GCD_THREADS = 256;

// One resultant res_y(f, g).  A is the operand of larger y-degree (m >= n);
// rows of A and B are listed top-down (row m of A first) so that the
// register arrays of the elimination are "top-aligned".
struct ResJob {
  int32_t m, n;        // y-degrees of A and B over Z[x], m >= 1, m >= n >= 0
  int32_t sign;        // 1: operands were swapped and m*n is odd (result negated)
  int32_t D;           // degree bound
  int32_t k;           // primes 0..k-1 of the table
  int32_t T;           // residues per prime (coefficients of f and g)
  int32_t L;           // output limbs per coefficient
  int32_t nl;          // limbs per input coefficient
  int32_t rows_off;    // first RowDesc of A (rstride groups), then those of B
  int32_t rstride;     // row groups per operand: ceil((width + 1) / 4), width = register class or m
  int64_t coef_off;    // input limbs, limb-major [nl][T] (uint32 index)
  int64_t res_off;     // residues [k][T] (uint32 index)
  int64_t val_off;     // coefficients mod p: [k][D+1]
  int64_t pts_off;     // values at the points: [k][npts_of(D)] (bivariate gcd: [k][D+1])
  int64_t nq_off;      // right behind them, [k][64 ceil((D+1)/64)]: Newton blocks of the bivariate gcd's interpolation;
                       // of resultants the rest of the limb sums that start at pts_off (crt_mfma.hip)
  int64_t dig_off;     // mixed-radix digits [D+1][k]
  int64_t out_off;     // output limbs [D+1][L]
};

// Rows of an operand are stored top-down (row of y^deg first) in groups of
// four: group g holds rows 4g..4g+3, zero-padded to the longest of the four.
// The evaluation takes even and odd powers of x apart (points come in pairs
// +-x), so a group is a sequence of 64-byte chunks, four powers of one parity
// by four rows: the coefficient of x^c of row 4g + q is residue
// off + grp_pos(c, len) + q.
struct RowDesc {
  int32_t off;  // first residue of the group within a prime's block of T
  int32_t len;  // coefficients per row of the group (0 for an all-zero group)
};
// Workgroups are dealt to the 8 XCDs (each with its own L2) round-robin by
// block index.  Renumbering so that XCD x runs a contiguous range of logical
// blocks keeps neighbouring work, which reads the same data (the residues of
// one prime, adjacent coefficients), in one L2.  A bijection on [0, nb).
constexpr int NXCD = 8;
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
  const int64_t q = nb / NXCD, r = nb % NXCD, x = b % NXCD;
  return x * q + (x < r ? x : r) + b / NXCD;
}

constexpr int ROWGRP = 4;
constexpr int HCHUNK = 4;   // powers of one parity per chunk; group lengths are padded to a multiple
__host__ __device__ inline int padded_group_len(int ml) { return (ml + HCHUNK - 1) / HCHUNK * HCHUNK; }
// position of x^c in a group of length len: pairs of chunks (even, odd powers)
// of eight, and for the top four of a length that is 4 mod 8 one chunk with
// two even powers and two odd ones
__host__ __device__ inline int grp_pos(int c, int len) {
  if (c >= (len & ~7)) return 4 * (len & ~7) + 8 * (c & 1) + 4 * ((c >> 1) & 1);
  return 16 * (2 * (c >> 3) + (c & 1)) + 4 * ((c >> 1) & 3);
}
// evaluation points: pairs +-q^i, i = 0..D/2 (one point more than needed when D is even)
__host__ __device__ inline int npts_of(int D) { return 2 * (D / 2 + 1); }

// Constant tables of a Chinese-remainder reconstruction over primes
// q_0..q_{k-1}: garner[i] = Montgomery form of (Q_i mod q_i)^-1 and
// wtab[j*wstride + i] = Montgomery form of Q_j mod q_i with Q_j = prod_{l<j} q_l;
// ptab row j (pstride limbs) = Q_j.
struct CrtTables {
  const PrimeC* primes;
  const uint32_t* garner;
  const uint32_t* wtab;
  const uint32_t* ptab;
  int32_t wstride, pstride;
};

// One gcd problem in Z[x]: a and b of degrees da, db >= 1; its primes are
// "slots" (table index per slot), filled in rounds of nslots starting at slot0.
struct GcdDesc {
  int32_t da, db;          // degrees of a and b
  int32_t nl;              // limbs per input coefficient
  int32_t wl;              // row length of w: min(da, db) + 1
  int32_t deriv;           // 1: b = a' (only a's limbs are stored; b's residues are formed from them)
  int32_t fused;           // 1: a's residues are given (plain, vals[slot * vstride + i]), b = a'; only
                           //    e and the degree of a mod p are written
  const uint32_t* vals;    // fused: residues of a, coefficient i of slot s at vals[s * vstride + i]
  int64_t vstride;
  int64_t d_off;           // fused: int32 per slot, degree of a mod p
  int64_t coef_off;        // input limbs [(da+1)+(db+1)][nl], or [da+1][nl] when deriv (uint32 index)
  int64_t slot_prime_off;  // int32 per slot: index of its prime in the modulus table
  int64_t res_off;         // residues [slot][da+db+2] (Montgomery)
  int64_t e_off;           // int32 per slot: degree of the gcd mod p, -2 if p divides both leading coefficients
  int64_t w_off;           // [slot][wl]   monic gcd mod p (plain)
  int64_t u_off;           // [slot][da+1] a / monic gcd mod p (plain)
  int64_t v_off;           // [slot][db+1] b / monic gcd mod p (plain)
  int32_t* ed_out;         // fused: if set, e and d are written at ed_out + e_off / d_off (host-mapped)
};

// gcd degree written for a prime dividing both leading coefficients (the prime is not used)
constexpr int32_t GCD_SLOT_UNUSABLE = -2;

// value left at an abnormal instance's point for the interpolation, which
// computes it by the general elimination (no residue is >= 2^30)
constexpr uint32_t ABN_MARK = 0xffffffffu;

__host__ __device__ constexpr int lx_of(int k) { return (30 * k + 31) / 32 + 2; }

// launchers (kernels_res.hip)
void upload_tables(const PrimeC* primes, const uint32_t* garner_c, const uint32_t* wtab,
                   const uint32_t* ptab, hipStream_t s);
hipError_t configure_kernels();
// Interpolation at the points 0..D of the bivariate gcd (interp_int.hip).
size_t interp_lds_bytes(int max_D);
// block-parallel: one workgroup per (resultant, prime, block of 64 coefficients),
// for degree bounds below 64 IFF_J and the first IFF_K primes (falling-factorial table)
constexpr int IFF_J = 16;
constexpr int IFF_K = 256;
inline bool interp_blk_fits(int max_D, int max_k) { return max_D + 1 <= 64 * IFF_J && max_k <= IFF_K; }
void launch_interp_blk(const ResJob* jobs_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks, uint32_t* ws,
                       hipStream_t s);
void launch_zero_u32(uint32_t* p, int64_t n, hipStream_t s);
// Evaluation points of the resultants: x_2i = q^i, x_2i+1 = -q^i mod p, q =
// q(p) with q^2 of order above MAX_D / 2.  Row p of the table: q^l for l < 32,
// then q^(32 b) at 32 + b.
constexpr int POINT_ROW = 256;
static_assert(32 + MAX_D / 64 < POINT_ROW, "a row holds the block powers of the largest degree bound");
__device__ __forceinline__ uint32_t point_mont(const uint32_t* points, int pi, int j, const PrimeC& c) {
  const uint32_t* r = points + (int64_t)pi * POINT_ROW;
  const int i = j >> 1;
  const uint32_t t = canon2(mmul(r[32 + (i >> 5)], r[i & 31], c.p, c.pinv), c.p);
  return j & 1 ? c.p - t : t;  // a power is never zero
}
// Powers of 2^32 for the reduction of multi-limb inputs, a row per prime:
// entry l <= 64 = 2^(32 l) 2^64 mod p, entry POW32_STEP = Montgomery form of 2^2048
constexpr int POW32_ROW = 68, POW32_STEP = 65;
const uint32_t* pow32_table();           // of the current device
void launch_pow32_init(hipStream_t s);   // once per device
// residues: workgroups of 64 coefficients for RED_PRIMES primes
constexpr int RED_PRIMES = 8;
inline int64_t reduce_blocks(int k, int T) {
  return (int64_t)((k + RED_PRIMES - 1) / RED_PRIMES) * ((T + 63) / 64);
}
void launch_points_init(hipStream_t s);  // points and interpolation tables (once per device)
const uint32_t* points_table();          // of the current device
// Interpolation at those points: a workgroup per prime of a group of jobs
// (job_list_d[gstart_d[g]] .. of group g, prefix: the largest prime count of
// each group).  lds: the largest group's interp_mfma_lds.
constexpr int IM_JOBS = 16;                    // jobs of a group
constexpr size_t IM_LDS = 48 * 1024;           // LDS a group of more than one job may take
constexpr int64_t IM_MIN_BLOCKS = 1024;        // workgroups wanted before jobs share one
size_t interp_mfma_lds(int max_D, int blocks); // largest degree bound, interp_mfma_blocks of all jobs
int interp_mfma_blocks(int D);                 // 64-coefficient blocks of both parities
hipError_t configure_interp_mfma();
void launch_interp_mfma(const ResJob* jobs_d, const int32_t* job_list_d, const int32_t* gstart_d,
                        const int64_t* gprefix_d, int ngroups, int64_t nblocks, size_t lds, const RowDesc* rows_d,
                        uint32_t* ws, hipStream_t s);
void launch_reduce(const ResJob* jobs_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks,
                   const uint32_t* ws, uint32_t* res_base, hipStream_t s);
// the evaluation kernel stages a prime's residues in LDS up to this size
constexpr int EE_LDS_MAX = 64 * 1024;
inline bool eval_elim_in_lds(int max_T) { return (size_t)max_T * sizeof(uint32_t) <= (size_t)EE_LDS_MAX; }
// Launch variant of the evaluation kernel for one register class:
//   wpe: minimum wavefronts per SIMD the register allocation is held to (1..4, 1 = unconstrained);
//   chunk: 0 = one workgroup per block; > 0 = persistent grid of `grid` workgroups taking `chunk`
//          blocks at a time from a counter that is zero at launch.
struct EEVariant {
  int32_t wpe = 1;
  int32_t chunk = 0;
  int64_t grid = 0;
};
constexpr int EE_WPE_MAX = 4;
// Revision of the evaluation kernels' code and of the tuner's choice rule,
// part of the autotuner's cache file name: a changed kernel is tuned again
// instead of taking stale choices.
constexpr int EE_KERNEL_REV = 8;
// workgroups of a variant resident on the whole device (0 if the query fails)
int eval_elim_grid(int cls, int wpe, int max_T);
// private (spill) bytes per lane of a variant's kernel (-1 if the query fails)
int eval_elim_scratch(int cls, int wpe, int max_T);
// reduce_in: the residues are reduced from the input limbs inside the kernel (LDS variant only)
void launch_eval_elim(int cls, const EEVariant& v, uint32_t* counter, const ResJob* jobs_d,
                      const int32_t* job_list_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks,
                      int max_T, const RowDesc* rows_d, uint32_t* ws, bool reduce_in, hipStream_t s);
void launch_elim_general_all(const ResJob* jobs_d, const int32_t* job_list_d,
                             const int64_t* inst_prefix_d, int njobs, int64_t ninst,
                             const RowDesc* rows_d, uint32_t* ws, hipStream_t s);
// interpolation at the points 0..D (bivariate gcd images)
void launch_interp(const ResJob* jobs_d, const int64_t* blk_prefix_d, int njobs, int64_t nblocks,
                   int max_D, uint32_t* ws, hipStream_t s);
// job_list_d: the jobs of the launch (block prefix over them), or null for jobs 0..njobs-1
void launch_crt_digits(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d,
                       int njobs, int64_t nblocks, uint32_t* ws, hipStream_t s);
void launch_crt_combine(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d,
                        int njobs, int64_t nblocks, int kmax, uint32_t* ws, hipStream_t s);
// Chinese remaindering with at most CRT_SMALL_K[cls] primes of the modulus
// table (images of the bivariate gcd; of resultants the first NCRT_RES
// classes, up to 64 primes, in large batches): one lane per coefficient
// (digits and binary value in one kernel); blocks of 64 coefficients, prefix
// over the launch's jobs
constexpr int NCRT_SMALL = 3, NCRT_RES = 2;
constexpr int64_t CRT_SMALL_MIN_COEFS = 64 * 64;  // a wavefront for every fourth CU
constexpr int CRT_SMALL_K[NCRT_SMALL] = {32, 64, 128};
inline int crt_small_class(int k) {
  for (int c = 0; c < NCRT_SMALL; ++c)
    if (k <= CRT_SMALL_K[c]) return c;
  return -1;
}
void launch_crt_small(int cls, const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d, int njobs,
                      int64_t nblocks, uint32_t* ws, hipStream_t s);
void launch_crt_small_init(hipStream_t s);  // transposed table of P_j mod p_i (once per device)
// Chinese remaindering on the matrix cores (more than CRT_MFMA_MIN - 1
// primes): digits and carry over groups of 16 coefficients (prefix of
// crt_mfma_groups over the launch's jobs), limb sums over tiles (prefix of
// crt_mfma_tiles).  The limb sums, [lx_of(k)][D+1] of 64 bits, take the points
// region and the one behind it: two words a sum, where the two regions hold
// at least 2 k (D + 1).
constexpr int CRT_MFMA_MIN = 65;
static_assert(lx_of(CRT_MFMA_MIN) <= CRT_MFMA_MIN && lx_of(KMAX) <= KMAX, "the limb sums fit the two regions");
static_assert(CRT_SMALL_K[NCRT_RES - 1] == CRT_MFMA_MIN - 1, "the classes of the resultants end where the matrix cores begin");
int64_t crt_mfma_groups(int n1);
int64_t crt_mfma_tiles(int n1, int k);
hipError_t configure_crt_mfma();
void launch_crt_mfma_init(const CrtTables& tb, hipStream_t s);  // operand tables (once per device)
void launch_crt_mfma_digits(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d,
                            const int64_t* prefix_d, int njobs, int64_t ngroups, int kmax, uint32_t* ws,
                            hipStream_t s);
void launch_crt_mfma_product(const ResJob* jobs_d, const int32_t* job_list_d, const int64_t* prefix_d, int njobs,
                             int64_t ntiles, uint32_t* ws, hipStream_t s);
void launch_crt_mfma_carry(const CrtTables& tb, const ResJob* jobs_d, const int32_t* job_list_d,
                           const int64_t* prefix_d, int njobs, int64_t ngroups, int kmax, uint32_t* ws,
                           hipStream_t s);
CrtTables global_crt_tables();  // the resident tables of the modulus table (after upload)

// gcd work items are (problem, slot) pairs indexing a device array of GcdDesc
void launch_gcd_reduce(const GcdDesc* descs, const int32_t* items, int nitems, int max_rows, int max_nl,
                       uint32_t* ws, hipStream_t s);   // residues of a, b per item (rows: stored coefficient rows)
int gcd_reg_slots(int maxd);             // register class of a degree (slots per lane), 0: LDS kernel
constexpr int GCD_MAX_DEG = 13000;       // the LDS kernel keeps 3 (deg + 1) words
void launch_gcd_euclid(const GcdDesc* descs, const int32_t* items, int nitems, int slots, int maxd, uint32_t* ws,
                       hipStream_t s);   // monic gcd and cofactors per item; one register class per launch
// selected slots sel_d[j] (primes sprimes_d[j]) into compact rows; scales_d[3j..3j+2] = beta,
// cont(a)^-1, cont(b)^-1 mod q_j (plain) multiply w, u, v
void launch_gcd_gather(const GcdDesc& G, const int32_t* sel_d, const uint32_t* scales_d, const PrimeC* sprimes_d,
                       int ks, int e, uint32_t* ws, int64_t wv, int64_t uv, int64_t vv, hipStream_t s);
hipError_t configure_gcd_kernels();
// blocked Euclid of the square-free check (a workgroup of eight wavefronts per
// (problem, prime), fused descriptors only) for the register classes 6, 9, 12, 16
bool gcd_lehmer_class(int slots);
size_t gcd_lehmer_lds_bytes(int slots);
void launch_gcd_lehmer(const GcdDesc* descs, const int32_t* items, int nitems, int slots, uint32_t* ws,
                       hipStream_t s);

// Per-(prime, point) images of a bivariate gcd (k_ygcd): A and B (rows in y
// of polynomials in x, dense rectangles of residues) evaluated at
// x_j = j + shift, W_j = gamma(x_j) * monic gcd_y(A(x_j, y), B(x_j, y)) mod p.
struct YGcdArgs {
  const PrimeC* primes;
  const uint32_t* res;   // Montgomery residues [k][T]
  int32_t T, k, npts;    // residues per prime, primes, points
  int32_t mA, dxA, offA; // A: row i, coefficient of x^t at offA + i (dxA + 1) + t
  int32_t mB, dxB, offB;
  int32_t offG, dg;      // gamma: coefficient of x^t at offG + t, degree dg
  int32_t emax;          // coefficients 0..emax of W are written
  int32_t cap;           // LDS columns hold cap + 1 words (cap >= mA, mB)
  uint32_t shift;
  int32_t* e_out;        // [k][npts]: degree of the gcd, -1 at a point where a leading coefficient vanishes
  uint32_t* w;           // coefficient i of W at w[w_off + i w_stride + pi npts + j] (Montgomery)
  int64_t w_off, w_stride;
};
size_t ygcd_lds_bytes(int cap);
hipError_t configure_ygcd_kernel();
void launch_ygcd(const YGcdArgs& a, hipStream_t s);

int fast_class_of(int maxy);  // index of the register class for a y-degree, -1 if none
int fast_class_cap(int cls);

}  // namespace snc
