// Workspace layout and launch sequence of the resultant pipeline, shared by
// the single-resultant call (direct launches, optional per-stage timing) and
// the batched call (one captured HIP graph per batch shape, replayed).
#include <hip/hip_runtime.h>

#include <atomic>
#include <functional>
#include <thread>

#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "runtime_internal.hpp"

int snc_ctx::stage_in(size_t bytes) {
  if (bytes <= h_in_bytes) return SNC_OK;
  if (h_in) (void)hipHostFree(h_in);
  h_in = nullptr;
  size_t nb = std::max(bytes, h_in_bytes * 2);
  if (hipHostMalloc(&h_in, nb, hipHostMallocDefault) != hipSuccess) { h_in_bytes = 0; h_in = nullptr; return SNC_EDEVICE; }
  h_in_bytes = nb;
  return SNC_OK;
}

int snc_ctx::stage_out(size_t bytes) {
  if (bytes <= h_out_bytes) return SNC_OK;
  if (h_out) (void)hipHostFree(h_out);
  h_out = nullptr;
  size_t nb = std::max(bytes, std::min(h_out_bytes * 2, STAGE_KEEP));
  if (hipHostMalloc(&h_out, nb, hipHostMallocDefault) != hipSuccess) { h_out_bytes = 0; h_out = nullptr; return SNC_EDEVICE; }
  h_out_bytes = nb;
  return SNC_OK;
}

void snc_ctx::release() {
  if (gexec) (void)hipGraphExecDestroy(gexec);
  gexec = nullptr;
  if (cap_stream) (void)hipStreamDestroy(cap_stream);
  cap_stream = nullptr;
  if (side_stream) (void)hipStreamDestroy(side_stream);
  side_stream = nullptr;
  if (ev_mid) (void)hipEventDestroy(ev_mid);
  ev_mid = nullptr;
  if (ev_tail) (void)hipEventDestroy(ev_tail);
  ev_tail = nullptr;
  if (fork_stream) (void)hipStreamDestroy(fork_stream);
  fork_stream = nullptr;
  if (ev_fork) (void)hipEventDestroy(ev_fork);
  ev_fork = nullptr;
  if (ev_join) (void)hipEventDestroy(ev_join);
  ev_join = nullptr;
  for (auto e : events) (void)hipEventDestroy(e);
  events.clear();
  if (h_in) (void)hipHostFree(h_in);
  if (h_out) (void)hipHostFree(h_out);
  h_in = h_out = nullptr;
  h_in_bytes = h_out_bytes = 0;
}

namespace snc {

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Essential lane-operations of one evaluation block (64 instances): Horner
// on the powers of one parity (0.75 per coefficient), the fused remainder steps (5 per entry of
// each remainder), the first remainder's elementary steps and the final
// powers and inversion.
static int64_t eval_block_cost(const ResPlan& P) {
  const int64_t m = P.m, n = P.n;
  return 3 * (int64_t)P.T / 4 + 5 * n * (n + 1) / 2 + 4 * n * std::max<int64_t>(m - n - 1, 0) + 300;
}

// Download and collection of a large output block in chunks: the copy of
// chunk c+1 runs while host threads widen chunk c into the caller's buffers.
constexpr size_t COLLECT_CHUNKED_WORDS = (size_t)1 << 20;
constexpr int COLLECT_CHUNKS = 8;

// Remaindering of a job: class of the one-lane-per-coefficient kernel, or
// CRT_B (lanes over primes), CRT_M (matrix cores)
constexpr int CRT_B = -1, CRT_M = -2;
static int crt_kind(const BatchLayout& lay, int k) {
  if (k >= CRT_MFMA_MIN) return CRT_M;
  return lay.crt_small_on ? crt_small_class(k) : CRT_B;
}

// Two tails when the output is large enough to be downloaded in chunks and
// the classes besides the one with the most output words take at least a
// tenth of the evaluation: the first tail's download (PCIe) then runs beside
// their evaluation.  Orders lay.dev so that each tail's jobs are consecutive.
// Pipelined runs overlap their downloads with the next run instead and take
// the tail of all jobs (97 pairs pipelined in two tails: 2.17 -> 2.45 ms).
static void choose_tails(const std::vector<ResPlan>& plans, BatchLayout& lay) {
  double words[NCLS + 1] = {0}, cost[NCLS + 1] = {0}, all_words = 0, all_cost = 0;
  for (int i : lay.dev) {
    const ResPlan& P = plans[i];
    const int c = P.cls >= 0 ? P.cls : NCLS;
    const double w = ((double)P.D + 1) * P.L, e = (double)P.k * npts_of(P.D) * (double)eval_block_cost(P);
    words[c] += w; all_words += w;
    cost[c] += e; all_cost += e;
  }
  int h = 0;
  for (int c = 1; c <= NCLS; ++c)
    if (words[c] > words[h]) h = c;
  lay.ntails = all_words >= (double)COLLECT_CHUNKED_WORDS && all_cost - cost[h] >= 0.1 * all_cost ? 2 : 1;
  lay.tail[0].j1 = (int)lay.dev.size();
  lay.tail[0].classes = (1u << NCLS) - 1;
  lay.tail[0].general = true;
  if (lay.ntails == 1) return;
  auto mid = std::stable_partition(lay.dev.begin(), lay.dev.end(),
                                   [&](int i) { return (plans[i].cls >= 0 ? plans[i].cls : NCLS) == h; });
  lay.tail[1] = lay.tail[TAIL_WHOLE] = lay.tail[0];
  lay.tail[0].j1 = lay.tail[1].j0 = (int)(mid - lay.dev.begin());
  lay.tail[0].classes = h < NCLS ? 1u << h : 0u;
  lay.tail[0].general = h == NCLS;
  lay.tail[1].classes &= ~lay.tail[0].classes;
  lay.tail[1].general = !lay.tail[0].general;
}

void layout_batch(const std::vector<ResPlan>& plans, BatchLayout& lay) {
  lay = BatchLayout();
  for (int i = 0; i < (int)plans.size(); ++i)
    if (!plans[i].trivial) lay.dev.push_back(i);
  const int NJ = (int)lay.dev.size();
  choose_tails(plans, lay);
  lay.jobs.resize(NJ);
  size_t off = 0;
  lay.jobs_off = off; off = align256(off + sizeof(ResJob) * NJ);
  int nrows = 0;
  for (int j = 0; j < NJ; ++j) nrows += 2 * plans[lay.dev[j]].rstride;
  lay.n_rows = nrows;
  lay.rows_off = off; off = align256(off + sizeof(RowDesc) * nrows);
  lay.pref_red = off; off = align256(off + 8 * (NJ + 1));
  // One lane per coefficient pays off from a wavefront for every fourth CU of the coefficients that would take
  // it; below, the lanes go over the primes of each coefficient.  Whole runs, lanes over primes / one lane: 4,200
  // coefficients of 4, 32 and 60 primes 77 / 74, 144 / 129 and 219 / 202 us, 14,000 of them 119 / 84, 302 / 226
  // and 460 / 332; 2,940 of up to 64 primes beside larger jobs 395 / 395.
  int64_t small_coefs = 0;
  for (int j = 0; j < NJ; ++j)
    if (plans[lay.dev[j]].k < CRT_MFMA_MIN) small_coefs += plans[lay.dev[j]].D + 1;
  lay.crt_small_on = small_coefs >= CRT_SMALL_MIN_COEFS;
  for (int x = 0; x < lay.tails(); ++x) {
    BatchTail& t = lay.tail[x];
    const size_t n = (size_t)(t.j1 - t.j0);
    for (int j = t.j0; j < t.j1; ++j) {
      const ResPlan& P = plans[lay.dev[j]];
      const int n1 = P.D + 1, kind = crt_kind(lay, P.k);
      if (kind >= 0) {
        t.n_crts_jobs[kind]++;
        t.nb_crts[kind] += (n1 + 63) / 64;
      } else if (kind == CRT_M) {
        t.n_crtm_jobs++;
        t.nb_crtm_grp += crt_mfma_groups(n1);
        t.nb_crtm_tile += crt_mfma_tiles(n1, P.k);
        t.max_k_crtm = std::max(t.max_k_crtm, P.k);
      } else {
        t.n_crtb_jobs++;
        t.nb_crtd += (n1 + CRT_COEF_PER_BLOCK - 1) / CRT_COEF_PER_BLOCK;
        t.nb_crtc += (n1 + CRT_COMB_PER_BLOCK - 1) / CRT_COMB_PER_BLOCK;
      }
    }
    t.list_im = off; off = align256(off + 4 * std::max<size_t>(n, 1));
    t.start_im = off; off = align256(off + 4 * (n + 1));
    t.pref_interp = off; off = align256(off + 8 * (n + 1));
    // one section each for the jobs of both kinds of the other remaindering
    const size_t nbm = (size_t)t.n_crtb_jobs + t.n_crtm_jobs;
    t.pref_crtd = off; t.pref_crtm_grp = off + 8 * (t.n_crtb_jobs + 1); off = align256(off + 8 * (nbm + 2));
    t.pref_crtc = off; t.pref_crtm_tile = off + 8 * (t.n_crtb_jobs + 1); off = align256(off + 8 * (nbm + 2));
    t.list_crtb = off; t.list_crtm = off + 4 * t.n_crtb_jobs; off = align256(off + 4 * std::max<size_t>(nbm, 1));
    for (int c = 0; c < NCRT_RES; ++c) {
      t.pref_crts[c] = off; off = align256(off + 8 * (t.n_crts_jobs[c] + 1));
      t.list_crts[c] = off; off = align256(off + 4 * std::max(t.n_crts_jobs[c], 1));
    }
  }
  for (int j = 0; j < NJ; ++j) {
    const ResPlan& P = plans[lay.dev[j]];
    if (P.cls >= 0) lay.n_ee_jobs[P.cls]++; else lay.n_gen_jobs++;
  }
  for (int c = 0; c < NCLS; ++c) {
    lay.pref_ee[c] = off; off = align256(off + 8 * (lay.n_ee_jobs[c] + 1));
    lay.list_ee[c] = off; off = align256(off + 4 * std::max(lay.n_ee_jobs[c], 1));
  }
  lay.pref_gen = off; off = align256(off + 8 * (lay.n_gen_jobs + 1));
  lay.list_gen = off; off = align256(off + 4 * std::max(lay.n_gen_jobs, 1));
  lay.coef_off = off;
  size_t cw = 0;
  for (int j = 0; j < NJ; ++j) { const ResPlan& P = plans[lay.dev[j]]; cw += (size_t)P.T * P.nl; }
  lay.coef_words = cw;
  off = align256(off + 4 * cw);
  lay.header_bytes = off;
  // per-job device regions
  size_t w = off / 4;
  size_t coefw = lay.coef_off / 4;
  int rows = 0;
  double reduce_again = 0;  // wavefront instructions of reducing a prime's inputs for every block but the first
  for (int j = 0; j < NJ; ++j) {
    const ResPlan& P = plans[lay.dev[j]];
    ResJob& J = lay.jobs[j];
    std::memset(&J, 0, sizeof J);
    J.m = P.m; J.n = P.n;
    J.sign = (P.swap && ((P.m * P.n) & 1)) ? 1 : 0;
    J.D = P.D; J.k = P.k; J.T = P.T; J.L = P.L; J.nl = P.nl;
    J.rows_off = rows; J.rstride = P.rstride;
    rows += 2 * P.rstride;
    J.coef_off = (int64_t)coefw; coefw += (size_t)P.T * P.nl;
    const size_t n1 = (size_t)P.D + 1;
    J.res_off = (int64_t)w; w += align_words((size_t)P.k * P.T);
    J.val_off = (int64_t)w; w += align_words((size_t)P.k * n1);
    const size_t np = (size_t)npts_of(P.D);
    J.pts_off = (int64_t)w; w += align_words((size_t)P.k * np);
    J.nq_off = (int64_t)w; w += align_words((size_t)P.k * ((n1 + 63) / 64) * 64);  // adjacent: one buffer of limb sums
    J.dig_off = (int64_t)w; w += align_words(n1 * P.k);
    lay.nb_red += reduce_blocks(P.k, P.T);
    reduce_again += (double)P.k * ((np - 1) / EE_BLOCK) * ((P.T + 63) / 64) * (3 * P.nl + 8);
    lay.max_k = std::max(lay.max_k, P.k);
    if (P.cls >= 0) {
      lay.nb_ee[P.cls] += (int64_t)P.k * ((np + EE_BLOCK - 1) / EE_BLOCK);
      lay.max_T_ee[P.cls] = std::max(lay.max_T_ee[P.cls], P.T);
    }
    else lay.n_gen_inst += (int64_t)P.k * np;
    lay.max_D = std::max(lay.max_D, P.D);
  }
  // Interpolation groups: rows of several jobs fill the 16-row operand tiles,
  // one job per workgroup keeps more workgroups in flight; jobs share one
  // while IM_MIN_BLOCKS workgroups remain (and the group's LDS lets three
  // share a CU).
  int64_t npairs = 0;
  for (const ResJob& J : lay.jobs) npairs += J.k;
  const int per = (int)std::min<int64_t>(IM_JOBS, std::max<int64_t>(1, npairs / IM_MIN_BLOCKS));
  for (int x = 0; x < lay.tails(); ++x) {
    BatchTail& tl = lay.tail[x];
    const int n = tl.j1 - tl.j0;
    tl.im_order.resize(n);
    for (int j = 0; j < n; ++j) tl.im_order[j] = tl.j0 + j;
    std::stable_sort(tl.im_order.begin(), tl.im_order.end(),
                     [&](int a, int b) { return lay.jobs[a].D > lay.jobs[b].D; });
    tl.im_start.assign(1, 0);
    for (int t = 0; t < n;) {
      const int top = lay.jobs[tl.im_order[t]].D;
      int u = t, blocks = 0, kmax = 0;
      for (; u < n && u - t < per; ++u) {
        const ResJob& J = lay.jobs[tl.im_order[u]];
        const int nb = blocks + interp_mfma_blocks(J.D);
        if (u > t && interp_mfma_lds(top, nb) > IM_LDS) break;
        blocks = nb;
        kmax = std::max(kmax, (int)J.k);
      }
      tl.im_lds = std::max(tl.im_lds, interp_mfma_lds(top, blocks));
      tl.nb_interp += kmax;
      tl.im_start.push_back(u);
      t = u;
    }
  }
  // Every job on the evaluation kernel's LDS variant: it can reduce the
  // inputs itself, once per 64-point block of a prime.  With long
  // coefficients the repeats cost more than a launch: past about 4e6 wavefront
  // instructions (7 us of the whole chip) the reduction runs before it, once
  // per prime.
  lay.reduce_in_eval = NJ > 0 && lay.n_gen_jobs == 0 && reduce_again < 4e6;
  for (int c = 0; c < NCLS; ++c)
    if (lay.n_ee_jobs[c] && !eval_elim_in_lds(lay.max_T_ee[c])) lay.reduce_in_eval = false;
  lay.ee_counter_off = w * 4; w += 64;
  lay.out_off = w * 4;
  size_t ow = 0;
  for (int j = 0; j < NJ; ++j) {
    const ResPlan& P = plans[lay.dev[j]];
    lay.jobs[j].out_off = (int64_t)(w + ow);
    ow += ((size_t)P.D + 1) * P.L;
  }
  lay.out_words = ow;
  w += align_words(ow);
  size_t nk = 0;
  for (const ResJob& J : lay.jobs) nk += J.k;
  lay.sq_off = w * 4;
  lay.sq_words = align_words(sizeof(GcdDesc) / 4 * std::max<size_t>(NJ, 1)) + align_words(2 * std::max<size_t>(nk, 1)) +
                 align_words(KMAX) + 2 * align_words(std::max<size_t>(nk, 1));
  w += lay.sq_words;
  lay.total_bytes = w * 4;
}

struct StageTimer {
  snc_ctx* c;
  hipStream_t s;
  bool on;
  int n = 0;
  void start() {
    if (!on) return;
    c->stage_names.clear(); c->stage_ms.clear(); c->stage_launches.clear();
    mark(nullptr, 0);
  }
  void mark(const char* name, int launches) {
    if (!on) return;
    if ((int)c->events.size() <= n) {
      hipEvent_t e;
      (void)hipEventCreate(&e);
      c->events.push_back(e);
    }
    (void)hipEventRecord(c->events[n], s);
    if (name) { c->stage_names.push_back(name); c->stage_launches.push_back(launches); }
    ++n;
  }
  void finish() {
    if (!on) return;
    for (int i = 1; i < n; ++i) {
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, c->events[i - 1], c->events[i]);
      c->stage_ms.push_back(ms);
    }
  }
};

// Device launch sequence for a laid-out batch (everything after the upload).
// part: PIPE_ALL, PIPE_TO_INTERP (reduction .. interpolation) or PIPE_CRT
void launch_pipeline(const BatchLayout& lay, uint8_t* ws, hipStream_t s, StageTimer* tm, int part,
                     const PipeFork& fk, int tail) {
  if (tail < 0) tail = lay.whole();
  const BatchTail& t = lay.tail[tail];
  uint32_t* wsw = (uint32_t*)ws;
  const ResJob* jobs = (const ResJob*)(ws + lay.jobs_off);
  const RowDesc* rows = (const RowDesc*)(ws + lay.rows_off);
  if (part != PIPE_CRT) {
    uint32_t* ee_counters = (uint32_t*)(ws + lay.ee_counter_off);
    if (tail != 1) {  // before everything
      if (!lay.reduce_in_eval)
        launch_reduce(jobs, (const int64_t*)(ws + lay.pref_red), (int)lay.jobs.size(), lay.nb_red, wsw, wsw, s);
      if (tm) tm->mark("reduce", lay.reduce_in_eval ? 0 : 1);
      bool persistent = false;
      for (int c = 0; c < NCLS; ++c) persistent |= lay.n_ee_jobs[c] && lay.ee_var[c].chunk > 0;
      if (persistent) launch_zero_u32(ee_counters, NCLS, s);  // a kernel, not a memset node
    }
    // one stage per register class (names: eval_elim_<width>), then the
    // jobs above the register classes
    static const char* const kEEStage[NCLS] = {"eval_elim_8", "eval_elim_16", "eval_elim_32", "eval_elim_40",
                                               "eval_elim_48", "eval_elim_64"};
    for (int c = 0; c < NCLS; ++c) {
      if (!lay.n_ee_jobs[c] || !(t.classes >> c & 1u)) continue;
      launch_eval_elim(c, lay.ee_var[c], ee_counters + c, jobs, (const int32_t*)(ws + lay.list_ee[c]),
                       (const int64_t*)(ws + lay.pref_ee[c]), lay.n_ee_jobs[c], lay.nb_ee[c], lay.max_T_ee[c], rows,
                       wsw, lay.reduce_in_eval, s);
      if (tm) tm->mark(kEEStage[c], 1);
    }
    if (lay.n_gen_jobs && t.general) {
      launch_elim_general_all(jobs, (const int32_t*)(ws + lay.list_gen), (const int64_t*)(ws + lay.pref_gen),
                              lay.n_gen_jobs, lay.n_gen_inst, rows, wsw, s);
      if (tm) tm->mark("eval_elim_general", 1);
    }
    launch_interp_mfma(jobs, (const int32_t*)(ws + t.list_im), (const int32_t*)(ws + t.start_im),
                       (const int64_t*)(ws + t.pref_interp), (int)t.im_start.size() - 1, t.nb_interp, t.im_lds, rows,
                       wsw, s);
    if (tm) tm->mark("interp", 1);
  }
  if (part == PIPE_TO_INTERP) return;
  static const char* const kCrtStage[NCRT_RES] = {"crt_small_32", "crt_small_64"};
  // The jobs on the matrix cores (or, without any, the small-prime class with
  // the most primes: few, long workgroups bound by their own latency) run on a
  // branch beside the other jobs instead of after them.
  int nsmall = 0, top = -1;
  for (int c = 0; c < NCRT_RES; ++c)
    if (t.n_crts_jobs[c]) { ++nsmall; top = c; }
  const CrtTables tb = global_crt_tables();
  auto small = [&](int c, hipStream_t st) {
    launch_crt_small(c, jobs, (const int32_t*)(ws + t.list_crts[c]), (const int64_t*)(ws + t.pref_crts[c]),
                     t.n_crts_jobs[c], t.nb_crts[c], wsw, st);
  };
  auto mfma = [&](hipStream_t st) {
    const int32_t* lm = (const int32_t*)(ws + t.list_crtm);
    const int64_t* pg = (const int64_t*)(ws + t.pref_crtm_grp);
    launch_crt_mfma_digits(tb, jobs, lm, pg, t.n_crtm_jobs, t.nb_crtm_grp, t.max_k_crtm, wsw, st);
    if (tm) tm->mark("crt_mfma_digits", 1);
    launch_crt_mfma_product(jobs, lm, (const int64_t*)(ws + t.pref_crtm_tile), t.n_crtm_jobs, t.nb_crtm_tile,
                            wsw, st);
    if (tm) tm->mark("crt_mfma_product", 1);
    launch_crt_mfma_carry(tb, jobs, lm, pg, t.n_crtm_jobs, t.nb_crtm_grp, t.max_k_crtm, wsw, st);
    if (tm) tm->mark("crt_mfma_carry", 1);
  };
  const bool beside = t.n_crtm_jobs ? nsmall >= 1 || t.n_crtb_jobs : nsmall >= 2;
  const bool branch = fk.stream && !tm && beside;
  if (branch) {
    (void)hipEventRecord(fk.fork, s);
    (void)hipStreamWaitEvent(fk.stream, fk.fork, 0);
    if (t.n_crtm_jobs) mfma(fk.stream);
    else small(top, fk.stream);
  }
  for (int c = 0; c < NCRT_RES; ++c) {
    if (!t.n_crts_jobs[c] || (branch && !t.n_crtm_jobs && c == top)) continue;
    small(c, s);
    if (tm) tm->mark(kCrtStage[c], 1);
  }
  if (t.n_crtb_jobs) {
    const int32_t* lb = (const int32_t*)(ws + t.list_crtb);
    launch_crt_digits(tb, jobs, lb, (const int64_t*)(ws + t.pref_crtd), t.n_crtb_jobs, t.nb_crtd, wsw, s);
    if (tm) tm->mark("crt_digits", 1);
    launch_crt_combine(tb, jobs, lb, (const int64_t*)(ws + t.pref_crtc), t.n_crtb_jobs, t.nb_crtc,
                       (int)std::min<int64_t>(lay.max_k, CRT_MFMA_MIN - 1), wsw, s);
    if (tm) tm->mark("crt_combine", 1);
  }
  if (branch) {
    (void)hipEventRecord(fk.join, fk.stream);
    (void)hipStreamWaitEvent(s, fk.join, 0);
  }
  if (t.n_crtm_jobs && !branch) mfma(s);
}

// Fill the upload block: job descriptors, row descriptors, block prefixes,
// class job lists and the packed input coefficients.
void fill_header(const BatchLayout& lay, const std::vector<ResPlan>& plans, const std::vector<Operand>& F,
                 const std::vector<Operand>& G, uint8_t* h) {
  const int NJ = (int)lay.dev.size();
  std::memcpy(h + lay.jobs_off, lay.jobs.data(), sizeof(ResJob) * NJ);
  RowDesc* rows = (RowDesc*)(h + lay.rows_off);
  uint32_t* coef = (uint32_t*)(h + lay.coef_off);
  int64_t* pr = (int64_t*)(h + lay.pref_red);
  int64_t* pe[NCLS];
  int32_t* le[NCLS];
  int ne[NCLS] = {0};
  for (int c = 0; c < NCLS; ++c) {
    pe[c] = (int64_t*)(h + lay.pref_ee[c]);
    le[c] = (int32_t*)(h + lay.list_ee[c]);
    pe[c][0] = 0;
  }
  std::vector<std::pair<int64_t, int>> by_cost[NCLS];  // (work per block, job) per register class
  int64_t* pg = (int64_t*)(h + lay.pref_gen);
  int32_t* lg = (int32_t*)(h + lay.list_gen);
  int ng = 0;
  pg[0] = 0;
  pr[0] = 0;
  size_t cw = 0;
  for (int j = 0; j < NJ; ++j) {
    const int idx = lay.dev[j];
    const ResPlan& P = plans[idx];
    const ResJob& J = lay.jobs[j];
    const Operand& A = P.swap ? G[idx] : F[idx];
    const Operand& B = P.swap ? F[idx] : G[idx];
    RowDesc* ra = rows + J.rows_off;
    int off = 0;
    auto emit = [&](const Operand& O, RowDesc* rd, int deg) {
      for (int g = 0; g < P.rstride; ++g) {
        rd[g].off = 0; rd[g].len = 0;
        const int t0 = g * ROWGRP;
        if (t0 > deg) continue;
        int ml = 0;
        for (int q = 0; q < ROWGRP && t0 + q <= deg; ++q) ml = std::max(ml, O.rowdeg[deg - t0 - q] + 1);
        ml = padded_group_len(ml);
        rd[g].off = off; rd[g].len = ml;
        for (int kx = 0; kx < ml; ++kx) {
          for (int q = 0; q < ROWGRP; ++q) {
            uint32_t* dst = coef + cw + (size_t)(off + grp_pos(kx, ml) + q);  // limb l at dst[l T]
            const int row = deg - t0 - q;
            if (t0 + q > deg || kx > O.rowdeg[row]) {
              for (int l = 0; l < P.nl; ++l) dst[(size_t)l * P.T] = 0u;
              continue;
            }
            const uint32_t* src = O.limbs + ((size_t)row * (O.dx + 1) + kx) * O.nl;
            const uint32_t ext = (src[O.nl - 1] >> 31) ? 0xffffffffu : 0u;
            for (int l = 0; l < P.nl; ++l) dst[(size_t)l * P.T] = l < O.nl ? src[l] : ext;
          }
        }
        off += ROWGRP * ml;
      }
    };
    emit(A, ra, P.m);
    emit(B, ra + P.rstride, P.n);
    cw += (size_t)P.T * P.nl;
    pr[j + 1] = pr[j] + reduce_blocks(P.k, P.T);
    if (P.cls >= 0) {
      by_cost[P.cls].push_back({eval_block_cost(P), j});
    } else {
      lg[ng] = j;
      pg[ng + 1] = pg[ng] + (int64_t)P.k * npts_of(P.D);
      ng++;
    }
  }
  for (int x = 0; x < lay.tails(); ++x) {
    const BatchTail& t = lay.tail[x];
    // the interpolation's job order, groups and their prime counts
    std::memcpy(h + t.list_im, t.im_order.data(), 4 * t.im_order.size());
    std::memcpy(h + t.start_im, t.im_start.data(), 4 * t.im_start.size());
    int64_t* pi = (int64_t*)(h + t.pref_interp);
    pi[0] = 0;
    for (size_t g = 0; g + 1 < t.im_start.size(); ++g) {
      int kmax = 0;
      for (int i = t.im_start[g]; i < t.im_start[g + 1]; ++i) kmax = std::max(kmax, (int)lay.jobs[t.im_order[i]].k);
      pi[g + 1] = pi[g] + kmax;
    }
    // the remaindering's job lists and prefixes
    int64_t* ps[NCRT_RES];
    int32_t* ls[NCRT_RES];
    int ns[NCRT_RES] = {0}, nb = 0, nm = 0;
    for (int c = 0; c < NCRT_RES; ++c) {
      ps[c] = (int64_t*)(h + t.pref_crts[c]);
      ls[c] = (int32_t*)(h + t.list_crts[c]);
      ps[c][0] = 0;
    }
    int32_t *lb = (int32_t*)(h + t.list_crtb), *lm = (int32_t*)(h + t.list_crtm);
    int64_t *pd = (int64_t*)(h + t.pref_crtd), *pc = (int64_t*)(h + t.pref_crtc);
    int64_t *pmg = (int64_t*)(h + t.pref_crtm_grp), *pmt = (int64_t*)(h + t.pref_crtm_tile);
    pd[0] = pc[0] = pmg[0] = pmt[0] = 0;
    for (int j = t.j0; j < t.j1; ++j) {
      const int k = lay.jobs[j].k;
      const int64_t n1 = (int64_t)lay.jobs[j].D + 1;
      const int kind = crt_kind(lay, k);
      if (kind >= 0) {
        ls[kind][ns[kind]] = j;
        ps[kind][ns[kind] + 1] = ps[kind][ns[kind]] + (n1 + 63) / 64;
        ns[kind]++;
      } else if (kind == CRT_M) {
        lm[nm] = j;
        pmg[nm + 1] = pmg[nm] + crt_mfma_groups((int)n1);
        pmt[nm + 1] = pmt[nm] + crt_mfma_tiles((int)n1, k);
        nm++;
      } else {
        lb[nb] = j;
        pd[nb + 1] = pd[nb] + (n1 + CRT_COEF_PER_BLOCK - 1) / CRT_COEF_PER_BLOCK;
        pc[nb + 1] = pc[nb] + (n1 + CRT_COMB_PER_BLOCK - 1) / CRT_COMB_PER_BLOCK;
        nb++;
      }
    }
  }
  // a class's jobs most expensive first: a persistent launch hands out the
  // cheapest blocks last (the order does not change any result)
  for (int c = 0; c < NCLS; ++c) {
    std::stable_sort(by_cost[c].begin(), by_cost[c].end(),
                     [](const std::pair<int64_t, int>& x, const std::pair<int64_t, int>& y) { return x.first > y.first; });
    for (const auto& e : by_cost[c]) {
      const ResJob& J = lay.jobs[e.second];
      le[c][ne[c]] = e.second;
      pe[c][ne[c] + 1] = pe[c][ne[c]] + (int64_t)J.k * ((npts_of(J.D) + EE_BLOCK - 1) / EE_BLOCK);
      ne[c]++;
    }
  }
}


#define HIPCHK(x)                                                                     \
  do {                                                                                \
    hipError_t e_ = (x);                                                              \
    if (e_ != hipSuccess) {                                                           \
      c->err = std::string(#x) + ": " + hipGetErrorString(e_);                        \
      return SNC_EDEVICE;                                                             \
    }                                                                                 \
  } while (0)

// Status of a call on `stream`.  A failed one may have copies and kernels in
// flight on both streams: they end before its buffers can be reused or freed.
static int end_run(snc_ctx* c, hipStream_t stream, int st) {
  if (st != SNC_OK) {
    (void)hipStreamSynchronize(stream);
    if (c->side_stream) (void)hipStreamSynchronize(c->side_stream);
  }
  return st;
}

int prepare_resultants(snc_ctx* c, int n, const snc_bipoly* f, const snc_bipoly* g, void* d_ws,
                       size_t ws_bytes, hipStream_t stream, bool use_graph, bool one_shot, snc_prepared** outp) {
  *outp = nullptr;
  HIPCHK(hipSetDevice(c->device));
  std::vector<Operand> F(n), G(n);
  snc_prepared* pr = new snc_prepared();
  pr->c = c;
  pr->n = n;
  pr->use_graph = use_graph;
  pr->P.resize(n);
  for (int i = 0; i < n; ++i) {
    int st = parse_bipoly(&f[i], F[i], c->err);
    if (!st) st = parse_bipoly(&g[i], G[i], c->err);
    if (!st) st = plan_resultant(F[i], G[i], pr->P[i], c->err);
    if (st) { c->err = "pair " + std::to_string(i) + ": " + c->err; delete pr; return st; }
  }
  layout_batch(pr->P, pr->lay);
  const BatchLayout& lay = pr->lay;
  if (!lay.dev.empty()) {
    if (!d_ws || ws_bytes < lay.total_bytes) {
      c->err = "workspace of " + std::to_string(ws_bytes) + " bytes, need " + std::to_string(lay.total_bytes);
      delete pr;
      return SNC_ENOMEM;
    }
    pr->ws = (uint8_t*)d_ws;
    if (c->stage_in(lay.header_bytes)) { c->err = "pinned staging allocation failed"; delete pr; return SNC_EDEVICE; }
    // a handle keeps a pinned block of its own; a single call takes the
    // context's (pinning and unpinning a block cost 200-400 us a call) up to
    // the size a context keeps
    pr->own_out = !one_shot || lay.out_words * 4 > snc_ctx::STAGE_KEEP;
    bool pinned;
    if (!pr->own_out) {
      pinned = c->stage_out(lay.out_words * 4) == SNC_OK;
      pr->h_out = c->h_out;
    } else {
      pinned = hipHostMalloc(&pr->h_out, std::max<size_t>(lay.out_words * 4, 4), hipHostMallocDefault) == hipSuccess;
    }
    if (!pinned) {
      pr->h_out = nullptr;
      c->err = "pinned staging allocation failed";
      delete pr;
      return SNC_EDEVICE;
    }
    fill_header(lay, pr->P, F, G, (uint8_t*)c->h_in);
    StageTimer tm{c, stream, c->timing && !use_graph};
    tm.start();
    hipError_t e = hipMemcpyAsync(pr->ws, c->h_in, lay.header_bytes, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) {
      // launch variants of the evaluation kernel: measured for a batched graph, looked up otherwise
      const int st = choose_eval_variants(c, pr->lay, pr->ws, stream, use_graph);
      if (st) { end_run(c, stream, st); destroy_prepared(pr); return st; }
    }
    // a single call waits once, for its results; the staging buffer is not
    // written again before that
    if (e == hipSuccess && !one_shot) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) {
      c->err = std::string("input upload: ") + hipGetErrorString(e);
      end_run(c, stream, SNC_EDEVICE);
      destroy_prepared(pr);
      return SNC_EDEVICE;
    }
  }
  *outp = pr;
  return SNC_OK;
}

// output sizes and the host-only (trivial) results; false with SNC_ERANGE sizes written back
static bool prepared_outputs(snc_prepared* pr, snc_upoly* out) {
  const std::vector<ResPlan>& P = pr->P;
  bool range_err = false;
  for (int i = 0; i < pr->n; ++i) {
    const int need_deg = P[i].trivial ? (P[i].trivial_value ? 0 : -1) : P[i].D;
    const int need_nl = P[i].trivial ? 1 : P[i].L;
    if (out[i].deg < need_deg || out[i].nlimbs < need_nl || (need_deg >= 0 && !out[i].limbs)) {
      out[i].deg = need_deg;
      out[i].nlimbs = need_nl;
      range_err = true;
    }
  }
  if (range_err) { pr->c->err = "output buffer too small"; return false; }
  for (int i = 0; i < pr->n; ++i) {
    if (!P[i].trivial) continue;
    if (P[i].trivial_value) {
      for (int l = 0; l < out[i].nlimbs; ++l) out[i].limbs[l] = l == 0 ? 1u : 0u;
      out[i].deg = 0;
    } else {
      out[i].deg = -1;
    }
  }
  return true;
}

// the pipeline of one tail (-1: of all jobs) on `stream`, as a HIP graph
// captured on first use
static int launch_prepared(snc_prepared* pr, hipStream_t stream, StageTimer& tm, int tail) {
  snc_ctx* c = pr->c;
  // with timing on, the same launches go straight to the stream between
  // events (a replayed graph cannot be timed per stage)
  if (!pr->use_graph || tm.on) {
    launch_pipeline(pr->lay, pr->ws, stream, tm.on ? &tm : nullptr, PIPE_ALL, PipeFork(), tail);
    HIPCHK(hipGetLastError());
    return SNC_OK;
  }
  const int x = tail < 0 ? pr->lay.whole() : tail;
  hipGraphExec_t& gx = pr->gexec[x];
  if (!gx) {
    if (!c->cap_stream) HIPCHK(hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    if (!c->fork_stream) HIPCHK(hipStreamCreateWithFlags(&c->fork_stream, hipStreamNonBlocking));
    if (!c->ev_fork) HIPCHK(hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming));
    if (!c->ev_join) HIPCHK(hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming));
    PipeFork fk;
    fk.stream = c->fork_stream;
    fk.fork = c->ev_fork;
    fk.join = c->ev_join;
    hipGraph_t graph = nullptr;
    HIPCHK(hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
    launch_pipeline(pr->lay, pr->ws, c->cap_stream, nullptr, PIPE_ALL, fk, x);
    HIPCHK(hipStreamEndCapture(c->cap_stream, &graph));
    hipError_t e = hipGraphInstantiate(&gx, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) { gx = nullptr; c->err = std::string("graph instantiate: ") + hipGetErrorString(e); return SNC_EDEVICE; }
  }
  HIPCHK(hipGraphLaunch(gx, stream));
  return SNC_OK;
}

// results of jobs j0 .. j1-1 with j = tid mod nthr from the staged output block into out
static void collect_jobs(const snc_prepared* pr, const uint32_t* ho, snc_upoly* out, int j0, int j1, int tid,
                         int nthr) {
  const BatchLayout& lay = pr->lay;
  const size_t base = lay.out_off / 4;
  for (int j = j0 + tid; j < j1; j += nthr) {
    const int i = lay.dev[j];
    const ResJob& J = lay.jobs[j];
    const uint32_t* src = ho + (J.out_off - base);
    int deg = -1;
    for (int t = J.D; t >= 0 && deg < 0; --t)
      for (int l = 0; l < J.L; ++l)
        if (src[(size_t)t * J.L + l]) { deg = t; break; }
    const int stride = out[i].nlimbs;
    if (stride == J.L) {
      std::memcpy(out[i].limbs, src, sizeof(uint32_t) * (size_t)(deg + 1) * J.L);
    } else {
      for (int t = 0; t <= deg; ++t) {
        const uint32_t* s = src + (size_t)t * J.L;
        uint32_t* d = out[i].limbs + (size_t)t * stride;
        const uint32_t ext = (s[J.L - 1] >> 31) ? 0xffffffffu : 0u;
        for (int l = 0; l < stride; ++l) d[l] = l < J.L ? s[l] : ext;
      }
    }
    out[i].deg = deg;
  }
}

static void prepared_collect(snc_prepared* pr, snc_upoly* out) {
  collect_jobs(pr, (const uint32_t*)pr->h_out, out, 0, (int)pr->lay.dev.size(), 0, 1);
}

// job ranges of about equal output words (the jobs' output regions are consecutive)
static std::vector<int> chunk_bounds(const BatchLayout& lay) {
  const int NJ = (int)lay.dev.size();
  std::vector<int> bnd{0};
  const size_t per = (lay.out_words + COLLECT_CHUNKS - 1) / COLLECT_CHUNKS;
  size_t acc = 0;
  for (int j = 0; j < NJ; ++j) {
    acc += (size_t)(lay.jobs[j].D + 1) * lay.jobs[j].L;
    const bool border = lay.ntails == 2 && j + 1 == lay.tail[1].j0;  // a chunk belongs to one tail
    if ((acc >= per * bnd.size() || border) && j + 1 < NJ && ((int)bnd.size() < COLLECT_CHUNKS || border))
      bnd.push_back(j + 1);
  }
  bnd.push_back(NJ);
  return bnd;
}

// downloads of the output block from src (device, laid out as the
// workspace's output region) to dst (pinned host) in the chunks of bnd within
// jobs j0 .. j1-1 on stream, one event recorded after each
static int enqueue_chunks(const snc_prepared* pr, const std::vector<int>& bnd, const uint8_t* src, void* dst,
                          std::vector<hipEvent_t>& ev, hipStream_t stream, int j0, int j1) {
  snc_ctx* c = pr->c;
  const BatchLayout& lay = pr->lay;
  const int NJ = (int)lay.dev.size();
  const int nch = (int)bnd.size() - 1;
  while ((int)ev.size() < nch) {
    hipEvent_t e;
    HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    ev.push_back(e);
  }
  const size_t base = lay.out_off / 4;
  for (int ch = 0; ch < nch; ++ch) {
    if (bnd[ch] < j0 || bnd[ch] >= j1) continue;
    const size_t w0 = lay.jobs[bnd[ch]].out_off - base;
    const size_t w1 = bnd[ch + 1] < NJ ? lay.jobs[bnd[ch + 1]].out_off - base : lay.out_words;
    HIPCHK(hipMemcpyAsync((uint32_t*)dst + w0, src + w0 * 4, (w1 - w0) * 4, hipMemcpyDeviceToHost, stream));
    HIPCHK(hipEventRecord(ev[ch], stream));
  }
  return SNC_OK;
}

// host threads widen each chunk of ho into the caller's buffers as soon as
// its event has completed
static int widen_chunks(snc_prepared* pr, const std::vector<int>& bnd, const std::vector<hipEvent_t>& ev,
                        const uint32_t* ho, snc_upoly* out) {
  snc_ctx* c = pr->c;
  const int nch = (int)bnd.size() - 1;
  const unsigned hc = std::thread::hardware_concurrency();
  const int nthr = (int)std::max(1u, std::min(8u, hc / 2));
  std::atomic<int> ready{0};
  std::vector<std::thread> workers;
  for (int t = 1; t < nthr; ++t)
    workers.emplace_back([&, t] {
      for (int ch = 0; ch < nch; ++ch) {
        while (ready.load(std::memory_order_acquire) <= ch) {
          if (ready.load(std::memory_order_acquire) < 0) return;
          std::this_thread::yield();
        }
        collect_jobs(pr, ho, out, bnd[ch], bnd[ch + 1], t, nthr);
      }
    });
  hipError_t err = hipSuccess;
  for (int ch = 0; ch < nch; ++ch) {
    err = hipEventSynchronize(ev[ch]);
    if (err != hipSuccess) { ready.store(-1, std::memory_order_release); break; }
    ready.store(ch + 1, std::memory_order_release);
    collect_jobs(pr, ho, out, bnd[ch], bnd[ch + 1], 0, nthr);
  }
  for (auto& w : workers) w.join();
  if (err != hipSuccess) { c->err = std::string("result download: ") + hipGetErrorString(err); return SNC_EDEVICE; }
  return SNC_OK;
}

// A run with a large output: each tail's results are downloaded as soon as it
// is done, the first tail's on the side stream beside the second's kernels
// (512 pairs: 35 of the 50 MB travel beside the evaluation of the smaller
// classes; 0.9 ms of download after the kernels before, 0.3 ms now).
static int run_chunked(snc_prepared* pr, hipStream_t stream, snc_upoly* out) {
  snc_ctx* c = pr->c;
  const BatchLayout& lay = pr->lay;
  const std::vector<int> bnd = chunk_bounds(lay);
  StageTimer tm{c, stream, false};
  for (int x = 0; x < lay.ntails; ++x) {
    int st = launch_prepared(pr, stream, tm, x);
    if (st) return st;
    hipStream_t down = stream;
    if (x + 1 < lay.ntails) {
      if (!c->side_stream) HIPCHK(hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking));
      // a copy follows: the event releases to the whole system
      if (!c->ev_tail) HIPCHK(hipEventCreateWithFlags(&c->ev_tail, hipEventDisableTiming));
      HIPCHK(hipEventRecord(c->ev_tail, stream));
      HIPCHK(hipStreamWaitEvent(c->side_stream, c->ev_tail, 0));
      down = c->side_stream;
    }
    st = enqueue_chunks(pr, bnd, pr->ws + lay.out_off, pr->h_out, pr->d2h_ev, down, lay.tail[x].j0, lay.tail[x].j1);
    if (st) return st;
  }
  return widen_chunks(pr, bnd, pr->d2h_ev, (const uint32_t*)pr->h_out, out);
}

static int run_whole(snc_prepared* pr, hipStream_t stream, snc_upoly* out) {
  snc_ctx* c = pr->c;
  StageTimer tm{c, stream, c->timing};
  tm.start();
  int st = launch_prepared(pr, stream, tm, -1);
  if (st) return st;
  HIPCHK(hipMemcpyAsync(pr->h_out, pr->ws + pr->lay.out_off, pr->lay.out_words * 4, hipMemcpyDeviceToHost, stream));
  tm.mark("d2h", 1);
  HIPCHK(hipStreamSynchronize(stream));
  tm.finish();
  prepared_collect(pr, out);
  return SNC_OK;
}

int run_prepared(snc_prepared* pr, hipStream_t stream, snc_upoly* out) {
  snc_ctx* c = pr->c;
  if (!prepared_outputs(pr, out)) return SNC_ERANGE;
  if (pr->lay.dev.empty()) return SNC_OK;
  HIPCHK(hipSetDevice(c->device));
  const bool chunked = !c->timing && pr->lay.out_words >= COLLECT_CHUNKED_WORDS;
  return end_run(c, stream, chunked ? run_chunked(pr, stream, out) : run_whole(pr, stream, out));
}

size_t prepared_stage_bytes(const snc_prepared* pr) {
  return pr->lay.dev.empty() ? 0 : 2 * align_words(pr->lay.out_words) * 4;
}

// one run, the copy of its output region to the slot on the device (short, on
// this stream: the next run's kernels can start right after it) and from there
// to the host on the side stream
static int enqueue_run(snc_prepared* pr, uint8_t* slot, int s, hipStream_t stream) {
  snc_ctx* c = pr->c;
  StageTimer tm{c, stream, false};
  const int st = launch_prepared(pr, stream, tm, -1);
  if (st) return st;
  HIPCHK(hipMemcpyAsync(slot, pr->ws + pr->lay.out_off, pr->lay.out_words * 4, hipMemcpyDeviceToDevice, stream));
  HIPCHK(hipEventRecord(pr->slot_copied[s], stream));
  HIPCHK(hipStreamWaitEvent(c->side_stream, pr->slot_copied[s], 0));
  return enqueue_chunks(pr, chunk_bounds(pr->lay), slot, pr->slot_host[s], pr->slot_ev[s], c->side_stream, 0,
                        (int)pr->lay.dev.size());
}

int submit_prepared(snc_prepared* pr, void* d_stage, size_t stage_bytes, hipStream_t stream, int64_t* ticket) {
  snc_ctx* c = pr->c;
  const size_t need = prepared_stage_bytes(pr);
  if (stage_bytes < need || (need && !d_stage)) {
    c->err = "snc_prepared_submit: staging buffer of " + std::to_string(stage_bytes) + " bytes, " +
             std::to_string(need) + " needed (snc_prepared_stage_bytes)";
    return SNC_ENOMEM;
  }
  int s = (int)(pr->next_ticket & 1);
  if (pr->slot_ticket[s] >= 0) s ^= 1;
  if (pr->slot_ticket[s] >= 0) {
    c->err = "snc_prepared_submit: two runs are outstanding; collect one first";
    return SNC_EAGAIN;
  }
  HIPCHK(hipSetDevice(c->device));
  const size_t bytes = pr->lay.out_words * 4;
  if (bytes && !pr->slot_host[s]) {
    HIPCHK(hipHostMalloc(&pr->slot_host[s], bytes, hipHostMallocDefault));
    HIPCHK(hipEventCreateWithFlags(&pr->slot_copied[s], hipEventDisableTiming));
  }
  if (!c->side_stream) HIPCHK(hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking));
  if (!pr->lay.dev.empty()) {
    const int st = end_run(c, stream, enqueue_run(pr, (uint8_t*)d_stage + (size_t)s * (need / 2), s, stream));
    if (st) return st;
  }
  pr->slot_ticket[s] = pr->next_ticket;
  *ticket = pr->next_ticket++;
  return SNC_OK;
}

int collect_prepared(snc_prepared* pr, int64_t ticket, snc_upoly* out) {
  snc_ctx* c = pr->c;
  const int s = ticket >= 0 && pr->slot_ticket[0] == ticket ? 0 : ticket >= 0 && pr->slot_ticket[1] == ticket ? 1 : -1;
  if (s < 0) {
    c->err = "snc_prepared_collect: ticket " + std::to_string(ticket) + " is not an outstanding run";
    return SNC_EINVAL;
  }
  if (!prepared_outputs(pr, out)) return SNC_ERANGE;
  int st = SNC_OK;
  if (!pr->lay.dev.empty()) {
    HIPCHK(hipSetDevice(c->device));
    st = widen_chunks(pr, chunk_bounds(pr->lay), pr->slot_ev[s], (const uint32_t*)pr->slot_host[s], out);
  }
  pr->slot_ticket[s] = -1;
  return st;
}

static int run_fork(snc_prepared* pr, hipStream_t stream, const std::function<int(hipStream_t)>& branch,
                    const std::function<void()>& on_results, snc_upoly* out) {
  snc_ctx* c = pr->c;
  if (!c->side_stream) HIPCHK(hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking));
  // the side stream runs on this device only: a device-scope release suffices
  if (!c->ev_mid) HIPCHK(hipEventCreateWithFlags(&c->ev_mid, hipEventDisableTiming | hipEventReleaseToDevice));
  // plain launches: the host queues the whole step (both streams) while the
  // first kernels run, which measured slightly faster than replaying graphs here
  launch_pipeline(pr->lay, pr->ws, stream, nullptr, PIPE_TO_INTERP);
  HIPCHK(hipGetLastError());
  // the branch is queued on this stream right behind the interpolation, so
  // it starts without a cross-stream wait; the Chinese remaindering and the
  // download of the results go to the side stream
  HIPCHK(hipEventRecord(c->ev_mid, stream));
  const int st = branch(stream);
  if (st) return st;
  HIPCHK(hipStreamWaitEvent(c->side_stream, c->ev_mid, 0));
  launch_pipeline(pr->lay, pr->ws, c->side_stream, nullptr, PIPE_CRT);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(pr->h_out, pr->ws + pr->lay.out_off, pr->lay.out_words * 4, hipMemcpyDeviceToHost,
                        c->side_stream));
  HIPCHK(hipStreamSynchronize(c->side_stream));
  prepared_collect(pr, out);
  on_results();
  HIPCHK(hipStreamSynchronize(stream));
  return SNC_OK;
}

int run_prepared_fork(snc_prepared* pr, hipStream_t stream, const std::function<int(hipStream_t)>& branch,
                      const std::function<void()>& on_results, snc_upoly* out) {
  if (!prepared_outputs(pr, out)) return SNC_ERANGE;
  if (pr->lay.dev.empty()) { on_results(); return SNC_OK; }
  snc_ctx* c = pr->c;
  HIPCHK(hipSetDevice(c->device));
  return end_run(c, stream, run_fork(pr, stream, branch, on_results, out));
}

int run_resultants(snc_ctx* c, int n, const snc_bipoly* f, const snc_bipoly* g, void* d_ws,
                   size_t ws_bytes, hipStream_t stream, snc_upoly* out, bool use_graph) {
  snc_prepared* pr = nullptr;
  int st = prepare_resultants(c, n, f, g, d_ws, ws_bytes, stream, use_graph, true, &pr);
  if (st) return st;
  st = end_run(c, stream, run_prepared(pr, stream, out));  // an output refused after the upload waits for it too
  destroy_prepared(pr);
  return st;
}

void destroy_prepared(snc_prepared* pr) {
  if (!pr) return;
  for (int s = 0; s < 2; ++s) {
    // an uncollected run's download must end before its buffers go
    if (pr->slot_ticket[s] >= 0 && !pr->slot_ev[s].empty()) (void)hipEventSynchronize(pr->slot_ev[s].back());
    if (pr->slot_host[s]) (void)hipHostFree(pr->slot_host[s]);
    if (pr->slot_copied[s]) (void)hipEventDestroy(pr->slot_copied[s]);
    for (hipEvent_t e : pr->slot_ev[s]) (void)hipEventDestroy(e);
  }
  for (hipGraphExec_t g : pr->gexec)
    if (g) (void)hipGraphExecDestroy(g);
  if (pr->h_out && pr->own_out) (void)hipHostFree(pr->h_out);
  if (pr->h_ed) (void)hipHostFree(pr->h_ed);
  for (hipEvent_t e : pr->d2h_ev) (void)hipEventDestroy(e);
  delete pr;
}

}  // namespace snc
