// Host runtime of the two baselines (standard and pre-computation permutation tests) and of
// the HSIC independence test (see include/etest.h).
#include "runtime.h"

#include <algorithm>
#include <cmath>
#include <string>

using namespace et;

// ------------------------------------------------- baselines: standard and pre-computation
namespace et {

// Free the workspaces, wait for the result that the last kernel wrote to pinned memory.
static etest_status finish_baseline(const DevResult* h, Batch* b, void* aux, hipStream_t st,
                                    hipError_t e, const char* what, etest_result* out,
                                    const Fork* fork = nullptr) {
  if (e == hipSuccess) e = hipGetLastError();
  free_batch(b, st, true);
  if (aux) (void)hipFreeAsync(aux, st);
  e = finish_stream(st, e, fork);
  if (e != hipSuccess) return set_error(ETEST_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
  return dev_to_result(*h, out);
}

// Standard test: the pooled rows are staged once, in their own order (every split centres on
// the same pooled mean); the B + 1 splits (drawn splits 0..B-1, identity B) are recomputed in
// passes of up to 256 tests, each reading its X*, Y* through a row map: Gram, tile sums, block
// sums and observed statistic.  (Staging every split's rows again, and storing its blocks, took
// 250 us and half of the Gram's 517 us of a 930 us test of 500 + 500 rows, p = 500, B = 200.)
static etest_status run_standard(const etest_request& r, hipStream_t st, etest_result* out) {
  init_pool_once();
  const int64_t n = r.nx + r.ny, W = (n + 31) / 32, B = r.B;
  etest_request q = r;
  q.B = 0;
  q.perm_stats = nullptr;
  Batch sb;
  sb.plans.push_back(make_plan(q, 0, PLAN_STAGE));
  TestPlan P0 = make_plan(q, 0, PLAN_SUMS);
  etest_status s = check_launch_sizes(&P0, 1);
  if (s != ETEST_OK) return s;
  // a pass holds at most 4 GiB of sums and 2^20 tiles (its Gram is one launch)
  const int64_t budget = 4LL << 30;
  const int64_t chunk = std::max<int64_t>(
      1, std::min<int64_t>({B + 1, 256, budget / std::max<int64_t>(1, (int64_t)P0.bytes),
                            (1 << 20) / P0.d.ntiles}));
  size_t aoff[4], asz[4] = {(size_t)(chunk * n * 4), (size_t)(chunk * W * 4),
                            (size_t)((B + 1) * 8), (size_t)(FLAG_WORDS * 4)};
  size_t atotal = 0;
  for (int k = 0; k < 4; ++k) {
    aoff[k] = atotal;
    atotal += align256(asz[k]);
  }
  DevResult* res = pinned_results(1);
  if (!res) return set_error(ETEST_ENOMEM, "pinned result buffer");
  void* aux = nullptr;
  hipError_t e = hipMallocAsync(&aux, atotal, st);
  if (e != hipSuccess || !aux) {
    (void)hipGetLastError();
    return set_error(ETEST_ENOMEM, "standard test buffers of " + std::to_string(atotal) + " bytes");
  }
  char* a = (char*)aux;
  int32_t* rowmaps = (int32_t*)(a + aoff[0]);
  uint32_t* words = (uint32_t*)(a + aoff[1]);
  double* stats = (double*)(a + aoff[2]);
  int32_t* flags = (int32_t*)(a + aoff[3]);
  Batch b;
  sb.desc_by_kernel = true;
  b.desc_pinned = true;
  s = place_batch(&sb, st, true);
  if (s == ETEST_OK) {
    P0.staged = &sb.descs[0];
    b.plans.assign((size_t)chunk, P0);
    for (int64_t k = 0; k < chunk; ++k) b.plans[(size_t)k].d.rowmap = rowmaps + k * n;
    s = place_batch(&b, st, true);
    if (s != ETEST_OK) free_batch(&sb, st, true);
  }
  if (s != ETEST_OK) {
    (void)hipFreeAsync(aux, st);
    (void)finish_stream(st, hipSuccess);
    return s;
  }
  {
    auto offs = [&](Slot k) { return sb.d_offs + (size_t)k * 2; };
    auto total = [&](Slot k) { return sb.offs[(size_t)k * 2 + 1]; };
    launch_colpart(total(S_COLPART), st, sb.d_descs, offs(S_COLPART), 1);
    launch_colmean(total(S_COLMEAN), st, sb.d_descs, offs(S_COLMEAN), 1);
    launch_stage(total(S_STAGE), st, sb.d_descs, offs(S_STAGE), 1);
  }
  const int gop = P0.d.gop;
  const Slot gram = gop == GOP_F64 ? S_GRAM_F64 : gop == GOP_F16PAIR ? S_GRAM_F32 : S_GRAM_BF16;
  auto offs = [&](Slot k) { return b.d_offs + (size_t)k * (chunk + 1); };
  const TestDesc* D = b.d_descs;
  e = hipMemsetAsync(flags, 0, FLAG_WORDS * 4, st);
  for (int64_t c0 = 0; e == hipSuccess && c0 <= B; c0 += chunk) {
    const int m = (int)std::min<int64_t>(chunk, B + 1 - c0);
    const int64_t drawn = std::max<int64_t>(0, std::min<int64_t>(m, B - c0));
    // the launch tables of a prefix of the tests are prefixes of the batch's tables
    auto total = [&](Slot k) { return b.offs[(size_t)k * (chunk + 1) + m]; };
    launch_member_public(r.nx, r.ny, r.seed, c0, drawn, words, st);
    launch_rowmap(words, drawn, m, n, r.nx, rowmaps, st);
    launch_sum_flags(D, m, sb.descs[0].flags, st);
    launch_gram_sums(gop, total(gram), st, D, offs(gram), m);
    launch_rowsum(total(S_ROWSUM), st, D, offs(S_ROWSUM), m);
    launch_observed(st, D, nullptr, m);
    launch_collect(D, m, c0, B, stats, flags, st);
    e = hipGetLastError();
  }
  if (e == hipSuccess) launch_count(stats, B, flags, r.perm_stats, res, st);
  free_batch(&sb, st, true);
  return finish_baseline(res, &b, aux, st, e, "standard test", out);
}

// Pre-computation test: the pooled Gram (D_WW: upper tiles, or with `dense` the whole
// nt x nt grid as Alg. 5 prints it), the split stream, then the per-split class sums of
// every stored entry and the statistics.
// Stage timing (etest_profile_enable): 0 staging, 1 blocks, 2 split stream, 5 class sums,
// 6 statistics + p-value.
static etest_status run_precomputed(const etest_request& r, hipStream_t st, etest_result* out,
                                    bool dense) {
  init_pool_once();
  Batch b;
  b.plans.push_back(make_plan(r, 0, dense ? PLAN_PRECOMP_DENSE : PLAN_PRECOMP));
  // one workgroup per (stored tile, 32-row strip, 64 split columns)
  const int64_t groups = (r.B + 1 + 63) / 64;
  if ((int64_t)b.plans[0].d.ntiles * PC_STRIPS > 2147483647LL / groups)
    return set_error(ETEST_EINVAL, "pre-computation test: tiles x strips x split groups must "
                                   "stay below 2^31");
  DevResult* res = pinned_results(1);
  if (!res) return set_error(ETEST_ENOMEM, "pinned result buffer");
  b.desc_by_kernel = true;
  etest_status s = place_batch(&b, st, true);
  if (s != ETEST_OK) {
    (void)finish_stream(st, hipSuccess);
    return s;
  }
  const TestDesc& d = b.descs[0];
  const TestDesc* D = b.d_descs;
  auto offs = [&](Slot k) { return b.d_offs + (size_t)k * 2; };
  auto total = [&](Slot k) { return b.offs[(size_t)k * 2 + 1]; };
  const StageEvents* ev = profile_events();
  // the split stream needs neither the data nor its blocks: beside them, as in the permutation
  // test (1000 + 1000 x 500, 200 splits: 149 us on one stream, of which it took 32)
  const Fork* fork = batch_fork(b, false);
  hipStream_t ms = fork ? fork->aux : st;
  auto mark = [&](int k, bool begin) {
    if (ev && (ev->mask >> k & 1u))
      (void)hipEventRecord(begin ? ev->begin[k] : ev->end[k], k == 2 ? ms : st);
  };
  if (fork) {
    (void)hipEventRecord(fork->start, st);
    (void)hipStreamWaitEvent(ms, fork->start, 0);
  }
  mark(2, true);
  launch_member(total(S_MEMBER), ms, D, offs(S_MEMBER), 1);
  mark(2, false);
  if (fork) (void)hipEventRecord(fork->done, ms);
  mark(0, true);
  launch_colpart(total(S_COLPART), st, D, offs(S_COLPART), 1);
  launch_colmean(total(S_COLMEAN), st, D, offs(S_COLMEAN), 1);
  launch_stage(total(S_STAGE), st, D, offs(S_STAGE), 1);
  mark(0, false);
  mark(1, true);
  launch_gram_slots(offs, total, st, D, 1, false);
  mark(1, false);
  if (fork) (void)hipStreamWaitEvent(st, fork->done, 0);
  mark(5, true);
  launch_precomp(r.prec == ETEST_PREC_F64, D, d.ntiles, r.B, d.part, st);
  mark(5, false);
  mark(6, true);
  launch_precomp_stat(D, d.ntiles, r.B, d.part, d.pstat, st);
  launch_count(d.pstat, r.B, d.flags, r.perm_stats, res, st);
  mark(6, false);
  etest_status rs = finish_baseline(res, &b, nullptr, st, hipSuccess, "pre-computation test", out,
                                    fork);
  profile_collect();
  return rs;
}

// HSIC independence test: the Gaussian kernel matrices of x and of y as two one-sample Grams
// in one batch (staging and blocks only), then dense zero-diagonal copies, row sums, the
// permutations, the per-permutation terms, the statistics and the p-value.
// Stage timing (etest_profile_enable): 0 staging, 1 blocks, 2 permutations, 3 dense
// matrices and row sums, 5 per-permutation terms, 6 statistics + p-value.
static etest_status run_hsic(const etest_hsic_request& h, hipStream_t st, etest_result* out) {
  init_pool_once();
  const int64_t n = h.n, B = h.B, nperm = h.B + 1;
  const bool f64 = h.prec == ETEST_PREC_F64;
  etest_request rx{}, ry{};
  rx.kind = ry.kind = ETEST_MMD;
  rx.prec = ry.prec = h.prec;
  rx.nx = ry.nx = n;
  rx.ny = ry.ny = 0;  // one sample: the Gram covers the x (or y) rows alone
  rx.p = h.p;
  ry.p = h.q;
  rx.gamma = h.gamma_x;
  ry.gamma = h.gamma_y;
  rx.X = rx.Y = h.X;
  ry.X = ry.Y = h.Y;
  Batch b;
  b.plans.push_back(make_plan(rx, 0, PLAN_BLOCKS));
  b.plans.push_back(make_plan(ry, 0, PLAN_BLOCKS));
  const size_t el = f64 ? 8 : 4;
  const int64_t ld = (n + 255) / 256 * 256, nparts = hsic_parts(f64, n);
  // Permutations go in passes whose tables and partial sums take at most 1 GiB.
  const int64_t pass = std::min<int64_t>(
      nperm, std::max<int64_t>(64, ((int64_t)1 << 30) / (4 * ld + 8 * nparts)));
  enum { H_KX, H_RX, H_RY, H_HS, H_FLAGS, H_PERMS, H_INV, H_PART, H_STATS, H_N };
  size_t sz[H_N] = {(size_t)(n * ld) * el, (size_t)n * 8, (size_t)n * 8, 2 * 8, FLAG_WORDS * 4,
                    (size_t)(pass * ld) * 2, (size_t)(pass * ld) * 2, (size_t)(pass * nparts) * 8,
                    (size_t)nperm * 8};
  size_t off[H_N], total = 0;
  for (int k = 0; k < H_N; ++k) {
    off[k] = total;
    total += align256(sz[k]);
  }
  DevResult* res = pinned_results(1);
  if (!res) return set_error(ETEST_ENOMEM, "pinned result buffer");
  void* aux = nullptr;
  hipError_t e = hipMallocAsync(&aux, total, st);
  if (e != hipSuccess || !aux) {
    (void)hipGetLastError();
    return set_error(ETEST_ENOMEM, "HSIC test buffers of " + std::to_string(total) + " bytes");
  }
  char* a = (char*)aux;
  b.desc_pinned = true;
  etest_status s = place_batch(&b, st, true);
  if (s != ETEST_OK) {
    (void)hipFreeAsync(aux, st);
    (void)finish_stream(st, hipSuccess);
    return s;
  }
  double* rxs = (double*)(a + off[H_RX]);
  double* rys = (double*)(a + off[H_RY]);
  double* hs = (double*)(a + off[H_HS]);
  int32_t* flags = (int32_t*)(a + off[H_FLAGS]);
  uint16_t* p16 = (uint16_t*)(a + off[H_PERMS]);
  uint16_t* inv16 = (uint16_t*)(a + off[H_INV]);
  double* part = (double*)(a + off[H_PART]);
  double* stats = (double*)(a + off[H_STATS]);
  const TestDesc* D = b.d_descs;
  auto offs = [&](Slot k) { return b.d_offs + (size_t)k * 3; };
  auto tot = [&](Slot k) { return b.offs[(size_t)k * 3 + 2]; };
  const StageEvents* ev = profile_events();
  // the first pass's permutations need neither the data nor the kernels: beside them (2000 pairs,
  // 200 permutations: 41 us of a 365 us test in line)
  const Fork* fork = batch_fork(b, false);
  hipStream_t ms = fork ? fork->aux : st;
  auto mark = [&](int k, bool begin) {
    if (ev && (ev->mask >> k & 1u))
      (void)hipEventRecord(begin ? ev->begin[k] : ev->end[k], k == 2 ? ms : st);
  };
  auto perms = [&](int64_t c0, hipStream_t s) {
    const int64_t m = std::min(pass, nperm - c0);
    launch_hsic_perms(n, ld, h.seed, c0, std::min(m, B - c0), m, p16, inv16, s);
  };
  if (fork) {
    (void)hipEventRecord(fork->start, st);
    (void)hipStreamWaitEvent(ms, fork->start, 0);
  }
  mark(2, true);
  perms(0, ms);
  mark(2, false);
  if (fork) (void)hipEventRecord(fork->done, ms);
  launch_clear_flags(st, D, nullptr, 2);
  mark(0, true);
  launch_colpart(tot(S_COLPART), st, D, offs(S_COLPART), 2);
  launch_colmean(tot(S_COLMEAN), st, D, offs(S_COLMEAN), 2);
  launch_stage(tot(S_STAGE), st, D, offs(S_STAGE), 2);
  mark(0, false);
  mark(1, true);
  launch_gram_slots(offs, tot, st, D, 2, false);
  mark(1, false);
  mark(3, true);
  launch_hsic_prep(f64, D, b.descs[0].nt, n, ld, a + off[H_KX], rxs, rys, hs, flags, st);
  mark(3, false);
  if (fork) (void)hipStreamWaitEvent(st, fork->done, 0);
  for (int64_t c0 = 0; c0 < nperm; c0 += pass) {
    const int64_t m = std::min(pass, nperm - c0);
    const bool first = c0 == 0, last = c0 + m == nperm;  // stage events: the first pass's
    if (!first) perms(c0, st);
    if (first) mark(5, true);
    launch_hsic_terms(f64, D, a + off[H_KX], n, ld, p16, inv16, m, part, st);
    if (first) mark(5, false);
    if (last) mark(6, true);
    launch_hsic_stat(part, nparts, n, ld, p16, rxs, rys, m, hs, stats + c0, st);
  }
  launch_count(stats, B, flags, h.perm_stats, res, st);
  mark(6, false);
  etest_status rs = finish_baseline(res, &b, aux, st, hipSuccess, "HSIC test", out, fork);
  profile_collect();
  return rs;
}

static etest_status validate_hsic(const etest_hsic_request& h) {
  // The unbiased HSIC is a small difference of three large terms (on high-dimensional data
  // about 1e-5 of the kernel entries under independence): 8-bit coordinates cannot carry it,
  // so the test has the FP64 and FP32 forms only.
  if (h.prec != ETEST_PREC_F64 && h.prec != ETEST_PREC_F32)
    return set_error(ETEST_EINVAL, "HSIC test: prec must be ETEST_PREC_F64 or ETEST_PREC_F32");
  if (h.n < 4 || h.n > HSIC_NMAX)
    return set_error(ETEST_EINVAL, "HSIC test needs 4 <= n <= " + std::to_string(HSIC_NMAX));
  if (h.p < 1 || h.q < 1 || h.p > 2147483647LL || h.q > 2147483647LL)
    return set_error(ETEST_EINVAL, "p and q must be >= 1");
  if (h.B < 0 || h.B >= 2147483647LL) return set_error(ETEST_EINVAL, "B out of range");
  if (!(h.gamma_x > 0.0) || !(h.gamma_y > 0.0) || !std::isfinite(h.gamma_x) ||
      !std::isfinite(h.gamma_y))
    return set_error(ETEST_EINVAL, "gamma_x and gamma_y must be finite and > 0");
  if (!h.X || !h.Y) return set_error(ETEST_EINVAL, "X and Y must not be NULL");
  if (h.reserved != 0) return set_error(ETEST_EINVAL, "reserved field must be 0");
  // bound on the work of one call: (permutation, block of HSIC_RB rows) pairs
  const int64_t nblk = (h.n + HSIC_RB - 1) / HSIC_RB;
  if ((h.B + 1) > 2147483647LL / nblk)
    return set_error(ETEST_EINVAL, "HSIC test: (B + 1) * ceil(n / " + std::to_string(HSIC_RB) +
                                       ") must stay below 2^31");
  return ETEST_OK;
}

}  // namespace et

extern "C" {

etest_status etest_hsic(const etest_hsic_request* req, void* stream, etest_result* out) {
  if (!req || !out) return set_error(ETEST_EINVAL, "NULL argument");
  etest_status s = validate_hsic(*req);
  if (s != ETEST_OK) return s;
  return run_hsic(*req, (hipStream_t)stream, out);
}

etest_status etest_permutations(int64_t n, uint64_t seed, int64_t b0, int64_t count,
                                int32_t* perms, void* stream) {
  if (n < 1 || n > HSIC_NMAX) return set_error(ETEST_EINVAL, "permutations need 1 <= n <= " + std::to_string(HSIC_NMAX));
  if (b0 < 0 || count < 0 || !perms) return set_error(ETEST_EINVAL, "bad range or NULL perms");
  hipStream_t st = (hipStream_t)stream;
  launch_permgen(n, seed, b0, count, count, perms, st);
  HIP_OK(finish_stream(st, hipGetLastError()), "permutations");
  return ETEST_OK;
}

etest_status etest_standard(const etest_request* req, void* stream, etest_result* out) {
  if (!req || !out) return set_error(ETEST_EINVAL, "NULL argument");
  etest_status s = validate_request(*req);
  if (s != ETEST_OK) return s;
  return run_standard(*req, (hipStream_t)stream, out);
}

etest_status etest_precomputed(const etest_request* req, void* stream, etest_result* out) {
  if (!req || !out) return set_error(ETEST_EINVAL, "NULL argument");
  etest_status s = validate_request(*req);
  if (s != ETEST_OK) return s;
  return run_precomputed(*req, (hipStream_t)stream, out, false);
}

etest_status etest_precomputed_dense(const etest_request* req, void* stream, etest_result* out) {
  if (!req || !out) return set_error(ETEST_EINVAL, "NULL argument");
  etest_status s = validate_request(*req);
  if (s != ETEST_OK) return s;
  return run_precomputed(*req, (hipStream_t)stream, out, true);
}

}  // extern "C"
