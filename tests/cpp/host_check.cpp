// Host runtime checked without a device, one check per argument (see fake_hip.h).
#include <functional>

#include "fake_hip.h"

using namespace et;

static char sample[8];  // stands for device inputs, which only kernels read

static etest_request request(int prec, int64_t n, int64_t B, int kind = ETEST_ED) {
  etest_request r{};
  r.kind = kind;
  r.prec = prec;
  r.nx = r.ny = n;
  r.p = 20;
  r.B = B;
  r.gamma = 0.1;
  r.X = r.Y = sample;
  return r;
}

// Every call that waits, on stream st: 1600 pooled rows, so that the split stream is forked.
struct Call {
  std::string name;
  std::function<etest_status(hipStream_t)> run;
};
static std::vector<Call> waiting_calls() {
  static std::vector<char> words(1 << 16);
  std::vector<Call> v;
  for (int prec : {ETEST_PREC_F64, ETEST_PREC_F32, ETEST_PREC_BF16_REFINED}) {
    const std::string p = " prec " + std::to_string(prec);
    const etest_request r = request(prec, 800, 300), small = request(prec, 100, 20);
    auto one = [&](const char* name, etest_status (*f)(const etest_request*, void*, etest_result*)) {
      v.push_back({name + p, [=](hipStream_t st) { etest_result o; return f(&r, st, &o); }});
    };
    one("run", etest_run);
    one("precomputed", etest_precomputed);
    one("precomputed_dense", etest_precomputed_dense);
    one("standard", etest_standard);
    v.push_back({"cross" + p, [=](hipStream_t st) { etest_cross_result o; return etest_cross(&r, st, &o); }});
    v.push_back({"blocks" + p, [=](hipStream_t st) {
      return etest_blocks(&small, words.data(), words.data(), words.data(), st);
    }});
    v.push_back({"from_membership" + p, [=](hipStream_t st) {
      etest_result o;
      return etest_perm_stats_from_membership(&r, (uint32_t*)words.data(), 40, (double*)words.data(), st, &o);
    }});
    v.push_back({"batch" + p, [=](hipStream_t st) {
      const etest_request q[2] = {r, small};
      etest_result o[2];
      return etest_batch(q, 2, st, o);
    }});
    v.push_back({"timed batch" + p, [=](hipStream_t st) {
      const etest_request q[2] = {r, small};
      etest_result o[2];
      etest_profile_enable(1);
      const etest_status s = etest_batch(q, 2, st, o);
      etest_profile_enable(0);
      return s;
    }});
  }
  for (int prec : {ETEST_PREC_F64, ETEST_PREC_F32})
    v.push_back({"hsic prec " + std::to_string(prec), [=](hipStream_t st) {
      etest_hsic_request h{};
      h.prec = prec;
      h.n = 1600;
      h.p = h.q = 20;
      h.B = 50;
      h.gamma_x = h.gamma_y = 0.1;
      h.X = h.Y = sample;
      etest_result o;
      return etest_hsic(&h, st, &o);
    }});
  v.push_back({"membership", [=](hipStream_t st) {
    return etest_membership(100, 100, 1, 0, 10, (uint32_t*)words.data(), st);
  }});
  v.push_back({"permutations", [=](hipStream_t st) {
    return etest_permutations(100, 1, 0, 10, (int32_t*)words.data(), st);
  }});
  return v;
}

// Runs f once with each of its fallible HIP calls failing in turn, then as it is.
static void each_failure(const Call& c, hipStream_t st, const std::function<void(int64_t, etest_status)>& f) {
  for (int64_t k = 1;; ++k) {
    fake::calls = 0;
    fake::fail_at = k;
    fake::last = hipSuccess;
    const etest_status s = c.run(st);
    const bool reached = fake::calls >= k;
    fake::fail_at = -1;
    f(reached ? k : 0, s);
    hipDeviceSynchronize();
    if (!reached) return;
  }
}

// A call that waits leaves nothing in flight, also where it fails: its kernels read the
// caller's buffers and write the thread's pinned result, which the next call uses.
static void check_failed_calls_wait() {
  hipStream_t st;
  hipStreamCreateWithFlags(&st, 0);
  for (const Call& c : waiting_calls())
    each_failure(c, st, [&](int64_t k, etest_status s) {
      CHECK(fake::in_flight() == 0, "%s: %d launches in flight, failure %d, status %d", c.name.c_str(),
            fake::in_flight(), (int)k, (int)s);
      CHECK(k > 0 || s == ETEST_OK, "%s: status %d: %s", c.name.c_str(), (int)s, etest_last_error());
    });
}

// A call that fails frees its workspaces; up to four graphs keep theirs.
static void check_failed_calls_free() {
  hipStream_t st;
  hipStreamCreateWithFlags(&st, 0);
  std::vector<Call> calls = waiting_calls();
  for (int64_t n : {100, 800})
    calls.push_back({"async", [=](hipStream_t s) {
      const etest_request r = request(ETEST_PREC_F32, n, 100);
      etest_result o;
      return ed_test_async(&r, &o, s);
    }});
  calls.push_back({"async batch", [=](hipStream_t s) {
    const etest_request q[2] = {request(ETEST_PREC_F32, 100, 20), request(ETEST_PREC_F64, 800, 20)};
    etest_result o[2];
    return etest_batch_async(q, 2, s, o);
  }});
  for (const Call& c : calls)
    each_failure(c, st, [&](int64_t k, etest_status s) {
      CHECK(fake::ordered.empty(), "%s: %d workspaces kept, failure %d, status %d", c.name.c_str(),
            (int)fake::ordered.size(), (int)k, (int)s);
      // and one per (device, stream) of the asynchronous calls
      CHECK(fake::plain.size() <= 5, "%s: %d held, failure %d, status %d", c.name.c_str(),
            (int)fake::plain.size(), (int)k, (int)s);
    });
}

// One thread, two devices in turn, the null stream of each: every launch, record and replay is
// on the current device, and no call fails for having run on the other one before.
static void check_two_devices(const std::set<std::string>& names) {
  for (int pass = 0; pass < 3; ++pass) {
    fake::device = pass % 2;
    for (const Call& c : waiting_calls()) {
      if (!names.count(c.name.substr(0, c.name.find(" prec")))) continue;
      const etest_status s = c.run(nullptr);
      CHECK(s == ETEST_OK, "%s on device %d: %s", c.name.c_str(), fake::device, etest_last_error());
      CHECK(fake::other_device == 0, "%s on device %d used the other", c.name.c_str(), fake::device);
      fake::other_device = 0;
      hipDeviceSynchronize();
    }
  }
}
static void check_fork_of_two_devices() {
  check_two_devices({"run", "from_membership", "precomputed", "precomputed_dense", "cross", "blocks"});
}

static void check_staging_of_two_devices() { check_two_devices({"standard", "hsic"}); }
static void check_graphs_of_two_devices() {
  check_two_devices({"batch"});
  // graphs in flight on one device, put out of the cache by calls on the other
  for (int k = 0; k < 8; ++k) {
    fake::device = k / 4;
    const etest_request r = request(ETEST_PREC_F32, 50 + k, 20);
    etest_result o;
    CHECK(etest_batch_async(&r, 1, nullptr, &o) == ETEST_OK, "async batch %d", k);
  }
  CHECK(fake::destroyed_in_flight == 0, "%d graphs destroyed in flight", fake::destroyed_in_flight);
}
static void check_timing_of_two_devices() { check_two_devices({"timed batch"}); }

// What every mode's kernels write lies in the plan's buffers: tile sums (6 TILE doubles a tile in
// the FP64 form, 3 TILE else, at the descriptor's stride), the buffers a mode leaves out, and the
// rows that a recomputation of the standard test reads from another plan.
static void check_plan_buffers() {
  const int64_t sizes[][3] = {{1, 1, 1}, {128, 128, 20}, {129, 300, 33}, {700, 90, 500}, {5000, 4000, 64}};
  for (int prec : {ETEST_PREC_F64, ETEST_PREC_F32, ETEST_PREC_BF16_REFINED})
    for (const auto& z : sizes)
      for (int mode = PLAN_EFFICIENT; mode <= PLAN_SUMS; ++mode) {
        const bool f64 = prec == ETEST_PREC_F64;
        etest_request r = request(prec, z[0], mode == PLAN_STAGE || mode == PLAN_SUMS ? 0 : 300);
        r.ny = z[1];
        r.p = z[2];
        TestPlan stage = make_plan(r, 0, PLAN_STAGE), P = make_plan(r, 0, mode);
        char* at = (char*)(uintptr_t)(1 << 20);
        assign_pointers(stage, at + ((size_t)1 << 40), nullptr);
        if (mode == PLAN_SUMS) P.staged = &stage.d;
        assign_pointers(P, at, nullptr);
        const TestDesc& d = P.d;
        char what[96];
        std::snprintf(what, sizeof what, "prec %d mode %d, %d + %d x %d", prec, mode, d.nx, d.ny, d.p);
        auto inside = [&](const void* p, size_t bytes, int buf) {
          const size_t o = (size_t)((const char*)p - at);
          return o >= P.off[buf] && o + bytes <= P.off[buf] + P.size[buf];
        };
        const size_t tile = f64 ? 8 : 4, npad = (size_t)d.nt * TILE;
        const size_t rows = npad * d.p_pad * gram_operand_bytes(d.gop);
        int64_t gram = 0, stagers = 0;
        for (int k : GRAM_SLOTS)
          if (k != S_GRAM_FIN) gram += P.wg[k];
        for (int k : {S_COLPART, S_COLMEAN, S_STAGE}) stagers += P.wg[k];
        CHECK((gram > 0) == (mode != PLAN_STAGE) && (stagers > 0) == (mode != PLAN_SUMS), "%s", what);
        if (mode == PLAN_SUMS) {
          CHECK(d.D == nullptr && d.W == stage.d.W && d.nrm == stage.d.nrm, "%s", what);
          CHECK(d.gather == 1 && d.gshape == GSHAPE_TILE && gram == d.ntiles, "%s", what);
          CHECK(P.size[B_D] + P.size[B_W] + P.size[B_NRM] + P.size[B_COLPART] + P.size[B_PLANES] == 0, "%s", what);
        } else {
          CHECK(d.gather == 0 && inside(d.W, rows, B_W) && inside(d.nrm, npad * tile, B_NRM), "%s", what);
          CHECK(f64 || (inside(d.colpart, (size_t)d.nrowchunks * d.p * 8, B_COLPART) &&
                        inside(d.colmean, (size_t)d.p * 8, B_COLMEAN)), "%s", what);
        }
        CHECK(inside(d.flags, FLAG_WORDS * 4, B_FLAGS), "%s", what);
        if (mode == PLAN_STAGE) {
          CHECK(P.size[B_D] + P.size[B_TSUM] + P.size[B_PLANES] == 0 && P.wg[S_ROWSUM] == 0, "%s", what);
          continue;
        }
        const size_t sums = ((size_t)(d.ntiles - 1) * d.tsum_stride + (f64 ? 6 : 3) * TILE) * 8;
        CHECK(d.tsum_stride >= (f64 ? 6 : 3) * TILE, "%s: stride %d", what, (int)d.tsum_stride);
        CHECK(inside(d.tsum, sums, f64 && mode == PLAN_EFFICIENT ? B_PLANES : B_TSUM), "%s: tile sums", what);
        CHECK(inside(d.tmax, (size_t)d.ntiles * TMAX_PER_TILE * 4, B_TMAX), "%s", what);
        if (mode != PLAN_SUMS) CHECK(inside(d.D, (size_t)d.ntiles * TILE * TILE * tile, B_D), "%s", what);
        if (P.wg[S_ROWSUM]) CHECK(inside(d.rsum, npad * 16, B_RSUM) && inside(d.obs, 64, B_OBS), "%s", what);
      }
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> checks = {
      {"failed_calls_wait", check_failed_calls_wait},
      {"failed_calls_free", check_failed_calls_free},
      {"fork_of_two_devices", check_fork_of_two_devices},
      {"staging_of_two_devices", check_staging_of_two_devices},
      {"graphs_of_two_devices", check_graphs_of_two_devices},
      {"timing_of_two_devices", check_timing_of_two_devices},
      {"plan_buffers", check_plan_buffers},
  };
  for (int k = 1; k < argc; ++k) checks.at(argv[k])();
  if (!fake::failures) std::printf("ok\n");
  return fake::failures ? 1 : 0;
}
