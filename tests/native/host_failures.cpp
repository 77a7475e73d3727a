// The host side of libnetsim (netsim.cpp) with every runtime call and kernel
// launch of a first run, a second run and an advance made to fail in turn, on the stand-in
// runtime of tests/native/runtime (the launches only queue work).  After a
// call that fails
//   join   no work it queued is still running: the caller may use the
//          handle's state on another stream at once;
//   keep   the next call succeeds, and does not go on from parts that the wave
//          kernel left in the middle of an event for a launch that never came;
//          destroying the handle leaves no device or pinned memory, stream or
//          event behind.
// Run by tests/test_native_checks.py.
#include <hip/hip_runtime.h>

#include <vector>

#include "device.h"
#include "netsim.h"

FakeHip fake;

// The wave kernel may have left parts in the middle of an event.
static bool in_event = false;
static hipError_t wave(hipStream_t s) {
  if (in_event) FakeHip::bug("a part left in the middle of an event is run from its start");
  const hipError_t e = fake.work(s);
  in_event = e == hipSuccess;
  return e;
}
static hipError_t workgroups(const netsim_dev::Params& P, hipStream_t s) {
  const hipError_t e = fake.work(s);
  if (e == hipSuccess && P.hand) in_event = false;
  return e;
}

namespace netsim_dev {
hipError_t launch_reset(const Params& P, const Initial& I, int64_t, int64_t, int NP, bool, hipStream_t s) {
  const hipError_t e = fake.work(s);
  if (e == hipSuccess) memcpy(P.ctl, I.ctl, sizeof(ScenCtl) * (size_t)NP);
  if (e == hipSuccess) in_event = false;
  return e;
}
hipError_t launch_reset_words(const Params&, const Results&, int, hipStream_t s) { return fake.work(s); }
hipError_t launch_releases(const Params&, int, int, hipStream_t s) { return fake.work(s); }
hipError_t launch_results(const Params&, const Results&, const int32_t*, const int32_t*, int64_t, hipStream_t s) {
  return fake.work(s);
}
hipError_t launch_count_active(const Params&, const int32_t*, int, hipStream_t s) { return fake.work(s); }
hipError_t launch_gather_rates(const Params&, const int32_t*, int, double*, hipStream_t s) { return fake.work(s); }
hipError_t launch_block(const Params& P, int, int, hipStream_t s) { return workgroups(P, s); }
hipError_t launch_solve(const Params&, int, int, hipStream_t s) { return fake.work(s); }
hipError_t launch_wave(const Params&, const int32_t*, int, int, int, size_t, hipStream_t s) { return wave(s); }
size_t wave_bytes(int nl, int, int sc, int pc) { return 38 * (size_t)nl + 76 * (size_t)sc + 12 * (size_t)pc; }
hipError_t launch_xwave(const Params&, const int32_t*, int, int, int, size_t, hipStream_t s) { return wave(s); }
size_t xwave_bytes(int nl, int sc, int pc) { return 34 * (size_t)nl + 62 * (size_t)sc + 12 * (size_t)pc; }
hipError_t launch_grid(const Params&, int, int, hipStream_t s) { return fake.work(s); }
hipError_t grid_capacity(int, int, int* blocks) {
  *blocks = 256;
  return hipSuccess;
}
hipError_t launch_cluster(const Params&, int, hipStream_t s) { return fake.work(s); }
hipError_t cluster_capacity(int, int* blocks) {
  *blocks = 256;
  return hipSuccess;
}
hipError_t launch_exact(const Params& P, int, int, hipStream_t s) { return workgroups(P, s); }
hipError_t history_restore(const Params&, int, int, int, int64_t, int64_t, int32_t, const HistEv&, int64_t,
                           const int32_t*, const double*, int32_t*, uint32_t*, hipStream_t s) {
  return fake.work(s);
}
int exact_link_bytes() { return 24; }
hipError_t grid_solve_begin(const Params&, const ScenCtl&, int, hipStream_t s) { return fake.work(s); }
hipError_t grid_solve_count(const Params&, const ScenCtl&, int, int, hipStream_t s, unsigned long long*) {
  return fake.work(s);
}
hipError_t grid_solve_links(const Params&, const ScenCtl&, int, hipStream_t s) { return fake.work(s); }
hipError_t grid_solve_freeze(const Params&, const ScenCtl&, int, int, hipStream_t s, unsigned long long*) {
  return fake.work(s);
}
bool grid_solve_fill_fits(const ScenCtl&) { return true; }
hipError_t grid_solve_fill(const Params&, const ScenCtl&, int, int, hipStream_t s) { return fake.work(s); }
int count_blocks(int, int) { return 1; }
int freeze_blocks(int) { return 1; }
hipError_t launch_flush(void*, size_t, uint32_t, hipStream_t s) { return fake.work(s); }
}  // namespace netsim_dev

// Two scenarios: one whose 300 flows start together (a workgroup's), one of
// 600 flows of which 10 start (a wave's, which may hand it over); `wide`
// flows more in the first (results in pinned memory).
static netsim_t* make(const netsim_options& opt, int wide) {
  const int64_t off[3] = {0, 4, 8};
  const double cap[8] = {1, 2, 3, 4, 5, 6, 7, 8};
  netsim_t* h = nullptr;
  if (netsim_create(&h, 2, off, cap, &opt) != NETSIM_OK) FakeHip::bug("create");
  for (int s = 0; s < 2; ++s) {
    const int n = s == 0 ? 300 + wide : 600, roots = s == 0 ? n : 10;
    const int64_t base = s == 0 ? 0 : 300 + wide;
    std::vector<double> bytes(n, 1.0), start(n, 0.0);
    std::vector<int64_t> po(n + 1), dep(n + 1, 0), ids;
    std::vector<int32_t> pl(n);
    for (int i = 0; i < n; ++i) {
      po[i + 1] = i + 1;
      pl[i] = i % 4;
      if (i >= roots) ids.push_back(base + i % roots);
      dep[i + 1] = (int64_t)ids.size();
    }
    if (netsim_add_flows(h, s, n, nullptr, nullptr, bytes.data(), start.data(), po.data(), pl.data(), dep.data(),
                         ids.data(), nullptr) != NETSIM_OK)
      FakeHip::bug("add_flows");
  }
  return h;
}

static int bad = 0;
static void expect(bool ok, const char* what, const char* mode, long at) {
  if (ok) return;
  ++bad;
  printf("%s: %s (call %ld made to fail)\n", mode, what, at);
}

int main(int argc, char** argv) {
  const bool join = argc > 1 && !strcmp(argv[1], "join");
  const struct { const char* name; int exact, history, wide; } modes[] = {
      {"default", 0, 0, 0}, {"exact", 1, 0, 0}, {"history", 0, 1, 0}, {"pinned results", 0, 0, 40000}};
  long tried = 0;
  for (const auto& m : modes) {
    netsim_options opt;
    netsim_default_options(&opt);
    opt.single_clock = 1;  // one part a scenario: one launch of the wave kernel
    opt.exact = m.exact;
    opt.history_mb = m.history;
    opt.exec = m.exact ? NETSIM_EXEC_AUTO : NETSIM_EXEC_BLOCK;
    for (int run = 0; run < 3; ++run)  // the first run (preparation), a later one, a later advance
      for (long at = 1;; ++at) {
        fake.fail_at = 0;
        netsim_t* h = make(opt, m.wide);
        ihipStream own;
        fake.streams.insert(&own);
        if (run && netsim_run(h, &own) != NETSIM_OK) FakeHip::bug("a run without failures");
        auto go = [&] { return run < 2 ? netsim_run(h, &own) : netsim_advance(h, 1e9, 0, &own); };
        fake.calls = 0;
        fake.fail_at = at;
        const netsim_status rc = go();
        const bool reached = fake.calls >= at;
        fake.fail_at = 0;
        if (join) {
          expect(fake.queued() == 0, "work still queued after the call", m.name, at);
        } else {
          expect(go() == NETSIM_OK, "the next run fails", m.name, at);
          expect(fake.queued() == 0, "work still queued after the next run", m.name, at);
        }
        netsim_destroy(h);
        fake.streams.erase(&own);
        if (!join)
          expect(fake.device.empty() && fake.pinned.empty() && fake.streams.empty() && fake.events.empty(),
                 "memory, streams or events left behind", m.name, at);
        for (void* p : fake.device) free(p);
        for (void* p : fake.pinned) free(p);
        fake = FakeHip();
        in_event = false;
        if (!reached) {
          if (rc != NETSIM_OK) FakeHip::bug("a run without failures");
          break;
        }
        ++tried;
      }
  }
  printf("%s: %ld failures tried, %d wrong\n", join ? "join" : "keep", tried, bad);
  return bad != 0;
}
