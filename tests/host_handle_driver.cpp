// Test driver (CPU only): the life of a handle on a HIP runtime that stands in for the real one. Device memory is host memory, a launch does
// nothing, and every event, pinned block and call that would wait for the device is counted. Host allocations fail where a
// test says so.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <set>
#include <thread>
#include <vector>

#include "gnr_internal.h"

static int failures = 0;
#define EXPECT(cond)                                                      \
  do {                                                                    \
    if (!(cond)) { std::printf("line %d: %s\n", __LINE__, #cond); ++failures; } \
  } while (0)

// ---- host allocations: the one that brings the count to zero fails
static thread_local long allocations_left = -1;
void *operator new(size_t n)
{
  if (allocations_left > 0 && --allocations_left == 0) throw std::bad_alloc();
  if (void *p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
  if (allocations_left > 0 && --allocations_left == 0) return nullptr;
  return std::malloc(n ? n : 1);
}
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

// ---- the runtime
static std::set<hipEvent_t> *events = new std::set<hipEvent_t>;
static int device = 0, elapsed_asked = 0, bad_events = 0, pinned = 0, pinned_freed = 0, waits = 0;
static bool pinned_fails = false, sync_fails = false;
extern "C" {
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpy(void *to, const void *from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++waits; return sync_fails ? hipErrorUnknown : hipSuccess; }
hipError_t hipDeviceSynchronize() { ++waits; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
  if (pinned_fails) return hipErrorOutOfMemory;
  *p = std::malloc(n); ++pinned;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { ++waits; ++pinned_freed; std::free(p); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e)
{
  *e = static_cast<hipEvent_t>(std::malloc(1));
  const long left = allocations_left;
  allocations_left = -1;   // (the books are not what is to fail)
  events->insert(*e);
  allocations_left = left;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
  if (!events->erase(e)) { ++bad_events; return hipErrorInvalidHandle; }
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { bad_events += !events->count(e); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
  ++elapsed_asked;
  bad_events += !events->count(a) + !events->count(b);
  *ms = 1.f;
  return hipSuccess;
}
}

// ---- the launches: the totals of a handle are its seed, so that one can tell whose they are
namespace gnr {
static int launches_fail = 0, steps_launched = 0;
static uint64_t *last_totals = nullptr;
int launch_reset(const Params &, int, void *) { return SIM_OK; }
int launch_steps(const Params &, int, int, size_t, uint32_t, uint32_t n, void *) { steps_launched += static_cast<int>(n); return SIM_OK; }
int launch_reduce(const Params &p, int, uint64_t *out, void *)
{
  if (launches_fail) return SIM_EHIP;
  std::memset(out, 0, (kTallyWords + static_cast<size_t>(3) * p.K * kNBin) * sizeof(uint64_t));
  out[SIM_T_A] = p.key0;
  last_totals = out;
  return SIM_OK;
}
int launch_digest(const Params &, int, int64_t, void *) { return SIM_OK; }
int static_workspace(void **, size_t *) { return SIM_EHIP; }
size_t step_lds_bytes(const Params &) { return 1024; }
int step_threads(Params, int) { return 64; }
bool step_dense(int, int, size_t) { return false; }
}  // namespace gnr

struct Made {
  std::vector<unsigned char> mem;
  sim_t *h = nullptr;
};

static Made make(int K)
{
  sim_class cls[SIM_MAXK];
  const double x[SIM_MAXK] = {}, q[SIM_MAXK] = {};
  std::memset(cls, 0, sizeof cls);
  for (sim_class &c : cls) { c.lambda = 0.1; c.in_law = c.out_law = SIM_CONST; c.in_p0 = 100.0; c.out_p0 = 10.0; }
  sim_config g;
  std::memset(&g, 0, sizeof g);
  g.K = K; g.N = 4; g.B = 4; g.C = 256; g.M = 1;
  g.c0 = 0.01; g.c_pre = 5e-5; g.c_dec = 2e-4;
  g.cls = cls; g.x_star = x; g.qp_star = q;
  g.queue_cap = 64; g.dbuf_cap = 64;
  size_t bytes = 0;
  Made m;
  EXPECT(sim_workspace_bytes(&g, 2, &bytes) == SIM_OK);
  m.mem.resize(bytes + 256);
  unsigned char *at = m.mem.data() + (256 - reinterpret_cast<uintptr_t>(m.mem.data()) % 256) % 256;
  EXPECT(sim_create(&g, 2, at, bytes, &m.h) == SIM_OK);
  return m;
}

static uint64_t arrivals(sim_t *h)
{
  static sim_stats_t st;
  EXPECT(sim_stats(h, &st, nullptr) == SIM_OK);
  return st.tally[0][SIM_T_A];
}

// A handle takes a pinned block that another has given back, or makes one, up to 32 a device; without one it copies.
static void blocks()
{
  const int steps = 10;
  std::vector<Made> live;
  std::set<uint64_t *> seen;
  for (int i = 0; i < 100; ++i) {
    live.push_back(make(1 + i % SIM_MAXK));
    EXPECT(sim_run(live.back().h, steps, 2, 1000 + i, nullptr) == SIM_OK);
  }
  EXPECT(pinned == 32);
  for (int i = 0; i < 100; ++i) {   // no two of them write to the same totals
    EXPECT(arrivals(live[i].h) == 1000u + static_cast<unsigned>(i));
    EXPECT(seen.insert(gnr::last_totals).second);
  }
  waits = 0;
  for (Made &m : live) EXPECT(sim_destroy(m.h) == SIM_OK);
  EXPECT(waits == 0 && pinned_freed == 0);
  live.clear();
  for (int i = 0; i < 40; ++i) {
    live.push_back(make(2));
    EXPECT(sim_run(live.back().h, steps, 2, 7, nullptr) == SIM_OK);
  }
  EXPECT(pinned == 32);
  for (Made &m : live) EXPECT(arrivals(m.h) == 7u);
  while (live.size() > 32) {
    EXPECT(sim_destroy(live.back().h) == SIM_OK);
    live.pop_back();
  }
  device = 1;   // blocks of another device are not for this one, and are given back from wherever a handle is destroyed
  Made there = make(2);
  EXPECT(pinned == 33);
  device = 0;
  EXPECT(sim_destroy(there.h) == SIM_OK);
  Made here = make(2);
  EXPECT(pinned == 33);
  device = 1;
  there = make(2);
  EXPECT(pinned == 33);
  pinned_fails = true;
  Made without = make(2);   // none free, none to be had
  EXPECT(sim_run(without.h, steps, 2, 9, nullptr) == SIM_OK && arrivals(without.h) == 9u);
  pinned_fails = false;
  Made with = make(2);      // ... which is no lasting refusal
  EXPECT(pinned == 34);
  // totals that a launch may write to yet go to nobody else
  EXPECT(sim_run(with.h, steps, 2, 11, nullptr) == SIM_OK && arrivals(with.h) == 11u);
  uint64_t *const his = gnr::last_totals;
  sim_stats_t st;
  gnr::launches_fail = 1;
  EXPECT(sim_stats(with.h, &st, nullptr) == SIM_EHIP);
  gnr::launches_fail = 0;
  EXPECT(arrivals(with.h) == 11u && gnr::last_totals == his);
  sync_fails = true;
  EXPECT(sim_stats(with.h, &st, nullptr) == SIM_EHIP);
  sync_fails = false;
  EXPECT(arrivals(with.h) == 11u && gnr::last_totals != his);
  EXPECT(sim_destroy(with.h) == SIM_OK);
  with = make(2);
  EXPECT(pinned == 35 && sim_run(with.h, steps, 2, 12, nullptr) == SIM_OK && arrivals(with.h) == 12u && gnr::last_totals != his);
  for (sim_t *h : {there.h, without.h, with.h, here.h}) EXPECT(sim_destroy(h) == SIM_OK);
  for (Made &m : live) EXPECT(sim_destroy(m.h) == SIM_OK);
  device = 0;
}

// Handles made and destroyed by several threads at once.
static void threads()
{
  device = 2;
  const int before = pinned;
  std::vector<std::thread> all;
  for (int t = 0; t < 8; ++t)
    all.emplace_back([] {
      for (int i = 0; i < 50; ++i) {
        Made m = make(2);
        EXPECT(sim_destroy(m.h) == SIM_OK);
      }
    });
  for (std::thread &t : all) t.join();
  EXPECT(pinned - before >= 1 && pinned - before <= 8);
  device = 0;
}

// A launch's pair of events is read once and kept or destroyed once, whichever host allocation fails on the way, and what the
// handle knows of its steps is what has been launched.
static void timing_events()
{
  for (int launches : {1, 3, 63, 64, 65, 130})
    for (int fail_at = 1; fail_at <= 4; ++fail_at)
      for (bool in_run : {false, true}) {
        Made m = make(2);
        gnr::steps_launched = 0;
        elapsed_asked = 0;
        int refused = 0, asked = 0;
        for (int i = 0; i < launches; ++i) {
          allocations_left = in_run ? fail_at : -1;
          const int rc = sim_run(m.h, 10, 2, 5, nullptr);
          allocations_left = -1;
          EXPECT(rc == SIM_OK || rc == SIM_ENOMEM);
          refused += rc != SIM_OK;
        }
        double ms = 0.0;
        int64_t n = 0;
        allocations_left = in_run ? -1 : fail_at;
        const int rc = sim_kernel_time(m.h, &n, &ms, 0, nullptr);
        allocations_left = -1;
        EXPECT(rc == SIM_OK || rc == SIM_ENOMEM);
        asked = elapsed_asked;
        EXPECT(sim_kernel_time(m.h, &n, &ms, 0, nullptr) == SIM_OK);
        EXPECT(n == launches - refused && ms == static_cast<double>(n));
        EXPECT(asked == n && elapsed_asked == n);
        EXPECT(gnr::steps_launched == 10 * n);
        EXPECT(sim_run(m.h, 10, 2, 5, nullptr) == SIM_OK);
        sim_stats_t st;
        EXPECT(sim_stats(m.h, &st, nullptr) == SIM_OK && st.steps == 10 * (n + 1));
        EXPECT(sim_kernel_time(m.h, &n, &ms, 0, nullptr) == SIM_OK && ms == static_cast<double>(n));
        EXPECT(sim_destroy(m.h) == SIM_OK);
        EXPECT(events->empty());
      }
  // a wait that fails leaves the pairs where they are
  Made m = make(2);
  sync_fails = true;
  for (int i = 0; i < 200; ++i) {
    const int rc = sim_run(m.h, 10, 2, 5, nullptr);
    EXPECT(rc == (i < 63 ? SIM_OK : SIM_EHIP));
  }
  sync_fails = false;
  double ms = 0.0;
  int64_t n = 0;
  EXPECT(sim_kernel_time(m.h, &n, &ms, 0, nullptr) == SIM_OK && n == 200 && ms == 200.0);
  EXPECT(sim_destroy(m.h) == SIM_OK);
}

int main()
{
  blocks();
  timing_events();
  threads();
  EXPECT(bad_events == 0);
  EXPECT(events->empty());
  if (failures == 0) std::printf("clean\n");
  return failures != 0;
}
