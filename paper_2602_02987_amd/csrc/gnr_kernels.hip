// Small kernels of the simulator (reset, totals over replications, state digest) and the launchers (gfx950).
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>

#include "gnr_step.h"

namespace gnr {

size_t step_lds_bytes(const Params &p)
{
  // The layout is carved out of a host block that is never read or written: only the total is wanted, but the
  // same code as on the device forms the pointers, and those stay inside a real object this way (the largest
  // configuration the library accepts needs less than a fifth of it).
  alignas(16) static unsigned char block[1 << 20];
  switch (size_class(p.threads, p.nwords)) {
    case 0: return lds_carve<static_words(0), true>(p, block).bytes;
    case 1: return lds_carve<static_words(1)>(p, block).bytes;
    case 2: return lds_carve<static_words(2)>(p, block).bytes;
    default: return lds_carve<static_words(3)>(p, block).bytes;
  }
}

constexpr size_t kLdsPerComputeUnit = 160 * 1024;

// Compute units of the current device (asked once per device; 256 if the runtime does not say).
static int compute_units()
{
  constexpr int kMaxDevices = 64;
  static std::atomic<int> known[kMaxDevices] = {};
  int d = 0;
  if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= kMaxDevices) return 256;
  int n = known[d].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, d) != hipSuccess || n < 1) n = 256;
    known[d].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Workgroups a compute unit holds at once when its SIMDs hold `per_simd` waves of the kernel each.
static int workgroups_at_once(int threads, size_t lds_bytes, int per_simd)
{
  const int by_waves = 4 * per_simd / (threads / 64);   // wave slots of the four SIMDs
  const int by_lds = static_cast<int>(kLdsPerComputeUnit / (lds_bytes ? lds_bytes : 1));
  const int wgs = by_waves < by_lds ? by_waves : by_lds;
  return wgs < 1 ? 1 : wgs;
}

// Rounds of workgroups a launch of `reps` workgroups needs: every workgroup runs for the whole launch, so one that finds
// no place at first waits for another to end.
static int launch_rounds(int reps, int threads, size_t lds_bytes, int per_simd)
{
  const int at_once = compute_units() * workgroups_at_once(threads, lds_bytes, per_simd);
  return (reps + at_once - 1) / at_once;
}

bool step_dense(int reps, int threads, size_t lds_bytes)
{
  return threads <= 512 && launch_rounds(reps, threads, lds_bytes, waves_per_simd(threads, true)) <
                               launch_rounds(reps, threads, lds_bytes, waves_per_simd(threads, false));
}

int step_threads(Params q, int reps)
{
  // A replication with many servers fills the LDS of a compute unit, runs alone there and wants all sixteen
  // waves to hide latency.
  if (q.N > 64 * kMostWordsEight) return 1024;
  // Smaller replications share a compute unit. A workgroup steps faster the more waves it has, as long as its waves have
  // blocks of servers to work on and all workgroups of the launch find a place at once (at most four waves per SIMD): the
  // largest workgroup that keeps the rounds lowest. Rounds count as they are while a full compute unit holds two waves a
  // SIMD or more; with fewer nothing hides a wave's latency, and a round counts by as much as waves are missing (100 steps,
  // 3500 servers of eight classes, same-slot decode, 700 replications: three waves a compute unit in one round 8.7 ms,
  // sixteen in two rounds 3.2; 3000 servers of two classes, 2048 replications: four in two rounds 6.6, twelve in three
  // 4.4; but eight in one round 3.3 against sixteen in two 4.1, 1000 servers of four classes, weighted router, 2048).
  // With fewer than two blocks to a wave the larger workgroup is left out where the launch needs more than two waves a SIMD
  // for it. That holds from four waves to eight (500 steps of 512 replications, 256 threads roomy, 512 dense: 600 servers
  // of two classes 4.4 and 4.7 ms, 700 of four 5.1 and 5.6). With deadline rings eight dense waves are taken from a block a wave
  // on: the walks of the rings and the class selection take waves of their own. It pays with the weighted router (700
  // servers of four classes 8.4 and 8.1 ms), no longer without (with patience 5.8 and 6.2, convergence instance of 500
  // servers 5.7 and 5.8).
  // Timed again with steps that overlap in workgroups of eight waves (300 steps, 385 launches of 40 to 4500 servers, 4 to 2000
  // replications, every router): with two to four blocks more waves pay, for the gate, the router and the waves that serve have waves of
  // their own then. Time with the rule that stood here over that with this one, two to four blocks: same-slot decode 1.12 to 1.25 with
  // 512 threads where a compute unit has one workgroup, 1.03 to 1.19 where it has two; both buffers with patience 1.12 to 1.29 and 1.07
  // to 1.21; weighted router 1.05 to 1.16 and 1.05 to 1.14; patience 1.04 to 1.23 and 1.00 to 1.15. The base router's 512 threads are
  // no faster than 256 there (0.93 to 1.02), which are 5 to 8 % faster than 128. With three or four workgroups a compute unit 256 dense
  // threads give 4 to 18 % with deadline rings and nothing or less without; with five to eight 128 give 8 to 20 % over 64. Eight dense
  // waves give same-slot decode 14 to 21 % with five to 22 blocks too.
  // What is left: two and more waves for one block 8 to 39 %, four dense waves instead of two with five to seven blocks and
  // deadline rings 3 to 23 %, sixteen waves instead of eight with the base router, five to 30 blocks and up to 256 replications up to 8 %,
  // eight instead of sixteen with same-slot decode and 32 to 47 blocks 3 to 7 %, four instead of eight dense ones with the base router
  // and 16 to 32 blocks up to 13 %.
  constexpr int kRound = 840;   // (divisible by one to eight waves)
  const int blocks = (q.N + 63) / 64;
  int best = 64, best_cost = 0;
  const bool few = blocks >= 2 && blocks <= 4, more_roles = q.dl_rings || q.route_mode != SIM_ROUTE_SOLO_FIRST;
  const int most = few ? (more_roles ? 8 : 4) : 2 * blocks - 1;
  for (int t = 64; t <= 1024 && t / 64 <= most; t *= 2) {
    q.threads = t;
    const size_t lds = step_lds_bytes(q);
    if (lds > kLdsPerComputeUnit) break;
    const int waves = t / 64, rounds = launch_rounds(reps, t, lds, 4), held = waves * workgroups_at_once(t, lds, 4);
    const int cost = rounds * (kRound / (held < 8 ? held : 8));
    // few blocks a wave, and dense (sixteen waves have no roomy form)
    const bool pays = t == 512 ? (q.dl_rings && blocks >= 8) || (few && more_roles) || q.route_mode == SIM_ROUTE_IMMEDIATE
                               : few && (t == 128 || (t == 256 && q.dl_rings));
    const bool thin = blocks < 2 * waves && !pays && (t > 512 || launch_rounds(reps, t, lds, 2) > rounds);
    if (best_cost == 0 || cost < best_cost || (cost == best_cost && !thin)) { best = t; best_cost = cost; }
  }
  return best;
}

// ------------------------------------------------------------------ reset ----
__global__ void gnr_reset_kernel(const Params p, const int reps)
{
  const size_t n_srv = static_cast<size_t>(reps) * p.N;
  const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
  const size_t t0 = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  for (size_t i = t0; i < n_srv; i += stride) {
    p.rec[i] = ServerRec{0, 0, 0, 0, kNever};
    p.t_rel[i] = kIdleRel; p.remptok[i] = 0;
  }
  for (size_t i = t0; i < n_srv * p.BS; i += stride) p.fin[i] = kFreeSlot;
  for (size_t i = t0; i < static_cast<size_t>(reps) * CS_WORDS; i += stride) p.cstate[i] = 0;
  for (size_t i = t0; i < static_cast<size_t>(reps) * kTallyWords; i += stride) p.tally[i] = 0;
  for (size_t i = t0; i < static_cast<size_t>(reps) * 3 * p.K * kNBin; i += stride) p.hist[i] = 0;
  if (p.dl_rings)
    for (size_t i = t0; i < static_cast<size_t>(reps) * p.K * (p.cal_mask + 1u); i += stride) {
      p.cal[i] = 0; p.dcal[i] = 0;
      if (p.dcal_m) p.dcal_m[i] = 0;
    }
}

// ------------------------------------------------------------------ reduce ----
// Totals over replications: a lane per output word, the waves of a workgroup take every blockDim/64-th replication and
// keep eight rows in flight each. The sums wait for memory alone: with one thread per word that walked the replications
// one after the other, each row cost a round trip (2048 replications of four classes: 1480 us; 1024 of two: 515 us; 256
// of six: 158 us), while the rows are 8 bytes a lane, whole lines a wave.
constexpr int kReduceWaves = 16, kReduceAhead = 8;
__global__ void __launch_bounds__(64 * kReduceWaves) gnr_reduce_kernel(const Params p, const int reps, uint64_t *__restrict__ out)
{
  __shared__ uint64_t part[kReduceWaves][64];
  const int nh = 3 * p.K * kNBin;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  uint64_t acc = 0;
  if (i < kTallyWords + nh) {
    const size_t stride = i < kTallyWords ? kTallyWords : nh;
    const uint64_t *col = i < kTallyWords ? p.tally + i : p.hist + (i - kTallyWords);
    int r = wave;
    for (; r + (kReduceAhead - 1) * nwaves < reps; r += kReduceAhead * nwaves) {
      uint64_t v[kReduceAhead];
#pragma unroll
      for (int u = 0; u < kReduceAhead; ++u) v[u] = col[static_cast<size_t>(r + u * nwaves) * stride];
#pragma unroll
      for (int u = 0; u < kReduceAhead; ++u) acc += v[u];
    }
    for (; r < reps; r += nwaves) acc += col[static_cast<size_t>(r) * stride];
  }
  part[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && i < kTallyWords + nh) {
    for (int w = 1; w < nwaves; ++w) acc += part[w][lane];
    out[i] = acc;
  }
}

// ------------------------------------------------------------------ digest ----
// Sum mod 2^64 of a chained 64-bit finaliser (Steele-Lea-Flood / Vigna splitmix64 output
// function) over tagged items of the integer state; slot items ignore the slot position.
__device__ __forceinline__ uint64_t mix64(uint64_t z)
{
  z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27; z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  return z;
}
__device__ __forceinline__ uint64_t chain(uint64_t h, uint64_t w) { return mix64(h + w + 0x9E3779B97F4A7C15ull); }

__global__ void gnr_digest_kernel(const Params p, const int64_t t_end)
{
  __shared__ unsigned long long total;
  const int r = blockIdx.x, tid = threadIdx.x, NT = blockDim.x;
  const int K = p.K, N = p.N;
  if (tid == 0) total = 0;
  __syncthreads();
  const int32_t *cs = p.cstate + static_cast<size_t>(r) * CS_WORDS;
  uint64_t d = 0;
  if (tid < K) {
    const int k = tid;
    uint64_t h = chain(1, static_cast<uint64_t>(k));
    h = chain(h, static_cast<uint64_t>(static_cast<int64_t>(cs[CS_QP + k])));
    h = chain(h, static_cast<uint64_t>(static_cast<int64_t>(cs[CS_X + k])));
    h = chain(h, static_cast<uint64_t>(static_cast<int64_t>(cs[CS_QD + k])));
    h = chain(h, static_cast<uint64_t>(static_cast<int64_t>(cs[CS_YM + k])));
    h = chain(h, static_cast<uint64_t>(static_cast<int64_t>(cs[CS_YS + k])));
    d += h;
  }
  for (int k = 0; k < K; ++k) {
    const uint32_t head = static_cast<uint32_t>(cs[CS_QHEAD + k]), len = static_cast<uint32_t>(cs[CS_QP + k]);
    const uint32_t *ring = p.qring + (static_cast<size_t>(r) * K + k) * p.queue_cap;
    const uint32_t *dlr = p.ab_classes ? p.qdl + (static_cast<size_t>(r) * K + k) * p.queue_cap : nullptr;
    for (uint32_t i = tid; i < len; i += NT) {
      uint32_t pos = head + i;
      if (pos >= p.queue_cap) pos -= p.queue_cap;
      uint64_t h = chain(chain(chain(2, static_cast<uint64_t>(k)), i), ring[pos]);
      if (dlr) h = chain(h, dlr[pos]);   // with abandonment the deadline is part of the state
      d += h;
    }
  }
  {
    const uint32_t head = static_cast<uint32_t>(cs[CS_DHEAD]), len = static_cast<uint32_t>(cs[CS_DCOUNT]);
    const uint64_t *ring = p.dring + static_cast<size_t>(r) * p.dbuf_cap;
    const uint32_t *dlr = p.ab_classes ? p.ddl + static_cast<size_t>(r) * p.dbuf_cap : nullptr;
    for (uint32_t i = tid; i < len; i += NT) {
      uint32_t pos = head + i;
      if (pos >= p.dbuf_cap) pos -= p.dbuf_cap;
      uint64_t h = chain(chain(3, i), ring[pos]);
      if (dlr) h = chain(h, dlr[pos]);
      d += h;
    }
  }
  if (p.route_mode == SIM_ROUTE_RANDOM_SPLIT || p.route_mode == SIM_ROUTE_WEIGHTED_SPLIT) {   // the mixed group's buffer
    const uint32_t head = static_cast<uint32_t>(cs[CS_DHEAD_M]), len = static_cast<uint32_t>(cs[CS_DCOUNT_M]);
    const uint64_t *ring = p.dring_m + static_cast<size_t>(r) * p.dbuf_cap;
    const uint32_t *dlr = p.ab_classes ? p.ddl_m + static_cast<size_t>(r) * p.dbuf_cap : nullptr;
    for (uint32_t i = tid; i < len; i += NT) {
      uint32_t pos = head + i;
      if (pos >= p.dbuf_cap) pos -= p.dbuf_cap;
      uint64_t h = chain(chain(6, i), ring[pos]);
      if (dlr) h = chain(h, dlr[pos]);
      d += h;
    }
  }
  for (int g = tid; g < N; g += NT) {
    const size_t sg = static_cast<size_t>(r) * N + g;
    const uint32_t pk = p.remptok[sg];
    const uint32_t rem = pk & 0xFFFFu;
    const uint32_t ptok = (pk >> 16) & 0x1FFFu;
    const ServerRec sr = p.rec[sg];
    const uint32_t tr = p.t_rel[sg];
    uint64_t h = chain(4, static_cast<uint64_t>(g));
    h = chain(h, static_cast<uint64_t>(tr == kIdleRel ? kIdle : t_end + static_cast<int64_t>(tr)));
    h = chain(h, sr.iter);
    h = chain(h, rem);
    h = chain(h, ptok);
    h = chain(h, rem ? sr.pf_job : 0ull);
    h = chain(h, sr.n_cls);
    h = chain(h, sr.n_join);
    d += h;
    const int nd = static_cast<int>(byte_sum(sr.n_cls));
    for (int j = 0; j < nd; ++j)
      d += chain(chain(chain(5, static_cast<uint64_t>(g)), p.fin[sg * p.BS + j]), p.job[sg * p.BS + j]);
  }
  atomicAdd(&total, static_cast<unsigned long long>(d));
  __syncthreads();
  if (tid == 0) p.digest[r] = total;
}

// ------------------------------------------------------------------ static workspace ----
// Device memory for handles whose caller cannot allocate any (sim_create_static). In host code the array's name
// is only a stand-in for the symbol: its address on a device comes from hipGetSymbolAddress, asked once per device
// with that device current, and that pointer is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[SIM_STATIC_WORKSPACE_BYTES];

int static_workspace(void **dev_ptr, size_t *bytes)
{
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *resolved[kMaxDevices] = {};
  int d = -1;
  if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= kMaxDevices) return SIM_EHIP;
  std::lock_guard<std::mutex> lock(mu);
  if (!resolved[d]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SIM_EHIP;
    resolved[d] = ptr;
  }
  *dev_ptr = resolved[d];
  *bytes = sizeof(scratch);
  return SIM_OK;
}

// ------------------------------------------------------------------ launchers ----
// The step kernel's policy variants, each compiled in a translation unit of its own (gnr_step_<variant>.hip).
StepKernel step_kernel_plain(int form, bool dense);
StepKernel step_kernel_rr(int form, bool dense);
StepKernel step_kernel_im(int form, bool dense);
StepKernel step_kernel_ab(int form, bool dense);
StepKernel step_kernel_ab_rr(int form, bool dense);
StepKernel step_kernel_ab_im(int form, bool dense);
StepKernel step_kernel_ws(int form, bool dense);

static int hip_ok(hipError_t e) { return e == hipSuccess ? SIM_OK : SIM_EHIP; }

int launch_reset(const Params &p, int reps, void *stream)
{
  hipLaunchKernelGGL(gnr_reset_kernel, dim3(1024), dim3(256), 0, static_cast<hipStream_t>(stream), p, reps);
  return hip_ok(hipGetLastError());
}

// Which compilation of the step kernel a launch takes. Of eight waves all work off the events, and who does not serve draws beside the
// ones that do, up to 40 words (2560 servers): 300 servers x 4 2.03 -> 1.88 ms per 300 steps, 1024 x 256 2.76 -> 2.58, 1500 x 40 2.82 ->
// 2.64, with patience 900 x 400 4.74 -> 4.57 per 400; with more words four draw beside the events: 3000 x 500 4.19 and 4.25, 4500 x 500
// 2.53 and 2.80 per 200. With same-slot decode, which has no jobs to serve, four draw whatever the size (900 x 400 3.14 and 3.82 per
// 400), with two buffers none.
static int step_form(int threads, int nwords)
{
  switch (threads) {
    case 64: return 0;
    case 128: return 1;
    case 256: return 2;
    case 512: return nwords <= 40 ? 3 : nwords <= kMostWordsEight ? 6 : -1;
    case 1024: return 2 + size_class(threads, nwords);
    default: return -1;
  }
}

int launch_steps(const Params &p, int reps, int threads, size_t lds_bytes, uint32_t step_begin, uint32_t n_steps,
                 void *stream)
{
  const int form = step_form(threads, p.nwords);
  if (form < 0) return SIM_EINVAL;
  const bool ab = p.dl_rings != 0;
  // The roomy form of a small size class holds two waves per SIMD, the dense form four: the dense one is taken when
  // the launch then needs fewer rounds of workgroups (every workgroup runs for the whole launch, so a workgroup
  // that finds no place at first waits for another to end).
  const bool dense = step_dense(reps, threads, lds_bytes);
  StepKernel kernel = nullptr;
  switch (p.route_mode) {
    case SIM_ROUTE_SOLO_FIRST: kernel = ab ? step_kernel_ab(form, dense) : step_kernel_plain(form, dense); break;
    case SIM_ROUTE_RANDOM_SPLIT: kernel = ab ? step_kernel_ab_rr(form, dense) : step_kernel_rr(form, dense); break;
    case SIM_ROUTE_IMMEDIATE: kernel = ab ? step_kernel_ab_im(form, dense) : step_kernel_im(form, dense); break;
    // (the weighted router is the randomized router's variant with deadline rings plus the class draws)
    case SIM_ROUTE_WEIGHTED_SPLIT: kernel = ab ? step_kernel_ws(form, dense) : nullptr; break;
    default: break;
  }
  if (!kernel) return SIM_EINVAL;
  if (lds_bytes > 64 * 1024) {   // more than the default dynamic LDS limit has to be asked for
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
    if (e != hipSuccess) return SIM_EHIP;
  }
  const StepArrays a = {p.arr_thr, p.len_tab, p.rec,    p.t_rel, p.remptok,
                        p.fin,     p.job,     p.qring,  p.dring, p.cstate, p.tally,  p.hist,
                        p.pat_tab, p.qdl,     p.ddl,    p.cal,   p.dcal,   p.dring_m, p.ddl_m, p.dcal_m};
  hipLaunchKernelGGL(kernel, dim3(reps), dim3(threads), lds_bytes, static_cast<hipStream_t>(stream), p.self, a, p.key0,
                     p.key1, step_begin, n_steps);
  return hip_ok(hipGetLastError());
}

int launch_reduce(const Params &p, int reps, uint64_t *out, void *stream)
{
  const int n = kTallyWords + 3 * p.K * kNBin;
  // a wave for every row group it can keep in flight, up to sixteen
  const int waves = reps >= kReduceAhead * kReduceWaves ? kReduceWaves : (reps + kReduceAhead - 1) / kReduceAhead;
  hipLaunchKernelGGL(gnr_reduce_kernel, dim3((n + 63) / 64), dim3(64 * waves), 0, static_cast<hipStream_t>(stream), p, reps, out);
  return hip_ok(hipGetLastError());
}

int launch_digest(const Params &p, int reps, int64_t t_end, void *stream)
{
  hipLaunchKernelGGL(gnr_digest_kernel, dim3(reps), dim3(256), 0, static_cast<hipStream_t>(stream), p, t_end);
  return hip_ok(hipGetLastError());
}

}  // namespace gnr
