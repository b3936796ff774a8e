// HIP kernels of the gate-and-route network simulator (gfx950, wave64).
//
// One workgroup owns one replication for a whole launch and loops over the steps itself. The servers are
// handled in blocks of 64 (one per lane), of which a wave looks at some pairs in the completion pass, and what a step gives
// a server is written by the last waves of the workgroup, a barrier later, or while the others go on. A server is touched only
// when its batch changes (an event): the identical iterations in between follow from its event time. Class-level
// counters (queue lengths, occupancies, tallies) live in LDS and are updated with integer atomics, which commute, by the
// lanes that have something to add (a few of a wave as a rule; sums that all lanes add to are spread over several words).
// Everything that the policy defines sequentially (order of simultaneous prefill completions, of gate admissions, of
// routed requests) is reproduced with 64-server ballot words in LDS and prefix popcounts over them.
#ifndef GNR_STEP_H
#define GNR_STEP_H
#include <hip/hip_runtime.h>

#include "gnr_internal.h"

namespace gnr {

// ------------------------------------------------------------------ primitives ----
// x ^ y ^ z in one instruction: left to itself the compiler makes two of every such pair. The arrival draw is one
// Philox block per server and step, 2.56e9 of them in 1000 steps of 10000 servers x 256 replications: alone they take
// 3.0 ms there with this instruction, 3.7 ms without.
__device__ __forceinline__ uint32_t xor3(uint32_t x, uint32_t y, uint32_t z)
{
  return static_cast<uint32_t>(__builtin_amdgcn_bitop3_b32(static_cast<int>(x), static_cast<int>(y), static_cast<int>(z), 0x96));
}

// Philox4x32-10 (Salmon et al., SC'11): rounds FIRST to 10 on the state (c0, c1, c2, c3), k0 and k1 being round FIRST's keys.
template <int FIRST>
__device__ __forceinline__ void philox_rounds(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                                              uint32_t c3, uint32_t (&w)[4])
{
#pragma unroll
  for (int round = FIRST; round <= 10; ++round) {
    const uint64_t a = static_cast<uint64_t>(0xD2511F53u) * c0;
    const uint64_t b = static_cast<uint64_t>(0xCD9E8D57u) * c2;
    const uint32_t n0 = xor3(static_cast<uint32_t>(b >> 32), c1, k0);
    const uint32_t n2 = xor3(static_cast<uint32_t>(a >> 32), c3, k1);
    c1 = static_cast<uint32_t>(b);
    c3 = static_cast<uint32_t>(a);
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}
__device__ __forceinline__ void philox4x32_10(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                                              uint32_t c3, uint32_t (&w)[4])
{
  asm volatile("" : "+s"(k0), "+s"(k1));   // (the round keys are formed anew: see draw_words)
  philox_rounds<1>(k0, k1, c0, c1, c2, c3, w);
}

// Histogram bin of a duration in ns (those from 2^48 on are in the last one): exact below 16, then 16 bins per octave. The bin is the exponent and
// the upper four bits of the mantissa of the duration as a double, which holds it exactly.
__device__ __forceinline__ int hbin(int64_t v)
{
  const double f = __builtin_ldexp(static_cast<double>(static_cast<uint32_t>(v >> 32)), 32) + static_cast<double>(static_cast<uint32_t>(v));
  const int b = static_cast<int>(static_cast<uint32_t>(__double_as_longlong(f) >> 32) >> 16) - 16 * (1023 + 3);
  const int bin = v < 16 ? (v < 0 ? 0 : static_cast<int>(v)) : b;
  return bin < kNBin ? bin : kNBin - 1;
}

// The same for a duration below 2^31.
__device__ __forceinline__ int hbin32(uint32_t v)
{
  const int b = static_cast<int>(static_cast<uint32_t>(__double_as_longlong(static_cast<double>(v)) >> 32) >> 16) - 16 * (1023 + 3);
  return v < 16 ? static_cast<int>(v) : b;
}

__device__ __forceinline__ uint32_t byte_sum(uint64_t packed)
{
  return static_cast<uint32_t>((packed * 0x0101010101010101ull) >> 56);
}
// Bytes k and k + 1 (k even), one a half of the word.
__device__ __forceinline__ uint64_t two_bytes_at(uint64_t packed, int k)
{
  const uint32_t w = static_cast<uint32_t>(packed >> (32 * (k >> 2))), sh = 8u * static_cast<uint32_t>(k & 2);
  return ((w >> sh) & 255u) | static_cast<uint64_t>((w >> (sh + 8u)) & 255u) << 32;
}
__device__ __forceinline__ uint32_t byte_at(uint64_t packed, int k) { return static_cast<uint32_t>(packed >> (8 * k)) & 255u; }

// Prefill word of a server: prompt tokens left | tokens in the running chunk << 16 | class << 29.
__device__ __forceinline__ int pk_rem(uint32_t pk) { return static_cast<int>(pk & 0xFFFFu); }
__device__ __forceinline__ int pk_ptok(uint32_t pk) { return static_cast<int>((pk >> 16) & 0x1FFFu); }

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Position of the n-th set bit (n counted from 0) of a word that has more than n bits set.
__device__ __forceinline__ int nth_set_bit(uint64_t word, int n)
{
  const int c32 = __popc(static_cast<uint32_t>(word));
  const bool up = n >= c32;
  uint32_t w = static_cast<uint32_t>(up ? word >> 32 : word);
  n -= up ? c32 : 0;
  int pos = up ? 32 : 0;
#pragma unroll
  for (int sh = 16; sh > 0; sh >>= 1) {
    const int c = __popc(w & ((1u << sh) - 1u)), by = n >= c ? sh : 0;
    n -= by ? c : 0;
    w >>= by;
    pos += by;
  }
  return pos;
}

// Index of the j-th set bit of a bitmap given the exclusive prefix popcounts of its words.
__device__ __forceinline__ int select_bit(const uint64_t *bm, const uint16_t *pre, int nwords, uint32_t j)
{
  int lo = 0, hi = nwords - 1;   // largest w with pre[w] <= j
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= j) lo = mid; else hi = mid - 1;
  }
  return lo * 64 + nth_set_bit(bm[lo], static_cast<int>(j - pre[lo]));
}

// A wave-uniform value pinned in a scalar register. Without this the compiler, short of registers, re-reads
// parameters from memory through the scalar cache wherever they are used (a round trip of hundreds of cycles in
// the middle of a hot loop) instead of keeping them.
__device__ __forceinline__ uint32_t pinned(uint32_t v)
{
  uint32_t own;
  asm volatile("s_mov_b32 %0, %1" : "=s"(own) : "s"(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)))));
  return own;
}

__device__ __forceinline__ int pinned(int v) { return static_cast<int>(pinned(static_cast<uint32_t>(v))); }
// The same for a pointer to global memory. (Arguments and parameters arrive up to sixteen words at a time; what stays a piece of
// such a load comes back with the fifteen others, an instruction each, when there was no register for it for a while.)
template <class T>
__device__ __forceinline__ T *pinned(T *p)
{
  uint64_t own;
  asm volatile("s_mov_b64 %0, %1" : "=s"(own) : "s"(reinterpret_cast<uint64_t>(p)));
  return (T *)(__attribute__((address_space(1))) T *)own;
}

// Sixteen bytes of a slot row, read with the non-temporal hint: a row is read when one of its decodes ends and not
// again before it would have left the caches, so it should not push out the server records, ring entries and tables
// that the rest of the step reads.
__device__ __forceinline__ uint4 stream_load(const uint32_t *p)
{
  typedef uint32_t word4 __attribute__((ext_vector_type(4)));
  const word4 x = __builtin_nontemporal_load(reinterpret_cast<const word4 *>(p));
  return make_uint4(x.x, x.y, x.z, x.w);
}

// Smallest r with r * d >= x, for 0 < x < 2^40 and a quotient below 2^17 (the iterations a server still has to complete
// before its event, x ns ahead): estimated in single precision (relative error below 2^-21, so off by less than one),
// then corrected exactly.
__device__ __forceinline__ uint32_t iterations_left(uint64_t x, uint32_t d)
{
  const float xf = static_cast<float>(static_cast<uint32_t>(x >> 16)) * 65536.0f + static_cast<float>(static_cast<uint32_t>(x) & 0xFFFFu);
  uint32_t r = static_cast<uint32_t>(xf * __builtin_amdgcn_rcpf(static_cast<float>(d)));
  if (static_cast<uint64_t>(r) * d < x) ++r;
  if (static_cast<uint64_t>(r) * d < x) ++r;
  if (r > 0 && static_cast<uint64_t>(r - 1) * d >= x) --r;
  return r;
}

// How many lanes below this one a mask has.
__device__ __forceinline__ int rank_in(uint64_t mask)
{
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u)));
}
// Whether a wave-uniform mask has this lane.
__device__ __forceinline__ bool lane_in(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }
// v with lane l's value replaced by a wave-uniform x (the compiler has no builtin for the instruction).
__device__ int writelane32(int x, int l, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint64_t writelane64(uint64_t v, uint64_t x, int l)
{
  const uint32_t lo = static_cast<uint32_t>(writelane32(static_cast<int>(x), l, static_cast<int>(v)));
  const uint32_t hi = static_cast<uint32_t>(writelane32(static_cast<int>(x >> 32), l, static_cast<int>(v >> 32)));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}
// A lane's 64-bit word as a wave-uniform value.
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l)
{
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), l));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// The lanes of `who` by class number (0 to 7): a lane finds those of any class from three ballots over the bits of the
// number, whatever the count of classes.
struct ClassSets {
  uint64_t who, bit[3];
  __device__ __forceinline__ uint64_t among(int c) const
  {
    return who & (c & 1 ? bit[0] : ~bit[0]) & (c & 2 ? bit[1] : ~bit[1]) & (c & 4 ? bit[2] : ~bit[2]);
  }
};
__device__ __forceinline__ ClassSets class_sets(int c, uint64_t who)
{
  return {who, {__ballot((c & 1) != 0), __ballot((c & 2) != 0), __ballot((c & 4) != 0)}};
}

// Inclusive prefix sum over the wave with data-parallel-primitive adds: shifts by 1, 2, 4 and 8 inside each
// row of 16 lanes, then the row totals are passed on (row 0 -> 1, 2 -> 3, then 1 -> 2 and 3). All 64 lanes
// must be active.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v)
{
  return v + static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
  v = dpp_add<0x111, 0xF>(v);   // row_shr 1
  v = dpp_add<0x112, 0xF>(v);   // row_shr 2
  v = dpp_add<0x114, 0xF>(v);   // row_shr 4
  v = dpp_add<0x118, 0xF>(v);   // row_shr 8
  v = dpp_add<0x142, 0xA>(v);   // row_bcast 15 into rows 1 and 3
  v = dpp_add<0x143, 0xC>(v);   // row_bcast 31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ void lds_add64(uint64_t *p, uint64_t v)
{
  atomicAdd(reinterpret_cast<unsigned long long *>(p), static_cast<unsigned long long>(v));
}

// ------------------------------------------------------------------ LDS layout ----
enum Scalar {
  SC_NIDLE = 0, SC_NCOMP,
  SC_HEAD = 2,    // [8] head of each class queue as the pass's admissions find it
  // two-buffer routers only:
  SC_NSOLO = 13,  // completed prefills of this step whose request goes to the solo group
  // deadline rings (abandonment, weighted router) only:
  SC_DLEN = 10,   // entries of the decode buffer ring between head and tail, abandoned ones included
  SC_DSCAN = 11,  // entries of that ring the routing passes of this step have gone past
  SC_COMPACT = 12,// bit k: class queue ring k (bits 8, 9: the decode buffer rings) must be compacted before the appends
  SC_DLEN_M = 15, // two buffers: SC_DLEN / SC_DSCAN of the mixed group's buffer ring
  SC_DSCAN_M = 60,
  SC_QLEN = 32,   // [8] entries of each class queue ring between head and tail, abandoned ones included
  // every variant:
  SC_TAKE = 16,   // [8] accepted arrivals this step
  SC_TAIL = 24,   // [8] ring position of the first accepted arrival
  SC_ADMK = 40,   // [8] admissions per class in this gate pass
  SC_NADM = 61,   // admissions of the pass (bit 16: another gate pass follows)
  SC_LEVELS = 62, // the pass's routing levels: how many, of them the solo group's (8 bits each), bit 16: another pass follows
  SC_LMIN = 63,   // lowest level of the solo and (16 bits up) of the mixed group
  SC_TAKE_T = 48, // [kRouteLevels] jobs each level of the routing pass takes
  SC_CNT_T = 52,  // [kRouteLevels] servers with exactly the level's decodes
  SC_W_T = 56,    // [kRouteLevels] jobs of the pass that come before each level
  SC_WORDS = 64
};
// Per class: arrivals of the step; prefills that end, decodes that cease to be mixed, become solo and cease to be solo. The class state
// itself stays as the last step left it until the pass is over. (Sums of what is added only: two classes are added to at once.)
enum PassSum { AC_ARRIVALS = 0, AC_X_OUT = 8, AC_YM_OUT = 16, AC_YS_IN = 24, AC_YS_OUT = 32, AC_WORDS = 40 };
constexpr int kLoadBins = kMaxB + 1;
// (a run has fewer than 2^29 steps, an iteration is no shorter than a step, and an event lies at most 65535 iterations ahead)
constexpr uint32_t kEvChunk = 1u << 30, kEvFin = 1u << 31, kEvIter = kEvChunk - 1u;
// Running sums of the executed iterations, each spread over a row of words (see tally_iterations): iterations and busy time
// of the solo and, one row further, the mixed ones; time between tokens per class.
enum TallySum { TA_ITERS = 0, TA_BUSY = 2, TA_TBT = 4 };
constexpr int kTallyRows = 16, kTallyRowsSmall = 8;
// Table sizes. Workgroups of one or two waves (N up to 5120) share a compute unit with others of their kind and are
// given smaller tables, so that eight of them fit its LDS: gate and routing passes then decide 64 admissions and stage
// 64 requests at a time (more passes when a step brings more), and a wave finishes its queued servers when more than
// 32 wait.
constexpr int kEvPerWave = 128;   // servers a wave can queue for finishing; when full the queue is drained early
constexpr int kHeldEvSmall = 96, kJobsLdsSmall = 64, kAdmChunkSmall = 64;
constexpr int kRouteLevels = 4;
constexpr int kJobsLds = 256;      // requests of a routing pass staged in LDS; later ones are read from the buffer

struct Lds {
  int32_t *cs;        // [CS_WORDS]
  uint32_t *acc;      // [AC_WORDS] what the completion pass of a step adds up: arrivals and changes of the class counters
  uint32_t *cthr;     // [8] class thresholds of the arrival draw
  double *gtab;       // [5][kMaxK] gate targets of the launch: n x*, 1/x*, x*, n q*, priority index
  int32_t *sc;        // [SC_WORDS]
  uint64_t *tl;       // [kTallyWords]
  uint64_t *tbth;     // [(K + 1) / 2][tbt_w] time between tokens: counts of two classes a word, 32 bits each
  uint64_t *bm_idle;  // [nwords] servers below Mp with no prefill in service (the gate looks at those below M), as of the ranks in pre
  uint64_t *bm_comp;  // [2][nwords_m] servers whose prefill completed this step (immediate decode: that may be admitted to again), steps in turn
  uint64_t *bm_busy;  // [nwords, or one more: even] servers running an iteration
  uint64_t *bm_others;// [the same] steps that overlap: of a wave's words the servers that others have been given, for the next completion pass
  uint64_t *bm_just;  // [2][nwords] servers that went idle in this step (steps in turn)
  uint64_t *jobs;     // [kJobsLds] the first requests a routing pass places, copied from the decode buffer
  uint64_t *fresh;    // [kJobsLds] abandonment, more than one wave: this step's first completed prefills (two buffers: half each)
  // two-buffer routers only: completed prefills of this step whose request goes to the solo group, and their ranks
  uint64_t *bm_solo;  // [2][nwords_m] (steps in turn)
  uint16_t *pre_s;    // [nwords]
  uint64_t *bm_lvl;   // [kRouteLevels][nwords] routing pass: servers of the routed group with at most (level) decodes
  uint16_t *pre_lvl;  // [kRouteLevels][nwords] exclusive prefix popcounts of bm_lvl, per level
  uint16_t *pre_c;    // [nwords] exclusive prefix popcounts of bm_comp; in the space of pre_lvl
  uint16_t *pre;      // [nwords] exclusive prefix popcounts of bm_idle (read until the pass's last segment ends)
  uint16_t *adm;      // [kAdmChunk] class | sequence-in-class << 3 of each admission
  uint32_t *lh;       // [2][kLoadBins] servers per decode count: solo group, mixed group
  uint16_t *ev_g;     // [waves][kEvPerWave] servers queued by a wave: at their event, or given work
  uint32_t *ev_t;     // [N] time of the server's event, bits 8..39 of the nanoseconds
  uint32_t *ev_it;    // [N] iterations the server has completed by then (while idle: has completed), bits 0..29;
                      //     kEvChunk: the iterations up to then carry a prefill chunk, kEvFin: a decode ends then
  uint8_t *loads;     // [N] decodes per server
  uint8_t *ev_lo;     // [N] time of the event, bits 0..7
  uint16_t *rem;      // [Mp] prompt tokens left of the prefill in service (0: none) when the running phase began
  uint64_t *ta;       // [TA_TBT + K, K even or one more][kTallyRows] sums of the executed iterations (enum TallySum)
  uint32_t *live_off; // [K][kAdmChunk] abandonment only: ring offset from the head of the m-th waiting request of a class
  // weighted router only: the class selections of a routing pass
  uint32_t *sel_u;    // [kJobsLds] random word of each selection
  uint16_t *sel_co;   // [kJobsLds] class | (how many selections before it chose the same class) << 3
  uint16_t *sel_j;    // [kJobsLds] list position of each selection, ordered by class, then by order within the class
  int32_t *sel_n;     // [8] requests the pass takes from the solo group's buffer, per class
  size_t bytes;       // of the whole block
};

// Carves the dynamic LDS block; 8-byte granules. NWS > 0: the arrays indexed by 64-server word are sized for NWS
// words and the per-wave arrays for sixteen waves, whatever the configuration has; every array but the per-server
// ones and those behind them then sits at an offset the compiler knows (an immediate in the LDS instruction)
// instead of one it has to keep in a register, or to spill and fetch back, at every access. Used for the
// workgroups of sixteen waves (N up to 64 NWS servers). NWS = 0: everything sized by the configuration.
// Whether workgroups of this size have the bitmaps that overlapping steps take in turn (see kOverlap in the step kernel).
__host__ __device__ constexpr bool steps_overlap(int threads) { return threads >= 512; }
constexpr int kMostWordsEight = 80;   // words of a workgroup of up to eight waves
constexpr int kStaticWordsLarge = kMaxN / 64;   // any N the library accepts
constexpr int kStaticWordsMedium = 160;          // N up to 10240: three kilobytes less
template <int NWS, bool SMALL = false>
__host__ __device__ __forceinline__ Lds lds_carve(const Params &p, unsigned char *base)
{
  constexpr int kJobsLds = SMALL ? kJobsLdsSmall : gnr::kJobsLds;             // (these shadow the large tables' sizes)
  constexpr int kAdmChunk = SMALL ? kAdmChunkSmall : gnr::kAdmChunk;
  Lds L;
  size_t off = 0;
  const size_t nw = NWS ? static_cast<size_t>(NWS) : static_cast<size_t>(p.nwords);
  const size_t waves = NWS ? 16u : static_cast<size_t>(p.threads / 64);
  const size_t turns = steps_overlap(static_cast<int>(64 * waves)) ? 2 : 1;   // bitmaps that steps take in turn
  const size_t nw_m = NWS ? nw : static_cast<size_t>((p.Mp + 63) / 64);   // words with servers that may hold a prefill
#define GNR_TAKE(field, type, count)                       \
  L.field = reinterpret_cast<type *>(base + off);          \
  off += (sizeof(type) * static_cast<size_t>(count) + 7) & ~size_t(7);
  GNR_TAKE(tl, uint64_t, kTallyWords)
  GNR_TAKE(jobs, uint64_t, kJobsLds)
  GNR_TAKE(cs, int32_t, CS_WORDS)
  GNR_TAKE(acc, uint32_t, AC_WORDS)
  GNR_TAKE(cthr, uint32_t, 8)
  GNR_TAKE(gtab, double, 5 * kMaxK)
  GNR_TAKE(sc, int32_t, SC_WORDS)
  GNR_TAKE(adm, uint16_t, kAdmChunk)
  GNR_TAKE(lh, uint32_t, 2 * kLoadBins)
  GNR_TAKE(ev_g, uint16_t, waves * kEvPerWave)
  GNR_TAKE(bm_idle, uint64_t, nw)
  GNR_TAKE(bm_busy, uint64_t, (nw + 1) & ~size_t(1))
  GNR_TAKE(bm_others, uint64_t, turns > 1 ? (nw + 1) & ~size_t(1) : 0)
  GNR_TAKE(bm_just, uint64_t, turns * nw)
  GNR_TAKE(bm_lvl, uint64_t, kRouteLevels * nw)
  GNR_TAKE(bm_comp, uint64_t, turns * nw_m)
  const size_t nw_two = p.route_mode == SIM_ROUTE_RANDOM_SPLIT || p.route_mode == SIM_ROUTE_WEIGHTED_SPLIT ? nw : 0;
  GNR_TAKE(bm_solo, uint64_t, nw_two ? turns * nw_m : 0)
  GNR_TAKE(pre_s, uint16_t, nw_two)
  // the ranks of a pass's levels are formed when those of the completions are no longer read (a barrier lies between)
  GNR_TAKE(pre_lvl, uint16_t, kRouteLevels * nw)
  L.pre_c = L.pre_lvl;
  GNR_TAKE(pre, uint16_t, nw)
  GNR_TAKE(fresh, uint64_t, p.dl_rings && waves > 1 ? kJobsLds : 0)
  GNR_TAKE(ta, uint64_t, (TA_TBT + (NWS ? kMaxK : (p.K + 1) & ~1)) * (SMALL ? kTallyRowsSmall : kTallyRows))
  // What is refused for want of room, and how many workgroups share a compute unit, follows from the total. Both were set
  // with the tables of a kernel that executed every iteration (two words and a row list per queued server, four-byte
  // ranks, ...), and the total is theirs in every configuration: the tables above never need more (one and two waves go up
  // to 5120 servers), and where they need less the rest is held free: 14,128 bytes of 148,368 with 10000 servers of six
  // classes, 4,064 of 38,800 with 2048 of eight, 1,432 of 20,112 with 1024 of four. A few bytes more cost a round or half
  // the waves (200 steps: 33 servers of eight classes with patience, 4096 replications, 10248 bytes in two rounds 4.7 ms,
  // 10032 in one 3.1; 100 steps: 900 servers of eight classes with patience, 2048 replications, 20488 bytes in two rounds
  // 5.5 ms, 20424 in one 3.1).
  constexpr size_t held_fixed = sizeof(uint64_t) * (kTallyWords + kJobsLds) + sizeof(int32_t) * (CS_WORDS + SC_WORDS + kMaxK) +
                                sizeof(double) * 5 * kMaxK + 6 * kAdmChunk + sizeof(uint32_t) * 2 * kLoadBins;
  const size_t held = held_fixed + waves * (8 * (SMALL ? kHeldEvSmall : kEvPerWave) + 256) + 80 * nw + 2 * ((4 * (nw + 1) + 7) & ~size_t(7));
  off = off < held ? held : off;
  // from here on the offsets depend on the configuration
  GNR_TAKE(ev_t, uint32_t, p.N)
  GNR_TAKE(ev_it, uint32_t, p.N)
  GNR_TAKE(loads, uint8_t, p.N)
  GNR_TAKE(ev_lo, uint8_t, p.N)
  GNR_TAKE(rem, uint16_t, p.Mp)
  GNR_TAKE(tbth, uint64_t, p.K * p.tbt_w)
  GNR_TAKE(live_off, uint32_t, p.dl_rings ? p.K * kAdmChunk : 0)
  GNR_TAKE(sel_u, uint32_t, p.route_mode == SIM_ROUTE_WEIGHTED_SPLIT ? kJobsLds : 0)
  GNR_TAKE(sel_co, uint16_t, p.route_mode == SIM_ROUTE_WEIGHTED_SPLIT ? kJobsLds : 0)
  GNR_TAKE(sel_j, uint16_t, p.route_mode == SIM_ROUTE_WEIGHTED_SPLIT ? kJobsLds : 0)
  GNR_TAKE(sel_n, int32_t, p.route_mode == SIM_ROUTE_WEIGHTED_SPLIT ? 8 : 0)
#undef GNR_TAKE
  L.bytes = off + (nw_two ? 32 : 0);   // (held like the rest, with two buffers)
  return L;
}
// Size classes of the step kernel: 0 workgroups of one or two waves (small tables, arrays sized by the
// configuration), 1 up to 512 threads (arrays sized by the configuration), 2 and 3 sixteen waves with the
// word-indexed arrays sized for 160 words and for the largest N.
__host__ __device__ constexpr int size_class(int threads, int nwords)
{
  return threads <= 128 ? 0 : threads <= 512 ? 1 : (nwords <= kStaticWordsMedium ? 2 : 3);
}
// Waves of an instantiation that are guaranteed to fit a SIMD together (the compiler keeps its registers within
// 512 / this many). A workgroup of 1024 threads needs four; the smaller classes are compiled twice: roomy, with up
// to 256 registers and two waves per SIMD, taken while every workgroup of the launch finds a place at that density, and
// dense, with 128 registers and four waves per SIMD, for launches that would otherwise run their workgroups in more
// rounds. Registers roomy / dense (spilled when dense): base and randomized router, same-slot decode 107 to 113 in two waves and
// more and 117 to 121 in one, as many in either form; with deadline rings 118 to 127, in one wave 128 to 136 / 128 (up to 1);
// weighted router 136 to 139 / 128 (4) and in one wave 150 / 128 (8). Without deadline rings the two forms of one and of eight waves
// do the same, with a few spilled scalars more or less; those of two and four waves differ in their priorities (kChainFirst).
__host__ __device__ constexpr int waves_per_simd(int max_threads, bool dense)
{
  return max_threads > 512 || dense ? 4 : 2;
}
__host__ __device__ constexpr int static_words(int size_class)
{
  return size_class <= 1 ? 0 : (size_class == 2 ? kStaticWordsMedium : kStaticWordsLarge);
}

// How many of a workgroup's waves, the last ones, work off the events. With draws beside them (10000 servers, 10, 11 and 12 of sixteen
// waves 13.57, 13.61 and 13.42 ms per 1000 steps; 3001 servers, 8, 10 and 12 of them 4.464, 4.481 and 4.459 per 500) twelve of
// sixteen; of eight half, with more than eight words a wave five.
__host__ __device__ __forceinline__ constexpr int event_waves(int nwaves, bool beside, int nwords)
{
  return !beside ? nwaves : nwaves == 16 ? 12 : nwords > 8 * nwaves ? nwaves * 11 / 16 : nwaves / 2;
}

// A wave looks at the pairs of bitmap words scan_first, scan_first + scan_stride, ... below scan_end (and below the last one) in a completion
// pass: the last n_drain waves share all of them, unless steps overlap and the last n_serve waves serve the step before. Where the others are
// three times as many these look at all words, else, where the events are not shared by all waves (`beside`), at two pairs for one of the waves
// that serve (10000 x 256, four or five of twelve serve), which have the last pairs. What does not divide falls to the waves that serve: a wave
// with more than 64 events takes twice as long. `rounded_up`: npairs over share.
// (The kernel and the check below have these statements in common as a macro: as a function, whichever way it was passed what it reads and writes,
// it left the kernel with other registers throughout; eight waves, base router, took 0.6 to 1 % longer.)
#define GNR_OVERLAPPING_SCAN(beside, rounded_up)                                                             \
  const int n_busy = n_serve < n_drain ? n_serve : n_drain, n_free = n_drain - n_busy;                       \
  const bool serves = wave >= nwaves - n_busy, some = n_free < 3 * n_busy;                                   \
  if (!some || beside) {                                                                                     \
    const int npairs = (nwords + 1) >> 1, share = 2 * n_free + n_busy;                                       \
    const int each = rounded_up;                                                                             \
    const int ends_at = !some ? npairs : npairs - n_busy * uniform(each);                                    \
    if (!serves) {                                                                                           \
      scan_stride = n_free;                                                                                  \
      scan_end = ends_at > 0 ? ends_at : 0;                                                                  \
    } else {                                                                                                 \
      scan_stride = n_busy;                                                                                  \
      scan_first = (ends_at > 0 ? ends_at : 0) + wave - (nwaves - n_busy);                                   \
    }                                                                                                        \
  }

struct Scan { int first, stride, end; };
// The same on the host: the pairs of the last n_drain of `nwaves` waves while the last n_serve serve (0: no steps overlap).
constexpr Scan scan_of(int wave, int nwaves, int nwords, int n_drain, int n_serve, bool beside)
{
  int scan_first = wave - (nwaves - n_drain), scan_stride = n_drain, scan_end = (nwords + 1) >> 1;
  auto uniform = [](int v) constexpr { return v; };
  if (n_serve > 0) {
    GNR_OVERLAPPING_SCAN(beside, (npairs + share - 1) / share)
  }
  return {scan_first, scan_stride, scan_end};
}

// What others have been given is noted for one round of the completion pass (bm_others): no wave may have more pairs than that.
constexpr int kPairsARound = 16;
constexpr bool a_round_is_enough(int nwaves, bool beside, int most_words)
{
  for (int words = 1; words <= most_words; ++words) {
    const int n_drain = event_waves(nwaves, beside, words);
    for (int n_serve = 0; n_serve <= n_drain; ++n_serve)   // (where more serve it is as with those)
      for (int wave = nwaves - n_drain; wave < nwaves; ++wave) {
        const Scan mine = scan_of(wave, nwaves, words, n_drain, n_serve, beside);
        if (mine.end - mine.first > kPairsARound * mine.stride) return false;
      }
  }
  return true;
}

// Bits of bitmap word w that belong to servers below `nbits`.
__device__ __forceinline__ uint64_t bits_below(int w, int nbits)
{
  const int left = nbits - (w << 6);
  return left >= 64 ? ~0ull : (left <= 0 ? 0ull : (1ull << left) - 1ull);
}

// Exclusive prefix popcounts of the first `nbits` bits of a bitmap, computed by one whole wave; returns the
// total in every lane.
__device__ __forceinline__ uint32_t rank_bitmap(const uint64_t *bm, uint16_t *pre, int nwords, int nbits)
{
  const int lane = threadIdx.x & 63;
  uint32_t running = 0;
  for (int base = 0; base < nwords; base += 64) {
    const int w = base + lane;
    const uint32_t v = w < nwords ? static_cast<uint32_t>(__popcll(bm[w] & bits_below(w, nbits))) : 0u;
    const uint32_t inc = wave_incl_scan(v);
    if (w < nwords) pre[w] = static_cast<uint16_t>(running + inc - v);
    running += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), 63));
  }
  return running;
}

// The same value of the lane that a data-parallel-primitive control pairs this one with.
template <int CTRL>
__device__ __forceinline__ double dpp_of(double v)
{
  const int64_t b = __double_as_longlong(v);
  const int lo = static_cast<int>(b), hi = static_cast<int>(b >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false), h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false);
  return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(static_cast<uint32_t>(h2)) << 32) | static_cast<uint32_t>(l2)));
}
// Sum, least and largest over groups of 2, 4 or 8 neighbouring lanes (lg = 1, 2, 3, wave-uniform); every lane gets it.
__device__ __forceinline__ uint32_t group_sum(uint32_t v, int lg)
{
  v = dpp_add<0xB1, 0xF>(v);               // quad_perm [1,0,3,2]
  if (lg > 1) v = dpp_add<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
  if (lg > 2) v = dpp_add<0x141, 0xF>(v);  // row_half_mirror
  return v;
}
__device__ __forceinline__ double group_min(double v, int lg)
{
  v = fmin(v, dpp_of<0xB1>(v));
  if (lg > 1) v = fmin(v, dpp_of<0x4E>(v));
  if (lg > 2) v = fmin(v, dpp_of<0x141>(v));
  return v;
}
__device__ __forceinline__ double readlane_f64(double v, int l)
{
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(b), l));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(b >> 32), l));
  return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}

// Adds the tallies of executed iterations to the workgroup's totals: per lane
// m executed iterations of duration d whose batch held the per-class decode counts `comp`; lanes with
// nothing to tally pass m = 0. Every lane adds to the running sums in LDS itself, each sum being spread over kTallyRows
// words, so that at most 64 / kTallyRows lanes meet on one: a lane pays three instructions a sum, where the sum over the wave
// that stood here before cost forty each, twenty-four sums a call with six classes (a quarter of all vector
// instructions of a step; 10000 servers, 256 replications, 1000 steps: 32.0 -> 30.5 ms). Folded when the launch ends.
// The counts of two classes share a word, and a class without decodes adds zeros: a pair of classes takes fourteen instructions
// without a branch where it took two branches and twenty-six (2048 servers of eight classes x 1024 17.24 -> 16.94 ms per 1000
// steps, 10000 x 256 16.76 -> 16.41, randomized router 6.71 -> 6.58 per 300, 256 x 1024 8.51 -> 8.39; with the bins taken from doubles).
template <int ROWS>
__device__ __forceinline__ void tally_iterations(uint64_t *ta, uint64_t *tbth, int tbt_w, int tbt_lo, int K, uint32_t m,
                                                 uint32_t d, bool chunk, uint64_t comp)
{
  if (m == 0) return;
  const uint64_t md = static_cast<uint64_t>(m) * d;   // < 2^16 * 2^31
  uint64_t *mine = ta + (threadIdx.x & (ROWS - 1));
  uint64_t *kind = mine + (chunk ? ROWS : 0);
  lds_add64(&kind[TA_ITERS * ROWS], m);
  lds_add64(&kind[TA_BUSY * ROWS], md);
  uint64_t *bin = tbth + (hbin32(d) - tbt_lo);
  // (taken anew, else the comparisons below are kept in lanes of vector registers from one step to the next)
  asm volatile("" : "+s"(K));
  // Two classes at a time (one that does not exist has no decodes), their counts in one word: an iteration is no shorter than a
  // step and a launch has kStepsPerLaunch of those, so a class emits fewer than 2^32 tokens in it.
#pragma unroll
  for (int k = 0; k < kMaxK; k += 2) {
    if (k < K) {   // wave-uniform
      const uint32_t c0 = __umul24(m, byte_at(comp, k)), c1 = __umul24(m, byte_at(comp, k + 1));
      lds_add64(&mine[(TA_TBT + k) * ROWS], static_cast<uint64_t>(c0) * d);
      lds_add64(&mine[(TA_TBT + k + 1) * ROWS], static_cast<uint64_t>(c1) * d);
      lds_add64(&bin[(k >> 1) * tbt_w], (static_cast<uint64_t>(c1) << 32) | c0);
    }
  }
}


// Sort key of a gate candidate: the m-th waiting request of class k (m counted from the head).
// Occupancy gate: (X_k + m - n x_k*)/x_k*, ties by the larger queue deviation Q_k - m - n q_k*;
// priority gate: larger static index first; FCFS gate: older arrival stamp first.
// Ties that remain go to the lower class. Within a class the key does not decrease with m, so the
// gate's one-at-a-time argmin is the merge of the classes' sequences in this order.
struct GateKey { double a, b; };

// `live_off` (abandonment only, else null): ring offset of the m-th request of class k that still waits.
// The gate's targets live in an LDS table for the launch, [5][kMaxK]: n x*, 1/x*, x*, n q*, priority index (a copy
// of the parameter block's, which would be read through the scalar cache, a long round trip, at every comparison of
// the ranking loops). The values of one class are fetched together, once, before they are used.
enum GateTab { GT_NX = 0, GT_INVX = 1, GT_XSTAR = 2, GT_NQ = 3, GT_PRIO = 4 };
struct ClassTargets { double nx, invx, xstar, nq, prio; };
__device__ __forceinline__ ClassTargets load_targets(const double *tab, int k)
{
  ClassTargets t;
  t.nx = tab[GT_NX * kMaxK + k]; t.invx = tab[GT_INVX * kMaxK + k]; t.xstar = tab[GT_XSTAR * kMaxK + k];
  t.nq = tab[GT_NQ * kMaxK + k]; t.prio = tab[GT_PRIO * kMaxK + k];
  return t;
}
// Arrival step of the m-th waiting request of class k; head_k: ring position of the class queue's head, fresh_k: entries
// from there on that are of steps before `now` (the others are this step's arrivals, which another wave may be writing).
__device__ __forceinline__ uint32_t gate_stamp(const uint32_t queue_cap, const uint32_t *qring, const uint32_t *live_off,
                                               uint32_t head_k, uint32_t fresh_k, uint32_t now, int k, int m, int adm_chunk)
{
  const uint32_t off = live_off ? live_off[k * adm_chunk + m] : static_cast<uint32_t>(m);
  uint32_t pos = head_k + off;
  if (pos >= queue_cap) pos -= queue_cap;
  return off < fresh_k ? qring[static_cast<size_t>(k) * queue_cap + pos] : now;
}
// Key of the m-th waiting request of class k, of which X_k = xs_k are in prefill and Q_p,k = qp_k wait; head_k,
// fresh_k, now: as for gate_stamp.
__device__ __forceinline__ GateKey gate_key(const int gate_mode, const uint32_t queue_cap, const ClassTargets &t,
                                            const uint32_t *qring, const uint32_t *live_off, int xs_k, int qp_k,
                                            uint32_t head_k, uint32_t fresh_k, uint32_t now, int k, int m, int adm_chunk)
{
  GateKey key;
  if (gate_mode == SIM_GATE_OCCUPANCY) {
    key.a = (static_cast<double>(xs_k + m) - t.nx) * t.invx;
    key.b = static_cast<double>(qp_k - m) - t.nq;
  } else if (gate_mode == SIM_GATE_PRIORITY) {
    key.a = -t.prio;
    key.b = 0.0;
  } else {
    key.a = static_cast<double>(gate_stamp(queue_cap, qring, live_off, head_k, fresh_k, now, k, m, adm_chunk));
    key.b = 0.0;
  }
  return key;
}

// true if candidate (k1, key1) is admitted before candidate (k2, key2), k1 != k2
__device__ __forceinline__ bool gate_before(const GateKey &x, int k1, const GateKey &y, int k2)
{
  if (x.a != y.a) return x.a < y.a;
  if (x.b != y.b) return x.b > y.b;
  return k1 < k2;
}

// The end of a server's prefill, kept until the lane has left the divergent part of the finishing code.
struct PrefillEnd { bool done; int k; uint32_t P; int64_t ttft; uint64_t nc; };

// ------------------------------------------------------------------ step kernel ----
// A server whose batch does not change runs identical iterations, so nothing is done for them one by one. What is kept
// is the server's next event: the end of the iteration at which its batch may change, because a decode ends there, a
// phase of its prefill ends there (the run of full chunks, then the last chunk) or work that arrived in the middle of an
// iteration joins there. Between the last event and the next the batch, and with it the iteration time, is fixed: the
// iterations completed by any time follow from the event time by one division, and they are tallied with their
// multiplicity when the event comes, when the batch is changed at an iteration boundary before it, or when the launch
// ends. A step therefore reads one clock per server, and a record and a slot row only where an event has come. On
// 10000 servers x 256 replications with full batches this took a step from 86 us (every due server's slot row read,
// 27 % of the rows a step, 6.2 TB/s while it lasted) to 42 us.
// The arrays of the simulation state, handed to the step kernel by value: pointers that arrive as kernel
// arguments are known to point to global memory, so their loads and stores are plain global accesses
// (counted apart from LDS traffic) instead of generic ones that a wait on LDS would also wait for.
struct StepArrays {
  const uint32_t *arr_thr;
  const uint16_t *len_tab;
  ServerRec *rec;
  uint32_t *t_rel, *remptok;
  uint32_t *fin;
  uint64_t *job;
  uint32_t *qring;
  uint64_t *dring;
  int32_t *cstate;
  uint64_t *tally, *hist;
  // abandonment only
  const uint16_t *pat_tab;
  uint32_t *qdl, *ddl, *cal, *dcal;
  // randomized router only
  uint64_t *dring_m;
  uint32_t *ddl_m, *dcal_m;   // ... with abandonment
};

// AB: the variant with abandonment (some class has a patience rate). Ring entries then carry the step at whose
// start the request leaves if it still waits. Such entries stay in the rings as dead entries until the head
// passes them: the counters Q_p, Q_d follow the abandonments eagerly through per-step calendars, the gate and
// the router skip dead entries when they take requests, and a ring is compacted when it would not hold the
// step's appends and at the end of every launch (so the state between launches holds waiting requests only).
// RR: the variant with the randomized decode router: every completed prefill is sent to the solo or to the
// mixed group by a random word, each group has its own buffer ring and is fed from that ring only. A routing
// pass then takes jobs from both rings: the staged list holds the solo ring's jobs first.
// IM: the variant with immediate same-slot decode (no router): a request whose prefill ends goes on decoding on
// its own server, placed there by the lane that finishes the server; a server is offered to the gate while it
// holds no prefill and fewer than B decodes.
template <int NT, int NWS, bool AB, bool RR, bool IM, bool WS = false, bool DENSE = false, bool BESIDE = NT == 1024 || (NT == 512 && IM)>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(waves_per_simd(NT, DENSE)))) gnr_step_kernel(const Params *__restrict__ params, const StepArrays a,
                                                        const uint32_t key0_arg, const uint32_t key1_arg,
                                                        const uint32_t step_begin_arg, const uint32_t n_steps_arg)
{
  const uint32_t key0 = pinned(key0_arg), key1 = pinned(key1_arg), step_begin = pinned(step_begin_arg), n_steps = pinned(n_steps_arg);
  const Params &p = *params;   // immutable after creation; read through the scalar cache on demand
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr bool SMALL = NT <= 128;
  constexpr int kJobsLds = SMALL ? kJobsLdsSmall : gnr::kJobsLds;             // (these shadow the large tables' sizes)
  constexpr int kAdmChunk = SMALL ? kAdmChunkSmall : gnr::kAdmChunk;
  constexpr int kTallyRowsHere = SMALL ? kTallyRowsSmall : kTallyRows;
  const Lds L = lds_carve<NWS, SMALL>(p, lds_raw);

  const int r = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // wave-uniform values are made scalar explicitly, so that loops and branches on them are scalar too
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int nwaves = NT >> 6;
  const int wave_base = wave << 6;
  // The instruction arbiter of a SIMD prefers its oldest wave: left alone, the first four waves of the workgroup
  // finish every sweep early and the last four late, and the barrier waits for those. Raising the priority of the
  // younger waves evens this out. Workgroups of up to four waves share their SIMDs with others of their kind: the draw of the
  // next step's arrivals has a lower priority than the rest (nobody waits for it as long as another wave serves), and
  // workgroups that follow one another by as many as there are compute units (256), and so come to share one, take turns at
  // a higher one. Left to the order of their age the youngest end last, alone with the SIMD: 1024 servers x 2048
  // replications 18.4 -> 17.9 ms per 1000 steps, 256 x 1024 9.42 -> 9.19, 2048 x 1024 18.6 -> 18.1 (turns of 128 steps the same,
  // of 16 steps half of it).
  // With sixteen waves the waves that draw (the first ones, which have time left) come last and those that serve first, at the highest
  // priority while they do: 10000 servers x 256 13.83 -> 13.63 ms per 1000 steps. In eight that all work off the events those that
  // serve have it and the others none before one another: convergence instance 17.76 -> 17.57 per 2000; where some of eight draw they
  // gain nothing by either (same-slot decode 14.31 -> 14.49) and keep the order of their age.
  constexpr bool kDrawLast = NT == 1024, kEqual = NT == 512 && !BESIDE, kServeFirst = kDrawLast || kEqual;
  // Four waves a SIMD, of workgroups of two and four: what follows the events, short segments that others wait for, goes before the
  // events and draws of the other workgroups (500 servers x 2000 3.32 -> 3.19 ms per 300 steps, 900 x 1000 same-slot decode 3.40 -> 3.30,
  // 1500 x 1800 randomized router 9.32 -> 9.15, 1024 x 2048 16.14 -> 16.05 per 1000, 2048 x 1024 16.18 -> 16.11; with two waves a
  // SIMD 256 x 1024 8.17 -> 8.37).
  constexpr bool kChainFirst = DENSE && NT >= 128 && NT <= 256;
  const int nwords_all = p.nwords;
  constexpr bool kBeside = BESIDE;   // some waves draw while the others work off the events
  const int n_drain = !kBeside || nwaves == 16 ? event_waves(nwaves, kBeside, 0) : event_waves(nwaves, kBeside, nwords_all);   // (mostly a constant)
  const int n_draw = nwaves - n_drain, drain_first = n_draw;
  uint32_t turn = 0;   // in workgroups of two to four waves
  auto own_priority = [&]() __attribute__((always_inline)) {
    if (kEqual) __builtin_amdgcn_s_setprio(1);
    else if (kDrawLast) {
      if (wave >= 12) __builtin_amdgcn_s_setprio(2);
      else if (wave >= n_draw) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
    } else if (turn) __builtin_amdgcn_s_setprio(2);
    else if (wave >= 4 || nwaves <= 4) __builtin_amdgcn_s_setprio(1);
  };
  own_priority();
  int K = pinned(p.K), N = pinned(p.N), B = pinned(p.B), M = pinned(p.M), BS = pinned(p.BS);
  const int nper = (N + NT - 1) / NT;
  int nwords = pinned(p.nwords);
  // Servers 0..M-1 are the mixed group for the gate and the router. Servers below Mp >= M may hold a prefill:
  // Mp is the largest M the run has had (a prefill in service stays when its server turns solo).
  int Mp = pinned(p.Mp);
  int nwords_m = (Mp + 63) >> 6;   // bitmap words that hold servers with prefill state
  // Iteration-time coefficients, chunk size and step length in ns (each below 2^31: the longest iteration is),
  // window of the on-chip time-between-tokens histogram, class thresholds of the arrival draw: used in every block.
  const uint32_t c0_ns = pinned(static_cast<uint32_t>(p.c0)), cpre_ns = pinned(static_cast<uint32_t>(p.cpre));
  const uint32_t cdec_ns = pinned(static_cast<uint32_t>(p.cdec)), dt_ns = pinned(static_cast<uint32_t>(p.dt));
  const int chunk_max = static_cast<int>(pinned(static_cast<uint32_t>(p.C)));
  const int tbt_w = static_cast<int>(pinned(static_cast<uint32_t>(p.tbt_w))), tbt_lo = static_cast<int>(pinned(static_cast<uint32_t>(p.tbt_lo)));
  int gate_mode = static_cast<int>(pinned(static_cast<uint32_t>(p.gate_mode)));
  const uint32_t queue_cap = pinned(p.queue_cap), dbuf_cap = pinned(p.dbuf_cap);

  const uint32_t *arr_thr = pinned(a.arr_thr);
  const uint16_t *len_tab = pinned(a.len_tab), *pat_tab = AB ? pinned(a.pat_tab) : nullptr;
  ServerRec *rec = pinned(a.rec + static_cast<size_t>(r) * N);
  uint32_t *t_rel = pinned(a.t_rel + static_cast<size_t>(r) * N);
  uint32_t *remptok = pinned(a.remptok + static_cast<size_t>(r) * N);
  uint32_t *fin = pinned(a.fin + static_cast<size_t>(r) * N * BS);
  uint64_t *job = pinned(a.job + static_cast<size_t>(r) * N * BS);
  uint32_t *qring = pinned(a.qring + static_cast<size_t>(r) * K * queue_cap);
  uint64_t *dring = pinned(a.dring + static_cast<size_t>(r) * dbuf_cap);
  uint64_t *hist = pinned(a.hist + static_cast<size_t>(r) * 3 * K * kNBin);
  uint16_t *ev_g = L.ev_g + wave * kEvPerWave;
  // abandonment only
  const uint32_t cal_n = p.cal_mask + 1u;
  uint32_t *qdl = AB ? pinned(a.qdl + static_cast<size_t>(r) * K * queue_cap) : nullptr;
  uint32_t *ddl = AB ? pinned(a.ddl + static_cast<size_t>(r) * dbuf_cap) : nullptr;
  uint32_t *cal = AB ? pinned(a.cal + static_cast<size_t>(r) * K * cal_n) : nullptr;
  uint32_t *dcal = AB ? pinned(a.dcal + static_cast<size_t>(r) * K * cal_n) : nullptr;
  const uint32_t *lo_tab = AB ? L.live_off : nullptr;
  uint64_t *dring_m = RR ? pinned(a.dring_m + static_cast<size_t>(r) * dbuf_cap) : nullptr;
  uint32_t *ddl_m = AB && RR ? pinned(a.ddl_m + static_cast<size_t>(r) * dbuf_cap) : nullptr;
  uint32_t *dcal_m = AB && RR ? pinned(a.dcal_m + static_cast<size_t>(r) * K * cal_n) : nullptr;

  // ---- load the replication's class state and rebuild the on-chip views of the server state
  for (int i = tid; i < CS_WORDS; i += NT) L.cs[i] = a.cstate[static_cast<size_t>(r) * CS_WORDS + i];
  for (int i = tid; i < kTallyWords; i += NT) L.tl[i] = 0;
  for (int i = tid; i < (K + 1) / 2 * p.tbt_w; i += NT) L.tbth[i] = 0;
  for (int i = tid; i < (TA_TBT + ((K + 1) & ~1)) * kTallyRowsHere; i += NT) L.ta[i] = 0;
  for (int i = tid; i < SC_WORDS; i += NT) L.sc[i] = 0;
  for (int i = tid; i < AC_WORDS; i += NT) L.acc[i] = 0;
  // an arrival's class is the number of thresholds its random word has reached; classes beyond K-1 do not exist:
  // their thresholds are the largest word, and the count is capped
  if (tid < kMaxK) L.cthr[tid] = tid + 1 < K ? p.cls_thr[tid] : 0xFFFFFFFFu;
  if (tid < kMaxK) {
    L.gtab[GT_NX * kMaxK + tid] = tid < K ? p.nx[tid] : 0.0;
    L.gtab[GT_INVX * kMaxK + tid] = tid < K ? p.invx[tid] : 0.0;
    L.gtab[GT_XSTAR * kMaxK + tid] = tid < K ? p.xstar[tid] : 0.0;
    L.gtab[GT_NQ * kMaxK + tid] = tid < K ? p.nq[tid] : 0.0;
    L.gtab[GT_PRIO * kMaxK + tid] = tid < K ? p.prio[tid] : 0.0;
  }
  for (int i = tid; i < 2 * kLoadBins; i += NT) L.lh[i] = 0;
  __syncthreads();
  if constexpr (AB) {   // between launches the rings hold waiting requests only
    if (tid < K) L.sc[SC_QLEN + tid] = L.cs[CS_QP + tid];
    if (tid == 0) {
      L.sc[SC_DLEN] = L.cs[CS_DCOUNT];
      if constexpr (RR) L.sc[SC_DLEN_M] = L.cs[CS_DCOUNT_M];
    }
  }
  // ---- a server's clock: the time of its event, 40 bits of the nanoseconds (an event is never set further ahead than
  //      2^38 ns: an early one only tallies and is set again)
  auto iteration_ns = [&](int ptok, uint32_t nd) __attribute__((always_inline)) -> uint32_t {   // below 2^31
    return c0_ns + cpre_ns * static_cast<uint32_t>(ptok) + cdec_ns * nd;
  };
  auto chunk_of = [&](int rem) __attribute__((always_inline)) -> int { return rem < chunk_max ? rem : chunk_max; };
  auto event_time = [&](int g, int64_t X) __attribute__((always_inline)) -> int64_t {   // relative to X
    return (static_cast<int64_t>(static_cast<int32_t>(L.ev_t[g] - static_cast<uint32_t>(X >> 8))) << 8) +
           (static_cast<int>(L.ev_lo[g]) - static_cast<int>(X & 255));
  };
  auto set_event = [&](int g, int64_t t, uint32_t it, bool chunk, bool fin_ev) __attribute__((always_inline)) {
    L.ev_t[g] = static_cast<uint32_t>(t >> 8);
    L.ev_lo[g] = static_cast<uint8_t>(t & 255);
    L.ev_it[g] = it | (chunk ? kEvChunk : 0u) | (fin_ev ? kEvFin : 0u);
  };
  // Work that a server was given in the middle of an iteration joins at its end, and that is the server's event then. Such a
  // server has decodes that are not yet in the batch, or a prefill that the running iteration does not carry.
  auto joins_next = [](uint64_t nj, int rem, bool chunk) __attribute__((always_inline)) { return nj != 0 || (rem > 0 && !chunk); };
  // How many iterations like the next one (`nd` decodes, a chunk of `rem` prompt tokens left, d ns long) a server runs
  // before its batch may change; `to_fin`: iterations up to the first end of one of its decodes.
  auto phase_length = [&](uint32_t nd, int rem, uint32_t d, uint32_t to_fin) __attribute__((always_inline)) -> uint32_t {
    uint32_t n = static_cast<uint32_t>(274877906944.0f * __builtin_amdgcn_rcpf(static_cast<float>(d)));   // 2^38 ns
    n = n < 65535u ? n : 65535u;   // (at least 137: an iteration is at most 2e9 ns long)
    if (nd && to_fin < n) n = to_fin;
    if (rem > 0) {   // the full chunks before the last one, or the last one
      uint32_t full = 1;
      if (rem > chunk_max) {
        const uint32_t left = static_cast<uint32_t>(rem - 1), c = static_cast<uint32_t>(chunk_max);
        full = static_cast<uint32_t>(static_cast<float>(left) * __builtin_amdgcn_rcpf(static_cast<float>(c)));
        if ((full + 1u) * c <= left) ++full;
        if (full * c > left) --full;
      }
      if (full < n) n = full;
    }
    return n;
  };
  constexpr bool kOverlap = steps_overlap(NT);
  static_assert(!kOverlap || a_round_is_enough(nwaves, kBeside, NT == 1024 ? NWS : kMostWordsEight), "pairs of words a wave looks at");
  // bitmaps that steps take in turn where they overlap: how far apart they are
  const int turn_words = !kOverlap ? 0 : NWS ? NWS : nwords, turn_words_m = !kOverlap ? 0 : NWS ? NWS : nwords_m;
  // classes that the gate may admit: under the occupancy gate those with a positive target
  const uint64_t admissible = __ballot(lane < K && (gate_mode != SIM_GATE_OCCUPANCY || L.gtab[GT_INVX * kMaxK + (lane & (kMaxK - 1))] > 0.0));
  auto bits64 = [](uint64_t *p) __attribute__((always_inline)) { return reinterpret_cast<unsigned long long *>(p); };

  // (what the next round reads is asked for a round ahead)
  struct Stored { uint64_t nc, nj; uint32_t it, nf, tr, pk; };
  auto stored = [&](int g) __attribute__((always_inline)) -> Stored {
    Stored v = {0, 0, 0, 0, kIdleRel, 0};
    if (g < N) {
      v.nc = rec[g].n_cls; v.nj = rec[g].n_join; v.it = rec[g].iter; v.nf = rec[g].next_fin;
      v.tr = t_rel[g];
      if (g < Mp) v.pk = remptok[g];
    }
    return v;
  };
  Stored asked = stored(tid);
  for (int i = 0; i < nper; ++i) {
    const int g = i * NT + tid;
    const bool valid = g < N;
    bool busy = false, idle_slot = false;
    const Stored have = asked;
    asked = stored(g + NT);
    if (valid) {
      const uint64_t nc = have.nc, nj = have.nj;
      const uint32_t it = have.it, nf = have.nf, tr = have.tr;
      const uint32_t nd = byte_sum(nc);
      L.loads[g] = static_cast<uint8_t>(nd);
      atomicAdd(&L.lh[(g < M ? kLoadBins : 0) + nd], 1u);
      int rem = 0, ptok = 0;
      if (g < Mp) {   // the prompt tokens left stay in LDS during the launch
        rem = pk_rem(have.pk);
        ptok = pk_ptok(have.pk);
        L.rem[g] = static_cast<uint16_t>(rem);
        idle_slot = rem == 0 && (!IM || static_cast<int>(nd) < B);
      }
      busy = tr != kIdleRel;
      const int64_t start = static_cast<int64_t>(step_begin) * dt_ns;   // the boundary the launch begins at
      if (busy) {
        const uint32_t d = iteration_ns(ptok, nd);
        const uint32_t n = joins_next(nj, rem, ptok > 0) ? 1u : phase_length(nd, ptok > 0 ? rem : 0, d, nf - it);
        set_event(g, start + tr + static_cast<int64_t>(n - 1u) * d, it + n, ptok > 0, nd && nf == it + n);
      } else {
        set_event(g, start, it, false, false);
      }
    }
    const uint64_t bi = __ballot(idle_slot), bb = __ballot(busy);
    const int wi = (i * NT + wave_base) >> 6;
    if (lane == 0 && wi < nwords) {
      L.bm_idle[wi] = bi; L.bm_busy[wi] = bb;
      L.bm_just[wi] = 0;
      L.bm_just[turn_words + wi] = 0;
      if constexpr (kOverlap) L.bm_others[wi] = 0;
      if (wi < nwords_m) {
        L.bm_comp[wi] = 0;
        L.bm_comp[turn_words_m + wi] = 0;
        if constexpr (RR) { L.bm_solo[wi] = 0; L.bm_solo[turn_words_m + wi] = 0; }
      }
    }
  }
  if (tid == 0 && (nwords & 1)) L.bm_busy[nwords] = 0;   // (clocks are looked at for two words at a time)
  __syncthreads();

  // ---- abandonment only: ring compaction, one wave per ring. Entries whose deadline is not after `now` are
  //      dropped, the others keep their order and move towards the head (a lane never writes ahead of what
  //      the wave has read). `pending`: entries already counted in the ring length but not yet written.
  auto compact_queue = [&](int k, uint32_t now, uint32_t pending) __attribute__((always_inline)) {
    uint32_t *ring = qring + static_cast<size_t>(k) * queue_cap;
    uint32_t *dlr = qdl + static_cast<size_t>(k) * queue_cap;
    const uint32_t hd = static_cast<uint32_t>(L.cs[CS_QHEAD + k]);
    uint32_t n = static_cast<uint32_t>(L.sc[SC_QLEN + k]) - pending;
    if (n > queue_cap) n = queue_cap;   // (a ring never holds more; keeps every access inside it regardless)
    uint32_t w = 0;
    for (uint32_t off = 0; off < n; off += 64) {   // wave-uniform
      const uint32_t i = off + lane;
      uint32_t pos = hd + i;
      if (pos >= queue_cap) pos -= queue_cap;
      const uint32_t st = i < n ? ring[pos] : 0u, dl = i < n ? dlr[pos] : 0u;
      const bool live = i < n && dl > now;
      const uint64_t bal = __ballot(live);
      if (live) {
        uint32_t wp = hd + w + static_cast<uint32_t>(rank_in(bal));
        if (wp >= queue_cap) wp -= queue_cap;
        ring[wp] = st; dlr[wp] = dl;
      }
      w += static_cast<uint32_t>(__popcll(bal));
    }
    if (lane == 0) {
      uint32_t tail = hd + w;
      if (tail >= queue_cap) tail -= queue_cap;
      L.sc[SC_QLEN + k] = static_cast<int32_t>(w + pending);
      L.sc[SC_TAIL + k] = static_cast<int32_t>(tail);
    }
  };
  // (`mixed`: the mixed group's buffer ring of the randomized router)
  auto compact_buffer = [&](uint32_t now, bool mixed) __attribute__((always_inline)) {
    uint64_t *ring = mixed ? dring_m : dring;
    uint32_t *dlr = mixed ? ddl_m : ddl;
    const uint32_t hd = static_cast<uint32_t>(L.cs[mixed ? CS_DHEAD_M : CS_DHEAD]);
    uint32_t n = static_cast<uint32_t>(L.sc[mixed ? SC_DLEN_M : SC_DLEN]);
    if (n > dbuf_cap) n = dbuf_cap;
    uint32_t w = 0;
    for (uint32_t off = 0; off < n; off += 64) {   // wave-uniform
      const uint32_t i = off + lane;
      uint32_t pos = hd + i;
      if (pos >= dbuf_cap) pos -= dbuf_cap;
      const uint64_t jw = i < n ? ring[pos] : 0ull;
      const uint32_t dl = i < n ? dlr[pos] : 0u;
      const bool live = i < n && dl > now;
      const uint64_t bal = __ballot(live);
      if (live) {
        uint32_t wp = hd + w + static_cast<uint32_t>(rank_in(bal));
        if (wp >= dbuf_cap) wp -= dbuf_cap;
        ring[wp] = jw; dlr[wp] = dl;
      }
      w += static_cast<uint32_t>(__popcll(bal));
    }
    if (lane == 0) L.sc[mixed ? SC_DLEN_M : SC_DLEN] = static_cast<int32_t>(w);
  };

  // arrival thresholds of the step that is drawn next: the first three lanes hold them. Those of the one after it are asked for
  const uint32_t mod_rows = p.mod_period > 0xFFFFFFFFll ? 0xFFFFFFFFu : (p.mod_period > 0 ? static_cast<uint32_t>(p.mod_period) : 1u);
  uint32_t thr_ahead = arr_thr[3 * static_cast<size_t>(step_begin % mod_rows) + (lane < 2 ? lane : 2)];
  uint32_t mod_row = (step_begin + 1u) % mod_rows;
  uint32_t thr_asked = arr_thr[3 * static_cast<size_t>(mod_row) + (lane < 2 ? lane : 2)];   // of mod_row
  // what `n` steps leave in the class counters at their end enters the sums over steps
  auto add_step_sums = [&](int k, uint32_t n, int qp, int qd, int x, int ym, int ys) __attribute__((always_inline)) {
    lds_add64(&L.tl[k * kNTally + SIM_T_SUM_QP], static_cast<uint64_t>(n) * static_cast<uint32_t>(qp));
    lds_add64(&L.tl[k * kNTally + SIM_T_SUM_QD], static_cast<uint64_t>(n) * static_cast<uint32_t>(qd));
    lds_add64(&L.tl[k * kNTally + SIM_T_SUM_X], static_cast<uint64_t>(n) * static_cast<uint32_t>(x));
    lds_add64(&L.tl[k * kNTally + SIM_T_SUM_YM], static_cast<uint64_t>(n) * static_cast<uint32_t>(ym));
    lds_add64(&L.tl[k * kNTally + SIM_T_SUM_YS], static_cast<uint64_t>(n) * static_cast<uint32_t>(ys));
  };
  uint32_t ended = 0;   // steps that have ended with the class counters as they are, not yet in those sums

  // Quiet steps. A step without an arrival and without an event leaves everything as it is but for the clock: the gate and
  // the router went on in the step before until no slot or no request was left for them, and nothing has changed since
  // (in the first step of a launch it may have: the targets or the split). With a few servers most steps are like that
  // (8 servers of two classes: three of four), and going through all of a step costs a wave 9 thousand cycles. So the
  // only wave of a small workgroup looks for the next step in which anything happens: one random block per lane tells the
  // arrivals of 64 / servers steps. With more than 32 servers a block would tell those of one step only (2^lg_n lanes a step,
  // and `ahead` would be shifted by its whole width), and the search is left out: of the steps of two classes 33 % are quiet
  // with 33 servers and 13 % with 64 (58 % with 16, 36 % with 32), of four classes at 0.95 of the capacity 11 and 1.5 %.
  constexpr int kQuietServers = 32;
  const bool quiet_search = NT == 64 && N <= kQuietServers;
  const int lg_n = N <= 1 ? 0 : 32 - __clz(N - 1);   // a step's servers take 2^lg_n lanes
  uint64_t ahead = 0;       // servers with arrivals in the steps drawn ahead, the step to come in the lowest 2^lg_n bits
  int steps_ahead = 0;      // how many
  uint32_t requests = 0;    // this lane's requests in the step it has drawn: how many, and three bits of class number each
  auto class_of = [&](uint32_t word) __attribute__((always_inline)) -> int {
    int k = 0;
#pragma unroll
    for (int c = 0; c + 1 < kMaxK; ++c) k += word >= L.cthr[c];
    return k < K ? k : K - 1;
  };
  auto draw_block = [&](uint32_t sd) __attribute__((always_inline)) {   // steps sd, sd + 1, ...
    const uint32_t s_lane = sd + (static_cast<uint32_t>(lane) >> lg_n);
    const int g = lane & ((1 << lg_n) - 1);
    const uint32_t *thr = arr_thr + (mod_rows > 1u ? 3 * static_cast<size_t>(s_lane % mod_rows) : 0);
    const uint32_t thr0 = thr[0], thr1 = thr[1], thr2 = thr[2];
    uint32_t w[4];
    philox4x32_10(key0, key1, s_lane, 0u, static_cast<uint32_t>(g), static_cast<uint32_t>(r), w);
    requests = g < N && w[0] >= thr0 ? 1u + (w[0] >= thr1) + (w[0] >= thr2) : 0u;
    ahead = __ballot(requests != 0);
    requests |= static_cast<uint32_t>(class_of(w[1]) << 2 | class_of(w[2]) << 5 | class_of(w[3]) << 8);
    steps_ahead = 64 >> lg_n;
  };
  // ---- arrivals: one random block per server and step, word 0 -> count, words 1.. -> classes. Word 0 alone is worked out
  //      for every server (its last rounds take half the products), for 64 of them (a bitmap word) at a time, two words with the same
  //      round keys, and a step ahead; the few servers that get requests are queued and their blocks drawn in full, one a lane.
  //      In workgroups of sixteen waves, and of eight where step_form says so, some waves draw while the others work off the events (a
  //      wave with all the events of two has its lanes full: 10000 servers of six classes have 450 a step, 28 a wave); their requests
  //      are counted behind the barriers that follow. 10000 servers x 256 replications 18.3 -> 17.15 ms per 1000 steps, 3001 x 77 5.60
  //      -> 5.39 per 500, 500 x 3 with same-slot decode 19.4 -> 18.8 per 2000. In smaller workgroups, where the events are the longest
  //      part, and in eight waves, where serving is, all waves work off the events and those that do not serve draw
  //      beside the ones that do (draws beside the events: 1024 x 2048 in two waves 16.8 -> 17.8 ms, 2048 x 1024 in four 17.2 -> 17.6,
  //      convergence instance in eight 17.45 -> 18.71 per 2000).
  constexpr int kHits = NT <= 64 ? 2 : 1;
  uint64_t hits[kHits] = {};
  bool drawn = false;   // the step to come has been drawn (kBeside: by this wave, and its requests are not yet counted)
  // The words first, first + stride, ...: lane j of `hits` gets the servers of the j-th one that have requests. (One wave alone
  // may have more than 64: then also of the j + 64-th.)
  auto draw_words = [&](uint32_t sd, int first, int stride) __attribute__((always_inline)) {
    const uint32_t thr0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(thr_ahead), 0));
    // the random block's first round has the server in one product only; the other one is the same for all
    const uint64_t ps = static_cast<uint64_t>(0xD2511F53u) * sd;
    const uint32_t c2_1 = static_cast<uint32_t>(ps >> 32) ^ static_cast<uint32_t>(r) ^ key1, c3_1 = static_cast<uint32_t>(ps);
    int j = 0;
    // Many words a wave: four at a time, with the round keys formed anew in vector registers. (An instruction that reads a scalar
    // register takes the vector unit four cycles, an exclusive-or of three vector registers two and a half, measured; 10000
    // servers x 256 replications, 32 words a wave, 14.9 -> 14.7 ms per 1000 steps; with a few words a wave it gains nothing.)
    if constexpr (NT == 1024 && kBeside) {
      if (nwords > 8 * nwaves) {   // wave-uniform
        constexpr int kAtOnce = 4;
        // ... and the second round's products with what is the same for all
        const uint64_t b_2 = static_cast<uint64_t>(0xCD9E8D57u) * c2_1;
        const uint32_t n0_2 = static_cast<uint32_t>(b_2 >> 32) ^ (key0 + 0x9E3779B9u), n2_2 = c3_1 ^ (key1 + 0xBB67AE85u);
        for (; first + (j + 2) * stride < nwords; j += kAtOnce) {   // wave-uniform
          uint32_t c0[kAtOnce], c1[kAtOnce], c2[kAtOnce], c3[kAtOnce];
#pragma unroll
          for (int u = 0; u < kAtOnce; ++u) {
            const int word = first + (j + u) * stride;
            const uint64_t pg = static_cast<uint64_t>(0xCD9E8D57u) * static_cast<uint32_t>((word << 6) + lane);
            const uint64_t a_2 = static_cast<uint64_t>(0xD2511F53u) * (static_cast<uint32_t>(pg >> 32) ^ key0);
            c0[u] = static_cast<uint32_t>(pg) ^ n0_2;
            c1[u] = static_cast<uint32_t>(b_2);
            c2[u] = static_cast<uint32_t>(a_2 >> 32) ^ n2_2;
            c3[u] = static_cast<uint32_t>(a_2);
          }
          uint32_t k0 = key0 + 2u * 0x9E3779B9u, k1 = key1 + 2u * 0xBB67AE85u;
          asm volatile("" : "+v"(k0), "+v"(k1));
#pragma unroll
          for (int round = 3; round <= 10; ++round) {
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) {
              const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * c0[u];
              const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * c2[u];
              c0[u] = xor3(static_cast<uint32_t>(pb >> 32), c1[u], k0);
              c2[u] = xor3(static_cast<uint32_t>(pa >> 32), c3[u], k1);
              c1[u] = static_cast<uint32_t>(pb);
              c3[u] = static_cast<uint32_t>(pa);
            }
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
            asm volatile("" : "+v"(k0), "+v"(k1));
          }
#pragma unroll
          for (int u = 0; u < kAtOnce; ++u) {
            const uint64_t hit = __ballot(c0[u] >= thr0);
            if (kHits == 1 || j < 64) hits[0] = writelane64(hits[0], hit, j + u);
            else hits[kHits - 1] = writelane64(hits[kHits - 1], hit, j + u - 64);
          }
        }
      }
    }
    for (; first + j * stride < nwords; j += 2) {   // wave-uniform; two words with the same round keys
      // the round keys are formed anew with scalar additions: as loop invariants there are twenty of them, and they are
      // kept in lanes of vector registers, from which each costs two vector instructions a round
      uint32_t k0 = key0, k1 = key1;
      asm volatile("" : "+s"(k0), "+s"(k1));
      uint64_t hit[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int word = first + (j + u) * stride;
        const uint64_t pg = static_cast<uint64_t>(0xCD9E8D57u) * static_cast<uint32_t>((word << 6) + lane);
        uint32_t w[4];
        philox_rounds<2>(k0 + 0x9E3779B9u, k1 + 0xBB67AE85u, static_cast<uint32_t>(pg >> 32) ^ k0, static_cast<uint32_t>(pg), c2_1, c3_1, w);
        hit[u] = __ballot(w[0] >= thr0);
      }
      if (kHits == 1 || j < 64)
        hits[0] = writelane64(writelane64(hits[0], hit[0], j), hit[1], j + 1);
      else
        hits[kHits - 1] = writelane64(writelane64(hits[kHits - 1], hit[0], j - 64), hit[1], j - 63);
    }
  };
  // Those servers' blocks in full: their requests are added to the step's arrivals.
  auto count_requests = [&](uint32_t sd, int first, int stride) __attribute__((always_inline)) {
    const uint32_t thr1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(thr_ahead), 1));
    const uint32_t thr2 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(thr_ahead), 2));
#pragma unroll
    for (int h = 0; h < kHits; ++h) {
      if (first + 64 * h * stride >= nwords) break;   // wave-uniform
      const int word = first + (lane + 64 * h) * stride;
      // (what has been counted is taken out, so that behind the last step, for which nothing is drawn, there is nothing to count)
      uint64_t &left = hits[kHits == 1 ? 0 : h];
      left &= bits_below(word, N);   // (of a lane without a word it is empty)
      int n = 0;
      for (uint64_t todo = __ballot(left != 0); todo;) {   // a lane queues one server of its word at a time
        if (left) {
          ev_g[n + rank_in(todo)] = static_cast<uint16_t>((word << 6) + __ffsll(static_cast<long long>(left)) - 1);
          left &= left - 1ull;
        }
        n += __popcll(todo);
        todo = __ballot(left != 0);
        if (n > kEvPerWave - 64 || !todo) {
          for (int e0 = 0; e0 < n; e0 += 64) {   // wave-uniform
            if (e0 + lane < n) {
              uint32_t w[4];
              philox4x32_10(key0, key1, sd, 0u, static_cast<uint32_t>(ev_g[e0 + lane]), static_cast<uint32_t>(r), w);
              const int count = 1 + (w[0] >= thr1) + (w[0] >= thr2);
#pragma unroll
              for (int i = 0; i < 3; ++i) {
                if (i >= count) break;
                atomicAdd(&L.acc[class_of(w[i + 1])], 1u);
              }
            }
          }
          n = 0;
        }
      }
    }
  };
  auto next_thresholds = [&]() __attribute__((always_inline)) {   // of the step that is drawn next
    if (mod_rows > 1u) {
      thr_ahead = thr_asked;
      mod_row = mod_row + 1u == mod_rows ? 0u : mod_row + 1u;
      thr_asked = arr_thr[3 * static_cast<size_t>(mod_row) + (lane < 2 ? lane : 2)];
    }
  };
  // What follows from these (conditions, products, masks) is formed anew in every segment of a step. Left to itself the compiler
  // forms all of it once, before the first step: 150 scalar values, kept in lanes of vector registers.
  auto anew = [&]() __attribute__((always_inline)) {
    asm volatile("" : "+s"(K), "+s"(N), "+s"(B), "+s"(M), "+s"(BS), "+s"(nwords), "+s"(Mp), "+s"(nwords_m), "+s"(gate_mode));
  };
  // Where steps overlap (kOverlap) no barrier separates a step's last segment from the next step's completion pass: the waves that
  // serve nobody go on at once. (A step of a workgroup of eight waves and more spent a quarter to a third of its time in waits, most of
  // it there: a few waves serve, 8 to 12 thousand cycles, while the others wait. 500 servers x 3, same-slot decode 18.4 -> 14.4 ms per
  // 2000 steps, convergence instance 19.6 -> 17.8, 3001 x 77 4.98 -> 4.50 per 500, 10000 x 256 15.6 -> 14.8 per 1000. In workgroups of
  // up to four waves, where everything that does not serve draws, it costs 2 to 5 %: 1024 x 2048 16.4 -> 17.0, 256 x 1024 8.1 -> 8.5.
  // Two buffers and more than 5120 servers need draws beside the events for it: 10000 x 256, randomized router 5.24 -> 4.76 per 300 with
  // both, 5.36 with the overlap alone, weighted router 7.35 -> 6.84 and 7.54; with patience 8000 x 200 3.24 -> 2.98 per 200.)
  // What makes it sound: the servers that are given work belong to the waves that serve them until the next barrier. Every other wave
  // leaves them out of the words it looks at (bm_others, of its own words; it follows from the pass's words, as for the waves
  // that serve); those whose event comes in the next step already (`late`: lanes, late_g: the server) are queued by the wave that has
  // served them. What serving reads is not changed by a completion pass: bitmaps of completions and of servers that went idle are kept
  // for two steps in turn, slots given away and become idle change the bitmap of idle ones behind the next barrier (take_slots).
  // Counters are added to by atomics on both sides. The calendars are asked behind that barrier.
  // A wave looks at the pairs of words first, first + stride, ... below the end (and below the last one)
  int scan_first = wave - drain_first, scan_stride = n_drain, scan_end = nwords;
  constexpr int kPairsAtOnce = 4;
  uint64_t late = 0;   // lanes whose server (late_g) this wave has served and whose event comes next
  int late_g = 0;

  // The first `left` members of a lane's word: all of them, or (one word a level) some.
  auto first_members = [&](uint64_t in, int left) __attribute__((always_inline)) -> uint64_t {
    const int c = __popcll(in);
    uint64_t out = left >= c ? in : 0ull;
    const uint64_t part = __ballot(left > 0 && left < c);
    if (part) {   // wave-uniform
      const int src = __ffsll(static_cast<long long>(part)) - 1;
      const uint64_t w = readlane64(in, src);
      out = writelane64(out, __ballot(lane_in(w) && rank_in(w) < __builtin_amdgcn_readlane(left, src)), src);
    }
    return out;
  };
  int slots_given = 0;       // idle prefill slots that the last gate pass has given away: the first ones of bm_idle, still in it
  bool slots_taken = false;  // (where steps do not overlap) bm_comp holds those slots
  // The slots given away leave the bitmap of idle ones, those of the step's completions (`news`) enter it; by one whole wave. (Not when
  // they are given away and become idle: waves that serve look at the bitmap while others are in the next completion pass.)
  // The ranks of the idle slots are formed on the way; returns how many the mixed group has.
  auto take_slots = [&](const uint64_t *news) __attribute__((always_inline)) -> uint32_t {
    uint32_t running = 0;
    for (int w0 = 0; w0 < nwords_m; w0 += 64) {   // wave-uniform
      const int w = w0 + lane;
      uint64_t idle = 0, fresh_bits = 0;
      int left = 0;
      if (w < nwords_m) {
        idle = L.bm_idle[w];
        left = slots_given - static_cast<int>(L.pre[w]);
        if (news) fresh_bits = news[w];
      }
      const uint64_t given = first_members(idle & bits_below(w, M), left);
      idle = (idle & ~given) | fresh_bits;
      const uint32_t n = static_cast<uint32_t>(__popcll(idle & bits_below(w, M))), upto = wave_incl_scan(n);
      if (w < nwords_m) {
        L.bm_idle[w] = idle;
        L.pre[w] = static_cast<uint16_t>(running + upto - n);
      }
      running += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(upto), 63));
    }
    return running;
  };
  auto clear_bitmaps = [&](int at, int at_m) __attribute__((always_inline)) {   // by one whole wave
    for (int w = lane; w < nwords; w += 64) L.bm_just[at + w] = 0;
    for (int w = lane; w < nwords_m; w += 64) {
      L.bm_comp[at_m + w] = 0;
      if constexpr (RR) L.bm_solo[at_m + w] = 0;
    }
  };
  const uint32_t step_end = step_begin + n_steps;

  int64_t T = 0;
  for (uint32_t s = step_begin; s < step_end; ++s, ++ended) {
    T = (static_cast<int64_t>(s) + 1) * dt_ns;
    anew();
    if constexpr (SMALL) {
      if (quiet_search) {   // (here all arrivals are drawn by the block)
        bool search = s != step_begin;
        if constexpr (AB)   // (while nobody waits nobody leaves)
          search = search && __ballot(lane < K && (L.cs[CS_QP + (lane & (kMaxK - 1))] | L.cs[CS_QD + (lane & (kMaxK - 1))]) != 0) == 0;
        if (search) {
          const uint32_t s_first = s;
          const int64_t never = static_cast<int64_t>(1) << 62;
          int64_t rel = (L.bm_busy[0] >> lane) & 1ull ? event_time(lane < N ? lane : 0, T) : never;   // (events lie after the step before)
          for (; s < step_end; ++s) {
            if (steps_ahead == 0) draw_block(s);
            if ((ahead & ((1ull << (1 << lg_n)) - 1ull)) || __ballot(rel <= 0)) break;
            rel -= dt_ns;
            ahead >>= 1 << lg_n;
            --steps_ahead;
          }
          if (s != s_first) {
            ended += s - s_first;
            T = (static_cast<int64_t>(s) + 1) * dt_ns;
            if (s == step_end) { T = static_cast<int64_t>(s) * dt_ns; break; }
          }
        }
        // this step is gone through now: the lanes that have drawn it add its requests to the arrivals
        if (steps_ahead == 0) draw_block(s);
        if ((lane >> lg_n) == (64 >> lg_n) - steps_ahead) {
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            if (i >= static_cast<int>(requests & 3u)) break;
            atomicAdd(&L.acc[(requests >> (2 + 3 * i)) & 7u], 1u);
          }
        }
        ahead >>= 1 << lg_n;
        --steps_ahead;
      }
    }
    if (nwaves > 1 && nwaves <= 4) {
      const uint32_t t2 = ((s >> 8) + (static_cast<uint32_t>(r) >> 8)) & 1u;
      if (kChainFirst || t2 != turn) { turn = t2; own_priority(); }
    }
    // abandonment only: how many waiting requests of class `tid` leave at the start of this step. Asked for here and used after the
    // completion pass, or, where steps overlap, behind it: those that the step before has taken out of the calendars must be out.
    uint32_t n_leave_p = 0, n_leave_d = 0, n_leave_dm = 0;
    auto ask_leaving = [&]() __attribute__((always_inline)) {
      if constexpr (AB) {
        if (tid < K) {
          n_leave_p = atomicExch(&cal[static_cast<size_t>(tid) * cal_n + (s & p.cal_mask)], 0u);
          n_leave_d = atomicExch(&dcal[static_cast<size_t>(tid) * cal_n + (s & p.cal_mask)], 0u);
          if constexpr (RR) n_leave_dm = atomicExch(&dcal_m[static_cast<size_t>(tid) * cal_n + (s & p.cal_mask)], 0u);
        }
      }
    };
    if constexpr (!kOverlap) ask_leaving();
    // the bitmaps that steps take in turn: this step's
    const int side = s & 1u ? turn_words : 0, side_m = s & 1u ? turn_words_m : 0;
    // ---- 2. events: one server per lane (uniform control flow; lanes beyond the queue idle). Tallies the iterations
    //      since the last event, removes the decodes that emitted their last token, advances the prefill. What the
    //      lanes need of their servers' records is asked for first, together with the slot rows of the servers whose
    //      event is the end of a decode: eight lanes read a row, 16 bytes per lane and load, eight rows at a time.
    auto drain_events = [&](int nev) __attribute__((always_inline)) {
      int lane_here = lane;   // (likewise: thirteen vector registers)
      asm volatile("" : "+v"(lane_here));
      __builtin_assume(lane_here >= 0 && lane_here < 64);
      for (int e0 = 0; e0 < nev; e0 += 64) {
        const bool queued = e0 + lane < nev;
        const int g = queued ? static_cast<int>(ev_g[e0 + lane]) : 0;
        const int wi = g >> 6;
        // (every lane reads: those without a server that of server 0)
        uint64_t nc = rec[g].n_cls, nj = rec[g].n_join, pf = rec[g].pf_job;
        const uint32_t it_tal = rec[g].iter;
        uint32_t nf = rec[g].next_fin;
        const uint32_t ev = L.ev_it[g], it = ev & kEvIter;
        int nd = static_cast<int>(L.loads[g]);
        int rem = static_cast<int>(L.rem[g < Mp ? g : 0]);   // (without a mixed group: of the array behind)
        rem = g < Mp ? rem : 0;
        // exact completion time, relative to T: within a step of it
        const int32_t rel = static_cast<int32_t>(((L.ev_t[g] - static_cast<uint32_t>(T >> 8)) << 8) + L.ev_lo[g] - (static_cast<uint32_t>(T) & 255u));
        const bool active = queued && rel <= 0;
        const uint64_t bit = active ? 1ull << (g & 63) : 0ull;
        const int nd_before = nd;
        const bool has_chunk = ev & kEvChunk;
        const bool mixed_now = rem > 0;
        const uint64_t nc_before = nc;
        // ---- the ends of decodes: one leaves per round, highest slot first (the last slot's request moves into its
        //      place); a second round follows only where several end together
        bool leaving = active && (ev & kEvFin);
        // The request that leaves (a trip to memory that follows the row's) is asked for where its slot is known and used at the
        // end, unless another of the server's ends in the same iteration: the next event does not depend on it.
        int gone_slot = -1;
        uint64_t gone_job = 0, last_job = 0;
        uint32_t last_fin = 0;
        auto leave = [&]() __attribute__((always_inline)) {
          if (gone_slot >= 0) {
            uint32_t *frow = fin + static_cast<size_t>(g) * BS;
            uint64_t *jrow = job + static_cast<size_t>(g) * BS;
            const int k = static_cast<int>(gone_job >> 29) & 7;
            const uint32_t stamp = static_cast<uint32_t>(gone_job) & 0x1FFFFFFFu;
            const uint32_t Pl = (static_cast<uint32_t>(gone_job >> 32) & 0xFFFFu) + 1, Dl = static_cast<uint32_t>(gone_job >> 48) + 1;
            const int64_t e2e = static_cast<int64_t>(static_cast<uint64_t>(s - stamp) * dt_ns) + rel;   // (T is boundary s + 1)
            lds_add64(&L.tl[k * kNTally + (mixed_now ? SIM_T_S_DM : SIM_T_S_DS)], 1);
            atomicAdd(&L.acc[(mixed_now ? AC_YM_OUT : AC_YS_OUT) + k], 1u);
            lds_add64(&L.tl[k * kNTally + SIM_T_TOKP_DEC], Pl);
            lds_add64(&L.tl[k * kNTally + SIM_T_TOKD_DEC], Dl);
            lds_add64(&L.tl[k * kNTally + SIM_T_E2E_SUM], static_cast<uint64_t>(e2e));
            atomicAdd(reinterpret_cast<unsigned long long *>(&hist[(1 * K + k) * kNBin + hbin(e2e)]), 1ull);
            nc -= 1ull << (8 * k);
            if (gone_slot < nd) { frow[gone_slot] = last_fin; jrow[gone_slot] = last_job; }
            frow[nd] = kFreeSlot;
          }
          gone_slot = -1;
        };
        for (uint64_t lm = __ballot(leaving); lm; lm = __ballot(leaving)) {
          // lane q gets the server, the decodes and the iteration of the q-th row (the other lanes' follow behind them)
          const int nrows = __popcll(lm), my_row = rank_in(lm);
          const int to = (leaving ? my_row : nrows + rank_in(~lm)) << 2;
          const int row_gn = __builtin_amdgcn_ds_permute(to, g | (nd << 16));
          const int row_it = __builtin_amdgcn_ds_permute(to, static_cast<int>(it));
          int slot = -1;
          bool more = false;
          uint32_t next = 0xFFFFFFFFu;
          for (int r0 = 0; r0 < nrows; r0 += 8) {   // wave-uniform
            const int row = r0 + (lane_here >> 3), l8 = lane_here & 7;
            const int o_gn = __shfl(row_gn, row & 63, 64);
            const int o_g = o_gn & 0xFFFF, o_nd = row < nrows ? o_gn >> 16 : 0;
            const uint32_t o_it = static_cast<uint32_t>(__shfl(row_it, row & 63, 64));
            const uint32_t *frow = fin + (static_cast<uint32_t>(o_g) * static_cast<uint32_t>(BS) + 4u * static_cast<uint32_t>(l8));
            uint4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              v[q] = make_uint4(kFreeSlot, kFreeSlot, kFreeSlot, kFreeSlot);
              if (32 * q < BS && 4 * (l8 + 8 * q) < o_nd) v[q] = stream_load(frow + 32 * q);
            }
            // (two instructions and a half a slot; with a comparison, a selected slot number and a count it took four and three quarters
            // and twelve registers: 1024 x 2048 16.25 -> 16.15 ms per 1000 steps, 10000 x 256 14.05 -> 13.95, randomized router 5.36 -> 5.31
            // per 300)
            uint32_t least = 0xFFFFFFFFu, ends = 0;   // ends: the lane's slots that end now, one a bit, the last one looked at lowest
            int n_seen = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if (q > 0 && 32 * q >= BS) break;   // wave-uniform: no such slots
              const uint32_t wv[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
              for (int w = 0; w < 4; ++w) {
                const uint32_t ahead = wv[w] - o_it - 1u;   // negative for one that ends now, at least 2^30 for a free slot
                ends = __builtin_amdgcn_alignbit(ends, ahead, 31);
                least = ahead < least ? ahead : least;
              }
              n_seen = 4 * q + 3;
            }
            const int at_high = n_seen - (__ffs(static_cast<int>(ends)) - 1);   // the highest of them: its place among those looked at
            int high = ends ? ((at_high & ~3) << 3) + 4 * l8 + (at_high & 3) : -1, count = __popc(ends);
            // over the eight lanes of the row: pairs, quads, then the two quads
            auto over_row = [](auto f, int v) __attribute__((always_inline)) {
              v = f(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));
              v = f(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));
              return f(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));
            };
            high = over_row([](int x, int y) { return x > y ? x : y; }, high);
            count = over_row([](int x, int y) { return x + y; }, count);
            // (a request has at most 32768 decodes: the end that follows is nearer than 65535 iterations, or there is none)
            least = static_cast<uint32_t>(over_row([](int x, int y) { return x < y ? x : y; }, static_cast<int>(least < 0xFFFFu ? least : 0xFFFFu)));
            const int found = (high & 0xFF) | (count > 1 ? 0x100 : 0) | static_cast<int>(least << 16);
            // back to the lane that owns the server
            const uint32_t mine = static_cast<uint32_t>(__shfl(found, ((my_row - r0) << 3) & 63, 64));
            if (leaving && my_row >= r0 && my_row < r0 + 8) { slot = static_cast<int8_t>(mine); more = mine & 0x100u; next = mine >> 16; }
          }
          if (leaving) {
            leaving = more;
            nf = next < 0xFFFFu ? it + 1u + next : kNever;
            if (slot >= 0) {
              --nd;
              gone_slot = slot;
              const size_t row0 = static_cast<size_t>(g) * BS;
              gone_job = job[row0 + slot]; last_job = job[row0 + nd];
              last_fin = fin[row0 + nd];
            }
          }
          if (IM || __ballot(leaving)) leave();   // wave-uniform
        }
        uint32_t m = 0, d = 0;
        bool chunk = false;
        uint64_t comp = 0;
        uint32_t wait_steps = 0;   // patience of a completed prefill's request in the decode buffer (0: without end)
        PrefillEnd pe; pe.done = false; pe.k = 0; pe.P = 0; pe.ttft = 0; pe.nc = 0;
        if (active) {
          comp = nc_before - nj;   // bytewise: no class joins more decodes than it holds
          const int ptok = has_chunk ? chunk_of(rem) : 0;   // the chunk of every iteration since the last event
          d = iteration_ns(ptok, byte_sum(comp));
          chunk = has_chunk;
          m = it - it_tal;
          if (nd != nd_before) {
            L.loads[g] = static_cast<uint8_t>(nd);
            const int hb = g < M ? kLoadBins : 0;
            atomicSub(&L.lh[hb + nd_before], 1u);
            atomicAdd(&L.lh[hb + nd], 1u);
            if constexpr (IM) {   // a full server (it holds no prefill then) has a slot again
              if (nd_before == B && g < Mp) atomicOr(bits64(kOverlap ? &L.bm_comp[side_m + wi] : &L.bm_idle[wi]), bit);
            }
          }
          // the prefill advances by the chunks of those iterations
          if (has_chunk) {
            rem -= static_cast<int>(m) * ptok;
            L.rem[g] = static_cast<uint16_t>(rem);
            if (rem == 0) {
              const uint64_t jw = pf;
              const int k = static_cast<int>(jw >> 29) & 7;
              const uint32_t stamp = static_cast<uint32_t>(jw) & 0x1FFFFFFFu;
              pe.done = true; pe.k = k; pe.nc = nc;
              pe.P = (static_cast<uint32_t>(jw >> 32) & 0xFFFFu) + 1;
              pe.ttft = static_cast<int64_t>(static_cast<uint64_t>(s - stamp) * dt_ns) + rel;
              atomicAdd(reinterpret_cast<unsigned long long *>(&hist[(0 * K + k) * kNBin + hbin(pe.ttft)]), 1ull);
              if constexpr (IM) {
                // the request keeps its slot: it joins the batch at the restart that follows this completion
                // (the gate admits only where a slot is left, so nd < B here; were it not, the request is dropped)
                if (nd >= B) {
                  lds_add64(&L.tl[k * kNTally + SIM_T_DROP_D], 1);
                  L.tl[kMaxK * kNTally + SIM_G_OVERFLOW] = 1;
                } else {
                  const uint32_t ends = it + static_cast<uint32_t>(jw >> 48) + 1;
                  fin[static_cast<size_t>(g) * BS + nd] = ends;
                  job[static_cast<size_t>(g) * BS + nd] = jw;
                  if (nd == 0 || ends < nf) nf = ends;
                  nc += 1ull << (8 * k);
                  const int hb = g < M ? kLoadBins : 0;
                  atomicSub(&L.lh[hb + nd], 1u);
                  atomicAdd(&L.lh[hb + nd + 1], 1u);
                  ++nd;
                  L.loads[g] = static_cast<uint8_t>(nd);
                  lds_add64(&L.tl[k * kNTally + SIM_T_U_DS], 1);
                  atomicAdd(&L.acc[AC_YS_IN + k], 1u);
                  if (nd < B) atomicOr(bits64(kOverlap ? &L.bm_comp[side_m + wi] : &L.bm_idle[wi]), bit);
                }
              } else {
                atomicOr(bits64(&L.bm_comp[side_m + wi]), bit);
                if constexpr (!kOverlap) atomicOr(bits64(&L.bm_idle[wi]), bit);
                if constexpr (AB || RR) {   // word 0 of its block: patience in the buffer, word 1: which of two buffers
                  uint32_t w[4];
                  philox4x32_10(key0, key1, s, static_cast<uint32_t>(kStreamPatienceD), static_cast<uint32_t>(g), static_cast<uint32_t>(r), w);
                  if constexpr (RR) { if (w[1] < p.solo_thr[k]) atomicOr(bits64(&L.bm_solo[side_m + wi]), bit); }
                  if constexpr (AB) { if ((p.ab_classes >> k) & 1u) wait_steps = pat_tab[static_cast<size_t>(k) * kTableSize + (w[0] >> 16)]; }
                }
              }
            }
          }
          // The next iteration starts where this one has ended, with what the server holds now. Work that this step still
          // brings is then found to come at an iteration boundary (see `serve`) and starts the iteration anew.
          const int ptok_next = rem > 0 ? chunk_of(rem) : 0;
          if (ptok_next == 0 && nd == 0) {
            set_event(g, T + rel, it, false, false);
            atomicAnd(bits64(&L.bm_busy[wi]), ~bit);
            atomicOr(bits64(&L.bm_just[side + wi]), bit);
          } else {
            const uint32_t dur = iteration_ns(ptok_next, static_cast<uint32_t>(nd));
            const uint32_t n = phase_length(static_cast<uint32_t>(nd), rem, dur, nf - it);
            set_event(g, T + rel + static_cast<int64_t>(static_cast<uint64_t>(n) * dur), it + n, ptok_next > 0, nd && nf == it + n);
          }
          // (in the place of the prompt tokens left, of which there are none, until the request joins its buffer)
          if constexpr (AB && !IM) { if (pe.done) L.rem[g] = static_cast<uint16_t>(wait_steps); }
        }
        tally_iterations<kTallyRowsHere>(L.ta, L.tbth, tbt_w, tbt_lo, K, m, d, chunk, comp);
        if constexpr (!IM) { leave(); pe.nc = nc; }
        if (active) {
          rec[g].n_cls = nc;
          rec[g].n_join = 0;
          rec[g].iter = it;
          rec[g].next_fin = nf;
        }
        // a prefill that ended: completion count, recognised prompt tokens, time to first token; the
        // co-resident decodes switch mixed -> solo
        if (pe.done) {
          int n_classes = K;   // (taken anew, as in tally_iterations)
          asm volatile("" : "+s"(n_classes));
          lds_add64(&L.tl[pe.k * kNTally + SIM_T_S_P], 1);
          atomicAdd(&L.acc[AC_X_OUT + pe.k], 1u);
          lds_add64(&L.tl[pe.k * kNTally + SIM_T_TOKP_PRE], pe.P);
          lds_add64(&L.tl[pe.k * kNTally + SIM_T_TTFT_SUM], static_cast<uint64_t>(pe.ttft));
          // (two classes at a time; how many switched in all follows from the other tallies when the launch ends: 500 servers x 3, same-slot
          // decode 14.32 -> 14.11 ms per 2000 steps, the others within 0.5 %. Adding zeros too, without the condition, costs the
          // randomized router 1.4 %)
#pragma unroll
          for (int c = 0; c < kMaxK; c += 2) {
            if (c >= n_classes) break;   // wave-uniform
            const uint64_t v = two_bytes_at(pe.nc, c);
            if (v) {
              lds_add64(reinterpret_cast<uint64_t *>(&L.acc[AC_YM_OUT + c]), v);
              lds_add64(reinterpret_cast<uint64_t *>(&L.acc[AC_YS_IN + c]), v);
            }
          }
        }
      }
    };

    // ---- completion pass: the arrivals (see draw_words), and which servers have their event in this step (one clock per server and
    //      step is all that is read). What a word has but one of is kept one word a lane.
    if (!quiet_search) {
      if constexpr (kBeside) {
        if (wave < n_draw) {
          if (s == step_begin) draw_words(s, wave, n_draw);
          if (s == step_begin || drawn) count_requests(s, wave, n_draw);
          next_thresholds();
          if (s + 1u < step_end) draw_words(s + 1u, wave, n_draw);
          drawn = true;
        }
      } else {
        if (!drawn) {
          draw_words(s, wave, nwaves);
          count_requests(s, wave, nwaves);
          next_thresholds();
        }
        drawn = false;
      }
    }
    if (wave >= drain_first || late) {   // wave-uniform
      const uint32_t T_hi = static_cast<uint32_t>(T >> 8);
      int nev = 0;   // servers queued by this wave (wave-uniform)
      if (late) {
        if (lane_in(late)) ev_g[rank_in(late)] = static_cast<uint16_t>(late_g);
        nev = __popcll(late);
      }
      // A lane looks at two neighbouring servers of a pair of words; what it finds enters the lower end of its masks, so that after
      // `seen` pairs the i-th pair's servers are bits 2 (seen - 1 - i) and the one above. (A server a lane, the ballots collected a word
      // a lane and the words queued one after another, took twice the vector instructions for a clock and fifteen more a word: 1024 x
      // 2048 16.76 -> 16.25 ms per 1000 steps, 2048 x 1024 17.05 -> 16.42, 3001 x 77 4.74 -> 4.53 per 500, randomized router 5.48 -> 5.36
      // per 300, 10000 x 256 14.14 -> 14.05.)
      const int last_pair = (nwords - 1) >> 1, npairs = scan_end <= last_pair ? scan_end : last_pair + 1;
      const uint32_t T_past = T_hi + 1u;
      const int last_clock = (N - 1) & ~1;
      for (int first = scan_first;; first += kPairsARound * scan_stride) {   // wave-uniform; the wave's pairs of words, sixteen a round
        if (first >= npairs && nev == 0) break;
        if constexpr (!kOverlap) {   // (its own words: nobody else is at them)
          const int w = 2 * (first + (lane >> 1) * scan_stride) + (lane & 1);
          if (lane < 32 && w < nwords) {
            L.bm_just[w] = 0;
            if (w < nwords_m) {
              if (slots_taken) L.bm_idle[w] &= ~L.bm_comp[w];
              L.bm_comp[w] = 0;
              if constexpr (RR) L.bm_solo[w] = 0;
            }
          }
        }
        uint32_t due = 0, own = 0;
        int seen = 0;
        // (servers past the last one are not busy; a clock a few ns ahead may pass here for its upper bits: the servers
        // queued are looked at exactly)
        for (; seen < kPairsARound && first + seen * scan_stride < npairs; seen += kPairsAtOnce) {   // wave-uniform; up to three pairs past the last one
          uint2 ev[kPairsAtOnce];
          uint32_t here[kPairsAtOnce];
          int n_bits[kPairsAtOnce];
#pragma unroll
          for (int u = 0; u < kPairsAtOnce; ++u) {
            const int pair = first + (seen + u) * scan_stride, at = pair < npairs ? pair : last_pair, g = (at << 7) + 2 * lane;
            n_bits[u] = pair < npairs ? 2 : 0;
            ev[u] = *reinterpret_cast<const uint2 *>(L.ev_t + (g < last_clock ? g : last_clock));
            const int byte = (at << 4) + (lane >> 2);
            here[u] = reinterpret_cast<const uint8_t *>(L.bm_busy)[byte];
            if constexpr (kOverlap) here[u] &= ~static_cast<uint32_t>(reinterpret_cast<const uint8_t *>(L.bm_others)[byte]);
          }
#pragma unroll
          for (int u = 0; u < kPairsAtOnce; ++u) {
            due = __builtin_amdgcn_alignbit(due, ev[u].y - T_past, 31);
            due = __builtin_amdgcn_alignbit(due, ev[u].x - T_past, 31);
            own = (own << 2) | __builtin_amdgcn_ubfe(here[u], static_cast<uint32_t>(lane & 3) << 1, static_cast<uint32_t>(n_bits[u]));
          }
        }
        due &= own;
        for (uint64_t todo = __ballot(due != 0); todo || nev > 0;) {   // a lane queues one of its servers at a time
          if (todo) {
            if (due) {
              const int b = __ffs(static_cast<int>(due)) - 1;
              ev_g[nev + rank_in(todo)] = static_cast<uint16_t>(((first + (seen - 1 - (b >> 1)) * scan_stride) << 7) + 2 * lane + (b & 1));
              due &= due - 1u;
            }
            nev += __popcll(todo);
            todo = __ballot(due != 0);
          }
          if (nev > kEvPerWave - 64 || !todo) { drain_events(nev); nev = 0; }
        }
      }
    }
    late = 0;
    slots_taken = false;
    __syncthreads();
    if constexpr (kChainFirst) __builtin_amdgcn_s_setprio(3);

    anew();
    // ================= arrivals into the class queues; ranks of completions and idle slots =================
    if constexpr (kOverlap) ask_leaving();
    // (the completions' ranks by a wave of their own where there is one; with deadline rings the first one needs their number. That and
    // the idle slots' ranks formed while they change, where steps overlap: 2048 servers x 1024 16.36 -> 16.23 ms per 1000 steps, 10000 x
    // 256 13.93 -> 13.81, randomized router 5.30 -> 5.25 per 300, 3001 x 77 4.50 -> 4.46 per 500)
    constexpr int kRankWave = !AB && nwaves >= 4 ? 3 : 0;
    const bool ranks_comp = kRankWave > 0 ? wave == kRankWave : tid < 64;
    uint32_t ncomp_all = 0;
    if constexpr (!IM) { if (ranks_comp) ncomp_all = rank_bitmap(L.bm_comp + side_m, L.pre_c, nwords_m, Mp); }
    if (tid < K) {
      const int k = tid;
      // (everything that is needed is read first: one trip to LDS)
      const uint32_t arrived = L.acc[AC_ARRIVALS + k];
      const int x_out = static_cast<int>(L.acc[AC_X_OUT + k]), ym_out = static_cast<int>(L.acc[AC_YM_OUT + k]);
      const int ys_more = static_cast<int>(L.acc[AC_YS_IN + k] - L.acc[AC_YS_OUT + k]);
      int qp = L.cs[CS_QP + k], qd = L.cs[CS_QD + k];
      const int x = L.cs[CS_X + k], ym = L.cs[CS_YM + k], ys = L.cs[CS_YS + k];
      uint32_t tail = static_cast<uint32_t>(L.cs[CS_QHEAD + k]);
      const uint32_t ring_len = AB ? static_cast<uint32_t>(L.sc[SC_QLEN + k]) : 0u;
      add_step_sums(k, ended, qp, qd, x, ym, ys);   // of the steps before
      L.acc[AC_ARRIVALS + k] = 0; L.acc[AC_X_OUT + k] = 0; L.acc[AC_YM_OUT + k] = 0; L.acc[AC_YS_IN + k] = 0; L.acc[AC_YS_OUT + k] = 0;
      L.cs[CS_X + k] = x - x_out; L.cs[CS_YM + k] = ym - ym_out; L.cs[CS_YS + k] = ys + ys_more;
      L.sc[SC_HEAD + k] = L.cs[CS_QHEAD + k];
      if constexpr (AB) {   // abandonments come first: they free room in the queue
        if (n_leave_p) {
          qp -= static_cast<int32_t>(n_leave_p);
          lds_add64(&L.tl[k * kNTally + SIM_T_AB_P], n_leave_p);
        }
        if (n_leave_d) {
          qd -= static_cast<int32_t>(n_leave_d);
          lds_add64(&L.tl[k * kNTally + SIM_T_AB_D], n_leave_d);
          atomicSub(&L.cs[CS_DCOUNT], static_cast<int32_t>(n_leave_d));
          if constexpr (WS) L.cs[CS_QDS + k] -= static_cast<int32_t>(n_leave_d);
        }
        if constexpr (RR) {
          if (n_leave_dm) {
            qd -= static_cast<int32_t>(n_leave_dm);
            lds_add64(&L.tl[k * kNTally + SIM_T_AB_D], n_leave_dm);
            atomicSub(&L.cs[CS_DCOUNT_M], static_cast<int32_t>(n_leave_dm));
          }
        }
        L.cs[CS_QD + k] = qd;
      }
      const uint32_t room = queue_cap - static_cast<uint32_t>(qp);
      const uint32_t take = arrived < room ? arrived : room;
      // entries between head and tail: the waiting requests, with abandonment also the dead entries
      const uint32_t in_ring = AB ? ring_len : static_cast<uint32_t>(qp);
      tail += in_ring;
      if (tail >= queue_cap) tail -= queue_cap;
      if constexpr (AB) {
        if (in_ring + take > queue_cap) atomicOr(&L.sc[SC_COMPACT], 1 << k);
        L.sc[SC_QLEN + k] = static_cast<int32_t>(in_ring + take);
      }
      L.sc[SC_TAKE + k] = static_cast<int32_t>(take);
      L.sc[SC_TAIL + k] = static_cast<int32_t>(tail);
      L.cs[CS_QP + k] = qp + static_cast<int32_t>(take);
      if (arrived) lds_add64(&L.tl[k * kNTally + SIM_T_A], take);
      if (arrived > take) {
        lds_add64(&L.tl[k * kNTally + SIM_T_DROP_P], arrived - take);
        L.tl[kMaxK * kNTally + SIM_G_OVERFLOW] = 1;
      }
    }
    ended = 0;
    if (ranks_comp) {
      const uint32_t ncomp = ncomp_all;
      if (lane == 0) {
        L.sc[SC_NCOMP] = static_cast<int32_t>(ncomp);
        if constexpr (AB) {
          // a buffer ring that cannot hold this step's completions behind its dead entries is compacted first
          // (this wave has already taken the step's abandonments off the counters above)
          const uint32_t room = dbuf_cap - static_cast<uint32_t>(L.cs[CS_DCOUNT]);
          if (static_cast<uint32_t>(L.sc[SC_DLEN]) + (ncomp < room ? ncomp : room) > dbuf_cap) atomicOr(&L.sc[SC_COMPACT], 256);
          if constexpr (RR) {   // how the completions split between the two rings is not known yet: either may get all
            const uint32_t room_m = dbuf_cap - static_cast<uint32_t>(L.cs[CS_DCOUNT_M]);
            if (static_cast<uint32_t>(L.sc[SC_DLEN_M]) + (ncomp < room_m ? ncomp : room_m) > dbuf_cap) atomicOr(&L.sc[SC_COMPACT], 512);
          }
        }
      }
    }
    if (NT == 64 ? tid < 64 : (tid >= 64 && tid < 128)) {
      uint32_t nidle;   // idle prefill slots of the mixed group
      if constexpr (kOverlap) nidle = take_slots(L.bm_comp + side_m);
      else nidle = rank_bitmap(L.bm_idle, L.pre, nwords_m, M);
      if (lane == 0) L.sc[SC_NIDLE] = static_cast<int32_t>(nidle);
    }
    if constexpr (kOverlap) {   // (what the step before had in these has been read)
      if (wave == nwaves - 1) clear_bitmaps(turn_words - side, turn_words_m - side_m);
    }
    slots_given = 0;
    if constexpr (RR) {   // (another wave where there is one)
      if (wave == (nwaves > 2 ? 2 : nwaves - 1)) {
        const uint32_t nsolo = rank_bitmap(L.bm_solo + side_m, L.pre_s, nwords_m, Mp);
        if (lane == 0) L.sc[SC_NSOLO] = static_cast<int32_t>(nsolo);
      }
    }
    __syncthreads();
    anew();
    // what follows is shared out: the first waves rank the gate's candidates, the others look for the router's servers
    const int n_gate = nwaves > 1 ? nwaves >> 1 : 1, route_first = nwaves > 1 ? n_gate : 0, n_route = nwaves - route_first;
    if constexpr (AB) {
      // a ring that cannot hold this step's appends behind its dead entries is compacted first
      const int flags = L.sc[SC_COMPACT];   // cleared at the end of the step
      if (flags) {   // the same for every thread
        for (int k = wave; k < K; k += nwaves)
          if ((flags >> k) & 1) compact_queue(k, s, static_cast<uint32_t>(L.sc[SC_TAKE + k]));
        if ((flags & 256) && wave == nwaves - 1) compact_buffer(s, false);
        if constexpr (RR) {
          if ((flags & 512) && wave == (nwaves > 1 ? nwaves - 2 : 0)) compact_buffer(s, true);
        }
        __syncthreads();
      }
    }
    if constexpr (AB) {
      // One thread per accepted arrival of any class, so that the table reads of all classes are in flight together;
      // the last waves take them, while the first ones move the completions below. The accepted arrivals of a class
      // are exchangeable: the j-th of this step draws its patience.
      uint32_t upto[kMaxK];   // accepted arrivals of the classes up to and including k
      {
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kMaxK; ++k) {
          if (k < K) run += static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(L.sc[SC_TAKE + k]));
          upto[k] = run;
        }
      }
      for (uint32_t i = static_cast<uint32_t>((nwaves - 1 - wave) * 64 + lane); i < upto[kMaxK - 1]; i += NT) {
        int k = 0;
        uint32_t before = 0;
#pragma unroll
        for (int c = 0; c + 1 < kMaxK; ++c)
          if (i >= upto[c]) { k = c + 1; before = upto[c]; }
        const uint32_t j = i - before;
        uint32_t pos = static_cast<uint32_t>(L.sc[SC_TAIL + k]) + j;
        if (pos >= queue_cap) pos -= queue_cap;
        qring[static_cast<size_t>(k) * queue_cap + pos] = s;
        uint32_t dl = kNever;
        if ((p.ab_classes >> k) & 1u) {
          uint32_t w[4];
          philox4x32_10(key0, key1, s, static_cast<uint32_t>(kStreamPatienceP + k), j, static_cast<uint32_t>(r), w);
          dl = s + pat_tab[static_cast<size_t>(k) * kTableSize + (w[0] >> 16)];
          atomicAdd(&cal[static_cast<size_t>(k) * cal_n + (dl & p.cal_mask)], 1u);
        }
        qdl[static_cast<size_t>(k) * queue_cap + pos] = dl;
      }
    } else {
      // (by the waves that look for the router's servers, a class each: the others have the gate's candidates to rank. With the
      // first waves writing them 2048 x 1024 took 16.85 instead of 16.09 ms per 1000 steps, 10000 x 256 16.9 instead of 16.25,
      // 3001 x 77 5.24 instead of 5.01 per 500, 256 x 1024 8.39 instead of 8.16)
      if (wave >= route_first) {
        const int sc_lane = L.sc[lane];   // one word per lane: one trip to LDS
        for (int k = nwaves - 1 - wave; k < K; k += n_route) {   // wave-uniform
          const uint32_t take = static_cast<uint32_t>(__builtin_amdgcn_readlane(sc_lane, SC_TAKE + k));
          const uint32_t tail = static_cast<uint32_t>(__builtin_amdgcn_readlane(sc_lane, SC_TAIL + k));
          for (uint32_t j = lane; j < take; j += 64) {
            uint32_t pos = tail + j;
            if (pos >= queue_cap) pos -= queue_cap;
            qring[static_cast<size_t>(k) * queue_cap + pos] = s;
          }
        }
      }
    }
    // completed prefills join the decode buffer in ascending server order
    int ncs = 0, ncm = 0;   // two buffers: how many joined the solo and the mixed group's
    {
      const uint32_t ncomp = static_cast<uint32_t>(L.sc[SC_NCOMP]);
      const uint32_t dc0 = static_cast<uint32_t>(L.cs[CS_DCOUNT]), dc1 = RR ? static_cast<uint32_t>(L.cs[CS_DCOUNT_M]) : 0u;
      const uint32_t dh0 = static_cast<uint32_t>(L.cs[CS_DHEAD]), dh1 = RR ? static_cast<uint32_t>(L.cs[CS_DHEAD_M]) : 0u;
      // ring entries before the tail (with abandonment the dead entries count)
      const uint32_t fill0 = AB ? static_cast<uint32_t>(L.sc[SC_DLEN]) : dc0, fill1 = AB && RR ? static_cast<uint32_t>(L.sc[SC_DLEN_M]) : dc1;
      // (64 to a wave, the last wave that ranks the gate's candidates first: it has the least to do next)
      const int comp_turn = wave < n_gate ? n_gate - 1 - wave : wave;
      for (uint32_t j0 = static_cast<uint32_t>(comp_turn) * 64u; j0 < ncomp; j0 += NT) {   // wave-uniform trip count
        const uint32_t j = j0 + lane;
        if (j < ncomp) {
          const int g = select_bit(L.bm_comp + side_m, L.pre_c, nwords_m, j);
          const uint64_t jw = rec[g].pf_job;
          const int k = static_cast<int>(jw >> 29) & 7;
          uint32_t dl = kNever;
          if constexpr (AB) {
            const uint32_t wait_steps = L.rem[g];
            L.rem[g] = 0;
            if (wait_steps) dl = s + wait_steps;
          }
          bool solo = true;   // the only buffer, or the solo group's
          uint32_t idx = j;   // its place among those that join that buffer
          if constexpr (RR) {
            const uint64_t to_solo = L.bm_solo[side_m + (g >> 6)], bit = 1ull << (g & 63);
            solo = to_solo & bit;
            const uint32_t before = L.pre_s[g >> 6] + static_cast<uint32_t>(__popcll(to_solo & (bit - 1ull)));
            idx = solo ? before : j - before;
          }
          if ((solo ? dc0 : dc1) + idx < dbuf_cap) {
            uint32_t pos = (solo ? dh0 + fill0 : dh1 + fill1) + idx;
            if (pos >= dbuf_cap) pos -= dbuf_cap;
            if (solo) dring[pos] = jw; else dring_m[pos] = jw;
            constexpr uint32_t kHere = RR ? kJobsLds / 2 : kJobsLds;
            if (idx < kHere) {
              if constexpr (!AB) L.jobs[(solo ? 0u : kHere) + idx] = jw;
              else if (!WS && nwaves > 1) L.fresh[(solo ? 0u : kHere) + idx] = jw;
            }
            if constexpr (AB) {
              const size_t at = static_cast<size_t>(k) * cal_n + (dl & p.cal_mask);
              if (solo) {
                ddl[pos] = dl;
                if (dl != kNever) atomicAdd(&dcal[at], 1u);
              } else {
                ddl_m[pos] = dl;
                if (dl != kNever) atomicAdd(&dcal_m[at], 1u);
              }
            }
            atomicAdd(&L.cs[CS_QD + k], 1);
            // the weighted router also counts what waits in the solo group's buffer per class
            if constexpr (WS) { if (solo) atomicAdd(&L.cs[CS_QDS + k], 1); }
          } else {
            lds_add64(&L.tl[k * kNTally + SIM_T_DROP_D], 1);
            L.tl[kMaxK * kNTally + SIM_G_OVERFLOW] = 1;
          }
        }
      }
      if constexpr (RR) {   // what each ring accepted (a prefix of what it was sent)
        const uint32_t room0 = dbuf_cap - dc0, room1 = dbuf_cap - dc1, to_solo = static_cast<uint32_t>(L.sc[SC_NSOLO]);
        ncs = uniform(static_cast<int>(to_solo < room0 ? to_solo : room0));
        ncm = uniform(static_cast<int>(ncomp - to_solo < room1 ? ncomp - to_solo : room1));
      }
    }

    // ================= 3.-5. prefill gate, decode routing and restart =================
    // Gate: the m-th waiting request of class k is a candidate; its position in the admission sequence is
    // the number of candidates that sort before it. Candidates are ranked in parallel; the idle prefill slot
    // of rank j (ascending server index) takes the candidate of rank j.
    // Routing: sequentially every job goes to the least-loaded feasible server, lowest index first: all
    // servers with the lowest decode count l get one job in index order, then all servers with at most l+1,
    // and so on. One pass fills up to kRouteLevels such levels at once. Level t takes take_t jobs, the first
    // of them job w_t of the pass; the server of rank q among those with at most lmin+t decodes takes job
    // w_t + q into slot lmin+t. Every lane places the jobs of its own server.
    // Both run side by side in passes of two segments with a barrier after each, the waves being shared out:
    //   A  the first half of the waves ranks the gate's candidates; the others take the pass's parameters from the load
    //      histograms and find the members of each level as bitmaps
    //   C  the last waves find the servers that are given work and serve them (admission, jobs, next event); the others
    //      draw the next step's arrivals; class counters
    // (A server at its event starts its next iteration in the completion pass, in the same lane. With a pass over all touched
    // servers at the end of the step, every wave in every segment and five barriers a step, 10000 servers x 256 replications
    // took 26.0 ms per 1000 steps instead of 22.0, 1024 x 2048 28.1 instead of 22.5.)
    // One pass is the rule; more follow only when more than kAdmChunk slots are idle or the jobs reach past
    // kRouteLevels levels or into the mixed group.
    {
      const int dcount0 = L.cs[CS_DCOUNT], dcount0_m = RR ? L.cs[CS_DCOUNT_M] : 0;
      int jrem, next = 0;
      {
        const int ncp = L.sc[SC_NCOMP], room = static_cast<int>(dbuf_cap) - dcount0;
        jrem = dcount0 + (ncp < room ? ncp : room);
      }
      const uint32_t dhead0 = static_cast<uint32_t>(L.cs[CS_DHEAD]);
      // randomized router only: jobs left, jobs placed and ring head of the solo [0] and the mixed [1] group's buffer
      int jremL[2] = {0, 0}, nextL[2] = {0, 0}, takenL[2] = {0, 0};
      const uint32_t dheadL[2] = {dhead0, RR ? static_cast<uint32_t>(L.cs[CS_DHEAD_M]) : 0u};
      if constexpr (RR) {
        jremL[0] = dcount0 + ncs;
        jremL[1] = dcount0_m + ncm;
        jrem = jremL[0] + jremL[1];
      }
      // abandonment only: ring entries of the decode buffer, this step's completions included
      uint32_t dlen_all = AB ? static_cast<uint32_t>(L.sc[SC_DLEN]) + static_cast<uint32_t>(RR ? ncs : jrem - dcount0) : 0u;
      if (dlen_all > dbuf_cap) dlen_all = dbuf_cap;   // (never more: the ring was compacted if it had to be)
      uint32_t dlen_all_m = AB && RR ? static_cast<uint32_t>(L.sc[SC_DLEN_M]) + static_cast<uint32_t>(ncm) : 0u;
      if (dlen_all_m > dbuf_cap) dlen_all_m = dbuf_cap;
      bool gate_on = true, route_on = jrem > 0;
      // weighted router: the random word of a selection follows from the step and the selection's number alone, so those
      // the first pass can need are drawn by waves with little to do, one a lane, while others fill the buffers
      const int ready0 = WS ? (jremL[0] < kJobsLds ? jremL[0] : kJobsLds) : 0;
      const int ready1 = WS ? (jremL[1] < kJobsLds - ready0 ? jremL[1] : kJobsLds - ready0) : 0;
      auto select_word = [&](int pool, int number) __attribute__((always_inline)) -> uint32_t {
        uint32_t w[4];
        philox4x32_10(key0, key1, s, static_cast<uint32_t>(kStreamSelect + pool), static_cast<uint32_t>(number),
                      static_cast<uint32_t>(r), w);
        return w[0];
      };
      for (int pass = 0; gate_on || route_on; ++pass) {
        if constexpr (kOverlap) {
          if (pass > 0 && slots_given > 0) {
            if (tid < 64) take_slots(nullptr);
            slots_given = 0;
            __syncthreads();
          }
        } else if (slots_taken) {   // (in a pass after the first)
          for (int w = tid; w < nwords_m; w += NT) L.bm_idle[w] &= ~L.bm_comp[w];
          slots_taken = false;
          __syncthreads();
        }
        if (gate_on && pass > 0) {
          if (tid < 64) {
            const uint32_t nidle = rank_bitmap(L.bm_idle, L.pre, nwords_m, M);
            if (tid == 0) L.sc[SC_NIDLE] = static_cast<int32_t>(nidle);
            if (tid < K) L.sc[SC_HEAD + tid] = L.cs[CS_QHEAD + tid];
          }
          __syncthreads();
        }
        if constexpr (WS) {
          if (pass == 0) {
            for (int j = NT - 1 - tid; j < ready0 + ready1; j += NT)   // the solo group's from the front, the other's from the back
              L.sel_u[j < ready0 ? j : kJobsLds - 1 - (j - ready0)] = select_word(j < ready0 ? 0 : 1, j < ready0 ? j : j - ready0);
            __syncthreads();   // the class selection reads them, and the buffer entries and counts written above
          }
        }
        // With abandonment the requests a routing pass places are first staged in LDS, by the waves that own the decode
        // buffers (each buffer has a wave of its own, on different SIMDs).
        const int ring_wave = nwaves >= 8 ? route_first : nwaves - 1;
        const int ring_wave_m = nwaves >= 8 ? route_first + 1 : nwaves - 1;
        // one wave walks a ring from where the last pass stopped and stages the next `need` waiting jobs
        // (in the first pass this step's completions may not have reached the ring: they are taken from `fresh`)
        const bool fresh_kept = AB && !WS && nwaves > 1 && pass == 0;
        auto stage_ring = [&](const uint64_t *ring, const uint32_t *dlr, uint32_t *calr, uint32_t hd, uint32_t len,
                              int scan_word, uint32_t need, int first_job) __attribute__((always_inline)) {
          uint32_t off = static_cast<uint32_t>(L.sc[scan_word]), found = 0, stop = off;   // (0 when a step begins)
          // four chunks of 64 entries per round: deadlines and requests are loaded together
          for (; off < len && found < need; off += 256) {   // wave-uniform
            uint32_t dl4[4];
            uint64_t jw4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint32_t i = off + 64u * u + lane;
              uint32_t pos = hd + i;
              if (pos >= dbuf_cap) pos -= dbuf_cap;
              dl4[u] = i < len ? dlr[pos] : 0u;   // (beyond the ring: counts as dead)
              jw4[u] = i < len ? ring[pos] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint32_t dl = dl4[u];
              const bool live = dl > s;
              const uint64_t bal = __ballot(live);
              const uint32_t rk = found + static_cast<uint32_t>(rank_in(bal));
              const bool mine = live && rk < need;
              if (mine) {
                L.jobs[first_job + rk] = jw4[u];
                if (dl != kNever)
                  atomicSub(&calr[static_cast<size_t>((jw4[u] >> 29) & 7u) * cal_n + (dl & p.cal_mask)], 1u);
              }
              const uint64_t last = __ballot(mine && rk + 1 == need);
              if (last) stop = off + 64u * u + static_cast<uint32_t>(__ffsll(static_cast<long long>(last)));   // one past the last staged entry
              found += static_cast<uint32_t>(__popcll(bal));
            }
          }
          // (what was not found among the entries of the steps before is the first of this step's completions, which follow
          // them; else see the gate's scan)
          if (lane == 0) L.sc[scan_word] = static_cast<int32_t>(found >= need ? stop : fresh_kept ? len + (need - found) : len);
        };
        // Weighted router: the pass's `need` placements in a pool each draw a class among those that still
        // wait in the pool's buffer (one after the other: a class that runs out drops from the later draws) and
        // take that class's requests in their order of arrival. The ring keeps the others where they are: an
        // entry that is taken gets a deadline that has passed, like an abandoned one.
        auto select_and_stage = [&](int pool, uint64_t *ring, uint32_t *dlr, uint32_t *calr, uint32_t hd, uint32_t len,
                                    int scan_word, int need, int first_job, int placed_before, int ready,
                                    int &nselv) __attribute__((always_inline)) {
          // Lane c knows of class c its selection weight, how many requests wait (a pass takes at most 256, larger counts
          // are capped) and how many the pass has selected. The draws do not depend on one another until a class runs out,
          // so they are evaluated 64 at a time, one per lane: a draw's class is the number of running sums of the waiting
          // classes' weights that it has reached, and its place within the class is how many lanes below it have the same
          // three bits of class number. The first draw that takes the last request of a class ends its round: the sums are
          // taken again without that class, and the next round starts behind it. (With a chain of scalar counts per class,
          // once for the rounds' ends, once for the classes left and once more for the places, a round took 2.8 thousand
          // cycles, now 1.3, of the one wave the others wait for: 10000 servers x 256, 300 steps, 8.84 -> 7.94 ms.)
          int cntv = 0, tookv = 0;
          uint32_t wtv = 0;
          if (lane < K) {
            const int solo_c = L.cs[CS_QDS + lane];
            cntv = pool == 0 ? solo_c : L.cs[CS_QD + lane] - solo_c;
            wtv = p.wsel[pool][lane];
          }
          cntv = cntv < 0 ? 0 : (cntv > 0xFFFF ? 0xFFFF : cntv);
          auto word_at = [&](int j) __attribute__((always_inline)) -> int { return pool == 0 ? j : kJobsLds - 1 - j; };
          for (int j = ready + lane; j < need; j += 64) L.sel_u[word_at(j)] = select_word(pool, placed_before + j);
          uint32_t cum[kMaxK], total;
          auto sum_weights = [&]() __attribute__((always_inline)) {
            const uint32_t cumv = wave_incl_scan(cntv > 0 ? wtv : 0u);
#pragma unroll
            for (int c = 0; c < kMaxK; ++c) cum[c] = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(cumv), c));
            total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(cumv), 63));
          };
          sum_weights();
          __builtin_amdgcn_wave_barrier();
          for (int done = 0; done < need;) {   // wave-uniform
            const int j = done + lane;
            const bool valid = j < need;
            const uint32_t u = valid ? L.sel_u[word_at(j)] : 0u;
            const uint32_t x = __umulhi(u, total);
            int pick = 0;
#pragma unroll
            for (int c = 0; c < kMaxK; ++c)
              if (c < K) pick += x >= cum[c] ? 1 : 0;
            if (pick > K - 1) pick = K - 1;   // (no class waits: cannot happen, the pass takes no more than wait)
            const ClassSets sets = class_sets(pick, __ballot(valid));
            const int ord = rank_in(sets.among(pick));
            const int known = __shfl(cntv | (tookv << 16), pick, 64);
            const uint64_t runs_out = __ballot(valid && ord + 1 == (known & 0xFFFF));
            const int n_valid = need - done < 64 ? need - done : 64;
            const int n_acc = runs_out ? __ffsll(static_cast<long long>(runs_out)) : n_valid;
            if (lane < n_acc) L.sel_co[first_job + j] = static_cast<uint16_t>(pick | (((known >> 16) + ord) << 3));
            if (lane < kMaxK) {
              const int n = __popcll(sets.among(lane) & (~0ull >> (64 - n_acc)));
              tookv += n;
              cntv -= n < cntv ? n : cntv;
            }
            if (runs_out) sum_weights();   // wave-uniform
            done += n_acc;
          }
          uint32_t place = wave_incl_scan(static_cast<uint32_t>(tookv)) - static_cast<uint32_t>(tookv);   // lane c: the first of class c
          __builtin_amdgcn_wave_barrier();
          for (int j0 = 0; j0 < need; j0 += 64) {   // wave-uniform
            const int j = j0 + lane;
            const int co = j < need ? L.sel_co[first_job + j] : 0;
            const int b = __shfl(static_cast<int>(place), co & 7, 64);
            if (j < need) L.sel_j[first_job + b + (co >> 3)] = static_cast<uint16_t>(j);
          }
          __builtin_amdgcn_wave_barrier();
          nselv = tookv;
          // walk the ring from the first entry that may still wait; the o-th waiting request of class c met on
          // the way is taken if the pass selected that class more than o times
          uint32_t off = static_cast<uint32_t>(L.sc[scan_word]), stop = off, first_left = 0xFFFFFFFFu;
          int left = need;
          place |= static_cast<uint32_t>(tookv) << 16;   // lane c: the next selection of class c, how many are left
          for (; off < len && left > 0; off += 256) {   // wave-uniform
            uint32_t dl4[4], pos4[4];
            uint64_t jw4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint32_t i = off + 64u * u + lane;
              uint32_t pos = hd + i;
              if (pos >= dbuf_cap) pos -= dbuf_cap;
              pos4[u] = pos;
              dl4[u] = i < len ? dlr[pos] : 0u;   // (beyond the ring: counts as gone)
              jw4[u] = i < len ? ring[pos] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (left > 0) {   // wave-uniform
                const uint32_t dl = dl4[u];
                const bool live = dl > s;
                const int c = static_cast<int>(jw4[u] >> 29) & 7;
                const ClassSets sets = class_sets(c, __ballot(live));
                const uint32_t ord = static_cast<uint32_t>(rank_in(sets.among(c)));
                const uint32_t next_c = static_cast<uint32_t>(__shfl(static_cast<int>(place), c, 64));
                const bool mine = live && ord < (next_c >> 16);
                if (lane < kMaxK) {
                  const uint32_t n = static_cast<uint32_t>(__popcll(sets.among(lane))), quota = place >> 16;
                  place += (n < quota ? n : quota) * 0xFFFF0001u;   // (one up in the lower half, one down in the upper)
                }
                if (mine) {
                  L.jobs[first_job + L.sel_j[first_job + (next_c & 0xFFFFu) + ord]] = jw4[u];
                  dlr[pos4[u]] = 0u;   // gone from the buffer
                  if (dl != kNever) atomicSub(&calr[static_cast<size_t>(c) * cal_n + (dl & p.cal_mask)], 1u);
                }
                const uint64_t stay = __ballot(live && !mine), took = __ballot(mine);
                if (first_left == 0xFFFFFFFFu && stay)
                  first_left = off + 64u * u + static_cast<uint32_t>(__ffsll(static_cast<long long>(stay))) - 1u;
                if (took) {
                  left -= __popcll(took);
                  stop = off + 64u * u + 64u - static_cast<uint32_t>(__clzll(static_cast<long long>(took)));   // one past the last taken entry
                }
              }
            }
          }
          // the next pass (and the head, at the end of the step) starts at the first entry that still waits
          if (lane == 0)
            L.sc[scan_word] = static_cast<int32_t>(first_left != 0xFFFFFFFFu ? first_left : (left > 0 ? len : stop));
        };
        auto stage_pass = [&](int total_pass) __attribute__((always_inline)) {
          // (each buffer has a wave of its own, on different SIMDs; in a large workgroup these waves leave the
          // level counts below to the others)
          if constexpr (RR) {
            if (wave == ring_wave) {
              if constexpr (WS) {
                int nsel_s = 0;
                if (takenL[0] > 0)
                  select_and_stage(0, dring, ddl, dcal, dheadL[0], dlen_all, SC_DSCAN, takenL[0], 0, nextL[0], pass == 0 ? ready0 : 0, nsel_s);
                // what the pass took from the solo group's buffer per class comes off that buffer's counts in
                // segment C: the other buffer's wave reads them meanwhile (what waits in the mixed group's buffer is
                // the class total less the solo buffer's share, and the total follows the placements later)
                if (lane < K) L.sel_n[lane] = nsel_s;
              } else {
                if (takenL[0] > 0)
                  stage_ring(dring, ddl, dcal, dheadL[0], fresh_kept ? dlen_all - static_cast<uint32_t>(ncs) : dlen_all, SC_DSCAN, static_cast<uint32_t>(takenL[0]), 0);
              }
            }
            if (wave == ring_wave_m && takenL[1] > 0) {
              if constexpr (WS) {
                int nsel_m;
                select_and_stage(1, dring_m, ddl_m, dcal_m, dheadL[1], dlen_all_m, SC_DSCAN_M, takenL[1], takenL[0], nextL[1], pass == 0 ? ready1 : 0, nsel_m);
              } else {
                stage_ring(dring_m, ddl_m, dcal_m, dheadL[1], fresh_kept ? dlen_all_m - static_cast<uint32_t>(ncm) : dlen_all_m, SC_DSCAN_M, static_cast<uint32_t>(takenL[1]), takenL[0]);
              }
            }
          } else {
            if (wave == ring_wave)
              stage_ring(dring, ddl, dcal, dhead0, fresh_kept ? dlen_all - static_cast<uint32_t>(jrem - dcount0) : dlen_all, SC_DSCAN, static_cast<uint32_t>(total_pass), 0);
          }
        };

        // ---------------- segment A ----------------
        anew();
        const int nidle = gate_on ? uniform(L.sc[SC_NIDLE]) : 0;
        if (gate_on && wave < n_gate) {
          const int limit = nidle < kAdmChunk ? nidle : kAdmChunk;
          // A candidate is ranked by 2, 4 or 8 neighbouring lanes (as many as there are classes), each of which counts
          // the candidates of one class that sort before it. A lane keeps its class for the pass: targets, counters and
          // how many candidates the class has.
          const int lg = K <= 2 ? 1 : K <= 4 ? 2 : 3;
          const int k2 = lane & ((1 << lg) - 1);
          const ClassTargets t2 = load_targets(L.gtab, k2);
          const int xs2 = L.cs[CS_X + k2], qp2 = L.cs[CS_QP + k2];
          const uint32_t head2 = static_cast<uint32_t>(L.cs[CS_QHEAD + k2]);
          auto fresh_of = [&](int k) __attribute__((always_inline)) -> uint32_t {   // (a later pass comes after a barrier)
            return pass > 0 ? 0xFFFFFFFFu : static_cast<uint32_t>((AB ? L.sc[SC_QLEN + k] : L.cs[CS_QP + k]) - L.sc[SC_TAKE + k]);
          };
          const uint32_t fresh2 = gate_mode == SIM_GATE_FCFS ? fresh_of(k2) : 0u;
          int cnt2 = ((admissible >> k2) & 1ull) && qp2 > 0 ? (qp2 < limit ? qp2 : limit) : 0;
          int ncand = __builtin_amdgcn_readfirstlane(static_cast<int>(group_sum(static_cast<uint32_t>(cnt2), lg)));
          const int nadm = ncand < limit ? ncand : limit;
          bool gate_more = false;
          // rare: more idle slots than one pass serves, and requests left to take them
          if (nadm == kAdmChunk && nidle > kAdmChunk) {
            const uint32_t left = ((admissible >> k2) & 1ull) ? static_cast<uint32_t>(qp2) : 0u;
            gate_more = uniform(static_cast<int>(group_sum(left, lg))) > nadm;
          }
          if (tid == 0) L.sc[SC_NADM] = nadm | (gate_more ? 0x10000 : 0);
          if (gate_mode == SIM_GATE_OCCUPANCY && (SMALL ? ncand << lg : ncand) > (n_gate << 6) && ncand > nadm &&
              __ballot(cnt2 > 0 && !(fabs(t2.nx) < 1e9)) == 0) {
            // Long queues offer up to `limit` candidates of every class, `limit` of which are admitted in all, and the others
            // need no rank. The keys of a class rise linearly, so a bound on the key tells how many of its candidates lie
            // below: the lanes try 64 bounds between the least key and one that is certainly high enough, and the classes
            // are cut behind the least bound with nadm candidates below it. Counted with a margin of one candidate a
            // class on the one side and cut with two on the other, so rounding cannot lose one that is admitted: no class
            // has a term of a milliard or more (below that a product's error, a part in 2^52 of it, is under 1e-6; with
            // larger targets nothing is cut). With six classes and 150 admissions a step the ranking went over 900
            // candidates, seven rounds of sixteen waves.
            const double inf = __longlong_as_double(0x7FF0000000000000ll);
            const double base2 = static_cast<double>(xs2) - t2.nx;
            const double least = group_min(cnt2 > 0 ? base2 * t2.invx : inf, lg);
            const double most = -group_min(cnt2 > 0 ? -((base2 + static_cast<double>(cnt2 - 1)) * t2.invx) : inf, lg);
            const double full = group_min(cnt2 >= nadm ? (base2 + static_cast<double>(nadm - 1)) * t2.invx : inf, lg);
            const double high = full < inf ? full : most;
            const double bound = least + (high - least) * (static_cast<double>(lane + 1) * 0.015625);
            int below = 0;
            for (int k = 0; k < K; ++k) {   // wave-uniform
              const double n = bound * readlane_f64(t2.xstar, k) - readlane_f64(base2, k);
              const int c = __builtin_amdgcn_readlane(cnt2, k);
              below += n > 0.0 ? (n < static_cast<double>(c) ? static_cast<int>(n) : c) : 0;
            }
            const uint64_t enough = __ballot(below >= nadm);
            if (enough) {
              const double cut = readlane_f64(bound, __ffsll(static_cast<long long>(enough)) - 1);
              const double n = cut * t2.xstar - base2 + 3.0;
              if (n < static_cast<double>(cnt2)) cnt2 = n > 0.0 ? static_cast<int>(n) : 0;
              ncand = __builtin_amdgcn_readfirstlane(static_cast<int>(group_sum(static_cast<uint32_t>(cnt2), lg)));
            }
          }
          if constexpr (AB) {
            // where the candidates sit in their rings: a wave per class walks from the head past the dead entries
            // (the last waves take this: the first ones rank the candidates below)
            for (int k = n_gate - 1 - wave; k < K; k += n_gate) {   // wave-uniform
              const uint32_t need = static_cast<uint32_t>(__builtin_amdgcn_readlane(cnt2, k));
              uint32_t qlen = static_cast<uint32_t>(L.sc[SC_QLEN + k]);
              if (qlen > queue_cap) qlen = queue_cap;
              // (in the first pass this step's arrivals may not have reached the ring: they wait behind the others, all of them)
              const uint32_t arrived = pass > 0 ? 0u : static_cast<uint32_t>(L.sc[SC_TAKE + k]);
              qlen -= arrived < qlen ? arrived : qlen;
              const uint32_t hd = static_cast<uint32_t>(L.cs[CS_QHEAD + k]);
              const uint32_t *dlr = qdl + static_cast<size_t>(k) * queue_cap;
              uint32_t found = 0;
              // four chunks of 64 entries per round: their deadlines are loaded together, one trip to memory
              for (uint32_t off = 0; off < qlen && found < need; off += 256) {   // wave-uniform
                uint32_t dl4[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  const uint32_t i = off + 64u * u + lane;
                  uint32_t pos = hd + i;
                  if (pos >= queue_cap) pos -= queue_cap;
                  dl4[u] = i < qlen ? dlr[pos] : 0u;   // (beyond the ring: counts as dead)
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  const uint32_t i = off + 64u * u + lane;
                  const bool live = dl4[u] > s;
                  const uint64_t bal = __ballot(live);
                  const uint32_t rk = found + static_cast<uint32_t>(rank_in(bal));
                  if (live && rk < need) L.live_off[k * kAdmChunk + rk] = i;
                  found += static_cast<uint32_t>(__popcll(bal));
                }
              }
              // (ring and arrivals hold as many live entries as the class counter says; if they ever did not, the
              // candidates beyond them would point at the head entry)
              for (uint32_t rk = found + lane; rk < need; rk += 64)
                L.live_off[k * kAdmChunk + rk] = rk - found < arrived ? qlen + (rk - found) : 0u;
              if (lane == 0 && need == 0) L.live_off[k * kAdmChunk] = 0;   // (no candidate: the head stays)
            }
            // only the FCFS gate reads the offsets while it ranks the candidates; the other gates first use them
            // after the barrier that ends this segment
            if (gate_mode == SIM_GATE_FCFS) __syncthreads();
          }
          // The searches of a candidate in the other classes run side by side on neighbouring lanes, which add up what they
          // find; the candidates of a class follow those of the class before it.
          if (nadm > 0) {   // wave-uniform
          const uint32_t cnt_class = lane < (1 << lg) ? static_cast<uint32_t>(cnt2) : 0u;
          const int first_lane = static_cast<int>(wave_incl_scan(cnt_class) - cnt_class);   // lane k: first candidate of class k
          int first_of[kMaxK], n_classes = K;
          asm volatile("" : "+s"(n_classes));   // (taken anew, as in tally_iterations)
#pragma unroll
          for (int kk = 1; kk < kMaxK; ++kk) first_of[kk] = kk < n_classes ? __builtin_amdgcn_readlane(first_lane, kk) : 0x7FFFFFFF;
          // First come, first served with few candidates: a lane per candidate fetches its arrival step, one trip to memory
          // for all of them, and the searches read each other's lanes. (Each step of a search is a trip to memory of its
          // own otherwise: 500 servers, three replications, 2000 steps, 20.9 -> 19.5 ms.)
          const bool few = gate_mode == SIM_GATE_FCFS && __ballot(cnt2 > (64 >> lg)) == 0;   // wave-uniform
          uint32_t stamp = kNever;
          if (few && (lane >> lg) < cnt2)
            stamp = gate_stamp(queue_cap, qring, lo_tab, head2, fresh2, s, k2, lane >> lg, kAdmChunk);
          // Occupancy gate: the key is linear in the sequence number, so the candidates of a class before this one end at an
          // estimate whose rounding errors are below 1e-8 while the terms are below 1e6: no comparison is needed unless it
          // lies next to a whole number (equal keys among them). With larger terms the exact comparisons on both sides of
          // the estimate are made, and if they say otherwise the rest is searched on the side they point to.
          auto search_near = [](auto before, double est, int most) __attribute__((always_inline)) -> int {
            int lo = 0, hi = most;
            const int g0 = est > 0.0 ? (est < static_cast<double>(hi) ? static_cast<int>(est) : hi) : 0;
            const int l2 = g0 > 1 ? g0 - 1 : 0, h2 = g0 + 2 < hi ? g0 + 2 : hi;
            const bool b0 = l2 == 0 || before(l2 - 1), b1 = h2 < hi && before(h2);
            if (b0) lo = b1 ? h2 + 1 : l2; else hi = l2 - 1;
            if (b0 && !b1) hi = h2;
            while (lo < hi) {
              const int mid = (lo + hi) >> 1;
              if (before(mid)) lo = mid + 1; else hi = mid;
            }
            return lo;
          };
          // A lane to a candidate, the classes one after another: half the instructions of a lane to each class, since a
          // candidate's own key is formed once. It pays where candidates are many (10000 servers x 256 replications past a load
          // peak 22.9 -> 22.5 ms per 1000 steps, 2048 x 1024 18.9 -> 18.7) and with two classes (1024 x 256 8.7 -> 8.6). Where a lane
          // to each class takes one round of the waves anyway, the chain over the classes is longer: 1024 x 256 of four classes
          // 10.5 -> 10.7, 1000 x 200 of six 10.2 -> 10.5, 2048 x 256 of eight 12.4 -> 13.2. (Both forms in one kernel, the few
          // candidates by class, take these back and cost two-class launches 1 to 2 %.) In workgroups of one or two waves, whose
          // first wave ranks alone and decides 64 admissions a pass, it gains nothing but with the fewest servers; a lane to each
          // class stays there. Its time with a lane to a candidate over that with a lane to each class: 8 servers of two classes 0.98,
          // 256 x 1024 and 700 x 2048 of two 1.003 and 1.005, 1024 x 2048 of two 0.999, of four 1.012, of eight 1.003, 128 x
          // 4096 of two 1.012 (the runs of one side differ by 0.5 %).
          if (!SMALL && gate_mode == SIM_GATE_OCCUPANCY) {   // wave-uniform
            const double base2 = static_cast<double>(xs2) - t2.nx;
            const uint64_t some = __ballot(cnt2 > 0), moderate = __ballot(fabs(t2.nx) < 1e6);
            for (int c0 = wave << 6; c0 < ncand; c0 += n_gate << 6) {   // wave-uniform
              const int c = c0 + lane;
              int k = 0;
#pragma unroll
              for (int kk = 1; kk < kMaxK; ++kk) k += c >= first_of[kk] ? 1 : 0;
              const int m = c - __shfl(first_lane, k, 64);
              const double own_nx = L.gtab[GT_NX * kMaxK + k], own_invx = L.gtab[GT_INVX * kMaxK + k];
              const double a = (static_cast<double>(L.cs[CS_X + k] + m) - own_nx) * own_invx;   // as gate_key has it
              int rank = m;
              for (int j = 0; j < K; ++j) {   // wave-uniform
                if (!((some >> j) & 1ull)) continue;
                const int cnt = __builtin_amdgcn_readlane(cnt2, j);
                const double reach = a * readlane_f64(t2.xstar, j), est = reach - readlane_f64(base2, j), up = ceil(est);
                int n = static_cast<int>(up);   // (of one too large for it no use is made)
                n = n < 0 ? 0 : (n < cnt ? n : cnt);
                const bool small_terms = fabs(reach) < 1e6 && ((moderate >> j) & 1ull);
                if (c < ncand && j != k && !(fabs((up - est) - 0.5) < 0.5 - 1e-6 && small_terms)) {
                  const ClassTargets tj = load_targets(L.gtab, j);
                  const int xj = __builtin_amdgcn_readlane(xs2, j), qj = __builtin_amdgcn_readlane(qp2, j);
                  const GateKey key = {a, static_cast<double>(L.cs[CS_QP + k] - m) - L.gtab[GT_NQ * kMaxK + k]};
                  auto before = [&](int i) __attribute__((always_inline)) -> bool {   // is the i-th of class j admitted before it
                    return gate_before(gate_key(SIM_GATE_OCCUPANCY, queue_cap, tj, qring, lo_tab, xj, qj, 0u, 0u, s, j, i, kAdmChunk), j, key, k);
                  };
                  if (small_terms) {   // next to a whole number: that one is compared
                    const int at = static_cast<int>(rint(est));
                    n = at < 0 ? 0 : (at < cnt ? at + (before(at) ? 1 : 0) : cnt);
                  } else {
                    n = search_near(before, est, cnt);
                  }
                }
                rank += j == k ? 0 : n;
              }
              if (c < ncand && rank < nadm) {
                L.adm[rank] = static_cast<uint16_t>(k | (m << 3));
                atomicAdd(&L.sc[SC_ADMK + k], 1);
              }
            }
          } else {
          const int mode_here = SMALL ? gate_mode : gate_mode == SIM_GATE_PRIORITY ? SIM_GATE_PRIORITY : SIM_GATE_FCFS;
          for (int c0 = wave << 6; c0 < (ncand << lg); c0 += n_gate << 6) {   // wave-uniform trip count
            const int c = (c0 + lane) >> lg;
            int k = 0, lo = 0;
#pragma unroll
            for (int kk = 1; kk < kMaxK; ++kk) k += c >= first_of[kk] ? 1 : 0;
            const int m = c - __shfl(first_lane, k, 64);
            if (few) {
              const uint32_t own = static_cast<uint32_t>(__shfl(static_cast<int>(stamp), (m << lg) + k, 64));
              auto before = [&](int j) __attribute__((always_inline)) -> bool {   // (behind a class's last candidate: never)
                const uint32_t other = static_cast<uint32_t>(__shfl(static_cast<int>(stamp), (j << lg) + k2, 64));
                return other < own || (other == own && k2 < k);
              };
              for (int n = 32 >> lg; n > 0; n >>= 1) lo += before(lo + n - 1) ? n : 0;   // wave-uniform
              lo += before(lo) ? 1 : 0;
              if (k2 == k) lo = m;
            } else if (c < ncand) {
              if (k2 == k) {
                lo = m;
              } else if (cnt2 > 0) {   // those before it form a prefix of the class
                // this candidate's own key: one trip to LDS
                const ClassTargets own = load_targets(L.gtab, k);
                const GateKey key = gate_key(mode_here, queue_cap, own, qring, lo_tab, L.cs[CS_X + k], L.cs[CS_QP + k],
                                             static_cast<uint32_t>(L.cs[CS_QHEAD + k]), fresh_of(k), s, k, m, kAdmChunk);
                auto before = [&](int j) __attribute__((always_inline)) -> bool {   // is the j-th of class k2 admitted before it
                  return gate_before(gate_key(mode_here, queue_cap, t2, qring, lo_tab, xs2, qp2, head2, fresh2, s, k2, j, kAdmChunk), k2, key, k);
                };
                if (SMALL && gate_mode == SIM_GATE_OCCUPANCY) {
                  const double reach = key.a * t2.xstar, est = reach - (static_cast<double>(xs2) - t2.nx), up = ceil(est);
                  if (fabs((up - est) - 0.5) < 0.5 - 1e-6 && fabs(reach) < 1e6 && fabs(t2.nx) < 1e6)
                    lo = up > 0.0 ? (up < static_cast<double>(cnt2) ? static_cast<int>(up) : cnt2) : 0;
                  else
                    lo = search_near(before, est, cnt2);
                } else if (gate_mode == SIM_GATE_PRIORITY) {   // one key for the whole class
                  lo = before(0) ? cnt2 : 0;
                } else {
                  int hi = cnt2;
                  while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (before(mid)) lo = mid + 1; else hi = mid;
                  }
                }
              }
            }
            const int rank = static_cast<int>(group_sum(static_cast<uint32_t>(lo), lg));
            if (c < ncand && k2 == 0 && rank < nadm) {
              L.adm[rank] = static_cast<uint16_t>(k | (m << 3));
              atomicAdd(&L.sc[SC_ADMK + k], 1);
            }
          }
          }
          }
        }
        if constexpr (AB) {   // (the barrier between the walk and the ranking, for the other waves)
          if (gate_on && wave >= n_gate && gate_mode == SIM_GATE_FCFS) __syncthreads();
        }
        // routing pass: up to kRouteLevels levels, first of the solo group (servers M..N-1), then, if that group
        // is full by then, of the mixed group (servers 0..M-1, one slot less). Level t of group G holds the
        // servers of G with at most lminG + (t - firstG) decodes.
        int nl = 0, total = 0;
        int lminG[2] = {0, 0}, nG[2] = {0, 0}, csumG[2] = {0, 0}, tlastG[2] = {0, 0};
        if (route_on && wave >= route_first) {
          // Placements on a mixed-group server must see every admission of the step (it decides whether the job
          // counts as mixed or solo decode): while the gate may need another pass, only the solo group is routed.
          bool gate_unfinished = false;
          if (nidle > kAdmChunk) {   // rare (wave-uniform): does the pass admit all it can
            int n = 0;
            for (int k = 0; k < K; ++k) {
              const int qp = uniform(L.cs[CS_QP + k]);
              if ((admissible >> k) & 1ull) n += qp < kAdmChunk ? qp : kAdmChunk;
            }
            gate_unfinished = n >= kAdmChunk;
          }
          // (every one of these waves computes the same values and stores them: no broadcast, no barrier)
          // (with abandonment a pass places no more jobs than are staged in LDS)
          const int jpass = AB && jrem > kJobsLds ? kJobsLds : jrem;
          int rem_jobs = jpass;
          // The load histograms of both groups (servers per decode count below the cap) are read once, one bin per
          // lane and register; the lowest non-empty level and the counts of the levels above it then come from
          // ballots and lane reads instead of a chain of LDS round trips.
          uint32_t hv[2][2];
#pragma unroll
          for (int gi = 0; gi < 2; ++gi) {
            hv[gi][0] = L.lh[gi * kLoadBins + lane];
            hv[gi][1] = L.lh[gi * kLoadBins + 64 + lane];
          }
          auto lowest_level = [&](int gi, int capg) __attribute__((always_inline)) -> int {
            const uint64_t nz0 = __ballot(lane < capg && hv[gi][0] != 0);
            if (nz0) return __ffsll(static_cast<long long>(nz0)) - 1;
            const uint64_t nz1 = __ballot(64 + lane < capg && hv[gi][1] != 0);
            return nz1 ? 63 + __ffsll(static_cast<long long>(nz1)) : -1;
          };
          auto level_count = [&](int gi, int level) __attribute__((always_inline)) -> uint32_t {   // level: wave-uniform, below 128
            const int lo = __builtin_amdgcn_readlane(static_cast<int>(hv[gi][0]), level & 63);
            const int hi = __builtin_amdgcn_readlane(static_cast<int>(hv[gi][1]), level & 63);
            return static_cast<uint32_t>(level < 64 ? lo : hi);
          };
          bool full[2] = {M >= N, M == 0};   // no slot of the group is left behind the pass (as far as it has looked)
          if constexpr (RR) {
            // each group takes jobs from its own ring; the pass's list holds the solo ring's jobs first and is
            // never longer than what is staged in LDS
            int listed = 0;
            takenL[0] = takenL[1] = 0;
#pragma unroll
            for (int gi = 0; gi < 2; ++gi) {
              const int glo = gi == 0 ? M : 0, ghi = gi == 0 ? N : M;
              const int capg = gi == 0 ? B : B - 1;
              int rem_g = jremL[gi] < kJobsLds - listed ? jremL[gi] : kJobsLds - listed;
              const int start_g = rem_g;
              if (glo >= ghi || nl >= kRouteLevels || rem_g <= 0 || (gi == 1 && gate_unfinished)) continue;   // wave-uniform
              const int lm = lowest_level(gi, capg);
              if (lm < 0) { full[gi] = true; continue; }
              lminG[gi] = lm;
              for (int u = 0; nl < kRouteLevels && rem_g > 0 && lm + u < capg; ++u) {
                const int cnt = static_cast<int>(level_count(gi, lm + u));
                csumG[gi] += cnt;
                const int tk = csumG[gi] < rem_g ? csumG[gi] : rem_g;
                if (lane == 0) { L.sc[SC_TAKE_T + nl] = tk; L.sc[SC_CNT_T + nl] = cnt; L.sc[SC_W_T + nl] = listed + (start_g - rem_g); }
                rem_g -= tk;
                tlastG[gi] = tk;
                ++nG[gi];
                ++nl;
              }
              full[gi] = rem_g > 0 && lm + nG[gi] >= capg;
              takenL[gi] = start_g - rem_g;
              listed += takenL[gi];
            }
            rem_jobs = jpass - listed;
          } else {
#pragma unroll
          for (int gi = 0; gi < 2; ++gi) {
            const int glo = gi == 0 ? M : 0, ghi = gi == 0 ? N : M;
            const int capg = gi == 0 ? B : B - 1;
            if (glo >= ghi || nl >= kRouteLevels || rem_jobs <= 0 || (gi == 1 && gate_unfinished)) continue;   // wave-uniform
            const int lm = lowest_level(gi, capg);
            if (lm < 0) { full[gi] = true; continue; }
            lminG[gi] = lm;
            for (int u = 0; nl < kRouteLevels && rem_jobs > 0 && lm + u < capg; ++u) {
              const int cnt = static_cast<int>(level_count(gi, lm + u));
              csumG[gi] += cnt;
              const int tk = csumG[gi] < rem_jobs ? csumG[gi] : rem_jobs;
              if (lane == 0) { L.sc[SC_TAKE_T + nl] = tk; L.sc[SC_CNT_T + nl] = cnt; L.sc[SC_W_T + nl] = jpass - rem_jobs; }
              rem_jobs -= tk;
              tlastG[gi] = tk;
              ++nG[gi];
              ++nl;
            }
            full[gi] = rem_jobs > 0 && lm + nG[gi] >= capg;
          }
          }
          total = jpass - rem_jobs;
          // another pass follows if jobs and slots for them may be left (the levels of a pass, what it stages, or a mixed group
          // that waits for the gate set its bounds)
          const bool more = RR ? (jremL[0] > takenL[0] && !full[0]) || (jremL[1] > takenL[1] && !full[1])
                               : jrem > total && !(full[0] && full[1]);
          if (lane == 0) {
            L.sc[SC_LEVELS] = nl | (nG[0] << 8) | (more ? 0x10000 : 0);
            L.sc[SC_LMIN] = lminG[0] | (lminG[1] << 16);
          }
          if (nl > 0) {
            // Waves that count the servers of each level, and this wave's place among them. With abandonment the
            // requests the pass places are first staged in LDS by the waves that own the decode buffers: a large
            // workgroup gives them no counting to do, so that the staging runs beside the gate's ranking.
            int cw = wave - route_first, cn = n_route;
            if constexpr (AB) {
              stage_pass(total);
              if (nwaves >= 8) {   // the first of these waves are the buffers'
                constexpr int n_ring = RR ? 2 : 1;
                cn = n_route - n_ring;
                cw = cw < n_ring ? nwords : cw - n_ring;   // (nothing to count)
              }
            }
            // A lane looks at sixteen servers, four decode counts at a time: the top bit of a byte of `at_most` less the counts
            // says that the server has no more than the level's (a count is at most 128, a level below that: no borrow), and
            // four of them become four bits of the bitmap in one dot product. (A comparison a server, its ballot written to a
            // lane, took three instructions a word and level, 157 words with 10000 servers; this takes 16 for sixteen words:
            // 10000 servers x 256 replications 20.4 -> 20.0 ms per 1000 steps, randomized router 6.74 -> 6.26 per 300, 1024 x
            // 2048 19.1 -> 18.5, 3001 x 77 7.16 -> 6.79 per 500.)
            // The words of a group that no level is of are left out.
            const int w_first = nG[1] > 0 ? 0 : M >> 6, w_end = nG[0] > 0 ? nwords : ((M + 63) >> 6);
            for (int p0 = 4 * w_first + (cw << 6); p0 < 4 * w_end; p0 += cn << 6) {   // wave-uniform; quarters of words
              const int part = p0 + lane, g0 = part << 4;
              if (part < 4 * w_end) {
                const int n_all = N - g0, n_mixed = M - g0;
                const uint32_t all = (1u << (n_all < 16 ? (n_all > 0 ? n_all : 0) : 16)) - 1u;
                const uint32_t mixed = (1u << (n_mixed < 16 ? (n_mixed > 0 ? n_mixed : 0) : 16)) - 1u, solo = all & ~mixed;
                uint2 ld[2] = {make_uint2(0u, 0u), make_uint2(0u, 0u)};
                if (n_all > 0) {   // (what is read past the last server, up to eight bytes, belongs to the array behind)
                  const uint2 *at = reinterpret_cast<const uint2 *>(L.loads + g0);
                  ld[0] = at[0]; ld[1] = at[1];
                }
#pragma unroll
                for (int t = 0; t < kRouteLevels; ++t) {
                  if (t < nl) {   // wave-uniform
                    const bool of_solo = t < nG[0];
                    const uint32_t at_most = (static_cast<uint32_t>(of_solo ? lminG[0] + t : lminG[1] + (t - nG[0])) | 0x80u) * 0x01010101u;
                    uint32_t half[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                      half[h] = __builtin_amdgcn_udot4((at_most - ld[h].x) & 0x80808080u, 0x08040201u, 0u, false);
                      half[h] = __builtin_amdgcn_udot4((at_most - ld[h].y) & 0x80808080u, 0x80402010u, half[h], false);
                    }
                    const uint32_t members = ((half[0] >> 7) | (half[1] << 1)) & (of_solo ? solo : mixed);
                    reinterpret_cast<uint16_t *>(L.bm_lvl)[4 * t * nwords + part] = static_cast<uint16_t>(members);
                  }
                }
              }
            }
          }
        }
        __syncthreads();

        // ---------------- segment C ----------------
        anew();
        const int sc_pass = L.sc[lane];   // one word a lane: one trip to LDS
        auto word_of = [&](int i) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(sc_pass, i); };
        const int nadm = gate_on ? word_of(SC_NADM) & 0xFFFF : 0;
        const bool gate_more = gate_on && (word_of(SC_NADM) & 0x10000);
        const int levels = route_on ? word_of(SC_LEVELS) : 0;
        const int nl_here = levels & 0xFF, nl_solo = (levels >> 8) & 0xFF;
        int take_r[kRouteLevels], w_r[kRouteLevels];
#pragma unroll
        for (int t = 0; t < kRouteLevels; ++t) { take_r[t] = word_of(SC_TAKE_T + t); w_r[t] = word_of(SC_W_T + t); }
        int placed = 0, placed_solo = 0;   // jobs the pass places, of them (two buffers) from the solo group's
#pragma unroll
        for (int t = 0; t < kRouteLevels; ++t) {
          if (t < nl_here) placed = w_r[t] + take_r[t];
          if (t < nl_solo) placed_solo = w_r[t] + take_r[t];
        }
        if (pass == 0 && tid == 0) {   // the completions of this step are in the buffer
          if constexpr (RR) { L.cs[CS_DCOUNT] = jremL[0]; L.cs[CS_DCOUNT_M] = jremL[1]; }
          else L.cs[CS_DCOUNT] = jrem;
        }
        if (gate_on && tid < K) {   // class counters follow the admissions of this pass
          const int k = tid, adm_k = L.sc[SC_ADMK + k];
          // ring entries the head moves past: the admitted requests; with abandonment also the dead entries
          // before the last of them (before the first waiting request when none was admitted)
          uint32_t past = static_cast<uint32_t>(adm_k);
          if constexpr (AB) {
            past = adm_k ? L.live_off[k * kAdmChunk + adm_k - 1] + 1u : L.live_off[k * kAdmChunk];
            if (past) {
              L.sc[SC_QLEN + k] -= static_cast<int32_t>(past);
              if (!adm_k) {
                uint32_t h = static_cast<uint32_t>(L.cs[CS_QHEAD + k]) + past;
                if (h >= queue_cap) h -= queue_cap;
                L.cs[CS_QHEAD + k] = static_cast<int32_t>(h);
              }
            }
          }
          if (adm_k) {
            uint32_t h = static_cast<uint32_t>(L.cs[CS_QHEAD + k]) + past;
            if (h >= queue_cap) h -= queue_cap;
            L.cs[CS_QHEAD + k] = static_cast<int32_t>(h);
            L.cs[CS_QP + k] -= adm_k;
            L.cs[CS_X + k] += adm_k;
            L.tl[k * kNTally + SIM_T_U_P] += static_cast<uint64_t>(adm_k);
            L.sc[SC_ADMK + k] = 0;
          }
        }
        // The servers that are given work: the admissions take the first nadm idle prefill slots, in every routing level the
        // first take_r of its members get a job. The last waves find these servers (a lane looks at a word), queue 64 of them
        // and serve those, one a lane; as long as no level is of the mixed group no server gets both, and admissions
        // and jobs are served by waves of their own. The other waves see to the next step's arrivals meanwhile.
        const int work = nadm + placed;   // (servers, or more: one may get an admission and jobs)
        const int n_adm = (nadm + 63) >> 6, n_job = (placed + 63) >> 6, n_both = (work + 63) >> 6;
        const bool apart = nadm > 0 && placed > 0 && nl_here == nl_solo && nwaves >= 4 && n_adm + n_job <= (nwaves >> 1);
        const int n_serve = apart ? n_adm + n_job : n_both < nwaves ? n_both : nwaves;
        // (left to the next completion pass, where all waves take part, if these would get more than sixteen words each)
        const bool draws_here = !kBeside && work > 0 && !drawn && s + 1u < step_end && n_serve < nwaves && 16 * (nwaves - n_serve) >= nwords;
        if (work > 0 && wave < nwaves - n_serve) {
          if constexpr (kBeside) {
            if (wave < n_draw && drawn) {
              count_requests(s + 1u, wave, n_draw);
              drawn = false;
            }
          } else if (draws_here) {
            __builtin_amdgcn_s_setprio(0);
            draw_words(s + 1u, wave, nwaves - n_serve);
            count_requests(s + 1u, wave, nwaves - n_serve);
            if constexpr (kChainFirst) __builtin_amdgcn_s_setprio(3); else own_priority();
          }
        } else if (work > 0) {
          if constexpr (kServeFirst) __builtin_amdgcn_s_setprio(3);
          // this wave is the my_serve-th of n_serve_kind that serve its kind
          const bool for_jobs = !apart || wave >= nwaves - n_job, for_adm = !apart || !for_jobs;
          const int n_serve_kind = !apart ? n_serve : for_jobs ? n_job : n_adm;
          const int my_serve = (apart && !for_jobs ? nwaves - n_job : nwaves) - 1 - wave;
          const int nadm_here = for_adm ? nadm : 0, nl_mine = for_jobs ? nl_here : 0;
          const int lvl_first = nl_here > nl_solo ? 0 : M >> 6, lvl_end = nl_solo > 0 ? nwords : (M + 63) >> 6;   // words with levels
          // Everything a step gives a server, and what follows from it, in one go: its admission, its jobs, and either the next
          // event (the server is idle or at an iteration boundary) or the end of the running iteration as its event.
          auto serve = [&](int nsrv) __attribute__((always_inline)) {   // (up to 64)
              const bool active = lane < nsrv;
              uint32_t m = 0, d = 0;   // iterations to tally
              bool chunk = false, comes_next = false;
              uint64_t comp = 0;
              if (active) {
                const int entry = ev_g[lane], g = entry & 0x7FFF, wi = g >> 6;
                const bool admitted = entry & 0x8000;   // the idle slot of rank j takes the candidate of rank j
                const uint64_t bit = 1ull << (g & 63);
                uint64_t nc = rec[g].n_cls, nj = rec[g].n_join;
                uint32_t it_tal = rec[g].iter, nf = rec[g].next_fin;
                const uint64_t idle = L.bm_idle[wi];
                const bool busy = L.bm_busy[wi] & bit, due = L.bm_just[side + wi] & bit;
                const int n_own = static_cast<int>(L.loads[g]);   // decodes of the server
                int rem = g < Mp ? static_cast<int>(L.rem[g]) : 0;
                const uint32_t ev = L.ev_it[g];
                uint32_t it = ev & kEvIter;
                const bool had_chunk = ev & kEvChunk, pin = joins_next(nj, rem, had_chunk);
                const int64_t rel = event_time(g, T);
                // ---- the admission
                int a_k = 0;
                uint32_t a_stamp = 0, a_in = 0, a_out = 0;
                if (admitted) {
                  const int j = static_cast<int>(L.pre[wi]) + __popcll(idle & (bit - 1ull));
                  const uint32_t e = L.adm[j];
                  a_k = static_cast<int>(e & 7u);
                  uint32_t pos = static_cast<uint32_t>(L.sc[SC_HEAD + a_k]) + (AB ? L.live_off[a_k * kAdmChunk + (e >> 3)] : (e >> 3));
                  if (pos >= queue_cap) pos -= queue_cap;
                  a_stamp = qring[static_cast<size_t>(a_k) * queue_cap + pos];
                  if constexpr (AB) {   // the request no longer waits: it leaves the calendar of its deadline
                    const uint32_t dl = qdl[static_cast<size_t>(a_k) * queue_cap + pos];
                    if (dl != kNever) atomicSub(&cal[static_cast<size_t>(a_k) * cal_n + (dl & p.cal_mask)], 1u);
                  }
                  uint32_t w[4];
                  philox4x32_10(key0, key1, s, 1u, static_cast<uint32_t>(g), static_cast<uint32_t>(r), w);
                  a_in = len_tab[(static_cast<size_t>(a_k) * 2 + 0) * kTableSize + (w[0] >> 16)];
                  a_out = len_tab[(static_cast<size_t>(a_k) * 2 + 1) * kTableSize + (w[1] >> 16)];
                }
                // ---- its jobs: which one of each level the server takes follows from its rank among the level's members (looked up here,
                //      while its record is on the way)
                uint64_t job_of[kRouteLevels];
                uint32_t takes = 0;
                const bool has_prefill = g < Mp && (admitted || !(idle & bit));
                const int gi = g >= M ? 0 : 1;
                const int lmins = word_of(SC_LMIN);
                const int first = gi == 0 ? 0 : nl_solo, my_lmin = gi == 0 ? lmins & 0xFFFF : lmins >> 16;
#pragma unroll
                for (int t = 0; t < kRouteLevels; ++t) {
                  if (t < nl_mine) {   // wave-uniform
                    const uint64_t in = wi >= lvl_first && wi < lvl_end ? L.bm_lvl[t * nwords + wi] : 0ull;
                    const int q = static_cast<int>(L.pre_lvl[t * nwords + wi]) + __popcll(in & (bit - 1ull));
                    if ((in & bit) && q < take_r[t]) {
                      const int j = w_r[t] + q;   // position in this pass
                      uint64_t &jw = job_of[t];
                      takes |= 1u << t;
                      if constexpr (AB) {
                        jw = L.jobs[j];
                        if (fresh_kept) {
                          const int i = RR && gi ? j - placed_solo : j;   // place in the group's buffer, live requests only
                          const int ci = i - (RR && gi ? dcount0_m : dcount0);
                          if (ci >= 0) {   // one of this step's completions: it leaves the calendar of its deadline
                            const uint32_t fill = RR && gi ? dlen_all_m - static_cast<uint32_t>(ncm) : dlen_all - static_cast<uint32_t>(RR ? ncs : jrem - dcount0);
                            uint32_t pos = (RR ? dheadL[gi] : dhead0) + fill + static_cast<uint32_t>(ci);
                            if (pos >= dbuf_cap) pos -= dbuf_cap;
                            if (pos >= dbuf_cap) pos -= dbuf_cap;
                            constexpr int kHere = RR ? kJobsLds / 2 : kJobsLds;
                            jw = L.fresh[(RR && gi ? kHere : 0) + (ci < kHere ? ci : 0)];
                            asm("" : "+v"(jw));   // (see below)
                            if (ci >= kHere) { if (!RR || gi == 0) jw = dring[pos]; else jw = dring_m[pos]; }
                            uint32_t dl;
                            if (!RR || gi == 0) dl = ddl[pos]; else dl = ddl_m[pos];
                            if (dl != kNever) {
                              uint32_t *at = &dcal[((jw >> 29) & 7u) * static_cast<size_t>(cal_n) + (dl & p.cal_mask)];
                              if constexpr (RR) { if (gi) at = &dcal_m[((jw >> 29) & 7u) * static_cast<size_t>(cal_n) + (dl & p.cal_mask)]; }
                              atomicSub(at, 1u);
                            }
                          }
                        }
                      } else {   // this step's completions are in LDS too, behind them what has waited in the ring
                        const int i = RR ? (gi == 0 ? nextL[0] + j : nextL[1] + j - placed_solo) : next + j;
                        const int ci = i - (RR && gi ? dcount0_m : dcount0);
                        constexpr int kHere = RR ? kJobsLds / 2 : kJobsLds;
                        const bool here = ci >= 0 && ci < kHere;
                        jw = L.jobs[here ? (RR && gi ? kHere : 0) + ci : 0];
                        asm("" : "+v"(jw));   // (else the two loads become one through a pointer to either memory)
                        if (!here) {
                          uint32_t pos = (RR ? dheadL[gi] : dhead0) + static_cast<uint32_t>(i);
                          if (pos >= dbuf_cap) pos -= dbuf_cap;
                          if (pos >= dbuf_cap) pos -= dbuf_cap;
                          if (!RR || gi == 0) jw = dring[pos]; else jw = dring_m[pos];
                        }
                      }
                    }
                  }
                }
                // ---- where the server stands: `it` iterations are completed; in the middle of one (`mid`: what it is given
                //      now joins when that one ends), at a boundary, the iterations before it then being tallied, or idle.
                //      A server that has had its event in this step is at the boundary it was started anew from.
                int64_t start = due ? rel : 0;   // (idle: back to back after a completion in this step, else from the step boundary)
                bool mid = false;
                uint32_t dur = 0;
                if (busy) {
                  uint32_t left = 1;   // iterations up to the event
                  mid = pin;
                  if (!pin) {
                    const int ptok = had_chunk ? chunk_of(rem) : 0;
                    dur = iteration_ns(ptok, static_cast<uint32_t>(n_own));
                    left = iterations_left(static_cast<uint64_t>(rel), dur);
                    start = rel - static_cast<int64_t>(static_cast<uint64_t>(left) * dur);   // end of the latest completed iteration
                    mid = start <= -static_cast<int64_t>(dt_ns);
                    if (!mid) {
                      m = it - left - it_tal;
                      d = dur;
                      chunk = had_chunk;
                      comp = nc;
                      rem -= static_cast<int>(m) * ptok;
                    }
                  }
                  it -= left;
                }
                if (!mid) { it_tal = it; nj = 0; }
                // ---- the request admitted; decodes beside it switch solo -> mixed
                if (admitted) {
                  rec[g].pf_job = static_cast<uint64_t>(a_stamp) | (static_cast<uint64_t>(a_k) << 29) |
                                  (static_cast<uint64_t>(a_in - 1) << 32) | (static_cast<uint64_t>(a_out - 1) << 48);
                  rem = static_cast<int>(a_in);   // an idle prefill slot implies that the running iteration holds no chunk
                  lds_add64(&L.tl[a_k * kNTally + SIM_T_WAIT_STEPS], static_cast<uint64_t>(s - a_stamp));
                  if (n_own) {
                    int n_classes = K;   // (taken anew, as in tally_iterations)
                    asm volatile("" : "+s"(n_classes));
                    // (two classes at a time: there are no fewer solo decodes of a class than these servers have, and nothing is
                    // taken from the class above)
#pragma unroll
                    for (int c = 0; c < kMaxK; c += 2) {
                      if (c >= n_classes) break;   // wave-uniform
                      const uint64_t v = two_bytes_at(nc, c);
                      if (v == 0) continue;
                      lds_add64(&L.tl[c * kNTally + SIM_T_M_SM], static_cast<uint32_t>(v));
                      lds_add64(&L.tl[(c + 1) * kNTally + SIM_T_M_SM], v >> 32);
                      lds_add64(reinterpret_cast<uint64_t *>(&L.cs[CS_YS + c]), 0ull - v);
                      lds_add64(reinterpret_cast<uint64_t *>(&L.cs[CS_YM + c]), v);
                    }
                  }
                }
                // ---- the jobs
                int nd = n_own;
#pragma unroll
                for (int t = 0; t < kRouteLevels; ++t) {
                  if ((takes >> t) & 1u) {
                    const uint64_t jw = job_of[t];
                    const int k = static_cast<int>(jw >> 29) & 7;
                    const int slot = my_lmin + (t - first);   // the server holds exactly this many decodes by now
                    const uint32_t ends = it + static_cast<uint32_t>(jw >> 48) + 1u + (mid ? 1u : 0u);
                    nf = nd == 0 || ends < nf ? ends : nf;
                    fin[static_cast<size_t>(g) * BS + slot] = ends;
                    job[static_cast<size_t>(g) * BS + slot] = jw;
                    nc += 1ull << (8 * k);
                    if (mid) nj += 1ull << (8 * k);   // not part of the iterations still to be tallied for this server
                    nd = slot + 1;
                    lds_add64(&L.tl[k * kNTally + (has_prefill ? SIM_T_U_DM : SIM_T_U_DS)], 1);
                    atomicAdd(&L.cs[(has_prefill ? CS_YM : CS_YS) + k], 1);
                    atomicSub(&L.cs[CS_QD + k], 1);
                  }
                }
                // ---- the next event
                if (!mid) {   // starts the next iteration with what it holds now
                  const int ptok = rem > 0 ? chunk_of(rem) : 0;
                  dur = iteration_ns(ptok, static_cast<uint32_t>(nd));
                  const uint32_t n = phase_length(static_cast<uint32_t>(nd), rem, dur, nf - it);
                  set_event(g, T + start + static_cast<int64_t>(static_cast<uint64_t>(n) * dur), it + n, ptok > 0, nd && nf == it + n);
                  if (!busy) atomicOr(bits64(&L.bm_busy[wi]), bit);
                } else if (!pin) {   // the end of the running iteration
                  set_event(g, T + start + dur, it + 1u, had_chunk, nd && nf == it + 1u);
                }
                if (admitted || (chunk && m)) L.rem[g] = static_cast<uint16_t>(rem);
                L.loads[g] = static_cast<uint8_t>(nd);
                rec[g].n_cls = nc;
                rec[g].n_join = nj;
                rec[g].iter = it_tal;
                rec[g].next_fin = nf;
                if constexpr (kOverlap) {
                  comes_next = event_time(g, T + dt_ns) <= 0;
                  late_g = g;
                }
              }
              if constexpr (kOverlap) late = __ballot(comes_next);
              tally_iterations<kTallyRowsHere>(L.ta, L.tbth, tbt_w, tbt_lo, K, m, d, chunk, comp);
          };
          // Which servers: the members of every level before a lane's word are counted, two levels in one sum.
          int lo = my_serve << 6, n_all = 0;   // this wave's are lo, lo + 1, ... of n_all
          do {   // (a second time round only where even all waves are too few)
            uint32_t before[2] = {0, 0};   // members of the levels in the words before
            n_all = 0;
            // (words of a group none of whose servers this wave serves are left out: 10000 x 256, 38 of 157 words mixed, 16.25 ->
            // 15.62 ms per 1000 steps)
            const int w_first = nadm_here > 0 || (nl_mine > 0 && nl_here > nl_solo) ? 0 : M >> 6;
            const int w_last = nl_mine > 0 && nl_solo > 0 ? nwords : nwords_m;
            for (int w0 = w_first; w0 < w_last; w0 += 64) {   // wave-uniform
              const int w = w0 + lane;
              uint64_t adm = 0, got = 0;
              if (nadm_here > 0 && w0 < nwords_m) {   // wave-uniform
                uint64_t slots = 0;
                int left = 0;
                if (w < nwords_m) {
                  slots = L.bm_idle[w] & bits_below(w, M);   // the gate admits to the mixed group only
                  left = nadm_here - static_cast<int>(L.pre[w]);
                }
                adm = first_members(slots, left);
                got = adm;
                // (other waves may still look at bm_idle: the slots given away are taken out of it later)
                if constexpr (!kOverlap) { if (my_serve == 0 && w < nwords_m) L.bm_comp[w] = adm; }
              }
#pragma unroll
              for (int t0 = 0; t0 < kRouteLevels; t0 += 2) {
                if (t0 < nl_mine && w0 < lvl_end && w0 + 64 > lvl_first) {   // wave-uniform
                  uint64_t in[2];
                  uint32_t n = 0;
#pragma unroll
                  for (int u = 0; u < 2; ++u) {
                    in[u] = t0 + u < nl_mine && w >= lvl_first && w < lvl_end ? L.bm_lvl[(t0 + u) * nwords + w] : 0ull;
                    n += static_cast<uint32_t>(__popcll(in[u])) << (16 * u);
                  }
                  const uint32_t upto = wave_incl_scan(n), rank = before[t0 / 2] + upto - n;
                  before[t0 / 2] += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(upto), 63));
#pragma unroll
                  for (int u = 0; u < 2; ++u) {
                    if (t0 + u < nl_mine) {   // wave-uniform
                      const uint32_t r_u = u ? rank >> 16 : rank & 0xFFFFu;
                      if (w < nwords) L.pre_lvl[(t0 + u) * nwords + w] = static_cast<uint16_t>(r_u);   // (the same from every wave that serves)
                      got |= first_members(in[u], take_r[t0 + u] - static_cast<int>(r_u));
                    }
                  }
                }
              }
              // the servers' places among all; those of this wave are queued: a word with many by a lane per server, of the others
              // every lane queues one server at a time
              const int c = __popcll(got);
              const uint32_t upto = wave_incl_scan(static_cast<uint32_t>(c));
              const int at = n_all + static_cast<int>(upto) - c - lo;
              n_all += __builtin_amdgcn_readlane(static_cast<int>(upto), 63);
              const bool here = c > 0 && at < 64 && at + c > 0;
              uint64_t left = here && c <= 6 ? got : 0ull;
              for (uint64_t many = __ballot(here && c > 6); many; many &= many - 1ull) {
                const int src = __ffsll(static_cast<long long>(many)) - 1;
                const uint64_t g_w = readlane64(got, src), a_w = readlane64(adm, src);
                const int to = __builtin_amdgcn_readlane(at, src) + rank_in(g_w);
                if (lane_in(g_w) && to >= 0 && to < 64)
                  ev_g[to] = static_cast<uint16_t>(((w0 + src) << 6) + lane + (lane_in(a_w) ? 0x8000 : 0));
              }
              for (int to = at; __ballot(left != 0); ++to) {
                if (left) {
                  const int b = __ffsll(static_cast<long long>(left)) - 1;
                  if (to >= 0 && to < 64) ev_g[to] = static_cast<uint16_t>((w << 6) + b + ((adm >> b) & 1ull ? 0x8000 : 0));
                  left &= left - 1ull;
                }
              }
            }
            if (n_all > lo) serve(n_all - lo < 64 ? n_all - lo : 64);
            lo += n_serve_kind << 6;
          } while (lo < n_all);
          if constexpr (kServeFirst) own_priority();
        }
        if (draws_here) {
          next_thresholds();
          drawn = true;
        }
        if (placed > 0) {
          if constexpr (WS) {   // what the pass took from the solo group's buffer, per class
            if (tid >= NT - 64 && lane < K) L.cs[CS_QDS + lane] -= L.sel_n[lane];
          }
          // (by atomics: where steps overlap other waves may be at the next step's events already, which change the same histograms.
          // Nobody reads them before the barriers that follow.)
          if (wave == route_first && lane == 0) {
#pragma unroll
            for (int gi = 0; gi < 2; ++gi) {
              if (nG[gi] > 0) {
                uint32_t *h = &L.lh[gi * kLoadBins + lminG[gi]];
                const int32_t *cnt = &L.sc[SC_CNT_T + (gi == 0 ? 0 : nG[0])];
                for (int t = 0; t < nG[gi]; ++t)   // the last level keeps the servers that got no job in it
                  atomicAdd(&h[t], static_cast<uint32_t>((t + 1 < nG[gi] ? 0 : csumG[gi] - tlastG[gi]) - cnt[t]));
                atomicAdd(&h[nG[gi]], static_cast<uint32_t>(tlastG[gi]));
              }
            }
          }
          jrem -= placed;
          next += placed;
          if constexpr (RR) {
            jremL[0] -= placed_solo; nextL[0] += placed_solo;
            jremL[1] -= placed - placed_solo; nextL[1] += placed - placed_solo;
          }
        }
        route_on = levels & 0x10000;
        gate_on = gate_more;
        if (nadm > 0) { slots_given = nadm; slots_taken = true; }
        // Where the step ends here, every wave goes on by itself, as long as the servers that are given work are known to the others.
        const bool apart_next = kOverlap && work > 0 && n_serve < nwaves && !gate_on && !route_on;
        if (gate_on || route_on || (work > 0 && !apart_next)) __syncthreads();   // (the same for every thread)
        if (!apart_next) late = 0;
        scan_first = wave - drain_first; scan_stride = n_drain; scan_end = nwords;
        if constexpr (kOverlap) {
          if (apart_next) {
            GNR_OVERLAPPING_SCAN(kBeside, static_cast<int>((static_cast<float>(npairs + share) - 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(share))))
          }
          if (wave < drain_first) scan_first = nwords;
          // (no wave has more than kPairsARound pairs: a_round_is_enough)
          const int pair_here = scan_first + (lane >> 1) * scan_stride, w = pair_here < scan_end ? 2 * pair_here + (lane & 1) : nwords;
          uint64_t others = 0;
          if (apart_next) {
            if (scan_first < nwords) {
              if (nadm > 0) {   // the first nadm idle slots
                uint64_t slots = 0;
                int left = 0;
                if (w < nwords_m) {
                  slots = L.bm_idle[w] & bits_below(w, M);
                  left = nadm - static_cast<int>(L.pre[w]);
                }
                others = first_members(slots, left);
              }
              // of each group all members of the levels below its last one, and the first take_r of the last one
  #pragma unroll
              for (int gi = 0; gi < 2; ++gi) {
                const int t_first = gi == 0 ? 0 : nl_solo, t_last = (gi == 0 ? nl_solo : nl_here) - 1;
                const int w_begin = gi == 0 ? M >> 6 : 0, w_end = gi == 0 ? nwords : (M + 63) >> 6;
                if (t_last >= t_first) {   // wave-uniform
                  const uint64_t *lvl = L.bm_lvl + t_last * nwords;
                  const int take = word_of(SC_TAKE_T + t_last);
                  int members = 0;
                  for (int t = t_first; t <= t_last; ++t) members += word_of(SC_CNT_T + t);
                  int cut_word = nwords;    // the word that has the last of the first `take`
                  uint64_t cut_set = 0;     // those of them in that word
                  if (take < members) {
                    int before = 0;
                    for (int w0 = w_begin; w0 < w_end; w0 += 64) {   // wave-uniform
                      const uint64_t in = w0 + lane < w_end ? lvl[w0 + lane] : 0ull;
                      const int c = __popcll(in), upto = before + static_cast<int>(wave_incl_scan(static_cast<uint32_t>(c)));
                      const uint64_t here = __ballot(upto >= take);
                      if (here) {
                        const int src = __ffsll(static_cast<long long>(here)) - 1;
                        const uint64_t set = readlane64(in, src);
                        const int n = take - (__builtin_amdgcn_readlane(upto, src) - __popcll(set));
                        cut_word = w0 + src;
                        cut_set = __ballot(lane_in(set) && rank_in(set) < n);
                        break;
                      }
                      before = __builtin_amdgcn_readlane(upto, 63);
                    }
                  }
                  if (w >= w_begin && w < w_end) {
                    others |= w < cut_word ? lvl[w] : w == cut_word ? cut_set : 0ull;
                    if (t_last > t_first) others |= lvl[w - nwords];
                  }
                }
              }
            }
          }
          if (lane < 2 * kPairsARound && w < nwords) L.bm_others[w] = others;
        }
      }
      if constexpr (AB) {
        if (tid == 0) {   // the head moves past everything the routing passes walked over
          const uint32_t past = static_cast<uint32_t>(L.sc[SC_DSCAN]);
          L.sc[SC_DSCAN] = 0;
          uint32_t h = dhead0 + past;
          if (h >= dbuf_cap) h -= dbuf_cap;
          L.cs[CS_DHEAD] = static_cast<int32_t>(h);
          L.cs[CS_DCOUNT] -= RR ? nextL[0] : next;
          L.sc[SC_DLEN] = static_cast<int32_t>(dlen_all - past);
          if constexpr (RR) {
            const uint32_t past_m = static_cast<uint32_t>(L.sc[SC_DSCAN_M]);
            L.sc[SC_DSCAN_M] = 0;
            h = dheadL[1] + past_m;
            if (h >= dbuf_cap) h -= dbuf_cap;
            L.cs[CS_DHEAD_M] = static_cast<int32_t>(h);
            L.cs[CS_DCOUNT_M] -= nextL[1];
            L.sc[SC_DLEN_M] = static_cast<int32_t>(dlen_all_m - past_m);
          }
          L.sc[SC_COMPACT] = 0;
        }
      } else if constexpr (RR) {
        if (tid == 0 && next > 0) {
          uint32_t h = dheadL[0] + static_cast<uint32_t>(nextL[0]);
          if (h >= dbuf_cap) h -= dbuf_cap;
          L.cs[CS_DHEAD] = static_cast<int32_t>(h);
          L.cs[CS_DCOUNT] -= nextL[0];
          h = dheadL[1] + static_cast<uint32_t>(nextL[1]);
          if (h >= dbuf_cap) h -= dbuf_cap;
          L.cs[CS_DHEAD_M] = static_cast<int32_t>(h);
          L.cs[CS_DCOUNT_M] -= nextL[1];
        }
      } else {
      if (tid == 0 && next > 0) {
        uint32_t h = dhead0 + static_cast<uint32_t>(next);
        if (h >= dbuf_cap) h -= dbuf_cap;
        L.cs[CS_DHEAD] = static_cast<int32_t>(h);
        L.cs[CS_DCOUNT] -= next;
      }
      }
    }
  }
  __syncthreads();
  // the sums over steps get the last step's counters (those of the others are in them)
  if (tid < K) add_step_sums(tid, ended, L.cs[CS_QP + tid], L.cs[CS_QD + tid], L.cs[CS_X + tid], L.cs[CS_YM + tid], L.cs[CS_YS + tid]);
  if (tid == 0) L.tl[kMaxK * kNTally + SIM_G_STEPS] += n_steps;
  if (tid < 8) L.acc[tid] = 0;   // prompt tokens already processed of the prefills in service
  if constexpr (AB) {   // the rings leave the launch without dead entries
    const uint32_t s_last = step_begin + n_steps - 1u;
    for (int k = wave; k < K; k += nwaves) compact_queue(k, s_last, 0u);
    if (wave == nwaves - 1) compact_buffer(s_last, false);
    if constexpr (RR) {
      if (wave == (nwaves > 1 ? nwaves - 2 : 0)) compact_buffer(s_last, true);
    }
  }
  // decodes that switched from mixed to solo: those that became mixed, less those that still are or ended mixed
  if (tid < K) {
    const uint64_t *t = L.tl + tid * kNTally;
    const int64_t more = static_cast<int64_t>(L.cs[CS_YM + tid]) - a.cstate[static_cast<size_t>(r) * CS_WORDS + CS_YM + tid];
    L.tl[tid * kNTally + SIM_T_M_MS] = t[SIM_T_U_DM] + t[SIM_T_M_SM] - t[SIM_T_S_DM] - static_cast<uint64_t>(more);
  }
  uint64_t *gt = a.tally + static_cast<size_t>(r) * kTallyWords;
  const uint64_t prompt_before = tid < K ? gt[tid * kNTally + SIM_T_TOKP_PRE] : 0ull;
  __syncthreads();

  // ---- tally what each server has completed since its last event; its clock and prefill as of now (a block's records are
  //      asked for a round ahead)
  struct Kept { uint64_t nc, nj, pf; uint32_t it; };
  auto kept = [&](int g) __attribute__((always_inline)) -> Kept {
    Kept v = {0, 0, 0, 0};
    if (g < N) { v.nc = rec[g].n_cls; v.nj = rec[g].n_join; v.pf = rec[g].pf_job; v.it = rec[g].iter; }
    return v;
  };
  Kept ahead_rec = kept((wave << 6) + lane);
  for (int blk = wave; blk < nwords; blk += nwaves) {
    const int g = (blk << 6) + lane;
    const uint64_t bit = 1ull << lane;
    const bool busy = L.bm_busy[blk] & bit;
    const Kept sr = ahead_rec;
    ahead_rec = kept(g + NT);
    uint32_t m = 0, d = 0, tr = kIdleRel;
    bool chunk = false;
    uint64_t comp = 0;
    int rem = g < Mp ? static_cast<int>(L.rem[g]) : 0, ptok = 0;
    if (busy) {
      comp = sr.nc - sr.nj;
      chunk = L.ev_it[g] & kEvChunk;
      ptok = chunk ? chunk_of(rem) : 0;
      const uint32_t dur = iteration_ns(ptok, byte_sum(comp));
      const int64_t rel = event_time(g, T);
      const uint32_t left = joins_next(sr.nj, rem, chunk) ? 1u : iterations_left(static_cast<uint64_t>(rel), dur);
      const uint32_t it = (L.ev_it[g] & kEvIter) - left;
      m = it - sr.it;
      d = dur;
      tr = static_cast<uint32_t>(rel - static_cast<int64_t>(static_cast<uint64_t>(left - 1u) * dur));
      if (m) rec[g].iter = it;
      if (ptok > 0) rem -= static_cast<int>(m) * ptok;
    }
    if (g < N) t_rel[g] = tr;
    if (g < Mp) {   // prompt tokens left, those of the running chunk
      uint32_t pk = 0;
      if (rem) {
        const uint32_t Pl = (static_cast<uint32_t>(sr.pf >> 32) & 0xFFFFu) + 1, k = static_cast<uint32_t>(sr.pf >> 29) & 7u;
        atomicAdd(&L.acc[k], Pl - static_cast<uint32_t>(rem));
        pk = static_cast<uint32_t>(rem) | (static_cast<uint32_t>(chunk ? chunk_of(rem) : 0) << 16) | (k << 29);
      }
      remptok[g] = pk;
    }
    tally_iterations<kTallyRowsHere>(L.ta, L.tbth, tbt_w, tbt_lo, K, m, d, chunk, comp);
  }
  __syncthreads();

  // ---- the sums of the executed iterations, folded; the time-between-tokens counts of this launch, whose total is the
  //      emitted-token tally. What is added to the totals in memory is added by atomics: nothing waits for an old value.
  if (tid < TA_TBT + K) {
    uint64_t tot = 0;
#pragma unroll
    for (int i = 0; i < kTallyRowsHere; ++i) tot += L.ta[tid * kTallyRowsHere + i];
    constexpr int kGlob = kMaxK * kNTally;
    L.tl[tid >= TA_TBT ? (tid - TA_TBT) * kNTally + SIM_T_TBT_SUM
                       : kGlob + (tid == TA_ITERS ? SIM_G_ITERS_SOLO : tid == TA_ITERS + 1 ? SIM_G_ITERS_MIX :
                                  tid == TA_BUSY ? SIM_G_BUSY_SOLO : SIM_G_BUSY_MIX)] = tot;
  }
  for (int i = tid; i < K * tbt_w; i += NT) {
    const int k = i / tbt_w, b = i - k * tbt_w;
    const uint32_t n = static_cast<uint32_t>(L.tbth[(k >> 1) * tbt_w + b] >> (32 * (k & 1)));
    if (n) {
      atomicAdd(reinterpret_cast<unsigned long long *>(&hist[(2 * K + k) * kNBin + tbt_lo + b]), static_cast<unsigned long long>(n));
      lds_add64(&L.tl[k * kNTally + SIM_T_TOK_EMIT], n);
    }
  }
  for (int i = tid; i < CS_WORDS; i += NT) a.cstate[static_cast<size_t>(r) * CS_WORDS + i] = L.cs[i];
  __syncthreads();

  for (int i = tid; i < kTallyWords; i += NT) {
    const uint64_t v = L.tl[i];
    if (v) {
      if (i == kMaxK * kNTally + SIM_G_OVERFLOW) atomicOr(reinterpret_cast<unsigned long long *>(&gt[i]), static_cast<unsigned long long>(v));
      else atomicAdd(reinterpret_cast<unsigned long long *>(&gt[i]), static_cast<unsigned long long>(v));
    }
  }
  // prompt tokens processed so far = prompt tokens of completed prefills + progress of those in service
  if (tid < K) gt[tid * kNTally + SIM_T_TOK_PREF] = prompt_before + L.tl[tid * kNTally + SIM_T_TOKP_PRE] + L.acc[tid];
}

// The step kernel of one policy variant: `form` is 0 to 3 for workgroups of 64, 128, 256 and 512 threads, in their roomy or
// dense form (see waves_per_simd), 4 and 5 for those of 1024, 6 for those of 512 some of whose waves draw (see step_form; with
// two buffers the same as 3, with same-slot decode 3 is the same as 6). Every workgroup size is compiled by itself, so that the count of waves and what follows from it are constants and not values kept in lanes of vector registers: compiled for
// two sizes each, with the count read at run time, the timed cases took 1 to 7 % longer (8 servers x 16 replications 16.7
// instead of 15.7 ms per 10^4 steps, 256 x 1024 9.15 instead of 8.61 per 1000, 1024 x 2048 17.85 instead of 17.20, 3001 x 77 5.80
// instead of 5.58 per 500). Each variant is compiled in a translation unit of its own.
using StepKernel = void (*)(const Params *, StepArrays, uint32_t, uint32_t, uint32_t, uint32_t);
#define GNR_STEP_VARIANT(name, AB, RR, IM, WS)                                                             \
  StepKernel name(int form, bool dense)                                                                    \
  {                                                                                                        \
    static const StepKernel roomy[7] = {gnr_step_kernel<64, 0, AB, RR, IM, WS>,                            \
                                        gnr_step_kernel<128, 0, AB, RR, IM, WS>,                           \
                                        gnr_step_kernel<256, 0, AB, RR, IM, WS>,                           \
                                        gnr_step_kernel<512, 0, AB, RR, IM, WS>,                           \
                                        gnr_step_kernel<1024, static_words(2), AB, RR, IM, WS>,            \
                                        gnr_step_kernel<1024, static_words(3), AB, RR, IM, WS>,            \
                                        gnr_step_kernel<512, 0, AB, RR, IM, WS, false, !(RR)>};            \
    static const StepKernel full[7] = {gnr_step_kernel<64, 0, AB, RR, IM, WS, true>,                       \
                                       gnr_step_kernel<128, 0, AB, RR, IM, WS, true>,                      \
                                       gnr_step_kernel<256, 0, AB, RR, IM, WS, true>,                      \
                                       gnr_step_kernel<512, 0, AB, RR, IM, WS, true>,                      \
                                       nullptr, nullptr,   /* (sixteen waves are dense as they are) */     \
                                       gnr_step_kernel<512, 0, AB, RR, IM, WS, true, !(RR)>};              \
    return dense && full[form] ? full[form] : roomy[form];                                                 \
  }

}  // namespace gnr
#endif

