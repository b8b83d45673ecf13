// grid.hip -- the whole minimization of one instance by a grid of co-resident
// workgroups, with no host decision between rounds.
//
// An instance too large for one workgroup's LDS and too small to fill the GPU
// spends its time between kernels: a host-planned round is about eight
// launches and one readback, ~60 us whatever the size.  Here one launch of up
// to one workgroup per CU keeps every workgroup resident, each thread owns
// the same ITEMS states from beginning to end, and grid barriers separate the
// steps.  A round (Section 3.3, Algorithm 4) is two steps:
//   group    gather the signature (own block, successor blocks), group equal
//            hashes of the workgroup's states in LDS, one insert per local
//            group into a global table of 64-bit slots;
//   resolve  every state reads its slot: the group's least member is the new
//            block id, confirmed by comparing the full signature with that
//            member's (the old ids are still there: ids are double-buffered),
//            so grouping is exact; a mismatch redoes the round with a new salt.
// The rounds are those of the round engine and of the fused kernel, so
// partitions, round counts and closure levels agree: plain rounds over the
// non-identity letters, doubling rounds for AUTO instances with one such
// letter (each level, Section 3.4, Algorithm 5, is squared in the round
// before the one that reads it), and rounds over a given list of rows (closure
// ON, or AUTO's closure letters after auto_rounds rounds: the kernel then ends
// with kFusedHandOff and a second launch goes on from its partition).
//
// What bounds it: latency.  A step is a chain of three or four dependent
// accesses (about 1 us each through the coherent part of the memory system)
// and a grid barrier (measured: 1.2 us for 16 workgroups, 1.5 us for 32, 2.2
// for 64 on one counter; above 32 arrivals go through eight counters, since a
// single one costs 28 ns per workgroup).  Per call, against the host-planned
// rounds (the one-workgroup kernel up to 16,384 states): Fib_20 (17,711
// states, 15 rounds) 932 -> 184 us; a permuted chain of 300,007 states (19
// rounds) 1,240 -> 400 us; random, n = 16,384, two letters, 140 -> 81 us; the
// 2^20-state bit-splitter 5.14 -> 1.60 ms, much of it reading rows and
// records (with records of four bytes an id 1.95).
#include "../../include/dfamin.h"
#include "internal.h"

#include <type_traits>

namespace dfamin {

namespace {

constexpr int kT = (int)kGridThreads;
constexpr uint32_t kWavesT = kGridThreads / 64;
constexpr uint32_t kSingleBit = 0x80000000u; // blk[]: a block of one state, which can never split
constexpr uint32_t kIdBits = 0x7fffffffu;
constexpr uint32_t kNoSlot = 0xffffffffu;
// barrier word: arrivals, collisions reported, payload sum
constexpr int kArriveShift = 48, kCollShift = 36;
constexpr unsigned long long kSumMask = (1ull << kCollShift) - 1ull;
constexpr unsigned long long kSpinTicks = 2000000ull;  // 20 ms of the 100 MHz clock

__device__ __forceinline__ uint64_t mix(uint64_t h, uint32_t w) {
  h ^= w;
  h *= 0x9E3779B97F4A7C15ull;
  return h ^ (h >> 29);
}
__device__ __forceinline__ uint64_t mix_end(uint64_t h) {
  h ^= h >> 32;
  h *= 0xD6E8FEB86659FD93ull;
  return h ^ (h >> 32);
}
__device__ __forceinline__ uint32_t sum64(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ uint32_t or64(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o, 64);
  return v;
}

template <typename T>
__device__ __forceinline__ T load_agent(T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Grid barrier that also sums a payload over the workgroups.  Four words
// rotate; workgroup 0 resets the one used two barriers ago, which no
// workgroup can still be reading.  Returns false (for the whole workgroup)
// when a wait ran out -- some workgroup is not resident, or its step took
// longer than 20 ms -- or another workgroup gave up: the caller leaves at once
// and the host takes another path.  What was written before the barrier is
// visible after it.
struct GridSync {
  GridBar* bar;
  uint32_t G, wg, gen;
  unsigned long long* s_val;  // LDS: [0] the sum, [1] 1 if the barrier was passed

  __device__ bool wait(unsigned long long payload, unsigned long long& sum) {
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      const uint32_t b = gen & 3u;
      const unsigned long long mine = (1ull << kArriveShift) | payload;
      if (G <= 32) {
        __hip_atomic_fetch_add(&bar->root[b].v, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        const uint32_t g = wg & 7u, members = (G - g + 7u) / 8u;
        const unsigned long long all =
            __hip_atomic_fetch_add(&bar->leaf[g][b].v, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
        if ((uint32_t)(all >> kArriveShift) == members)
          __hip_atomic_fetch_add(&bar->root[b].v, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      unsigned long long v;
      bool ok = true;
      unsigned long long t0 = 0;
      for (uint32_t spins = 0;; ++spins) {
        v = load_agent(&bar->root[b].v);
        if ((uint32_t)(v >> kArriveShift) == G) break;
        if ((spins & 15u) == 15u) {
          const unsigned long long t = wall_clock64();
          if (!t0) t0 = t;
          if (load_agent(&bar->abort) || t - t0 > kSpinTicks) {
            store_agent(&bar->abort, 1u);
            ok = false;
            break;
          }
        }
        __builtin_amdgcn_s_sleep(1);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (wg == 0) {
        const uint32_t r = (b + 2u) & 3u;
        store_agent(&bar->root[r].v, 0ull);
        if (G > 32)
          for (uint32_t g = 0; g < 8; ++g) store_agent(&bar->leaf[g][r].v, 0ull);
      }
      s_val[0] = v & ((1ull << kArriveShift) - 1ull);
      s_val[1] = ok ? 1ull : 0ull;
    }
    ++gen;
    __syncthreads();
    sum = s_val[0];
    return s_val[1] != 0;
  }

  // Every workgroup's last act: the last one leaves the words as the next
  // launch expects them (all zero), also after an abort.
  __device__ void leave() {
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      const uint32_t old = __hip_atomic_fetch_add(&bar->exits, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old + 1u == G) {
        for (uint32_t b = 0; b < 4; ++b) {
          store_agent(&bar->root[b].v, 0ull);
          for (uint32_t g = 0; g < 8; ++g) store_agent(&bar->leaf[g][b].v, 0ull);
        }
        store_agent(&bar->abort, 0u);
        store_agent(&bar->exits, 0u);
      }
    }
  }
};

// Slot: [hash fragment:32 | least member:31 | shared:1], 0 = empty.  A new
// group costs one CAS; a joiner lowers the member with one atomicMin or sets
// the shared bit with one atomicOr, so a hot slot never loops on a CAS.
//
// A group's slots are tried in one order: the kBucket slots of its home
// bucket from its home slot on, cyclically, then the next bucket.  A slot's
// fragment never changes once set, so a slot read as occupied by another
// fragment can be passed over for good, while one read as empty is settled by
// the CAS.  After a first miss the rest of the bucket is read at once: the
// slowest of a thousand threads then waits for two or three accesses, where
// probing slot by slot it walked the longest cluster of the table (a 16,384
// state round: 13.9 us of probing became 6).
constexpr uint32_t kBucketSlots = 8;
__device__ __forceinline__ uint32_t grid_insert(unsigned long long* table, uint32_t S, uint64_t h, uint32_t g,
                                                bool multi, bool read_first, uint32_t* fault) {
  const uint32_t hi = (uint32_t)(h >> 32), frag = hi ? hi : 1u;
  const uint32_t home = (uint32_t)(((h & 0xffffffffull) * S) >> 32);
  uint32_t bk = home & ~(kBucketSlots - 1u), at = home & (kBucketSlots - 1u);
  const unsigned long long mine =
      ((unsigned long long)frag << 32) | ((unsigned long long)g << 1) | (multi ? 1ull : 0ull);
  auto join = [&](uint32_t p, unsigned long long cur) {
    const uint32_t cg = (uint32_t)(cur >> 1) & kIdBits;
    if (g < cg) atomicMin(&table[p], mine | 1ull);
    else if (!(cur & 1ull)) atomicOr(&table[p], 1ull);
    return p;
  };
  {
    unsigned long long cur = read_first ? load_agent(&table[home]) : 0ull;
    if (cur == 0ull) cur = atomicCAS(&table[home], 0ull, mine);
    if (cur == 0ull) return home;
    if ((uint32_t)(cur >> 32) == frag) return join(home, cur);
  }
  uint32_t done = 1u << at;  // slots of the bucket known to hold other groups
  for (uint32_t buckets = 0; buckets <= S / kBucketSlots; ++buckets) {
    unsigned long long c[kBucketSlots];
#pragma unroll
    for (uint32_t i = 0; i < kBucketSlots; ++i) c[i] = load_agent(&table[bk + i]);
    uint32_t match = 0, empty = 0;
#pragma unroll
    for (uint32_t i = 0; i < kBucketSlots; ++i) {
      if (c[i] == 0ull) empty |= 1u << i;
      else if ((uint32_t)(c[i] >> 32) == frag) match |= 1u << i;
    }
    match &= ~done;
    empty &= ~done;
    if (match) {  // (one at most: a group has one slot)
      const uint32_t i = (uint32_t)__ffs(match) - 1u;
      return join(bk + i, load_agent(&table[bk + i]));
    }
    while (empty) {
      // the first empty slot from the home slot on
      const uint32_t rot = (empty >> at) | (empty << (kBucketSlots - at));
      const uint32_t i = (at + (uint32_t)__ffs(rot & ((1u << kBucketSlots) - 1u)) - 1u) & (kBucketSlots - 1u);
      const unsigned long long cur = atomicCAS(&table[bk + i], 0ull, mine);
      if (cur == 0ull) return bk + i;
      if ((uint32_t)(cur >> 32) == frag) return join(bk + i, cur);
      empty &= ~(1u << i);
    }
    bk = bk + kBucketSlots >= S ? 0u : bk + kBucketSlots;
    at = 0;
    done = 0;
  }
  *fault = 1u;  // cannot happen: the table has more slots than states
  return 0u;
}

// A row or id array at a workgroup-uniform address, indexed by 32-bit byte
// offsets (n <= 2^21 entries): one scalar base and one offset register per
// load, where 64-bit addresses per lane cost two.
__device__ __forceinline__ const uint32_t* uniform_ptr(unsigned long long a) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return reinterpret_cast<const uint32_t*>(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ uint32_t at32(const uint32_t* p, uint32_t i) {
  return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(p) + (i << 2));
}
__device__ __forceinline__ uint2 at64(const uint2* p, uint32_t i) {
  return *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(p) + (i << 3));
}

// Three block ids (below 2^21, see grid_shape) in a record of 8 bytes.
__device__ __forceinline__ uint2 pack3(uint32_t a, uint32_t b, uint32_t c) {
  return make_uint2(a | b << 21, b >> 11 | c << 10);
}

// ITEMS states per thread.  A workgroup owns the kT*ITEMS states from
// base on, item e of thread t being base + e*kT + t, so workgroup order is
// state order (the numbering at the end is a prefix over workgroups).  A
// state's own id, and its successors under up to CH letters (or its successor
// at the current doubling level), stay in registers from round to round: a
// group step then starts with the gathers.
template <int ITEMS>
__global__ __launch_bounds__(kT) void k_grid(GridJob J) {
  constexpr int CH = 8 / ITEMS;                           // letters kept in registers
  // Letters per chunk of longer signatures: one record's.  (Longer chunks for
  // fewer states per thread, 9 at one and 6 at two, load more past the last
  // letter and hold more registers: 2^19 states, 18 letters, 1.04 against 0.83
  // ms, 32,768 states and 14 letters 0.35 against 0.32.)
  constexpr int CL = 3;
  constexpr uint32_t kLds = 2u * ITEMS * kT;  // slots for grouping the workgroup's states
  __shared__ unsigned long long lkey[kLds];
  __shared__ uint32_t lmin[kLds], lval[kLds];  // least state; member count, then the slot
  __shared__ unsigned long long s_val[2], s_rows[kFusedMaxLetters];
  __shared__ uint32_t s_w[kWavesT * ITEMS + 1], s_or[2], s_cnt, s_coll, s_fault;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t n = J.n, wg = blockIdx.x, G = gridDim.x, S = J.S;
  const uint32_t base = wg * (uint32_t)(kT * ITEMS);
  const uint8_t* acc = reinterpret_cast<const uint8_t*>(J.accept);
  auto state = [&](int e) { return base + (uint32_t)(e * kT) + tid; };
  GridSync sync{J.bar, G, wg, 0u, s_val};
  unsigned long long sum = 0;
  if (tid == 0) {
    s_or[0] = s_or[1] = 0;
    s_cnt = s_coll = s_fault = 0;
  }
  __syncthreads();

  // ---- tables cleared; validation (every entry < n), identity letters,
  // accept bits as the first block names ({F, Q\F}, Section 3.2)
  {
    uint4* t4 = reinterpret_cast<uint4*>(J.table[0]);  // both tables, one after the other
    for (uint64_t i = (uint64_t)wg * kT + tid; i < (uint64_t)S; i += (uint64_t)G * kT) t4[i] = make_uint4(0, 0, 0, 0);
  }
  uint32_t cur = J.cur0, count = J.count0, rounds = J.rounds0, refine = J.refine0;
  uint32_t mask = 0;
  uint32_t own[ITEMS];  // block id | kSingleBit
  if (!J.resume) {
    uint32_t nonid = 0, any = 0;  // any: bit 0 some rejecting state, bit 1 some accepting, bit 2 a bad entry
    if (!J.rows)
      for (uint32_t a0 = 0; a0 < J.k; a0 += CH) {
        uint32_t v[CH][ITEMS];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const uint32_t* rp = reinterpret_cast<const uint32_t*>(J.delta) + (size_t)min(a0 + c, J.k - 1u) * n;
#pragma unroll
          for (int e = 0; e < ITEMS; ++e) v[c][e] = state(e) < n ? at32(rp, state(e)) : state(e);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
          for (int e = 0; e < ITEMS; ++e) {
            if (state(e) < n && v[c][e] >= n) any |= 4u;
            if (v[c][e] != state(e)) nonid |= 1u << min(a0 + c, J.k - 1u);
          }
      }
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
      const uint32_t q = state(e);
      own[e] = kSingleBit;
      if (q >= n) continue;
      own[e] = (acc[q >> 3] >> (q & 7u)) & 1u;
      J.blk[0][q] = own[e];
      any |= 1u << own[e];
    }
    nonid = or64(nonid);
    any = or64(any);
    if (lane == 0) {
      if (nonid) atomicOr(&s_or[0], nonid);
      if (any) atomicOr(&s_or[1], any);
    }
    __syncthreads();
    if (tid == 0) {
      J.wgw[2 * wg] = s_or[0];
      J.wgw[2 * wg + 1] = s_or[1];
    }
  } else {
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) own[e] = state(e) < n ? J.blk[cur][state(e)] : kSingleBit;
  }
  int32_t status = sync.wait(0, sum) ? kFusedOk : kGridAborted;
  if (!J.resume && status == kFusedOk) {
    uint32_t w0 = 0, w1 = 0;
    for (uint32_t i = tid; i < G; i += kT) {
      w0 |= load_agent(&J.wgw[2 * i]);
      w1 |= load_agent(&J.wgw[2 * i + 1]);
    }
    w0 = or64(w0);
    w1 = or64(w1);
    if (lane == 0) {
      if (w0) atomicOr(&s_or[0], w0);
      if (w1) atomicOr(&s_or[1], w1);
    }
    __syncthreads();
    mask = s_or[0];
    if (s_or[1] & 4u) status = kFusedBad;
    count = (uint32_t)__popc(s_or[1] & 3u);
  }
  const bool list = J.rows != nullptr;
  const uint32_t knon = list ? J.nrows : (uint32_t)__popc(mask);
  const bool autom = J.closure == DFAMIN_CLOSURE_AUTO;
  const bool dbl = !list && autom && knon == 1;
  if (!list && tid < 32u && ((mask >> tid) & 1u))
    s_rows[__popc(mask & ((1u << tid) - 1u))] = (unsigned long long)(J.delta + 4ull * tid * n);
  if (dbl && J.no_doubling && status == kFusedOk) status = kFusedHandOff;
  __syncthreads();
  const uint64_t* lrows = J.rows;
  auto row = [&](uint32_t t) { return uniform_ptr(list ? (unsigned long long)lrows[t] : s_rows[t]); };

  uint32_t l = 0, used = 0;  // doubling: the level of this round, the highest a splitting round read
  uint64_t jlen = 0;         // the partition is P_jlen
  uint32_t tsel = 0, retries = 0;
  uint64_t salt = J.salt;
  uint32_t slot[ITEMS], clr[ITEMS];  // this round's slot; the slot of the last round this thread has to clear
#pragma unroll
  for (int e = 0; e < ITEMS; ++e) clr[e] = kNoSlot;

  // LDS grouping and the table inserts, from the hashes h on.
  auto clear_lds = [&]() {
    uint4* k4 = reinterpret_cast<uint4*>(lkey);
    uint4* m4 = reinterpret_cast<uint4*>(lmin);
    uint4* v4 = reinterpret_cast<uint4*>(lval);
    for (uint32_t i = tid; i < kLds / 2; i += kT) k4[i] = make_uint4(0, 0, 0, 0);
    for (uint32_t i = tid; i < kLds / 4; i += kT) {
      m4[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
      v4[i] = make_uint4(0, 0, 0, 0);
    }
  };
  auto group = [&](uint64_t (&h)[ITEMS]) {
    unsigned long long* table = J.table[tsel];
    // few groups: most inserts join a slot that already has a lower member
    // and the shared bit, and a read then saves the atomic
    const bool read_first = (uint64_t)count * 64u < n;
    uint32_t lp[ITEMS];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
      const bool act = !(own[e] & kSingleBit);
      uint64_t hh = mix_end(h[e]);
      if (J.hash_mask) hh = mix_end(hh & J.hash_mask);
      h[e] = hh;
      // The lanes that agree with the wave's first active lane go in as one:
      // where blocks are large most of a wave does, and a thousand LDS
      // atomics on one word are what the step would wait for.
      const unsigned long long am = __ballot(act);
      const int f = am ? __builtin_ctzll(am) : 0;
      const uint32_t fl = __shfl((uint32_t)hh, f, 64), fh = __shfl((uint32_t)(hh >> 32), f, 64);
      const bool like = act && (uint32_t)hh == fl && (uint32_t)(hh >> 32) == fh;
      const unsigned long long lm = __ballot(like);
      lp[e] = 0;
      if (act && (!like || (int)lane == f)) {
        const unsigned long long lk = hh ? hh : 1ull;
        uint32_t p = (uint32_t)(hh >> 20) & (kLds - 1u);
        while (true) {
          const unsigned long long prev = atomicCAS(&lkey[p], 0ull, lk);
          if (prev == 0ull || prev == lk) break;
          p = (p + 1u) & (kLds - 1u);
        }
        atomicMin(&lmin[p], state(e));
        atomicAdd(&lval[p], like ? (uint32_t)__popcll(lm) : 1u);
        lp[e] = p;
      }
      const uint32_t fp = __shfl(lp[e], f, 64);
      if (like) lp[e] = fp;
    }
    __syncthreads();
    // one insert per local group, by its least member (the only one to read
    // the group's count, which the slot then replaces)
#pragma unroll
    for (int e = 0; e < ITEMS; ++e)
      if (!(own[e] & kSingleBit) && lmin[lp[e]] == state(e))
        lval[lp[e]] = grid_insert(table, S, h[e], state(e), lval[lp[e]] > 1u, read_first, &s_fault);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) slot[e] = (own[e] & kSingleBit) ? kNoSlot : lval[lp[e]];
  };
  // Ends the resolve step: new ids (nid) are known; counts leaders, and
  // after the barrier decides what comes next.  True: another round.
  uint32_t r[ITEMS];  // the group's least member
  bool shared[ITEMS];
  auto read_slots = [&]() {
    const unsigned long long* table = J.table[tsel];
    unsigned long long w[ITEMS];
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) w[e] = slot[e] != kNoSlot ? table[slot[e]] : 0ull;
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
      r[e] = slot[e] != kNoSlot ? (uint32_t)(w[e] >> 1) & kIdBits : state(e);
      shared[e] = (w[e] & 1ull) != 0;
    }
  };
  auto new_id = [&](int e) {
    return slot[e] == kNoSlot ? own[e] : (r[e] | (shared[e] ? 0u : kSingleBit));
  };
  auto finish = [&](uint32_t coll) {
    uint32_t leaders = 0;
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
      const bool lead = state(e) < n && r[e] == state(e);
      leaders += lead ? 1u : 0u;
      clr[e] = lead ? slot[e] : kNoSlot;
    }
    leaders = sum64(leaders);
    const bool anyc = __any(coll != 0u);
    if (lane == 0) {
      if (leaders) atomicAdd(&s_cnt, leaders);
      if (anyc) s_coll = 1u;
    }
    __syncthreads();
    const uint32_t wleaders = s_cnt;
    const unsigned long long pay = (unsigned long long)wleaders | ((unsigned long long)(s_coll | s_fault) << kCollShift);
    __syncthreads();
    if (tid == 0) {
      J.wgw[wg] = wleaders;
      s_cnt = s_coll = 0;
    }
    if (!sync.wait(pay, sum)) {
      status = kGridAborted;
      return false;
    }
    tsel ^= 1u;
    if (sum >> kCollShift) {  // two signatures shared a hash: the same round again
      if (++retries > kMaxSaltRetries) {
        status = kFusedFault;
        return false;
      }
      salt = mix_end(salt + 0x9E3779B97F4A7C15ull);
      return true;
    }
    retries = 0;
    return true;
  };
  // After a round that was not redone: false when it was the last.
  auto settle = [&](uint32_t cnew, uint64_t step) {
    ++rounds;
    cur ^= 1u;  // (when nothing split, the same blocks under their least members)
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) own[e] = new_id(e);
    if (cnew == count) return false;
    ++refine;
    used = max(used, l);
    count = cnew;
    jlen += step;
    return count != n;
  };
  auto clear_old = [&]() {
    unsigned long long* old_table = J.table[tsel ^ 1u];
#pragma unroll
    for (int e = 0; e < ITEMS; ++e)
      if (clr[e] != kNoSlot) old_table[clr[e]] = 0ull;
  };

  // Doubling, one letter: pr[] holds (block id, successor at the level the
  // next round reads) side by side, so a round gathers both the successor's
  // block and the next level's square in one access.
  auto doubling_rounds = [&]() {
    const uint32_t* row0 = row(0);
    uint32_t sx[ITEMS];  // successor at this round's level
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) sx[e] = state(e) < n ? at32(row0, state(e)) : 0u;
    bool first = true;  // ids still are accept bits in blk[0], the level is the row itself
    while (true) {
      if (rounds >= J.max_rounds) {
        status = kFusedRoundCap;
        break;
      }
      const uint2* pc = J.pr[cur];
      uint2* pn = J.pr[cur ^ 1u];
      const bool up = l < J.levels && (1ull << (l + 1)) <= jlen + (1ull << l) + 1ull;  // the next round reads l + 1
      clear_lds();
      clear_old();
      uint32_t bb[ITEMS], nx[ITEMS];
      uint64_t h[ITEMS];
      if (first) {
        const uint32_t* b0 = J.blk[0];
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
          bb[e] = at32(b0, sx[e]);
          nx[e] = at32(row0, sx[e]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
          const uint2 v = at64(pc, sx[e]);
          bb[e] = v.x & kIdBits;
          nx[e] = v.y;
        }
      }
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) {
        if (!up) nx[e] = sx[e];
        h[e] = mix(mix(salt, own[e]), bb[e]);
      }
      group(h);
      if (!sync.wait(0, sum)) {
        status = kGridAborted;
        break;
      }
      read_slots();
      uint32_t coll = 0;
      uint32_t sr[ITEMS];
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) {
        sr[e] = sx[e];
        if (r[e] == state(e) || slot[e] == kNoSlot) continue;
        const uint2 v = first ? make_uint2(at32(J.blk[0], r[e]), at32(row0, r[e])) : at64(pc, r[e]);
        coll |= (uint32_t)(v.x != own[e]);
        sr[e] = v.y;
      }
#pragma unroll
      for (int e = 0; e < ITEMS; ++e)
        if (sr[e] != sx[e]) coll |= (uint32_t)(((first ? at32(J.blk[0], sr[e]) : at64(pc, sr[e]).x) & kIdBits) != bb[e]);
#pragma unroll
      for (int e = 0; e < ITEMS; ++e)
        if (state(e) < n) pn[state(e)] = make_uint2(new_id(e), nx[e]);
      if (!finish(coll)) break;
      if (sum >> kCollShift) continue;
      first = false;
      if (!settle((uint32_t)(sum & kSumMask), 1ull << l)) break;
      if (up) ++l;
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) sx[e] = nx[e];
    }
  };
  // Several letters (or rows).  FIT: at most CH, whose successors and their
  // blocks stay in registers.
  auto multi_rounds = [&](auto fitc) {
    constexpr bool fit = decltype(fitc)::value;
    const uint32_t kp = knon;
    uint32_t sc[fit ? CH : 1][ITEMS], b[fit ? CH : 1][ITEMS];
    if constexpr (fit) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t* rp = (uint32_t)c < kp ? row((uint32_t)c) : nullptr;
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) sc[c][e] = (rp && state(e) < n) ? at32(rp, state(e)) : 0u;
      }
    }
    // longer signatures: the blocks gathered in the group step are kept for
    // the comparison in the resolve step
    uint2* rec = fit ? nullptr : J.rec;
    [[maybe_unused]] uint2* rows3 = fit ? nullptr : J.rows3;
    [[maybe_unused]] bool packed = false;  // rows3 is written
    while (true) {
      if (!list && autom && knon >= 2 && rounds == J.auto_rounds) {
        status = kFusedHandOff;  // still splitting: the host builds its closure letters
        break;
      }
      if (rounds >= J.max_rounds) {
        status = kFusedRoundCap;
        break;
      }
      const uint32_t* bc = J.blk[cur];
      uint32_t* bn = J.blk[cur ^ 1u];
      uint64_t h[ITEMS];
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) h[e] = mix(salt, own[e]);
      if constexpr (fit) {
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
          for (int e = 0; e < ITEMS; ++e)
            b[c][e] = ((uint32_t)c < kp && !(own[e] & kSingleBit)) ? at32(bc, sc[c][e]) & kIdBits : 0u;
        clear_lds();
        clear_old();
#pragma unroll
        for (int c = 0; c < CH; ++c)
          if ((uint32_t)c < kp) {
#pragma unroll
            for (int e = 0; e < ITEMS; ++e) h[e] = mix(h[e], b[c][e]);
          }
      } else {
        // chunks of CL letters; the next chunk's row entries go out before
        // this chunk's gathers.  At one state per thread they come as records,
        // too, from the second round on (rows3), as the first one wrote them:
        // a third of the loads and two thirds of the bytes.
        auto load = [&](uint32_t t0, uint32_t (&x)[CL][ITEMS], auto packedc) {
          if constexpr (decltype(packedc)::value) {
            const uint2* rp = rows3 + (size_t)(min(t0, kp - 1u) / 3u) * n;
#pragma unroll
            for (int e = 0; e < ITEMS; ++e) {
              const uint2 w = (own[e] & kSingleBit) ? make_uint2(0, 0) : at64(rp, state(e));
              x[0][e] = w.x & 0x1fffffu;
              x[1][e] = (w.x >> 21 | w.y << 11) & 0x1fffffu;
              x[2][e] = w.y >> 10;
            }
          } else {
#pragma unroll
            for (int c = 0; c < CL; ++c) {
              const uint32_t* rp = row(min(t0 + c, kp - 1u));
#pragma unroll
              for (int e = 0; e < ITEMS; ++e) x[c][e] = (own[e] & kSingleBit) ? 0u : at32(rp, state(e));
            }
          }
        };
        auto gather = [&](auto packedc) {
          uint32_t s[CL][ITEMS];
          load(0u, s, packedc);
          clear_lds();
          clear_old();
          for (uint32_t t0 = 0; t0 < kp; t0 += CL) {
            uint32_t sn[CL][ITEMS] = {}, v[CL][ITEMS];
            if (t0 + CL < kp) load(t0 + CL, sn, packedc);
#pragma unroll
            for (int c = 0; c < CL; ++c)
#pragma unroll
              for (int e = 0; e < ITEMS; ++e) v[c][e] = (own[e] & kSingleBit) ? 0u : at32(bc, s[c][e]) & kIdBits;
            if constexpr (ITEMS == 1 && !decltype(packedc)::value)
              if (rows3 && !(own[0] & kSingleBit))
                rows3[(size_t)(t0 / 3u) * n + state(0)] = pack3(s[0][0], s[1][0], s[2][0]);
#pragma unroll
            for (int c = 0; c < CL; ++c)
              if (t0 + c < kp) {
#pragma unroll
                for (int e = 0; e < ITEMS; ++e) h[e] = mix(h[e], v[c][e]);
              }
            // (letters past the last one repeat it: the same in every record)
            if (rec) {
              uint2* rp = rec + (size_t)(t0 / 3u) * n;
#pragma unroll
              for (int e = 0; e < ITEMS; ++e)
                if (!(own[e] & kSingleBit)) rp[state(e)] = pack3(v[0][e], v[1][e], v[2][e]);
            }
#pragma unroll
            for (int c = 0; c < CL; ++c)
#pragma unroll
              for (int e = 0; e < ITEMS; ++e) s[c][e] = sn[c][e];
          }
        };
        if constexpr (ITEMS == 1) {
          if (packed) gather(std::true_type{});
          else gather(std::false_type{});
          packed = rows3 != nullptr;
        } else {
          gather(std::false_type{});
        }
      }
      group(h);
      if (!sync.wait(0, sum)) {
        status = kGridAborted;
        break;
      }

      // ---- resolve
      read_slots();
      uint32_t coll = 0;
      bool chk[ITEMS];
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) {
        chk[e] = slot[e] != kNoSlot && r[e] != state(e);
        if (chk[e]) coll |= (uint32_t)(at32(bc, r[e]) != own[e]);
      }
      if constexpr (fit) {
        uint32_t o[CH][ITEMS];
#pragma unroll
        for (int c = 0; c < CH; ++c)
          if ((uint32_t)c < kp) {
            const uint32_t* rp = row((uint32_t)c);
#pragma unroll
            for (int e = 0; e < ITEMS; ++e) o[c][e] = chk[e] ? at32(rp, r[e]) : 0u;
          }
#pragma unroll
        for (int c = 0; c < CH; ++c)
          if ((uint32_t)c < kp) {
#pragma unroll
            for (int e = 0; e < ITEMS; ++e)
              if (chk[e]) coll |= (uint32_t)((at32(bc, o[c][e]) & kIdBits) != b[c][e]);
          }
      } else if (rec) {
        for (uint32_t t = 0; t < grid_records(kp); ++t) {
          const uint2* rp = rec + (size_t)t * n;
          uint2 x[ITEMS], y[ITEMS];
#pragma unroll
          for (int e = 0; e < ITEMS; ++e) {
            x[e] = chk[e] ? at64(rp, state(e)) : make_uint2(0, 0);
            y[e] = chk[e] ? at64(rp, r[e]) : make_uint2(0, 0);
          }
#pragma unroll
          for (int e = 0; e < ITEMS; ++e) coll |= (uint32_t)(x[e].x != y[e].x || x[e].y != y[e].y);
        }
      } else {  // no room for records: both signatures gathered again
        for (uint32_t t = 0; t < kp; ++t) {
          const uint32_t* rp = row(t);
#pragma unroll
          for (int e = 0; e < ITEMS; ++e)
            if (chk[e])
              coll |= (uint32_t)((at32(bc, at32(rp, r[e])) & kIdBits) != (at32(bc, at32(rp, state(e))) & kIdBits));
        }
      }
#pragma unroll
      for (int e = 0; e < ITEMS; ++e)
        if (state(e) < n) bn[state(e)] = new_id(e);
      if (!finish(coll)) break;
      if (sum >> kCollShift) continue;
      if (!settle((uint32_t)(sum & kSumMask), 1ull)) break;
    }
  };
  if (status == kFusedOk) {
    if (dbl) doubling_rounds();
    else if (knon <= (uint32_t)CH) multi_rounds(std::true_type{});
    else multi_rounds(std::false_type{});
  }

  if (status == kFusedOk) {
    // ---- canonical numbering by least member (J.rank is free by now)
    uint32_t* out = reinterpret_cast<uint32_t*>(J.out);
    if (count == n) {
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) {
        const uint32_t q = state(e);
        if (q < n) {
          out[q] = q;
          if (J.want_ids) J.blk[0][q] = q;
        }
        if (q == J.q0) J.res->initial_block = q;
      }
    } else {
      // leaders of the workgroups before this one
      uint32_t before = 0;
      for (uint32_t i = tid; i < wg; i += kT) before += load_agent(&J.wgw[i]);
      before = sum64(before);
      if (lane == 0 && before) atomicAdd(&s_cnt, before);
      unsigned long long m[ITEMS];
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) {
        m[e] = __ballot(state(e) < n && (own[e] & kIdBits) == state(e));
        if (lane == 0) s_w[e * kWavesT + wave] = (uint32_t)__popcll(m[e]);
      }
      __syncthreads();
      if (wave == 0) {  // exclusive offsets of the wave counts, in state order
        uint32_t run = s_cnt;
        for (uint32_t c0 = 0; c0 < kWavesT * ITEMS; c0 += 64) {
          const uint32_t c = c0 + lane;
          const uint32_t x = c < kWavesT * ITEMS ? s_w[c] : 0u;
          uint32_t v = x;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(v, o, 64);
            if ((int)lane >= o) v += u;
          }
          if (c < kWavesT * ITEMS) s_w[c] = run + v - x;
          run += __shfl(v, 63, 64);
        }
      }
      __syncthreads();
      uint32_t* rank = J.rank;
#pragma unroll
      for (int e = 0; e < ITEMS; ++e)
        if ((m[e] >> lane) & 1ull)
          rank[state(e)] = s_w[e * kWavesT + wave] + (uint32_t)__popcll(m[e] & ((1ull << lane) - 1ull));
      if (!sync.wait(0, sum)) {
        status = kGridAborted;
      } else {
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
          const uint32_t q = state(e);
          if (q >= n) continue;
          const uint32_t c = at32(rank, own[e] & kIdBits);
          out[q] = c;
          if (J.want_ids) J.blk[0][q] = own[e] & kIdBits;
          if (q == J.q0) J.res->initial_block = c;
        }
      }
    }
  }
  if (tid == 0 && wg == 0) {
    J.res->num_blocks = count;
    J.res->refine_rounds = refine;
    J.res->rounds = rounds;
    J.res->levels_used = used;
    J.res->doubling = dbl ? 1u : 0u;
    J.res->letters = mask;
    J.res->cur = cur;
    J.res->status = status;
  }
  if (tid == 0 && status == kGridAborted) J.res->aborted = 1u;
  sync.leave();
}

// Breadth-first levels from a frontier, one barrier per level instead of one
// launch, readback and host decision (whole minimal-DFA calls, four letters:
// 30,000 states 740 -> 370 us, 262,144 states 1,558 -> 1,177 us), until the
// frontier is wide enough for a launch per level.  Each workgroup
// stages the states it visits first in LDS and appends them with one atomic
// per chunk of rows, as k_bfs_level does; the barrier's sum is the next
// frontier's size, so no counter is read.  Bound: the latency of a level's
// three dependent accesses (frontier, row entry, visited word) and the
// barrier while frontiers are small, random access where they are large.
constexpr uint32_t kBfsRows = 8;
__global__ __launch_bounds__(kT) void k_bfs_grid(BfsJob B) {
  __shared__ unsigned long long s_val[2];
  __shared__ uint32_t s_new[kT * kBfsRows];
  __shared__ uint32_t s_cnt, s_base;
  const uint32_t tid = threadIdx.x, wg = blockIdx.x, G = gridDim.x;
  GridSync sync{B.bar, G, wg, 0u, s_val};
  uint32_t f = B.fcount, levels = B.levels, reached = B.reached, cur = B.cur;
  bool ok = true;
  if (B.seed) {  // visited = {q0}; the one state of the first frontier is q0 itself
    for (uint64_t i = (uint64_t)wg * kT + tid; i < B.words; i += (uint64_t)G * kT)
      B.visited[i] = i == B.q0 >> 5 ? 1u << (B.q0 & 31u) : 0u;
    if (wg == 0 && tid < 2) B.counter[32u * tid] = 0u;
    if (wg == 0 && tid == 0) B.list[cur][0] = B.q0;
    unsigned long long sum = 0;
    ok = sync.wait(0, sum);
  }
  while (ok && f && f <= B.max_frontier && levels < B.max_levels) {
    const uint32_t* frontier = B.list[cur];
    uint32_t* next = B.list[cur ^ 1u];
    uint32_t* counter = B.counter + (levels & 1u) * 32u;  // zero: reset a level ago, or by the host
    uint32_t found = 0;
    for (uint64_t j0 = (uint64_t)wg * kT; j0 < f; j0 += (uint64_t)G * kT) {
      const bool valid = j0 + tid < f;
      const uint32_t q = valid ? frontier[j0 + tid] : 0u;
      for (uint32_t r0 = 0; r0 < B.nrows; r0 += kBfsRows) {
        if (tid == 0) s_cnt = 0;
        __syncthreads();
        if (valid) {
          uint32_t t[kBfsRows], v[kBfsRows];
#pragma unroll
          for (uint32_t r = 0; r < kBfsRows; ++r)
            t[r] = r0 + r < B.nrows ? reinterpret_cast<const uint32_t*>(B.rows[r0 + r])[q] : q;
#pragma unroll
          for (uint32_t r = 0; r < kBfsRows; ++r) v[r] = B.visited[t[r] >> 5];
#pragma unroll
          for (uint32_t r = 0; r < kBfsRows; ++r) {
            const uint32_t bit = 1u << (t[r] & 31u);
            // (a visited word read before is stale at worst: the atomic decides)
            if (!(v[r] & bit) && !(atomicOr(&B.visited[t[r] >> 5], bit) & bit))
              s_new[atomicAdd(&s_cnt, 1u)] = t[r];
          }
        }
        __syncthreads();
        const uint32_t cnt = s_cnt;
        if (tid == 0 && cnt) s_base = atomicAdd(counter, cnt);
        __syncthreads();
        for (uint32_t x = tid; x < cnt; x += kT) next[s_base + x] = s_new[x];
        found += cnt;
        __syncthreads();
      }
    }
    unsigned long long sum = 0;
    if (!sync.wait(found, sum)) {
      ok = false;
      break;
    }
    if (wg == 0 && tid == 0) store_agent(counter, 0u);  // next used two levels on, a barrier away
    f = (uint32_t)(sum & kSumMask);
    reached += f;
    ++levels;
    cur ^= 1u;
  }
  if (tid == 0 && wg == 0) {
    B.res->num_blocks = f;
    B.res->rounds = levels;
    B.res->refine_rounds = reached;
    B.res->cur = cur;
    B.res->status = ok ? kFusedOk : kGridAborted;
  }
  if (tid == 0 && !ok) B.res->aborted = 1u;
  sync.leave();
}

}  // namespace

// 1,024 threads and the fewest states per thread that fit the CUs: more
// workgroups with fewer states each beat fewer barrier arrivals (n = 150,000
// chain: 314 us with 147 workgroups of one state per thread, 399 with 74 of
// two), while 512 or 256 threads for small n changed nothing.  At four states
// per thread the kernel uses 64 bytes of scratch a thread; at eight many
// registers spill, whose dirty lines every barrier has to write back, and the
// gathers no longer fit the caches: random DFAs of 2^21 states took 790 us
// against the round engine's 600 (at 2^20: 332 against 415), so larger
// instances stay with the round engine.
bool grid_shape(uint32_t n, uint32_t cus, uint32_t* items, uint32_t* wgs) {
  uint32_t it = 1;
  while (it <= kGridMaxItems && (uint64_t)it * kGridThreads * cus < n) it *= 2;
  if (it > kGridMaxItems || n > 1u << 21) return false;  // (records hold 21-bit ids)
  *items = it;
  *wgs = (n + it * kGridThreads - 1) / (it * kGridThreads);
  return true;
}

void launch_grid(const GridJob& J, uint32_t items, uint32_t wgs, hipStream_t s) {
  const dim3 g(wgs), b(kT);
  switch (items) {
    case 1: hipLaunchKernelGGL(k_grid<1>, g, b, 0, s, J); break;
    case 2: hipLaunchKernelGGL(k_grid<2>, g, b, 0, s, J); break;
    default: hipLaunchKernelGGL(k_grid<4>, g, b, 0, s, J); break;
  }
}

void launch_bfs_grid(const BfsJob& B, uint32_t wgs, hipStream_t s) {
  hipLaunchKernelGGL(k_bfs_grid, dim3(wgs), dim3(kT), 0, s, B);
}

}  // namespace dfamin
