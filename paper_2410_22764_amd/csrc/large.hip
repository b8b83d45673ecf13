// large.hip -- the early rounds of one large instance (more states than the
// grid kernel takes).
//
// From P_0 the blocks of such an instance multiply: a random automaton of
// 2^24 states and four letters has 2 blocks, 32, 2^21 and then 2^24, and the
// last two rounds take nearly all of the time.  Two observations shorten
// them.
//
// The second round (k_label2).  The label of the first round is the accept
// bit of q and of its successors, so the successors' labels and q's own
// accept bit determine q's own label: the signature is an exact key of
// 1 + kp + kp * kp bits, which is itself a block label.  No grouping is needed,
// only the number of keys that occur, and that only where the next round does
// not make it needless.
//
// The round in which nearly every state becomes a block of its own
// (k_uniq_*).  A state whose hash of a part of its signature -- own block and
// the first few letters -- no other state shares is alone under the whole
// signature, whatever the hash: a shared hash only means that the state has
// to be looked at again.  So few letters are gathered, the (hash, state)
// pairs are spread over buckets of one workgroup's LDS each, and only the
// states that share a hash there (hundreds of 2^24) go through the round
// engine's kernels with their whole signatures.  A sample of blocks, taken
// as the round before ends, tells whether that will be so.
//
// Random automata, before and after: 2^24 states and four letters 3.90 ->
// 1.67 ms, 4,100,000 and four 1.02 -> 0.50, 8,388,608 and seven 2.03 -> 0.96,
// 4,000,037 and five 0.86 -> 0.55.  Automata with copied states or skewed
// classes take the ordinary rounds after the sample (10 to 60 us).
#include "internal.h"

#include <algorithm>

namespace dfamin {

namespace {

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

// Second round, K = 4 letters.  A successor's label is its accept bit, which q's
// own label holds already, and those of its successors: K bits, so the array
// gathered from has four bits per state (nib), and the key is q's own label
// and K bits per letter.  Bound: those gathers.  The workgroups keep a tile's
// successors in registers and go through the array a window (2 MiB, half an
// XCD's L2) at a time, roughly in step, the rows and labels passing by the
// caches, so that more of the gathers hit.  2^24 states, four letters: 440 us,
// 150 G gathers/s (one-byte labels gathered without windows 900, with them
// 620; the round through a count table of atomics 1,220).
constexpr int kL2Items = 8;
constexpr uint32_t kL2Window = 21;  // log2 of its bytes
__global__ __launch_bounds__(kBlock) void k_label2(const InstDesc* __restrict__ desc,
                                                   const uint64_t* __restrict__ rows,
                                                   const uint8_t* __restrict__ nib,
                                                   uint32_t* __restrict__ label) {
  constexpr int K = 4;
  const InstDesc D = desc[0];
  const uint32_t n = D.n, nwin = ((n - 1u) >> (kL2Window + 1u)) + 1u;
  const uint8_t* __restrict__ acc = reinterpret_cast<const uint8_t*>(D.accept);
  const uint64_t* __restrict__ R = rows + D.rows_off;
  for (uint64_t base = (uint64_t)blockIdx.x * (kBlock * kL2Items); base < n;
       base += (uint64_t)gridDim.x * (kBlock * kL2Items)) {
    uint32_t s[K][kL2Items], key[kL2Items];
#pragma unroll
    for (int e = 0; e < kL2Items; ++e) {
      const uint64_t q = base + e * kBlock + threadIdx.x;
#pragma unroll
      for (int t = 0; t < K; ++t)
        s[t][e] = q < n ? __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(R[t]) + q) : 0xffffffffu;
      key[e] = q < n ? ((acc[q >> 3] >> (q & 7u)) & 1u) | ((nib[q >> 1] >> ((q & 1u) * 4u)) & 15u) << 1 : 0u;
    }
    for (uint32_t w = 0; w < nwin; ++w) {
      uint32_t v[K][kL2Items];
#pragma unroll
      for (int t = 0; t < K; ++t)
#pragma unroll
        for (int e = 0; e < kL2Items; ++e)
          v[t][e] = nib[(s[t][e] >> (kL2Window + 1u)) == w ? s[t][e] >> 1 : w << kL2Window];
#pragma unroll
      for (int t = 0; t < K; ++t)
#pragma unroll
        for (int e = 0; e < kL2Items; ++e)
          if ((s[t][e] >> (kL2Window + 1u)) == w)
            key[e] |= ((v[t][e] >> ((s[t][e] & 1u) * 4u)) & 15u) << (1u + K + t * K);
    }
#pragma unroll
    for (int e = 0; e < kL2Items; ++e) {
      const uint64_t q = base + e * kBlock + threadIdx.x;
      if (q < n) __builtin_nontemporal_store(kSlotLabel | key[e], &label[q]);
    }
  }
}

// The keys that occur: a workgroup marks those of its share of the states in
// a bit map in LDS (2^20 bits: each half of the keys has workgroups of its
// own) and writes the map out; k_seen_count then merges them.  A byte per
// key in global memory, read and set by every state, took 240 us of 2^24
// states.
constexpr uint32_t kSeenWords = 1u << 15, kSeenThreads = 1024, kHalves = 2;
__global__ __launch_bounds__(kSeenThreads) void k_seen_bits(const uint32_t* __restrict__ label, uint32_t n,
                                                            uint32_t* __restrict__ maps,
                                                            uint32_t* __restrict__ part,
                                                            const Ctrl* __restrict__ ctrl, UniqTest lazy) {
  if (lazy.go(ctrl->u_count, ctrl->u_dup)) return;
  __shared__ uint32_t map[kSeenWords];
  for (uint32_t i = threadIdx.x; i < kSeenWords; i += kSeenThreads) map[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < kGroupCounters) part[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t half = blockIdx.x % kHalves, share = blockIdx.x / kHalves, shares = gridDim.x / kHalves;
  const uint64_t first = (uint64_t)n * share / shares, last = (uint64_t)n * (share + 1) / shares;
  for (uint64_t q0 = first; q0 < last; q0 += 8 * kSeenThreads) {
    uint32_t k[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint64_t q = q0 + e * kSeenThreads + threadIdx.x;
      k[e] = q < last ? label[q] & ~kSlotLabel : 0xffffffffu;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if ((k[e] >> 20) == half) {
        uint32_t* w = &map[(k[e] & 0xfffffu) >> 5];
        const uint32_t bit = 1u << (k[e] & 31u);
        if (!(*w & bit)) atomicOr(w, bit);
      }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kSeenWords; i += kSeenThreads)
    maps[(uint64_t)blockIdx.x * kSeenWords + i] = map[i];
}

// One word of the key space per thread, merged over the shares.
__global__ __launch_bounds__(kBlock) void k_seen_count(const uint32_t* __restrict__ maps, uint32_t maps_n,
                                                       uint32_t* __restrict__ part,
                                                       const Ctrl* __restrict__ ctrl, UniqTest lazy) {
  if (lazy.go(ctrl->u_count, ctrl->u_dup)) return;
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;  // (kSeenWords is a multiple of kBlock)
  uint32_t v = 0;
#pragma unroll 16
  for (uint32_t w = i / kSeenWords; w < maps_n; w += kHalves) v |= maps[(uint64_t)w * kSeenWords + (i % kSeenWords)];
  const uint32_t c = sum64((uint32_t)__popc(v));
  if ((threadIdx.x & 63u) == 0 && c) atomicAdd(&part[blockIdx.x % kGroupCounters], c);
}

// (where lazy says go, the parts have not been counted)
__global__ void k_label2_end(const uint32_t* __restrict__ part, uint32_t before, uint32_t m,
                             uint32_t* __restrict__ changed_inst, Ctrl* __restrict__ ctrl, UniqTest lazy) {
  const bool split = lazy.go(ctrl->u_count, ctrl->u_dup);
  const uint32_t formed = split ? 0u : sum64(part[threadIdx.x]);
  if (threadIdx.x) return;
  if (!split) ctrl->prev_shared = formed;
  if (!changed_inst) return;
  ctrl->any_changed = 0u;
  ctrl->collision = 0u;
  ctrl->m_next = m;
  if (split || formed > before) changed_inst[0] = 1u;
}

// Own block and first t letters of q, hashed.  SRC: 1 = one-byte numbers, 4 =
// block words.
template <int SRC>
__device__ __forceinline__ uint32_t src_at(const void* p, uint32_t i) {
  return SRC == 1 ? (uint32_t) reinterpret_cast<const uint8_t*>(p)[i] : reinterpret_cast<const uint32_t*>(p)[i];
}

// The sample: every state of some signatures, counted (u_count), its hash put
// into a table, the repeats counted (u_dup).  One-byte numbers (large blocks):
// own number 0 and the first letter's below `sel`; block words: the blocks
// whose hash has the bits of `sel` clear.
constexpr int kSampleThreads = 512, kSampleItems = 8;
constexpr uint32_t kSampleWgs = 256, kMine = kUniqSample / kSampleWgs;  // twice what a workgroup expects
template <int SRC>
__global__ __launch_bounds__(kSampleThreads) void k_uniq_sample(const InstDesc* __restrict__ desc,
                                                                const uint64_t* __restrict__ rows,
                                                                const void* __restrict__ src, uint32_t t,
                                                                uint32_t sel, uint32_t* __restrict__ table,
                                                                Ctrl* __restrict__ ctrl) {
  __shared__ uint32_t s_q[kMine], s_cnt, s_dup;
  const InstDesc D = desc[0];
  const uint64_t* __restrict__ R = rows + D.rows_off;
  if (threadIdx.x == 0) s_cnt = s_dup = 0;
  __syncthreads();
  constexpr uint64_t kTile = kSampleThreads * kSampleItems;
  for (uint64_t base = blockIdx.x * kTile; base < D.n; base += gridDim.x * kTile) {
    uint32_t own[kSampleItems], in = 0;
#pragma unroll
    for (int e = 0; e < kSampleItems; ++e) {
      const uint64_t q = base + e * kSampleThreads + threadIdx.x;
      own[e] = q < D.n ? src_at<SRC>(src, (uint32_t)q) : 0xffffffffu;
    }
#pragma unroll
    for (int e = 0; e < kSampleItems; ++e) {
      const uint64_t q = base + e * kSampleThreads + threadIdx.x;
      if (q < D.n && (SRC == 1 ? own[e] == 0u : ((own[e] * 0x9E3779B1u >> 8) & sel) == 0u)) in |= 1u << e;
    }
    if constexpr (SRC == 1) {
      uint32_t v[kSampleItems];
#pragma unroll
      for (int e = 0; e < kSampleItems; ++e) {
        const uint64_t q = base + e * kSampleThreads + threadIdx.x;
        v[e] = ((in >> e) & 1u) ? reinterpret_cast<const uint32_t*>(R[0])[q] : 0u;
      }
#pragma unroll
      for (int e = 0; e < kSampleItems; ++e)
        if (((in >> e) & 1u) && src_at<SRC>(src, v[e]) >= sel) in &= ~(1u << e);
    }
#pragma unroll
    for (int e = 0; e < kSampleItems; ++e) {
      if (!((in >> e) & 1u)) continue;
      const uint32_t at = atomicAdd(&s_cnt, 1u);
      if (at < kMine) s_q[at] = (uint32_t)(base + e * kSampleThreads + threadIdx.x);
    }
    if (s_cnt > kMine) break;  // (too many: the other waves see it here or a tile later)
  }
  __syncthreads();
  const uint32_t mine = s_cnt;
  if (threadIdx.x == 0 && mine) atomicAdd(&ctrl->u_count, mine > kMine ? kUniqSample + 1u : mine);
  if (mine > kMine) return;
  if (threadIdx.x < mine) {
    const uint32_t q = s_q[threadIdx.x];
    uint64_t h = mix(kUniqSeed, src_at<SRC>(src, q));
    uint32_t v[kMaxLabelLetters];  // (t <= kMaxLabelLetters; the loads of all letters together)
#pragma unroll
    for (uint32_t a = 0; a < kMaxLabelLetters; ++a)
      v[a] = a < t ? reinterpret_cast<const uint32_t*>(R[a])[q] : 0u;
#pragma unroll
    for (uint32_t a = 0; a < kMaxLabelLetters; ++a)
      if (a < t) v[a] = src_at<SRC>(src, v[a]);
#pragma unroll
    for (uint32_t a = 0; a < kMaxLabelLetters; ++a)
      if (a < t) h = mix(h, v[a]);
    const uint32_t w = (uint32_t)(mix_end(h) >> 16) | 1u;
    uint32_t p = (w * 0x85EBCA6Bu) >> 16;
    while (true) {  // (at most half full)
      p &= kUniqTable - 1u;
      const uint32_t prev = atomicCAS(&table[p], 0u, w);
      if (prev == 0u) break;
      if (prev == w) {
        atomicAdd(&s_dup, 1u);
        break;
      }
      ++p;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && s_dup) atomicAdd(&ctrl->u_dup, s_dup);
}

// (hash, state) pairs to buckets by the hash's top bits.  Bound: the gathers
// of t letters from the whole block array (64 MiB at 2^24 states: 59 G/s, 280
// of 420 us for one letter); a tile's pairs go out in runs of eight or more per
// bucket, straight from registers, merged in L2.
constexpr int kPartThreads = 512, kPartItems = 16;
template <int SRC>
__global__ __launch_bounds__(kPartThreads) void k_uniq_part(const InstDesc* __restrict__ desc,
                                                            const uint64_t* __restrict__ rows,
                                                            const void* __restrict__ src, uint32_t t,
                                                            uint2* __restrict__ entries,
                                                            uint32_t* __restrict__ cursor, uint32_t pbits,
                                                            Ctrl* __restrict__ ctrl) {
  __shared__ uint32_t cnt[kUniqBuckets];
  const InstDesc D = desc[0];
  const uint64_t* __restrict__ R = rows + D.rows_off;
  const uint32_t n = D.n, P = 1u << pbits;
  for (uint32_t b = threadIdx.x; b < P; b += kPartThreads) cnt[b] = 0;
  const uint64_t base = (uint64_t)blockIdx.x * (kPartThreads * kPartItems);
  uint64_t h[kPartItems];
#pragma unroll
  for (int e = 0; e < kPartItems; ++e) {
    const uint64_t q = base + e * kPartThreads + threadIdx.x;
    h[e] = mix(kUniqSeed, q < n ? src_at<SRC>(src, (uint32_t)q) : 0u);
  }
  for (uint32_t a = 0; a < t; ++a) {
    const uint32_t* __restrict__ row = reinterpret_cast<const uint32_t*>(R[a]);
    uint32_t s[kPartItems];
#pragma unroll
    for (int e = 0; e < kPartItems; ++e) {
      const uint64_t q = base + e * kPartThreads + threadIdx.x;
      s[e] = q < n ? row[q] : 0u;
    }
#pragma unroll
    for (int e = 0; e < kPartItems; ++e) s[e] = src_at<SRC>(src, s[e]);
#pragma unroll
    for (int e = 0; e < kPartItems; ++e) h[e] = mix(h[e], s[e]);
  }
  __syncthreads();
  uint32_t rank[kPartItems];
#pragma unroll
  for (int e = 0; e < kPartItems; ++e) {
    const uint64_t q = base + e * kPartThreads + threadIdx.x;
    h[e] = mix_end(h[e]);
    rank[e] = q < n ? atomicAdd(&cnt[h[e] >> (64u - pbits)], 1u) : 0u;
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < P; b += kPartThreads) {
    const uint32_t c = cnt[b];
    cnt[b] = c ? atomicAdd(&cursor[b], c) : 0u;
  }
  __syncthreads();
  bool over = false;
#pragma unroll
  for (int e = 0; e < kPartItems; ++e) {
    const uint64_t q = base + e * kPartThreads + threadIdx.x;
    if (q >= n) continue;
    const uint32_t b = (uint32_t)(h[e] >> (64u - pbits)), at = cnt[b] + rank[e];
    if (at < kUniqCap) entries[(uint64_t)b * kUniqCap + at] = make_uint2((uint32_t)h[e], (uint32_t)q);
    else over = true;
  }
  if (over) ctrl->u_over = 1u;
}

// A bucket in LDS.  Each pair throws (fragment, index) at a table with one
// minimum and reads back the winner of its slot: itself, a pair of the same
// hash (both share it), or of another (it throws again elsewhere; after four
// throws it counts as sharing, which only costs it a second look).  100 us of
// 2^24 states; inserting as many groups into
// a table takes 620 us of device atomics (27 G/s).
constexpr int kGroupThreads = 1024, kGroupItems = (int)kUniqCap / kGroupThreads;
__global__ __launch_bounds__(kGroupThreads) void k_uniq_group(const uint2* __restrict__ entries,
                                                              const uint32_t* __restrict__ cursor,
                                                              uint32_t* __restrict__ list, Ctrl* __restrict__ ctrl) {
  constexpr uint32_t kTab = 16384;
  __shared__ uint32_t hs[kUniqCap], tab[kTab], hit[kUniqCap / 32], s_rest, s_base;
  const uint32_t tid = threadIdx.x, count = min(cursor[blockIdx.x], kUniqCap);
  const uint2* __restrict__ E = entries + (uint64_t)blockIdx.x * kUniqCap;
  uint32_t q[kGroupItems], todo = 0, both = 0;
#pragma unroll
  for (int e = 0; e < kGroupItems; ++e) {
    const uint32_t x = e * kGroupThreads + tid;
    q[e] = 0;
    if (x >= count) continue;
    const uint2 v = E[x];
    hs[x] = v.x;
    q[e] = v.y;
    todo |= 1u << e;
  }
  for (uint32_t i = tid; i < kUniqCap / 32; i += kGroupThreads) hit[i] = 0;
  if (tid == 0) s_rest = 0;
  for (uint32_t r = 0; r < 4; ++r) {
    for (uint32_t i = tid; i < kTab; i += kGroupThreads) tab[i] = 0xffffffffu;
    __syncthreads();
    const uint32_t mul = 0x9E3779B1u + 0x3C6EF372u * r;
    auto aim = [&](uint32_t x, uint32_t& pos, uint32_t& word) {
      uint32_t y = hs[x] * mul;
      y ^= y >> 15;
      pos = y & (kTab - 1u);
      word = ((y >> 14) & 0x1ffffu) << 15 | x;
    };
#pragma unroll
    for (int e = 0; e < kGroupItems; ++e) {
      if (!((todo >> e) & 1u)) continue;
      uint32_t pos, word;
      aim(e * kGroupThreads + tid, pos, word);
      atomicMin(&tab[pos], word);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kGroupItems; ++e) {
      if (!((todo >> e) & 1u)) continue;
      const uint32_t x = e * kGroupThreads + tid;
      uint32_t pos, word;
      aim(x, pos, word);
      const uint32_t w = tab[pos] & 0x7fffu;
      if (w == x) {
        todo &= ~(1u << e);
      } else if (hs[w] == hs[x]) {
        todo &= ~(1u << e);
        both |= 1u << e;
        atomicOr(&hit[w >> 5], 1u << (w & 31u));
      }
    }
    __syncthreads();
  }
  both |= todo;
  uint32_t rest = 0;
#pragma unroll
  for (int e = 0; e < kGroupItems; ++e) {
    const uint32_t x = e * kGroupThreads + tid;
    if (x < count && ((hit[x >> 5] >> (x & 31u)) & 1u)) both |= 1u << e;
    rest += (both >> e) & 1u;
  }
  uint32_t at = rest ? atomicAdd(&s_rest, rest) : 0u;
  __syncthreads();
  if (tid == 0 && s_rest) s_base = atomicAdd(&ctrl->u_rest, s_rest);
  __syncthreads();
  at += s_base;
#pragma unroll
  for (int e = 0; e < kGroupItems; ++e)
    if ((both >> e) & 1u) list[at++] = q[e];
}

// block[q] = q for every state: those alone in this round are blocks of their
// own from now on (the others' ids are written behind this).  Nothing is
// written where the round has to be redone.
__global__ __launch_bounds__(kBlock) void k_uniq_apply(uint32_t n, uint32_t* __restrict__ block,
                                                       uint32_t* __restrict__ changed_inst,
                                                       const Ctrl* __restrict__ ctrl) {
  if (ctrl->collision) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) changed_inst[0] = 1u;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint64_t q = ((uint64_t)blockIdx.x * 8 + e) * kBlock + threadIdx.x;
    if (q < n) block[q] = (uint32_t)q;
  }
}

inline uint32_t groups_of(uint64_t items, uint64_t per) { return (uint32_t)((items + per - 1) / per); }

}  // namespace

void launch_label2(const InstDesc* desc, const uint64_t* rows, uint32_t n, const uint8_t* nib, uint32_t* label,
                   uint32_t cus, hipStream_t s) {
  hipLaunchKernelGGL(k_label2, dim3(std::min(groups_of(n, kBlock * kL2Items), 8u * cus)), dim3(kBlock), 0, s, desc,
                     rows, nib, label);
}

namespace {
void label2_count(uint32_t n, const uint32_t* label, uint32_t* maps, uint32_t* part, const Ctrl* ctrl,
                  UniqTest lazy, hipStream_t s) {
  // (a map takes as long to clear, write and merge as 50,000 states to mark)
  uint32_t wgs = 32;
  while (wgs < kLabel2Maps && n / wgs > 40000u) wgs *= 2;
  hipLaunchKernelGGL(k_seen_bits, dim3(wgs), dim3(kSeenThreads), 0, s, label, n, maps, part, ctrl, lazy);
  hipLaunchKernelGGL(k_seen_count, dim3(kHalves * kSeenWords / kBlock), dim3(kBlock), 0, s, maps, wgs, part, ctrl,
                     lazy);
}
}  // namespace

void launch_label2_count(uint32_t n, const uint32_t* label, uint32_t* maps, uint32_t* part, Ctrl* ctrl,
                         hipStream_t s) {
  label2_count(n, label, maps, part, ctrl, UniqTest{}, s);
  hipLaunchKernelGGL(k_label2_end, dim3(1), dim3(64), 0, s, part, 0u, n, nullptr, ctrl, UniqTest{});
}

void launch_label2_end(uint32_t n, const uint32_t* label, uint32_t* maps, uint32_t before, uint32_t* part,
                       UniqTest lazy, uint32_t* changed_inst, Ctrl* ctrl, hipStream_t s) {
  label2_count(n, label, maps, part, ctrl, lazy, s);
  hipLaunchKernelGGL(k_label2_end, dim3(1), dim3(64), 0, s, part, before, n, changed_inst, ctrl, lazy);
}

void launch_uniq_sample(const InstDesc* desc, const uint64_t* rows, const void* src, int width, uint32_t letters,
                        uint32_t sel, uint32_t* table, Ctrl* ctrl, hipStream_t s) {
  const dim3 g(kSampleWgs), b(kSampleThreads);
  if (width == 1) hipLaunchKernelGGL(k_uniq_sample<1>, g, b, 0, s, desc, rows, src, letters, sel, table, ctrl);
  else hipLaunchKernelGGL(k_uniq_sample<4>, g, b, 0, s, desc, rows, src, letters, sel, table, ctrl);
}

void launch_uniq_round(const InstDesc* desc, const uint64_t* rows, uint32_t n, const void* src, int width,
                       uint32_t letters, void* entries, uint32_t* cursor, uint32_t pbits, uint32_t* list, Ctrl* ctrl,
                       hipStream_t s) {
  const dim3 g(groups_of(n, kPartThreads * kPartItems)), b(kPartThreads);
  uint2* e = static_cast<uint2*>(entries);
  if (width == 1)
    hipLaunchKernelGGL(k_uniq_part<1>, g, b, 0, s, desc, rows, src, letters, e, cursor, pbits, ctrl);
  else
    hipLaunchKernelGGL(k_uniq_part<4>, g, b, 0, s, desc, rows, src, letters, e, cursor, pbits, ctrl);
  hipLaunchKernelGGL(k_uniq_group, dim3(1u << pbits), dim3(kGroupThreads), 0, s, e, cursor, list, ctrl);
}

void launch_uniq_apply(uint32_t n, uint32_t* block, uint32_t* changed_inst, const Ctrl* ctrl, hipStream_t s) {
  hipLaunchKernelGGL(k_uniq_apply, dim3(groups_of(n, kBlock * 8)), dim3(kBlock), 0, s, n, block, changed_inst, ctrl);
}

}  // namespace dfamin
