// fused.hip -- the whole minimization of a small instance in one workgroup.
//
// An instance of up to 16,384 states keeps its partition (block id = least
// member state, 16 bits), the closure level a doubling round reads, and the
// grouping table of a round in LDS.  One workgroup runs validation, the
// initial partition {F, Q\F}, every signature round (Section 3.3,
// Algorithm 4: group equal (own block, successor blocks) signatures, new id =
// least member, stop when the block count does not grow) and the canonical
// numbering, with barriers between the steps and no host decision between
// rounds.  The transition rows stay in global memory (they are read once per
// round and the second time from L2).
//
// Rounds follow the round engine exactly, so both give the same partition
// and the same counts:
//   * closure OFF: rounds over the non-identity letters;
//   * closure AUTO with one non-identity letter a: doubling rounds.  From
//     P_j the round gathers the level a^(2^l), 2^l <= j+1 (l capped at L),
//     which gives P_(j+2^l); each level is the square of the previous one
//     (pointer jumping, Section 3.4, Algorithm 5), computed in LDS in the
//     round that first reads it;
//   * closure AUTO with two or more non-identity letters: plain rounds; an
//     instance still splitting after auto_rounds rounds is handed back
//     (kFusedHandOff) and the caller runs it through the round engine,
//     which then builds its closure letters.
#include "../../include/dfamin.h"
#include "internal.h"

#include <type_traits>

namespace dfamin {

namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
// inclusive prefix sum over the wave's lanes
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  const uint32_t lane = threadIdx.x & 63u;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(v, o);
    if (lane >= (uint32_t)o) v += t;
  }
  return v;
}

__device__ __forceinline__ uint32_t mix_step(uint32_t h, uint32_t c) {
  h = (h ^ c) * 0x9E3779B1u;
  return h ^ (h >> 15);
}
__device__ __forceinline__ uint32_t mix_final(uint32_t h) {
  h ^= h >> 13;
  h *= 0x85EBCA6Bu;
  return h ^ (h >> 16);
}

// Grouping by minimum.  A round's states all throw (hash fragment, state id)
// words at a table with one LDS minimum each -- no answer is waited for --
// and read their slot back after a barrier: where the fragment is theirs the
// slot holds their group's least member, which is confirmed on the full
// signature; a state whose slot went to a smaller fragment (or whose
// confirmation fails) throws again at another slot.  At 16,384 states, of
// which most form groups of their own, three throws place all but a few
// hundred, about 12 us; claiming slots with a compare-and-swap and probing on,
// one answer after another, took 38 us of a 46 us round.
//
// Slot word: bits 31..17 a 15-bit fragment, bits 16..1 the state id, bit 0
// set once another member has found the slot's state (after the throws, so
// that it does not take part in the minimum).
constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr uint32_t kThrows = 6;  // per hash of the signatures; then a new one

// row[i] through a uniform base and a 32-bit offset register
__device__ __forceinline__ uint32_t ld(const uint32_t* __restrict__ row, uint32_t i) {
  return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(row) + (i << 2));
}

template <int MAXN, int NT>
__global__ void __launch_bounds__(NT, 4) k_fused(const FusedJob* __restrict__ jobs, FusedRes* __restrict__ res,
                                              uint32_t njobs, FusedJob one) {
  constexpr int ITEMS = MAXN / NT;
  constexpr uint32_t NW = NT / 64;
  constexpr int LC = ITEMS >= 8 ? 1 : 8 / ITEMS;  // letters gathered together
  static_assert(MAXN % NT == 0 && MAXN <= (1 << 16), "state ids are 16-bit in LDS");
  static_assert(ITEMS <= 32, "a bit per state of a thread");
  // table slots: 128 fewer than 1.5 MAXN leave room for the shared words in
  // 160 KB at MAXN = 16,384
  constexpr uint32_t SMAX = (3u * MAXN) / 2u - 128u;
  static_assert(SMAX >= ITEMS * NW + MAXN / 2, "wave counts and 16-bit ranks fit the table");
  // One struct, the 16-bit arrays first: an LDS access reaches 64 KB from its
  // base register by an immediate offset, so a thread's states cost no
  // address register each.
  struct Lds {
    uint16_t blk[MAXN];  // block id (least member) per state
    uint16_t lvl[MAXN];  // doubling: the closure level a^(2^built); else labels
    uint32_t sh[64];     // 0 bad, 1 non-identity letters, 2 min F, 3 min Q\F, 4/5 leaders (alternate
                         // rounds), 8..10 states left after a throw
    uint32_t slot[SMAX]; // grouping table; numbering scratch between rounds
  };
  __shared__ __align__(16) Lds lds;
  uint16_t* const blk = lds.blk;
  uint16_t* const lvl = lds.lvl;
  uint32_t* const sh = lds.sh;
  uint32_t* const slot = lds.slot;
  const uint32_t j = blockIdx.x;
  if (j >= njobs) return;
  // One job may come as an argument.  (Two statements: a pointer to either
  // would put the job's fields, and every row address made from them, into
  // vector registers.)
  FusedJob J = one;
  if (jobs) J = jobs[j];
  const uint32_t n = J.n, k = J.k, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t* __restrict__ delta = reinterpret_cast<const uint32_t*>(J.delta);
  const uint8_t* __restrict__ acc = reinterpret_cast<const uint8_t*>(J.accept);
  auto state = [&](int i) { return tid + (uint32_t)i * NT; };
  FusedRes R{};
  if (tid == 0) {
    sh[0] = 0;
    sh[1] = 0;
    sh[2] = kNone;
    sh[3] = kNone;
    sh[4] = sh[5] = 0;
    sh[8] = sh[9] = sh[10] = 0;
  }
  __syncthreads();

  // ---- validation (every entry < n) and identity letters (Section 2).
  // Thread tid owns states tid + i*NT, i < ITEMS (n <= MAXN); its loads of
  // one row go out together, so each row costs one memory latency.
  uint32_t fbits = 0;  // accept bit of owned state i in bit i
  uint32_t live = 0;   // bit i: owned state i exists and its block may still split
  {
    uint32_t bad = 0, nonid = J.validated ? J.mask : 0u;
    for (uint32_t a = 0; a < (J.validated ? 0u : k); a += LC) {
      uint32_t v[LC][ITEMS];
#pragma unroll
      for (int c = 0; c < LC; ++c) {
        const uint32_t* __restrict__ row = delta + (size_t)min(a + c, k - 1u) * n;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) v[c][i] = state(i) < n ? ld(row + i * NT, tid) : state(i);
      }
#pragma unroll
      for (int c = 0; c < LC; ++c) {
        uint32_t d = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          bad |= (uint32_t)(state(i) < n && v[c][i] >= n);
          d |= (uint32_t)(v[c][i] != state(i));
        }
        if (d) nonid |= 1u << min(a + c, k - 1u);
      }
    }
    uint8_t ab[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) ab[i] = state(i) < n ? acc[state(i) >> 3] : 0u;
    uint32_t mf = kNone, mn = kNone;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint32_t q = state(i);
      if (q >= n) continue;
      live |= 1u << i;
      if ((ab[i] >> (q & 7)) & 1u) {
        mf = min(mf, q);
        fbits |= 1u << i;
      } else {
        mn = min(mn, q);
      }
    }
    bad = wave_or(bad);
    nonid = wave_or(nonid);
    mf = wave_min(mf);
    mn = wave_min(mn);
    if (lane == 0) {
      if (bad) atomicOr(&sh[0], 1u);
      if (nonid) atomicOr(&sh[1], nonid);
      atomicMin(&sh[2], mf);
      atomicMin(&sh[3], mn);
    }
  }
  __syncthreads();
  if (sh[0]) {  // the same for every thread: the output is not touched
    if (tid == 0) {
      R.status = kFusedBad;
      res[j] = R;
    }
    return;
  }
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane(v); };
  const uint32_t mask = uniform(sh[1]);
  const uint32_t knon = __popc(mask);
  const bool autom = J.closure == DFAMIN_CLOSURE_AUTO;
  const bool dbl = autom && knon == 1;
  const uint32_t minF = uniform(sh[2]), minN = uniform(sh[3]);
  const uint32_t* __restrict__ rowA = delta + (size_t)(mask ? __ffs(mask) - 1 : 0) * n;  // the doubling letter
  // ---- initial partition {F, Q\F}; ids are least members (Section 3.2)
  uint32_t count = (minF < n ? 1u : 0u) + (minN < n ? 1u : 0u);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (!((live >> i) & 1u)) continue;
    const bool f = (fbits >> i) & 1u;
    blk[state(i)] = (uint16_t)(f ? minF : minN);
    // a doubling instance keeps its closure level in lvl[]; any other
    // starts with its accept bit there, the exact label of its class
    lvl[state(i)] = dbl ? (uint16_t)ld(rowA + i * NT, tid) : (uint16_t)f;
  }
  // slots of a hash round: up to eight per state (a small instance's throws
  // then nearly all hit), 1.5 per state at MAXN
  const uint32_t S = min(SMAX, max(64u, 8u * n));
  uint32_t rounds = 0, refine = 0, built = 0, used = 0;
  uint64_t jlen = 0;  // this partition is P_jlen (states agree on words of length <= jlen)
  // Exact-key rounds: while the signature in labels of lw bits each (block
  // numbers 0..B-1, or the accept bit in the first round) fits in
  // floor(log2 S) bits, it is itself the slot index: one throw, no fragment,
  // no comparison of signatures.  lvl[] then holds each state's label.
  const uint32_t lgS = 31u - (uint32_t)__clz(S);
  uint32_t lw = 1;
  auto fits_direct = [&](uint32_t bits) { return !dbl && bits <= lgS; };
  bool direct = fits_direct((knon + 1u) * lw);
  uint32_t was = live;  // live at the start of the round
  // Number of least members below state(i), for each owned i that is one
  // (states in order): wave counts in element order, then a scan by wave 0.
  auto rank_leaders = [&](uint32_t (&rk)[ITEMS], uint32_t& lead) {
    lead = 0;
    unsigned long long m[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const bool is = state(i) < n && blk[state(i)] == state(i);
      m[i] = __ballot(is);
      lead |= (is ? 1u : 0u) << i;
      if (lane == 0) slot[i * NW + wave] = (uint32_t)__popcll(m[i]);
    }
    __syncthreads();
    if (wave == 0) {
      uint32_t run = 0;
      for (uint32_t c0 = 0; c0 < ITEMS * NW; c0 += 64) {
        const uint32_t c = c0 + lane, x = c < ITEMS * NW ? slot[c] : 0u;
        const uint32_t incl = wave_incl_scan(x);
        if (c < ITEMS * NW) slot[c] = run + incl - x;
        run += __shfl(incl, 63);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      rk[i] = slot[i * NW + wave] + (uint32_t)__popcll(m[i] & ((1ull << lane) - 1ull));
  };
  int32_t status = kFusedOk;
  __syncthreads();

  // ---- rounds (a copy of the loop for doubling instances: less to keep in
  // registers than in one loop for both)
  auto run = [&](auto dblc) {
  constexpr bool DBL = decltype(dblc)::value;
  while (true) {
    if (!DBL && autom && knon >= 2 && rounds == J.auto_rounds) {
      status = kFusedHandOff;  // still splitting: its closure letters come from the round engine
      break;
    }
    if (rounds >= J.max_rounds) {
      status = kFusedRoundCap;
      break;
    }
    uint32_t l = 0;
    if constexpr (DBL) {
      l = 63u - (uint32_t)__clzll(jlen + 1ull);
      if (l > J.levels) l = J.levels;
      for (; built < l; ++built) {  // level built+1 = level built, squared
        uint16_t nxt[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
          if (state(i) < n) nxt[i] = lvl[lvl[state(i)]];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
          if (state(i) < n) lvl[state(i)] = nxt[i];
        __syncthreads();
      }
    }
    // key[i]: the exact key or the signature's hash; once the state has its
    // group, its new id (least member)
    uint32_t key[ITEMS];
    const uint32_t T = !DBL && direct ? 1u << ((knon + 1u) * lw) : S;  // slots of this round
    // few groups: most throws would lose to a word already there, and a
    // read, which many lanes share, then saves the serialized minimum
    const bool read_first = count * 8u < n;
    uint32_t todo = live;
    // Successors of the states to place, LC letters at a time (their loads
    // go out together; small tiles have few per letter).
    auto for_letters = [&](auto use) {
      for (uint32_t mm = mask; mm;) {
        uint32_t s[LC][ITEMS], cnt = 0;
#pragma unroll
        for (int c = 0; c < LC; ++c) {
          if (!mm) break;
          const uint32_t* row = delta + (size_t)(__ffs(mm) - 1) * n;
          mm &= mm - 1u;
          ++cnt;
#pragma unroll
          for (int i = 0; i < ITEMS; ++i) s[c][i] = ((todo >> i) & 1u) ? ld(row + i * NT, tid) : 0u;
        }
        use(s, cnt);
      }
    };
    for (uint32_t hashes = 0; ; ++hashes) {
      if (!DBL && direct) {
        const uint16_t* lab = lvl;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) key[i] = state(i) < n ? lab[state(i)] : 0u;
        {
          uint32_t at = lw;
          for_letters([&](const uint32_t (&s)[LC][ITEMS], uint32_t cnt) {
#pragma unroll
            for (int c = 0; c < LC; ++c) {
              if ((uint32_t)c >= cnt) break;
#pragma unroll
              for (int i = 0; i < ITEMS; ++i) key[i] |= (uint32_t)lab[s[c][i]] << at;
              at += lw;
            }
          });
        }
      } else {
        const uint32_t seed = 0x6A09E667u + hashes * 0x9E3779B9u;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
          if ((todo >> i) & 1u) key[i] = mix_step(seed, blk[state(i)]);
        if constexpr (DBL) {
#pragma unroll
          for (int i = 0; i < ITEMS; ++i)
            if ((todo >> i) & 1u) key[i] = mix_step(key[i], blk[lvl[state(i)]]);
        } else {
          for_letters([&](const uint32_t (&s)[LC][ITEMS], uint32_t cnt) {
#pragma unroll
            for (int c = 0; c < LC; ++c) {
              if ((uint32_t)c >= cnt) break;
#pragma unroll
              for (int i = 0; i < ITEMS; ++i)
                if ((todo >> i) & 1u) key[i] = mix_step(key[i], blk[s[c][i]]);
            }
          });
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
          if ((todo >> i) & 1u) key[i] = mix_final(key[i]);
      }
      bool left = true;
      for (uint32_t t = 0; left && t < kThrows; ++t) {
        for (uint32_t x = tid; x < T / 4u; x += NT)
          reinterpret_cast<uint4*>(slot)[x] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
        if (tid < (T & 3u)) slot[(T & ~3u) + tid] = kEmpty;
        __syncthreads();
        // this throw's slot and fragment
        // (the multiplier is made opaque in each of the three steps: the
        // compiler would otherwise keep every state's slot and fragment from
        // one step to the next, and spill; at 16 states per thread 23
        // registers still do)
        uint32_t mul = 0x9E3779B1u + 0x3C6EF372u * t;  // odd: a bijection of h
        asm volatile("" : "+s"(mul));
        auto aim = [&](uint32_t h, uint32_t& pos, uint32_t& frag) {
          if (!DBL && direct) {
            pos = h;
            frag = 0;
          } else {
            uint32_t y = h * mul;
            y ^= y >> 16;
            frag = min(y >> 17, 0x7FFEu);
            pos = ((y & 0x1FFFFu) * T) >> 17;  // (T < 2^15)
          }
        };
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          if (!((todo >> i) & 1u)) continue;
          uint32_t pos, frag;
          aim(key[i], pos, frag);
          const uint32_t word = (frag << 17) | (state(i) << 1);
          if (!read_first || slot[pos] > word) atomicMin(&slot[pos], word);
        }
        __syncthreads();
        asm volatile("" : "+s"(mul));
        uint32_t reps = 0, cand = 0;  // owned states that are their slot's least member; that found one
        uint32_t rep[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          rep[i] = 0;
          if (!((todo >> i) & 1u)) continue;
          uint32_t pos, frag;
          aim(key[i], pos, frag);
          const uint32_t v = slot[pos];
          if ((v >> 17) != frag) continue;
          rep[i] = (v >> 1) & 0xFFFFu;
          if (rep[i] == state(i)) reps |= 1u << i;
          else cand |= 1u << i;
        }
        // Confirmed on the full signature, a letter at a time for half the
        // thread's states together (state by state, each one's row loads
        // waited for, took 13 us of a 16,384-state round; now 5).
        if ((DBL || !direct) && __any(cand != 0u)) {
#pragma unroll
          for (int i = 0; i < ITEMS; ++i)
            if (((cand >> i) & 1u) && blk[rep[i]] != blk[state(i)]) cand &= ~(1u << i);
          if constexpr (DBL) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
              if (((cand >> i) & 1u) && blk[lvl[rep[i]]] != blk[lvl[state(i)]]) cand &= ~(1u << i);
          } else {
            constexpr int HALF = (ITEMS + 1) / 2;
            for (uint32_t mm = mask; mm; mm &= mm - 1u) {
              const uint32_t* row = delta + (size_t)(__ffs(mm) - 1) * n;
#pragma unroll
              for (int i0 = 0; i0 < ITEMS; i0 += HALF) {
                uint32_t a[HALF], b[HALF];
#pragma unroll
                for (int i = 0; i < HALF; ++i) {
                  const bool on = i0 + i < ITEMS && ((cand >> (i0 + i)) & 1u);
                  a[i] = on ? ld(row, rep[i0 + i]) : 0u;
                  b[i] = on ? ld(row + (i0 + i) * NT, tid) : 0u;
                }
#pragma unroll
                for (int i = 0; i < HALF; ++i)
                  if (blk[a[i]] != blk[b[i]]) cand &= ~(1u << (i0 + i));
              }
            }
          }
        }
        asm volatile("" : "+s"(mul));
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          if (!((cand >> i) & 1u)) continue;
          uint32_t pos, frag;
          aim(key[i], pos, frag);
          if (!(slot[pos] & 1u)) atomicOr(&slot[pos], 1u);
          key[i] = rep[i];
        }
        todo &= ~cand;
        __syncthreads();
        asm volatile("" : "+s"(mul));
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          if (!((reps >> i) & 1u)) continue;
          uint32_t pos, frag;
          aim(key[i], pos, frag);
          if (!(slot[pos] & 1u)) live &= ~(1u << i);  // alone: this block can never split
          key[i] = state(i);
        }
        todo &= ~reps;
        // (a word of its own per throw, cleared two throws ahead)
        if (__any(todo != 0u) && lane == 0) sh[8 + t % 3u] = 1u;
        __syncthreads();
        left = uniform(sh[8 + t % 3u]) != 0u;
        if (tid == 0) sh[8 + (t + 2u) % 3u] = 0u;
      }
      if (!left) break;
      // signatures that share a whole hash: another one separates them.  (Every
      // state finds its group in the end; the bound is only a backstop.)
      if (hashes >= 64u) {
        status = kFusedFault;
        break;
      }
    }
    if (status != kFusedOk) break;
    // new id = the group's least member; count the groups.  (A state that was
    // alone before this round keeps its own id.)
    uint32_t leaders = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint32_t q = state(i);
      if (q >= n) continue;
      if ((was >> i) & 1u) blk[q] = (uint16_t)key[i];
      leaders += (uint32_t)(((was >> i) & 1u) ? key[i] == q : 1u);
    }
    was = live;
    leaders = wave_sum(leaders);
    if (lane == 0) atomicAdd(&sh[4 + (rounds & 1u)], leaders);
    __syncthreads();
    const uint32_t cnew = uniform(sh[4 + (rounds & 1u)]);
    if (tid == 0) sh[4 + ((rounds + 1u) & 1u)] = 0;
    ++rounds;
    if (cnew == count) break;  // no block split: stable
    ++refine;
    used = max(used, l);  // the highest level a splitting round read
    count = cnew;
    jlen += DBL ? (1ull << l) : 1ull;
    if (count == n) break;  // every block a singleton: stable without another round
    // the next round's labels: block numbers, if its signature fits
    const uint32_t wn = max(1u, 32u - (uint32_t)__clz(count - 1u));
    if (!DBL) direct = fits_direct((knon + 1u) * wn);
    if (!DBL && direct) {
      uint32_t rk[ITEMS], lead;
      rank_leaders(rk, lead);
      uint16_t* ranks = reinterpret_cast<uint16_t*>(slot + ITEMS * NW);
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if ((lead >> i) & 1u) ranks[state(i)] = (uint16_t)rk[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (state(i) < n) lvl[state(i)] = ranks[blk[state(i)]];
      lw = wn;
    }
    __syncthreads();
  }
  };
  if (dbl) run(std::true_type{});
  else run(std::false_type{});
  if (status != kFusedOk) {
    if (tid == 0) {
      R.status = status;
      res[j] = R;
    }
    return;
  }

  // ---- canonical numbering: out[q] = rank of q's block's least member.
  // The ranks take the least members' place in blk[] once every thread has
  // its states' ids.
  uint32_t id[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) id[i] = state(i) < n ? blk[state(i)] : 0u;
  const uint32_t id0 = blk[J.q0];
  {
    uint32_t rk[ITEMS], lead;
    rank_leaders(rk, lead);  // (its barriers come before the writes below)
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if ((lead >> i) & 1u) blk[state(i)] = (uint16_t)rk[i];
  }
  __syncthreads();
  uint32_t* __restrict__ out = reinterpret_cast<uint32_t*>(J.out);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (state(i) < n) out[state(i)] = blk[id[i]];
  if (tid == 0) {
    R.status = kFusedOk;
    R.num_blocks = count;
    R.initial_block = blk[id0];
    R.refine_rounds = refine;
    R.levels_used = used;
    R.doubling = dbl ? 1u : 0u;
    res[j] = R;
  }
}

// Larger instances of a batch (16,384 < n <= 65,536), one workgroup each: the
// same rounds and the same grouping by minimum, with the block ids (16-bit)
// and the table sharing the LDS -- 30,000 slots at 20,000 states, 7,700 at
// 65,536 -- and hashes, lists and signatures in global scratch (796 instances
// at once move 3.3 GB into and 2.8 GB out of L2 a launch for it).  Where a
// round may form more groups than the table takes, its states are first sorted
// into slices of the hash (all members of a group share one), and each throw
// takes one more slice along with what the last throw left.  Bound: LDS operations and the row reads of each round, on as
// many CUs as there are instances; a round of the round engine moves the same
// states through device atomics (27 G/s) and a dozen launches instead.  A
// random instance of 65,536 states and two letters takes 1.0 ms (six rounds
// of 40 us hashing and, in three, 150 us of throws), 256 of them 1.8 ms
// (round engine: 4.0), 512 chains of that size 5.3 ms (22.9); a batch of 4,096
// instances up to 65,536 states went from 10.2 to 3.3 ms.  New ids take the old
// ones' place as groups form (written to scratch and copied at the round's end:
// 2.2 and 6.2 ms).
constexpr uint32_t kBigThreads = 1024, kBigWaves = kBigThreads / 64;
constexpr uint32_t kBigLds = 40960 - 64;  // 32-bit words
constexpr uint32_t kSlices = 16;
constexpr int kBigChunk = 8;              // states of a thread whose loads go out together

__global__ void __launch_bounds__(kBigThreads, 4) k_fused_big(const FusedJob* __restrict__ jobs,
                                                              FusedRes* __restrict__ res, uint32_t njobs) {
  __shared__ __align__(16) uint32_t lds[kBigLds];
  // words 0..63: 0 bad, 1 letters, 2 min F, 3 min Q\F, 4/5 leaders, 6/7 list lengths
  uint32_t* const sh = lds;
  uint32_t* const hist = lds + 64;                      // per wave and slice: counts, then list positions
  uint32_t* const first = hist + kBigWaves * kSlices;   // start of each slice, and the end
  uint16_t* const blk = reinterpret_cast<uint16_t*>(lds + 64 + kBigWaves * kSlices + 32);
  const uint32_t j = blockIdx.x;
  if (j >= njobs) return;
  const FusedJob J = jobs[j];
  const uint32_t n = J.n, k = J.k, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t blkw = ((n + 7u) / 8u) * 4u;  // words of blk[], 16-byte multiple
  uint32_t* const slot = lds + 64 + kBigWaves * kSlices + 32 + blkw;
  const uint32_t S = kBigLds - (64 + kBigWaves * kSlices + 32) - blkw;  // below 2^15
  const uint32_t* __restrict__ delta = reinterpret_cast<const uint32_t*>(J.delta);
  const uint8_t* __restrict__ acc = reinterpret_cast<const uint8_t*>(J.accept);
  // scratch: hash per state, the emission's ids (in a round: a byte per state
  // that a list throw found alone), the sorted list, two leftover lists
  // ((hash, state) pairs), two levels, the signatures
  const uint32_t n4 = (n + 3u) & ~3u;
  uint32_t* H = reinterpret_cast<uint32_t*>(J.scratch);
  uint32_t* NB = H + n4;
  uint2* L = reinterpret_cast<uint2*>(NB + n4);
  uint2* LO[2] = {L + n4, L + 2 * n4};
  uint16_t* LV[2] = {reinterpret_cast<uint16_t*>(L + 3 * n4), reinterpret_cast<uint16_t*>(L + 3 * n4) + n4};
  // Signatures as 16-bit block ids, eight to a record of 16 bytes: what a
  // confirmation compares, two reads instead of two per letter.
  uint4* REC = reinterpret_cast<uint4*>(LV[1] + n4);
  const uint32_t iters = (n + kBigThreads - 1) / kBigThreads;  // at most 64
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane(v); };
  FusedRes R{};
  if (tid < 64) sh[tid] = tid == 2 || tid == 3 ? kNone : 0u;
  __syncthreads();

  unsigned long long live = 0;  // bit i: state tid + i*1024 exists and its block may still split
  {
    uint32_t bad = 0, nonid = 0;
    if (J.validated) {
      nonid = J.mask;
    } else {
      for (uint32_t a = 0; a < k; ++a) {
        const uint32_t* __restrict__ row = delta + (size_t)a * n;
        uint32_t d = 0;
        for (uint32_t i0 = 0; i0 < iters; i0 += kBigChunk) {
          uint32_t v[kBigChunk];
#pragma unroll
          for (int i = 0; i < kBigChunk; ++i) {
            const uint32_t q = tid + (i0 + i) * kBigThreads;
            v[i] = q < n ? ld(row, q) : q;
          }
#pragma unroll
          for (int i = 0; i < kBigChunk; ++i) {
            const uint32_t q = tid + (i0 + i) * kBigThreads;
            bad |= (uint32_t)(q < n && v[i] >= n);
            d |= (uint32_t)(v[i] != q);
          }
        }
        if (d) nonid |= 1u << a;
      }
    }
    uint32_t mf = kNone, mn = kNone;
    for (uint32_t i = 0; i < iters; ++i) {
      const uint32_t q = tid + i * kBigThreads;
      if (q >= n) break;
      live |= 1ull << i;
      if ((acc[q >> 3] >> (q & 7)) & 1u) mf = min(mf, q);
      else mn = min(mn, q);
    }
    bad = wave_or(bad);
    nonid = wave_or(nonid);
    mf = wave_min(mf);
    mn = wave_min(mn);
    if (lane == 0) {
      if (bad) atomicOr(&sh[0], 1u);
      if (nonid) atomicOr(&sh[1], nonid);
      atomicMin(&sh[2], mf);
      atomicMin(&sh[3], mn);
    }
  }
  __syncthreads();
  if (sh[0]) {
    if (tid == 0) {
      R.status = kFusedBad;
      res[j] = R;
    }
    return;
  }
  const uint32_t mask = uniform(sh[1]), knon = __popc(mask);
  const bool autom = J.closure == DFAMIN_CLOSURE_AUTO;
  const bool dbl = autom && knon == 1;
  const uint32_t minF = uniform(sh[2]), minN = uniform(sh[3]);
  uint32_t count = (minF < n ? 1u : 0u) + (minN < n ? 1u : 0u);
  {
    const uint32_t* __restrict__ rowA = delta + (size_t)(mask ? __ffs(mask) - 1 : 0) * n;
    for (uint32_t i = 0; i < iters; ++i) {
      const uint32_t q = tid + i * kBigThreads;
      if (q >= n) break;
      blk[q] = (uint16_t)(((acc[q >> 3] >> (q & 7)) & 1u) ? minF : minN);
      if (dbl) LV[0][q] = (uint16_t)ld(rowA, q);
    }
  }
  uint32_t rounds = 0, refine = 0, used = 0, l = 0, alive = n;
  uint64_t jlen = 0;
  int32_t status = kFusedOk;
  uint8_t* const AB = reinterpret_cast<uint8_t*>(NB);
  __syncthreads();

  // (a copy of the loop for doubling instances: less to keep in registers
  // than in one loop for both; no letter but identities: {F, Q\F} is stable)
  auto run = [&](auto dblc) {
  constexpr bool DBL = decltype(dblc)::value;
  while (knon) {
    if (autom && !DBL && knon >= 2 && rounds == J.auto_rounds) {
      status = kFusedHandOff;
      break;
    }
    if (rounds >= J.max_rounds) {
      status = kFusedRoundCap;
      break;
    }
    const uint16_t* lv = LV[l & 1u];
    uint16_t* lvn = nullptr;  // the next round's level, squared beside this round's hashes
    if (DBL && l < J.levels && (1ull << (l + 1)) <= jlen + (1ull << l) + 1ull) lvn = LV[(l + 1u) & 1u];
    // the first round's signatures (accept bits) index the table themselves
    const bool direct = !DBL && rounds == 0 && knon + 1u <= 31u - (uint32_t)__clz(S);
    // groups this round may form: as many as states left to place, but a
    // doubling round at most about squares its blocks, and from few blocks
    // forms far fewer (a guess: too low costs throws, nothing else)
    const uint32_t est = direct ? 1u : (DBL ? (uint32_t)min((uint64_t)alive, 4ull * count) : alive);
    const uint32_t P = est <= S + S / 2u ? 1u : min(kSlices, (uint32_t)((10ull * est + 7ull * S - 1) / (7ull * S)));
    const bool read_first = count * 8u < n;
    const uint32_t seed0 = 0x6A09E667u;
    auto slice = [&](uint32_t h) { return ((h >> 16) * P) >> 16; };
    auto aim_at = [&](uint32_t h, uint32_t mul, uint32_t& pos, uint32_t& frag) {
      uint32_t y = h * mul;
      y ^= y >> 16;
      frag = min(y >> 17, 0x7FFEu);
      pos = ((y & 0x1FFFFu) * S) >> 17;
    };
    if (P > 1 && tid < kBigWaves * kSlices) hist[tid] = 0;
    if (P == 1)
      for (uint32_t x = tid; x < S; x += kBigThreads) slot[x] = kEmpty;
    if (tid < 2) sh[6 + tid] = 0;
    __syncthreads();
    // ---- hashes (and the next level).  A doubling signature's two ids are
    // its exact 32-bit key, which the hash only permutes.  With one slice the
    // first throw happens right here.
    const uint32_t recs = (knon + 8u) / 8u;  // records per signature
    auto hash_one = [&](uint32_t q, uint32_t seed) {  // (a rehash, from the records: rare)
      const uint32_t* r = reinterpret_cast<const uint32_t*>(REC) + (size_t)q * (4u * recs);
      uint32_t h = seed;
      for (uint32_t a = 0; a <= knon; ++a) h = mix_step(h, (r[a >> 1] >> (16u * (a & 1u))) & 0xFFFFu);
      return mix_final(h);
    };
    auto throw_at = [&](uint32_t h, uint32_t q, uint32_t mul) {
      uint32_t pos = h, frag = 0;
      if (!direct) aim_at(h, mul, pos, frag);
      const uint32_t word = (frag << 17) | (q << 1);
      if (!read_first || slot[pos] > word) atomicMin(&slot[pos], word);
    };
    for (uint32_t i0 = 0; i0 < iters; i0 += kBigChunk) {
      uint32_t h[kBigChunk], s[kBigChunk];
      const uint32_t bits = (uint32_t)(live >> i0) & ((1u << kBigChunk) - 1u);
      if (DBL) {
        uint32_t nx[kBigChunk];
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i) {
          const uint32_t q = tid + (i0 + i) * kBigThreads;
          s[i] = q < n ? lv[q] : 0u;
        }
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i) nx[i] = lvn ? lv[s[i]] : 0u;
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i) {
          const uint32_t q = tid + (i0 + i) * kBigThreads;
          if (lvn && q < n) lvn[q] = (uint16_t)nx[i];
          h[i] = mix_final((((q < n ? (uint32_t)blk[q] : 0u) << 16) | blk[s[i]]) * 0x9E3779B1u);
        }
      } else {
        uint32_t w[kBigChunk];  // two ids of the record being filled
        uint32_t at = 1;
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i) {
          const uint32_t q = tid + (i0 + i) * kBigThreads;
          w[i] = q < n ? (uint32_t)blk[q] : 0u;
          h[i] = direct ? (uint32_t)(w[i] == minF) : mix_step(seed0, w[i]);
        }
        for (uint32_t mm = mask; mm; mm &= mm - 1u, ++at) {
          const uint32_t* row = delta + (size_t)(__ffs(mm) - 1) * n;
#pragma unroll
          for (int i = 0; i < kBigChunk; ++i)
            s[i] = ((bits >> i) & 1u) ? ld(row, tid + (i0 + i) * kBigThreads) : 0u;
#pragma unroll
          for (int i = 0; i < kBigChunk; ++i) {
            const uint32_t b = blk[s[i]];
            h[i] = direct ? h[i] | ((uint32_t)(b == minF) << at) : mix_step(h[i], b);
            w[i] |= b << (16u * (at & 1u));
          }
          // (letter pairs go out as they fill: word at/2 of the state's records)
          if (!direct && ((at & 1u) || !(mm & (mm - 1u)))) {
#pragma unroll
            for (int i = 0; i < kBigChunk; ++i) {
              if ((bits >> i) & 1u)
                reinterpret_cast<uint32_t*>(REC)[(size_t)(tid + (i0 + i) * kBigThreads) * (4u * recs) + (at >> 1)] = w[i];
              w[i] = 0;
            }
          }
        }
      }
#pragma unroll
      for (int i = 0; i < kBigChunk; ++i) {
        if (!((bits >> i) & 1u)) continue;
        if (!direct && !DBL) h[i] = mix_final(h[i]);
        H[tid + (i0 + i) * kBigThreads] = h[i];
        if (P > 1) atomicAdd(&hist[wave * kSlices + slice(h[i])], 1u);
        else throw_at(h[i], tid + (i0 + i) * kBigThreads, 0x9E3779B1u);
      }
    }
    __syncthreads();
    if (P > 1) {
      // list positions: slice by slice, wave by wave
      if (tid < 64) {
        uint32_t run = 0;
        for (uint32_t c0 = 0; c0 < kBigWaves * kSlices; c0 += 64) {
          const uint32_t c = c0 + lane;  // (slice, wave) in list order
          uint32_t& cell = hist[(c % kBigWaves) * kSlices + c / kBigWaves];
          const uint32_t x = cell, incl = wave_incl_scan(x);
          cell = run + incl - x;
          if (c % kBigWaves == 0) first[c / kBigWaves] = run + incl - x;
          run += __shfl(incl, 63);
        }
        if (lane == 0) first[kSlices] = run;
      }
      __syncthreads();
      for (uint32_t i0 = 0; i0 < iters; i0 += kBigChunk) {
        const uint32_t bits = (uint32_t)(live >> i0) & ((1u << kBigChunk) - 1u);
        uint32_t h[kBigChunk];
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i) h[i] = ((bits >> i) & 1u) ? H[tid + (i0 + i) * kBigThreads] : 0u;
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i)
          if ((bits >> i) & 1u)
            L[atomicAdd(&hist[wave * kSlices + slice(h[i])], 1u)] = make_uint2(h[i], tid + (i0 + i) * kBigThreads);
      }
      __syncthreads();
    }
    // ---- throws
    // A state that has its group takes its new id at once: the signatures are
    // in the records (doubling: in the hashes), the old ids no longer needed.
    uint32_t next = 0, left = 0, lo = 0, idle = 0, rehash = 0;  // next: slices thrown so far
    uint32_t leaders = 0, alone = 0;
    bool lists = false;  // some throw took its states from a list
    while (next < P || left) {
      // entries of this throw: what is left, then the next slice (or, with
      // one slice, every live state in order)
      const bool order = P == 1 && next == 0;
      uint32_t b0 = 0, add = 0;
      if (P > 1 && next < P) {
        b0 = uniform(first[next]);
        add = uniform(next + 1 < kSlices ? first[next + 1] : first[kSlices]) - b0;
      }
      const uint32_t total = order ? n : left + add;
      const uint2* old = LO[lo];
      uint2* fresh = LO[lo ^ 1u];
      auto entry = [&](uint32_t x) -> uint2 {
        if (order) return make_uint2(H[x], x);
        return x < left ? old[x] : L[b0 + x - left];
      };
      auto valid = [&](uint32_t x, uint32_t i) { return x < total && (!order || ((live >> i) & 1u)); };
      const uint32_t mul = 0x9E3779B1u + 0x3C6EF372u * (next + idle);  // odd: a bijection of h
      auto aim = [&](uint32_t h, uint32_t& pos, uint32_t& frag) {
        if (direct) {
          pos = h;
          frag = 0;
        } else {
          aim_at(h, mul, pos, frag);
        }
      };
      if (!order) {
        for (uint32_t x = tid; x < S; x += kBigThreads) slot[x] = kEmpty;
        if (!lists)
          for (uint32_t x = tid; x < n4 / 4u; x += kBigThreads) NB[x] = 0u;
        lists = true;
      }
      if (tid == 0) sh[6 + (lo ^ 1u)] = 0;
      __syncthreads();
      const uint32_t its = (total + kBigThreads - 1) / kBigThreads;
      constexpr int UT = 8, U = DBL ? 8 : 4;
      if (!order) {
        for (uint32_t i0 = 0; i0 < its; i0 += UT) {
          uint2 e[UT];
#pragma unroll
          for (int i = 0; i < UT; ++i) {
            const uint32_t x = tid + (i0 + i) * kBigThreads;
            e[i] = x < total ? entry(x) : make_uint2(0, kNone);
          }
#pragma unroll
          for (int i = 0; i < UT; ++i)
            if (e[i].y != kNone) throw_at(e[i].x, e[i].y, mul);
        }
        __syncthreads();
      }
      unsigned long long reps = 0;
      for (uint32_t i0 = 0; i0 < its; i0 += U) {
        uint2 e[U];
        uint32_t rep[U], cand = 0, todo = 0;
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const uint32_t x = tid + (i0 + i) * kBigThreads;
          e[i] = valid(x, i0 + i) ? entry(x) : make_uint2(0, kNone);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
          rep[i] = 0;
          if (e[i].y == kNone) continue;
          todo |= 1u << i;
          uint32_t pos, frag;
          aim(e[i].x, pos, frag);
          const uint32_t v = slot[pos];
          if ((v >> 17) != frag) continue;
          rep[i] = (v >> 1) & 0xFFFFu;
          if (rep[i] == e[i].y) {
            reps |= 1ull << (i0 + i);
            todo &= ~(1u << i);
          } else {
            cand |= 1u << i;
          }
        }
        if (!direct && __any(cand != 0u)) {
          if (DBL) {  // the hash is the signature
            uint32_t a[U];
#pragma unroll
            for (int i = 0; i < U; ++i) a[i] = ((cand >> i) & 1u) ? H[rep[i]] : e[i].x;
#pragma unroll
            for (int i = 0; i < U; ++i)
              if (a[i] != e[i].x) cand &= ~(1u << i);
          } else {
            for (uint32_t r = 0; r < recs; ++r) {
              uint4 a[U], b[U];
#pragma unroll
              for (int i = 0; i < U; ++i) {
                const bool on = (cand >> i) & 1u;
                a[i] = REC[(size_t)(on ? rep[i] : 0u) * recs + r];
                b[i] = REC[(size_t)(on ? e[i].y : 0u) * recs + r];
              }
              // (ids beyond the signature's last are never written: not compared)
              const uint32_t ids = min(8u, knon + 1u - 8u * r);
#pragma unroll
              for (int i = 0; i < U; ++i) {
                bool same = a[i].x == b[i].x || ids == 0u;
                if (ids > 2u) same = same && a[i].y == b[i].y;
                if (ids > 4u) same = same && a[i].z == b[i].z;
                if (ids > 6u) same = same && a[i].w == b[i].w;
                if (!same) cand &= ~(1u << i);
              }
            }
          }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
          if (!((cand >> i) & 1u)) continue;
          uint32_t pos, frag;
          aim(e[i].x, pos, frag);
          if (!(slot[pos] & 1u)) atomicOr(&slot[pos], 1u);
          blk[e[i].y] = (uint16_t)rep[i];
        }
        todo &= ~cand;
        // what is left joins the next throw's list
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const bool go = (todo >> i) & 1u;
          const unsigned long long m = __ballot(go);
          if (!m) continue;
          uint32_t p = 0;
          if (lane == (uint32_t)__builtin_ctzll(m)) p = atomicAdd(&sh[6 + (lo ^ 1u)], (uint32_t)__popcll(m));
          p = __shfl(p, __builtin_ctzll(m));
          if (go) fresh[p + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = e[i];
        }
      }
      __syncthreads();
      for (unsigned long long b = reps; b; b &= b - 1ull) {  // alone unless a member marked the slot
        const uint2 e = entry(tid + (uint32_t)__builtin_ctzll(b) * kBigThreads);
        uint32_t pos, frag;
        aim(e.x, pos, frag);
        blk[e.y] = (uint16_t)e.y;
        ++leaders;
        if (slot[pos] & 1u) continue;
        ++alone;
        if (order) live &= ~(b & (0ull - b));
        else AB[e.y] = 1;
      }
      left = uniform(sh[6 + (lo ^ 1u)]);
      lo ^= 1u;
      if (next < P) ++next;
      else ++idle;
      __syncthreads();
      if (idle > 4096u) {  // (each throw places at least one group: a backstop)
        status = kFusedFault;
        break;
      }
      if (!DBL && left && next >= P && (idle & 7u) == 7u) {
        // signatures that share a whole hash: another one separates them
        ++rehash;
        for (uint32_t x = tid; x < left; x += kBigThreads) {
          const uint32_t q = LO[lo][x].y;
          LO[lo][x].x = hash_one(q, seed0 + rehash * 0x9E3779B9u);
        }
        __syncthreads();
      }
    }
    if (status != kFusedOk) break;
    // ---- groups counted (a state alone before this round is one); the owners
    // of states found alone from a list drop them
    if (lists)
      for (uint32_t i0 = 0; i0 < iters; i0 += kBigChunk) {
        uint8_t v[kBigChunk];
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i)
          v[i] = ((live >> (i0 + i)) & 1ull) ? AB[tid + (i0 + i) * kBigThreads] : 0;
#pragma unroll
        for (int i = 0; i < kBigChunk; ++i)
          if (v[i]) live &= ~(1ull << (i0 + i));
      }
    leaders = wave_sum(leaders);
    alone = wave_sum(alone);
    if (lane == 0) {
      atomicAdd(&sh[4], leaders);
      atomicAdd(&sh[5], alone);
    }
    __syncthreads();
    const uint32_t cnew = uniform(sh[4]) + (n - alive);
    alive -= uniform(sh[5]);
    __syncthreads();
    if (tid < 2) sh[4 + tid] = 0;
    ++rounds;
    if (cnew == count) break;  // no block split: stable
    ++refine;
    used = max(used, l);
    count = cnew;
    jlen += DBL ? (1ull << l) : 1ull;
    if (lvn) ++l;
    if (count == n) break;
  }
  };
  if (dbl) run(std::true_type{});
  else run(std::false_type{});
  if (status != kFusedOk) {
    if (tid == 0) {
      R.status = status;
      res[j] = R;
    }
    return;
  }

  // ---- canonical numbering: the least members' ranks (in NB) by wave
  // counts in state order
  __syncthreads();
  for (uint32_t i = 0; i < iters; ++i) {
    const uint32_t q = tid + i * kBigThreads;
    const unsigned long long m = __ballot(q < n && blk[q] == q);
    if (lane == 0) slot[i * kBigWaves + wave] = (uint32_t)__popcll(m);
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t run = 0;
    for (uint32_t c0 = 0; c0 < iters * kBigWaves; c0 += 64) {
      const uint32_t c = c0 + lane, x = c < iters * kBigWaves ? slot[c] : 0u;
      const uint32_t incl = wave_incl_scan(x);
      if (c < iters * kBigWaves) slot[c] = run + incl - x;
      run += __shfl(incl, 63);
    }
  }
  __syncthreads();
  // (each thread keeps its own states' ids in NB while the ranks replace the
  // least members' entries of blk[])
  const uint32_t id0 = blk[J.q0];
  for (uint32_t i = 0; i < iters; ++i) {
    const uint32_t q = tid + i * kBigThreads;
    if (q < n) NB[q] = blk[q];
  }
  __syncthreads();
  for (uint32_t i = 0; i < iters; ++i) {
    const uint32_t q = tid + i * kBigThreads;
    const bool lead = q < n && blk[q] == q;  // (only this thread writes blk[q])
    const unsigned long long m = __ballot(lead);
    if (lead) blk[q] = (uint16_t)(slot[i * kBigWaves + wave] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)));
  }
  __syncthreads();
  uint32_t* __restrict__ out = reinterpret_cast<uint32_t*>(J.out);
  for (uint32_t i0 = 0; i0 < iters; i0 += kBigChunk) {
    uint32_t v[kBigChunk];
#pragma unroll
    for (int i = 0; i < kBigChunk; ++i) {
      const uint32_t q = tid + (i0 + i) * kBigThreads;
      v[i] = q < n ? NB[q] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kBigChunk; ++i) {
      const uint32_t q = tid + (i0 + i) * kBigThreads;
      if (q < n) out[q] = blk[v[i]];
    }
  }
  if (tid == 0) {
    R.status = kFusedOk;
    R.num_blocks = count;
    R.initial_block = blk[id0];
    R.refine_rounds = refine;
    R.levels_used = used;
    R.doubling = dbl ? 1u : 0u;
    res[j] = R;
  }
}

}  // namespace

void launch_fused(const FusedJob* jobs, FusedRes* res, uint32_t njobs, int cls, hipStream_t s,
                  const FusedJob* one) {
  if (!njobs) return;
  const FusedJob arg = one ? *one : FusedJob{};
  if (one) {
    jobs = nullptr;
    njobs = 1;
  }
  // Threads per class: as many as the states can use.  512 threads of four
  // states beat 256 of eight (2,000 instances of up to 2,048 states: 380
  // against 404 us a call), 1,024 of eight 512 of sixteen (up to 8,192: 632
  // against 656).  One instance alone takes 1,024 threads from 513 states on
  // (2,000 states, two letters: 43 us a call, with 256 threads 63).
  const dim3 g(njobs);
  switch (cls) {
    case 0: hipLaunchKernelGGL((k_fused<512, 256>), g, dim3(256), 0, s, jobs, res, njobs, arg); break;
    case 1:
      if (one) hipLaunchKernelGGL((k_fused<2048, 1024>), g, dim3(1024), 0, s, jobs, res, njobs, arg);
      else hipLaunchKernelGGL((k_fused<2048, 512>), g, dim3(512), 0, s, jobs, res, njobs, arg);
      break;
    case 2:
      if (one && one->n <= 4096) hipLaunchKernelGGL((k_fused<4096, 1024>), g, dim3(1024), 0, s, jobs, res, njobs, arg);
      else hipLaunchKernelGGL((k_fused<8192, 1024>), g, dim3(1024), 0, s, jobs, res, njobs, arg);
      break;
    default: hipLaunchKernelGGL((k_fused<16384, 1024>), g, dim3(1024), 0, s, jobs, res, njobs, arg); break;
  }
}

void launch_fused_big(const FusedJob* jobs, FusedRes* res, uint32_t njobs, hipStream_t s) {
  if (!njobs) return;
  hipLaunchKernelGGL(k_fused_big, dim3(njobs), dim3(kBigThreads), 0, s, jobs, res, njobs);
}

}  // namespace dfamin
