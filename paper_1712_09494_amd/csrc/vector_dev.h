// Keys that are state vectors of W 64-bit words (W = 2 or 4).  GPUexplore
// keeps each state as a vector of words in its bucketed table (Sec. 3.2,
// Sec. 4.2); the Cuckoo table of Sec. 4.1 moves keys with single-word
// exchanges, which a multi-word key cannot use directly.
//
// Layout.  Every member vector is written once into the table's arena (W
// words per entry, append-only).  Table slots, stash and overflow list hold
// 64-bit handles: the top 30 bits of the vector's hash H and a 34-bit arena
// index.  Bucket and slot positions are functions of those 30 hash bits, so
// a handle carries everything an eviction chain needs and a chain never reads
// the arena.  A handle is never all ones (arena indices stay below 2^34 - 1),
// so the empty marker needs no special key.
//
// Find-or-put, with no kernel reading a vector another lane is still writing
// and no lane waiting for another:
//   1. find or claim, one walk per vector: along its bucket sequence (then
//      stash, then overflow set) or, in a Cuckoo table, the stash and
//      overflow set and then its candidate slots h_1..h_c.  A stored handle
//      with the vector's hash bits is compared with the arena words (equal:
//      present, report 0); an empty slot gets a placeholder -- the hash bits
//      and the batch index -- by compare-and-swap.  Copies of a vector walk
//      the same slots in the same order, so a second copy meets the first
//      one's placeholder and compares the two batch rows (complete before the
//      kernel starts): equal means it reports 0.  No handle is committed and
//      no exchange runs in this kernel, so placeholders stay where they were
//      put.  One atomic per new vector; claims are listed per wave region;
//   2. commit: each claimed slot takes an arena entry (one counter atomic per
//      wave), gets the vector's words written there and its placeholder
//      replaced by the final handle;
// and for Cuckoo tables, the vectors that found every candidate taken:
//   3. evict: deduplicated in the scratch set by batch index (equal vectors
//      compared word by word in the batch); each winner reports 1, takes an
//      arena entry, writes its words and runs the exchange chain of Sec. 4.1
//      from h_1 with its handle (then stash, overflow set);
//   4. scrub the scratch set (the single-word Cuckoo scrub kernel).
// The stash and the overflow list of a vector table are open-addressed sets
// of handles, probed from positions given by the hash bits.
// Lookups stop early by the same rules as the single-word tables: a bucket
// with an empty slot ends the bucket sequence (slots fill as a prefix and are
// never emptied), and a Cuckoo lookup stops at an empty candidate when the
// handle's c slot indices are distinct.
#pragma once
#include "cuckoo_dev.h"

namespace ht {

constexpr uint64_t kArenaMask = (1ull << kArenaBits) - 1;
// Arena indices stay below 2^33; bit 33 of a handle marks a placeholder whose
// low 33 bits are a batch index (find-or-claim kernel, replaced in commit).
constexpr uint64_t kPlaceBit = 1ull << 33;
constexpr uint64_t kBatchMask = kPlaceBit - 1;

// Hash of a vector: the words folded through mix64 in order, seeded per table.
template <int W>
__device__ __forceinline__ uint64_t vec_hash(const uint64_t (&v)[W], uint64_t seed) {
  uint64_t h = mix64(v[0] ^ seed);
#pragma unroll
  for (int j = 1; j < W; ++j) h = mix64(h ^ mix64(v[j] + 0x9e3779b97f4a7c15ull * (uint64_t)j));
  return h;
}

__device__ __forceinline__ uint64_t handle_hb(uint64_t hd) { return hd >> kArenaBits; }
__device__ __forceinline__ uint64_t handle_idx(uint64_t hd) { return hd & kArenaMask; }

// W words from a 16-byte aligned address.
template <int W>
__device__ __forceinline__ void load_vec(const uint64_t* p, uint64_t (&v)[W]) {
#pragma unroll
  for (int j = 0; j < W; j += 2) {
    const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(p + j);
    v[j] = x.x;
    v[j + 1] = x.y;
  }
}

template <int W>
__device__ __forceinline__ bool vec_eq(const uint64_t (&a)[W], const uint64_t (&b)[W]) {
  bool e = true;
#pragma unroll
  for (int j = 0; j < W; ++j) e &= a[j] == b[j];
  return e;
}

// Handle hd holds vector v: hash bits first, then the arena words.  Empty
// slots and placeholders hold no arena entry.
template <int W>
__device__ __forceinline__ bool vec_holds(const DevTable& t, uint64_t hd, uint64_t hb, const uint64_t (&v)[W]) {
  if (hd == kEmpty || (hd & kPlaceBit) || handle_hb(hd) != hb) return false;
  uint64_t a[W];
  load_vec<W>(t.arena + handle_idx(hd) * W, a);
  return vec_eq<W>(a, v);
}

// q-th bucket of the bucket sequence: h_1..h_c, then the walk of consecutive
// buckets after h_c (wrapping at the end of the table), given the (q-1)-th.
__device__ __forceinline__ uint64_t vec_bucket(const DevTable& t, uint64_t hb, uint32_t q, uint64_t prev) {
  if (q < t.nhash) return hidx<false>(t, hb, q);
  return prev + 1 == t.nrange ? 0 : prev + 1;
}

// Masks over eight slots: handles (committed or placeholders) with hash bits
// hb, and empty slots.  Taken without a branch, so that the lanes of a wave
// meet at their compare-and-swaps instead of waiting for one another slot
// after slot (2^20 vectors of four words a call into 8-slot buckets: 83 -> 74
// us, queries of 2^20 64 -> 46; 64-slot buckets 148 -> 121 and 122 -> 95).
__device__ __forceinline__ uint32_t vec_eight(const uint64_t (&x)[8], uint64_t hb, uint32_t& empty) {
  uint32_t same = 0;
  empty = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const bool e = x[q] == kEmpty;
    empty |= (e ? 1u : 0u) << q;
    same |= (!e && handle_hb(x[q]) == hb ? 1u : 0u) << q;
  }
  return same;
}

template <int W>
__device__ bool vec_lookup_bucketed(const DevTable& t, uint64_t hb, const uint64_t (&v)[W]) {
  const uint32_t B = t.bucket_slots;
  const uint32_t steps = t.nhash + t.walk;
  uint64_t b = 0;
  for (uint32_t q = 0; q < steps; ++q) {
    b = vec_bucket(t, hb, q, b);
    const uint64_t* bk = t.slots + b * B;
    for (uint32_t c0 = 0; c0 < B; c0 += 8) {
      uint64_t x[8];
      load8(bk + c0, x);
      uint32_t em;
      for (uint32_t m = vec_eight(x, hb, em); m; m &= m - 1)
        if (vec_holds<W>(t, bk[c0 + __builtin_ctz(m)], hb, v)) return true;
      if (em) return false;                     // prefix: the rest of the sequence is unused
    }
  }
  return false;
}

template <int W>
__device__ bool vec_lookup_cuckoo(const DevTable& t, uint64_t hb, const uint64_t (&v)[W]) {
  const bool dist = hashes_distinct<false>(t, hb);
  for (uint32_t j = 0; j < t.nhash; ++j) {
    const uint64_t hd = t.slots[hidx<false>(t, hb, j)];
    if (hd == kEmpty) {
      if (dist) return false;
      continue;
    }
    if (vec_holds<W>(t, hd, hb, v)) return true;
  }
  return false;
}

// Start of the overflow set's probe sequence (linear probing, any length).
__device__ __forceinline__ uint32_t overflow_start(const DevTable& t, uint64_t hb) {
  return (uint32_t)mulhi64(mix64(hb ^ t.stash_seed ^ 0x5851f42d4c957f2dull), t.overflow_slots);
}

// Stash and overflow set: probe from the hash bits' position until an empty slot.
template <int W>
__device__ bool vec_stash_query(const DevTable& t, uint64_t hb, const uint64_t (&v)[W], uint32_t sc,
                                uint32_t oc) {
  if (sc) {
    const uint32_t S = t.stash_slots;
    uint32_t p = stash_start(t, hb);
    for (uint32_t i = 0; i < S; ++i) {
      const uint64_t hd = t.stash[p];
      if (hd == kEmpty) break;
      if (vec_holds<W>(t, hd, hb, v)) return true;
      p = (p + 1) & (S - 1);
    }
  }
  if (oc) {
    const uint32_t m = t.overflow_slots;
    uint32_t p = overflow_start(t, hb);
    for (uint32_t i = 0; i < m; ++i) {
      const uint64_t hd = t.overflow[p];
      if (hd == kEmpty) break;
      if (vec_holds<W>(t, hd, hb, v)) return true;
      p = p + 1 == m ? 0 : p + 1;
    }
  }
  return false;
}

template <int W>
__device__ __forceinline__ bool vec_find(const DevTable& t, uint64_t hb, const uint64_t (&v)[W], uint32_t sc,
                                         uint32_t oc) {
  const bool f = t.kind == HT_KIND_BUCKETED ? vec_lookup_bucketed<W>(t, hb, v) : vec_lookup_cuckoo<W>(t, hb, v);
  return f || ((sc | oc) && vec_stash_query<W>(t, hb, v, sc, oc));
}

// Place a handle of a vector known to be absent (no comparison needed).
__device__ inline void vec_stash_put(const DevTable& t, uint64_t hd) {
  const uint32_t S = t.stash_slots;
  uint32_t p = stash_start(t, handle_hb(hd));
  for (uint32_t i = 0; i < S; ++i) {
    if (cas64(&t.stash[p], kEmpty, hd) == kEmpty) {
      add_agent(&t.ctr->stash_count, 1u);
      return;
    }
    p = (p + 1) & (S - 1);
  }
  const uint32_t m = t.overflow_slots;
  p = overflow_start(t, handle_hb(hd));
  for (uint32_t i = 0; i < m; ++i) {
    if (cas64(&t.overflow[p], kEmpty, hd) == kEmpty) {
      add_agent(&t.ctr->overflow_count, 1u);
      return;
    }
    p = p + 1 == m ? 0 : p + 1;
  }
  add_agent(&t.ctr->lost, 1u);
}

// The exchange chain of Sec. 4.1 from h_1 with handle x, whose vector is absent
// and has every candidate taken.
__device__ __forceinline__ void vec_chain(const DevTable& t, uint64_t x, unsigned long long& nevict) {
  uint64_t slot = hidx<false>(t, handle_hb(x), 0);
  for (uint32_t step = 0;; ++step) {
    const uint64_t old = exch64(&t.slots[slot], x);
    if (old == kEmpty) return;
    x = old;
    ++nevict;
    if (step + 1 >= t.max_chain || !cuckoo_next<false>(t, t.nhash, handle_hb(x), slot)) break;
  }
  vec_stash_put(t, x);
}

// Arena entries for the U wants of each lane: one counter atomic per call and
// range.  A wave starts at its own range and moves on while a range is full,
// so every entry of every range is handed out.  ~0 when all are taken.
template <int U>
__device__ __forceinline__ void arena_take(const DevTable& t, bool (&want)[U], uint64_t wave, uint64_t (&idx)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) idx[u] = ~0ull;
  for (uint32_t a = 0; a < (uint32_t)kSpread; ++a) {
    uint64_t rank[U], total = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t wm = ballot(want[u]);
      rank[u] = total + lanes_below(wm);
      total += (uint64_t)__popcll(wm);
    }
    if (!total) break;
    const uint32_t rg = (uint32_t)((wave + a) % kSpread);
    unsigned long long first = 0;
    if (lane_id() == 0) first = add_agent(&t.ctr->arena_next[rg * kLineWords], (unsigned long long)total);
    first = shfl64(first, 0);
    const uint64_t avail = first < t.arena_cap ? t.arena_cap - first : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (want[u] && rank[u] < avail) {
        idx[u] = (uint64_t)rg * t.arena_cap + first + rank[u];
        want[u] = false;
      }
    }
  }
}

// List entry of a vector whose Cuckoo candidates were all taken at claim
// time: it goes to the evict kernel.
constexpr uint64_t kLeftover = ~1ull;

struct EvictLds {
  uint32_t list[kBlock / kWave][2 * kWave];   // a wave's gathered leftovers
};

// Kernel 3 (Cuckoo): the leftover vectors are deduplicated in the scratch
// set by batch index (equal vectors compared word by word in the batch);
// each winner reports 1, takes an arena entry, writes its words and runs the
// exchange chain of Sec. 4.1 from h_1 with its handle.  Every list entry's
// meta word becomes its scratch-set slot (or ~0) for the scrub kernel.
// The time is that of the chains, one dependent exchange after another, so a
// wave first gathers its leftovers from among the claims of its list and runs
// up to 64 of them at once (calls of 2^20 vectors up to load 0.7, two and four
// words: 51.6 and 55.4 us a call in list order, 44.0 and 43.6 so).
template <int W>
__global__ __launch_bounds__(kBlock) HT_EIGHT_WAVES
void vec_evict_kernel(DevTable t, const uint64_t* __restrict__ keys, uint64_t n, uint8_t* __restrict__ out,
                      CuckooScratch s) {
  const uint64_t wave = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  const int lane = lane_id();
  const uint64_t begin = wave * s.per_wave;
  const uint32_t cnt = begin < n ? s.wcnt[wave] : 0u;
  unsigned long long nnew = 0, nevict = 0;
  __shared__ EvictLds gathered;
  uint32_t* list = gathered.list[threadIdx.x / kWave];
  uint32_t e0 = 0, have = 0;
  for (;;) {
    while (have < (uint32_t)kWave && e0 < cnt) {
      const uint32_t e = e0 + (uint32_t)lane;
      const bool left = e < cnt && s.wkey[begin + e] == kLeftover;
      if (e < cnt && !left) s.wmeta[begin + e] = ~0ull;
      const uint64_t mm = ballot(left);
      if (left) list[have + lanes_below(mm)] = e;
      have += (uint32_t)__popcll(mm);
      e0 += kWave;
    }
    if (!have) break;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's own list
    const uint32_t take = have < (uint32_t)kWave ? have : (uint32_t)kWave;
    have -= take;
    bool winner = false;
    uint64_t hb = 0;
    uint64_t v[W];
#pragma unroll
    for (int j = 0; j < W; ++j) v[j] = 0;
    if ((uint32_t)lane < take) {
      const uint32_t e = list[have + lane];
      const uint64_t m = s.wmeta[begin + e];
      const uint64_t i = m & kBatchMask;
      hb = m >> 33;
      load_vec<W>(keys + i * W, v);
      uint64_t p = mix64(hb ^ s.dset_seed) & s.dset_mask;
      for (;;) {
        const uint64_t old = cas64(&s.dset[p], kEmpty, i);
        if (old == kEmpty) {
          winner = true;
          break;
        }
        if (old < n) {                   // the set holds indices of this batch only
          uint64_t u[W];
          load_vec<W>(keys + old * W, u);
          if (vec_eq<W>(u, v)) break;    // an equal vector of the batch won
        }
        p = (p + 1) & s.dset_mask;
      }
      if (out) out[i] = winner ? 1 : 0;
      s.wmeta[begin + e] = winner ? p : ~0ull;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (!ballot(winner)) continue;
    bool want[1] = {winner};
    uint64_t took[1];
    arena_take<1>(t, want, wave, took);
    const uint64_t idx = took[0];
    if (winner) {
      ++nnew;
      if (idx == ~0ull) {
        add_agent(&t.ctr->lost, 1u);     // only after more members than slots + stash + overflow
      } else {
#pragma unroll
        for (int j = 0; j < W; j += 2)
          *reinterpret_cast<ulonglong2*>(t.arena + idx * W + j) = make_ulonglong2(v[j], v[j + 1]);
        vec_chain(t, (hb << kArenaBits) | idx, nevict);
      }
    }
  }
  wave_count(t.ctr->size, nnew, (uint32_t)wave);
  wave_count(t.ctr->evictions, nevict, (uint32_t)wave);
}

// The lane that claims for this lane's vector: itself, or a lane of the wave
// with an equal vector (see wave_meet).
template <int W>
__device__ __forceinline__ uint32_t vec_meet(uint32_t* places, uint64_t hb, const uint64_t (&v)[W]) {
  const Meeting with = wave_meet(places, (uint32_t)hb);
  bool equal = with.maybe;
  if (ballot(equal)) {
#pragma unroll
    for (int j = 0; j < W; ++j) equal &= shfl64(v[j], with.lead) == v[j];
  }
  return equal ? with.lead : (uint32_t)lane_id();
}

// One slot of a claim walk, given the value read there: 1 = the placeholder
// is now here, 2 = an equal vector of the batch holds this slot, 0 = go on.
template <int W>
__device__ __forceinline__ int vec_claim_seen(uint64_t* p, uint64_t hd, uint64_t ph, uint64_t hb,
                                              const uint64_t (&v)[W], const uint64_t* __restrict__ keys,
                                              uint64_t n) {
  if (hd == kEmpty) {
    hd = cas64(p, kEmpty, ph);
    if (hd == kEmpty) return 1;
  }
  if ((hd & kPlaceBit) && hd != kEmpty && handle_hb(hd) == hb) {
    const uint64_t j = hd & kBatchMask;
    if (j < n) {
      uint64_t u[W];
      load_vec<W>(keys + j * W, u);
      if (vec_eq<W>(u, v)) return 2;
    }
  }
  return 0;
}

// One slot of a walk that only looks up: 3 = a member stored by an earlier call
// (a committed handle) holds the vector, 2 = an equal vector of the batch does,
// 0 = go on.
template <int W>
__device__ __forceinline__ int vec_find_seen(const DevTable& t, uint64_t hd, uint64_t hb, const uint64_t (&v)[W],
                                             const uint64_t* __restrict__ keys, uint64_t n) {
  const bool place = (hd & kPlaceBit) != 0;
  if (hd == kEmpty || handle_hb(hd) != hb || (place && (hd & kBatchMask) >= n)) return 0;
  uint64_t u[W];
  load_vec<W>(place ? keys + (hd & kBatchMask) * W : t.arena + handle_idx(hd) * W, u);
  return !vec_eq<W>(u, v) ? 0 : place ? 2 : 3;
}

// One slot of a walk that both looks up and claims: the answers of the two
// above.  No handle is committed while this runs (the commit kernel comes
// after), so a failed compare-and-swap only ever returns a placeholder.
template <int W>
__device__ __forceinline__ int vec_find_or_claim_seen(const DevTable& t, uint64_t* p, uint64_t hd, uint64_t ph,
                                                      uint64_t hb, const uint64_t (&v)[W],
                                                      const uint64_t* __restrict__ keys, uint64_t n) {
  if (hd != kEmpty && !(hd & kPlaceBit)) return vec_holds<W>(t, hd, hb, v) ? 3 : 0;
  return vec_claim_seen<W>(p, hd, ph, hb, v, keys, n);
}

// Kernel 1: lookup and claim in one walk.  Bucketed: slots
// fill as a prefix of each vector's bucket sequence, then the stash, then
// the overflow set, and none is ever emptied, so the walk meets a stored copy
// of the vector before the first empty slot it could claim.  Cuckoo: the
// stash and overflow set are looked up first (a chain that ends there can
// leave the vector's other candidates empty); then the candidates h_1..h_c
// in order, a stored copy never lying past an empty candidate when the c
// indices are distinct (else all c are looked up before any claim); a vector
// with every candidate taken is left for the evict kernel.  Either way one
// walk per vector answers "present" or claims a free location, and copies
// within the batch meet at one placeholder.  Claimed locations (and Cuckoo
// leftovers, as kLeftover) are listed per wave region as (location, hash
// bits << 33 | batch index) for the commit and evict kernels.
template <int W>
__global__ __launch_bounds__(kBlock, 8) HT_EIGHT_WAVES
void vec_find_or_claim_kernel(DevTable t, const uint64_t* __restrict__ keys, uint64_t n, uint8_t* __restrict__ out,
                              CuckooScratch s) {
  const uint64_t wave = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  const int lane = lane_id();
  const uint64_t begin = wave * s.per_wave;
  uint64_t end = begin + s.per_wave;
  if (end > n) end = n;
  const uint32_t B = t.bucket_slots;
  const uint32_t steps = t.nhash + t.walk;
  const uint64_t nslots = t.nrange * B;
  const uint32_t sc = t.ctr->stash_count;
  const uint32_t oc = t.ctr->overflow_count;
  __shared__ MeetLds places;
  uint32_t* const meet = places.wave[threadIdx.x / kWave];
  uint32_t nlist = 0;
  unsigned long long nnew = 0;
  for (uint64_t base = begin; base < end; base += kWave) {
    const uint64_t i = base + lane;
    bool claimed = false, leftover = false;
    uint64_t loc = ~0ull, hb = 0;
    if (i < end && t.kind == HT_KIND_CUCKOO) {
      uint64_t v[W];
      load_vec<W>(keys + i * W, v);
      hb = vec_hash<W>(v, t.vseed) >> kArenaBits;
      const uint64_t ph = (hb << kArenaBits) | kPlaceBit | i;
      int st = (sc | oc) && vec_stash_query<W>(t, hb, v, sc, oc) ? 3 : 0;
      if (!st && !hashes_distinct<false>(t, hb)) {
        for (uint32_t j = 0; j < t.nhash && !st; ++j) {
          const uint64_t hd = t.slots[hidx<false>(t, hb, j)];
          if (hd != kEmpty && !(hd & kPlaceBit) && vec_holds<W>(t, hd, hb, v)) st = 3;
        }
      }
      for (uint32_t j = 0; j < t.nhash && !st; ++j) {
        const uint64_t sl = hidx<false>(t, hb, j);
        const uint64_t hd = t.slots[sl];
        if (hd != kEmpty) {
          st = vec_find_seen<W>(t, hd, hb, v, keys, n);
          continue;
        }
        const uint32_t lead = vec_meet<W>(meet, hb, v);
        const bool copy = lead != (uint32_t)lane;
        if (!copy) st = vec_claim_seen<W>(t.slots + sl, kEmpty, ph, hb, v, keys, n);
        if (st == 1) loc = sl;
        const uint32_t led = shfl32((uint32_t)st, lead);
        if (copy && led) st = 2;
      }
      claimed = st == 1;
      leftover = st == 0;                        // every candidate taken: the evict kernel decides
      nnew += claimed ? 1u : 0u;
      if (out && !leftover) out[i] = claimed ? 1 : 0;
    } else if (i < end) {
      uint64_t v[W];
      load_vec<W>(keys + i * W, v);
      hb = vec_hash<W>(v, t.vseed) >> kArenaBits;
      const uint64_t ph = (hb << kArenaBits) | kPlaceBit | i;
      int st = 0;
      uint64_t b = 0;
      for (uint32_t q = 0; q < steps && !st; ++q) {
        b = vec_bucket(t, hb, q, b);
        for (uint32_t c0 = 0; c0 < B && !st; c0 += 8) {
          // stored handles with the same hash bits first (they lie before the
          // first empty slot), then the empty slots from the lowest on: every
          // lane at its own first empty slot together, one lane for the equal
          // vectors of the wave
          uint64_t* bk = t.slots + b * B + c0;
          uint64_t x[8];
          load8(bk, x);
          uint32_t em;
          for (uint32_t m = vec_eight(x, hb, em); m && !st; m &= m - 1) {
            const uint32_t k = (uint32_t)__builtin_ctz(m);
            st = vec_find_seen<W>(t, bk[k], hb, v, keys, n);   // read again: the mask alone is kept
          }
          if (em && !st) {
            const uint32_t lead = vec_meet<W>(meet, hb, v);
            const bool copy = lead != (uint32_t)lane;
            for (; em && !st && !copy; em &= em - 1) {
              const uint32_t k = (uint32_t)__builtin_ctz(em);
              st = vec_claim_seen<W>(bk + k, kEmpty, ph, hb, v, keys, n);
              if (st == 1) loc = b * B + c0 + k;
            }
            const uint32_t led = shfl32((uint32_t)st, lead);
            if (copy && led) st = 2;
          }
        }
      }
      if (!st) {
        const uint32_t S = t.stash_slots;
        uint32_t p = stash_start(t, hb);
        for (uint32_t k = 0; k < S && !st; ++k) {
          st = vec_find_or_claim_seen<W>(t, t.stash + p, t.stash[p], ph, hb, v, keys, n);
          if (st == 1) {
            loc = nslots + p;
            add_agent(&t.ctr->stash_count, 1u);
          }
          p = (p + 1) & (S - 1);
        }
      }
      if (!st) {
        const uint32_t m = t.overflow_slots;
        uint32_t p = overflow_start(t, hb);
        for (uint32_t k = 0; k < m && !st; ++k) {
          st = vec_find_or_claim_seen<W>(t, t.overflow + p, t.overflow[p], ph, hb, v, keys, n);
          if (st == 1) {
            loc = nslots + t.stash_slots + p;
            add_agent(&t.ctr->overflow_count, 1u);
          }
          p = p + 1 == m ? 0 : p + 1;
        }
      }
      if (!st) add_agent(&t.ctr->lost, 1u);
      claimed = st == 1;
      nnew += claimed ? 1u : 0u;
      if (out) out[i] = claimed ? 1 : 0;
    }
    const bool listed = claimed || leftover;
    const uint64_t mm = ballot(listed);
    if (listed) {
      const uint64_t slot = begin + nlist + lanes_below(mm);
      s.wkey[slot] = claimed ? loc : kLeftover;
      s.wmeta[slot] = (hb << 33) | i;
    }
    nlist += (uint32_t)__popcll(mm);
  }
  if (lane == 0 && begin < n) s.wcnt[wave] = nlist;
  wave_count(t.ctr->size, nnew, (uint32_t)wave);
}

__device__ __forceinline__ uint64_t* vec_location(const DevTable& t, uint64_t loc) {
  const uint64_t nslots = t.nrange * t.bucket_slots;
  if (loc < nslots) return t.slots + loc;
  loc -= nslots;
  if (loc < t.stash_slots) return t.stash + loc;
  return t.overflow + (loc - t.stash_slots);
}

// Kernel 2: the claimed slots get arena entries, the vectors' words and
// their final handles.  A wave takes up to three turns of its list together,
// list entries and batch rows loaded before the one arena atomic: turn by
// turn each waited for three dependent round trips (2^20 vectors a call, two
// and four words: 26.3 and 33.2 us a call turn by turn, 23.9 and 27.5 so).
template <int W>
__global__ __launch_bounds__(kBlock) void vec_commit_kernel(DevTable t, const uint64_t* __restrict__ keys, uint64_t n,
                                                             CuckooScratch s) {
  constexpr int U = 3;
  const uint64_t wave = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  const uint64_t begin = wave * s.per_wave;
  const uint32_t cnt = begin < n ? s.wcnt[wave] : 0u;
  for (uint32_t e0 = 0; e0 < cnt; e0 += U * kWave) {
    uint64_t loc[U], m[U], v[U][W], idx[U];
    bool have[U], want[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = e0 + u * kWave + (uint32_t)lane_id();
      loc[u] = e < cnt ? s.wkey[begin + e] : kLeftover;
      m[u] = e < cnt ? s.wmeta[begin + e] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      have[u] = want[u] = loc[u] < kLeftover;    // a location: neither that nor ~0
      if (have[u]) load_vec<W>(keys + (m[u] & kBatchMask) * W, v[u]);
    }
    arena_take<U>(t, want, wave, idx);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!have[u]) continue;
      if (idx[u] == ~0ull) {
        add_agent(&t.ctr->lost, 1u);             // cannot happen: every claimed location has an entry
        continue;
      }
#pragma unroll
      for (int j = 0; j < W; j += 2)
        *reinterpret_cast<ulonglong2*>(t.arena + idx[u] * W + j) = make_ulonglong2(v[u][j], v[u][j + 1]);
      store_coherent(vec_location(t, loc[u]), ((m[u] >> 33) << kArenaBits) | idx[u]);
    }
  }
}

template <int W>
__global__ __launch_bounds__(kBlock) HT_EIGHT_WAVES
void vec_query_kernel(DevTable t, const uint64_t* __restrict__ keys, uint64_t n, uint8_t* __restrict__ out) {
  const uint32_t sc = t.ctr->stash_count;
  const uint32_t oc = t.ctr->overflow_count;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
    uint64_t v[W];
    load_vec<W>(keys + i * W, v);
    const uint64_t H = vec_hash<W>(v, t.vseed);
    out[i] = vec_find<W>(t, H >> kArenaBits, v, sc, oc) ? 1 : 0;
  }
}

// Members: the arena entries named by the handles in `handles[0, nh)`.
template <int W>
__global__ __launch_bounds__(kBlock) void vec_dump_kernel(const uint64_t* __restrict__ handles, uint64_t nh,
                                                           const uint64_t* __restrict__ arena,
                                                           uint64_t* __restrict__ dst, uint64_t cap,
                                                           unsigned long long* count) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  const int lane = lane_id();
  for (uint64_t base = (uint64_t)blockIdx.x * kBlock + (threadIdx.x & ~63u); base < nh; base += stride) {
    const uint64_t i = base + lane;
    const uint64_t hd = i < nh ? handles[i] : kEmpty;
    const bool keep = hd != kEmpty && !(hd & kPlaceBit);
    const uint64_t m = ballot(keep);
    if (!m) continue;
    unsigned long long b = 0;
    if (lane == 0) b = add_agent(count, (unsigned long long)__popcll(m));
    b = shfl64(b, 0);
    if (keep) {
      const uint64_t pos = b + lanes_below(m);
      if (pos < cap) {
#pragma unroll
        for (int j = 0; j < W; ++j) dst[pos * W + j] = arena[handle_idx(hd) * W + j];
      }
    }
  }
}

}  // namespace ht
