// Tiled find-or-put: a batch that is large against its table is sorted by
// table region first, and each region is then worked on in LDS.
//
// A lane that find-or-puts its key straight into the table pays a random
// line read (54 G/s on this chip, 80 G/s within 16 MB) and, for a new key, a
// memory-side compare-and-swap (21-27 G/s), however often the batch comes
// back to the same line.  When the batch has a key for every line or two of
// the table it is cheaper to stream the table once:
//   1. partition: a block takes a chunk of C consecutive keys and sorts them
//      by the tile of h_1's bucket (a tile is a run of whole buckets that fits
//      in LDS); the sorted chunk, each key's place in the chunk and the start
//      of each tile's run are stored;
//   2. tile: a block loads one tile into LDS, inserts the keys of every
//      chunk's run for it with LDS compare-and-swaps, stores a flag per key
//      beside the sorted keys and writes the tile back;
//   3. finish: a block puts one chunk's flags back into batch order; the keys
//      whose bucket was full go on from h_2 in the table itself, with the
//      ordinary compare-and-swap probe.
// Placement is that of the direct kernels (the lowest empty slot of the first
// bucket of the probe sequence that is not full): all copies of a key are in
// one tile and meet at one slot, and a bucket seen full stays full, so exactly
// one copy reports new and the lookups' early exits hold.  No other call may
// work on the table at the same time (the tile is written back with plain
// stores).
// The same passes for Cuckoo tables (h_1 in LDS, the rest and the eviction
// chains as before) were no faster: 2^20 keys into 2^21 slots 84 against 87
// us, slower at every smaller size and above 2^23 keys, since most of the
// keys' lines are those of h_2 and the chains.
#pragma once
#include "bucketed_dev.h"
#include "tile.h"

namespace ht {

constexpr uint32_t kTileBlock = 1024;       // threads of the tile kernels
constexpr uint32_t kTileMore = 0xff;        // flag of a key that goes on at h_2
constexpr uint32_t kTileCopy = 0xfe;        // flag of a copy left out by the partition

// First slot of key k's h_1 bucket.
__device__ __forceinline__ uint64_t tile_home(const DevTable& t, uint64_t k) {
  return hidx<false>(t, k, 0) * t.bucket_slots;
}

// ---- partition ---------------------------------------------------------------

template <uint32_t C>
struct TilePartLds {
  uint64_t key[C];
  uint16_t idx[C];
  uint32_t hist[kTileMax];
  uint32_t wsum[kTileBlock / kWave];
  uint32_t crowded;         // a run far longer than keys without copies make
  uint32_t ncopy;
};

// Sort chunk `c` of the job's batch by tile.  COPIES: leave copies out (see
// tile_partition_chunk).  Without it the answer is false, and nothing is
// stored, when a run is too long.
template <uint32_t C, bool COPIES>
__device__ __forceinline__ bool tile_sort_chunk(const TileJob& j, uint32_t c, TilePartLds<C>& l) {
  constexpr uint32_t PER = C / kTileBlock;
  const uint32_t tid = threadIdx.x;
  const uint64_t base = (uint64_t)c * C;
  const uint32_t m = j.n - base < C ? (uint32_t)(j.n - base) : C;
  uint64_t k[PER];
#pragma unroll
  for (uint32_t r = 0; r < PER; ++r) {
    const uint32_t i = r * kTileBlock + tid;
    k[r] = i < m ? j.keys[base + i] : 0;
  }
  for (uint32_t i = tid; i < j.tiles; i += kTileBlock) l.hist[i] = 0;
  if (tid == 0) l.crowded = l.ncopy = 0;
  uint32_t rank[PER];                        // place in its run; of a copy the place of the key it copies
  uint32_t copies = 0;                       // bit r: key r is a copy
  if constexpr (COPIES) {
    // l.key: the chunk in its order, l.idx: the words that keys share by hash
    uint32_t word[PER];
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r) {
      const uint32_t i = r * kTileBlock + tid;
      word[r] = (uint32_t)mix64(k[r] ^ (j.t.stash_seed + c)) & (C - 1);
      if (i < m) {
        l.key[i] = k[r];
        l.idx[word[r]] = (uint16_t)i;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r) {
      const uint32_t i = r * kTileBlock + tid;
      rank[r] = i < m ? l.idx[word[r]] : i;
      if (rank[r] != i && l.key[rank[r]] == k[r]) copies |= 1u << r;
    }
  }
  __syncthreads();
  uint32_t tl[PER];
#pragma unroll
  for (uint32_t r = 0; r < PER; ++r) {
    tl[r] = (uint32_t)(tile_home(j.t, k[r]) >> j.shift);
    if (!COPIES) rank[r] = 0;
    if (r * kTileBlock + tid < m && !(COPIES && copies >> r & 1u))
      rank[r] = __hip_atomic_fetch_add(&l.hist[tl[r]], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  // exclusive scan of the counts: consecutive counters per thread, then over
  // the wave and the block
  const uint32_t per = (j.tiles + kTileBlock - 1) / kTileBlock;
  const uint32_t a = tid * per < j.tiles ? tid * per : j.tiles;
  const uint32_t z = a + per < j.tiles ? a + per : j.tiles;
  uint32_t mine = 0, most = 0;
  for (uint32_t i = a; i < z; ++i) {
    const uint32_t v = l.hist[i];
    mine += v;
    most = v > most ? v : most;
  }
  const uint32_t incl = wave_inclusive32(mine);
  if (lane_id() == kWave - 1) l.wsum[tid / kWave] = incl;
  if (!COPIES && most > j.run_most) l.crowded = 1;
  __syncthreads();
  if (!COPIES && l.crowded) return false;
  uint32_t run = incl - mine, total = m;     // total: keys in runs
  for (uint32_t w = 0; w < tid / kWave; ++w) run += l.wsum[w];
  if constexpr (COPIES) {
    total = 0;
    for (uint32_t w = 0; w < kTileBlock / kWave; ++w) total += l.wsum[w];
  }
  uint16_t* off = j.off + (uint64_t)c * (j.tiles + 1);
  for (uint32_t i = a; i < z; ++i) {
    const uint32_t v = l.hist[i];
    l.hist[i] = run;
    off[i] = (uint16_t)run;
    run += v;
  }
  if (tid == 0) off[j.tiles] = (uint16_t)total;
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < PER; ++r) {
    const uint32_t i = r * kTileBlock + tid;
    if (i < m) {
      uint32_t p = l.hist[tl[r]] + rank[r];
      uint64_t key = k[r];
      if (COPIES && copies >> r & 1u) {
        p = total + __hip_atomic_fetch_add(&l.ncopy, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        key = rank[r];
      }
      l.key[p] = key;
      l.idx[p] = (uint16_t)i;
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < PER; ++r) {
    const uint32_t i = r * kTileBlock + tid;
    if (i < m) {
      j.skey[base + i] = l.key[i];
      j.sidx[base + i] = l.idx[i];
      if (COPIES && i >= total) j.sflag[base + i] = (uint8_t)kTileCopy;
    }
  }
  return true;
}

// A run far longer than its share comes from copies of a few keys, and would
// make one block of the tile pass the time of the whole call: such a chunk is
// sorted without its copies.  Each key writes its place in the chunk to an LDS
// word that is its by hash, and the keys that read another place with their
// own key there are copies: they go behind the runs, with the place of the key
// they copy, and the finish pass gives them its answer (copies of one key, 16
// bytes of table each: 2^20 in 731 us with every copy in its run and 33 so,
// 2^24 in 16.7 and 0.36 ms).
template <uint32_t C>
__device__ __forceinline__ void tile_partition_chunk(const TileJob& j, uint32_t c, TilePartLds<C>& l) {
  if (tile_sort_chunk<C, false>(j, c, l)) return;
  __syncthreads();
  tile_sort_chunk<C, true>(j, c, l);
}

// ---- tile ---------------------------------------------------------------------

__device__ __forceinline__ uint64_t lds_cas(uint64_t* p, uint64_t want, uint64_t v) {
  __hip_atomic_compare_exchange_strong(p, &want, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
  return want;
}

// Find-or-put of key k in the B slots at `bk` in LDS: 1 placed, 0 present,
// kTileMore when they are full of other keys.  The tile pass is bound by the
// instructions and turns of this loop where a batch fills its table (keys of
// one bucket meet and retry: 9 of the 19 us for 2^20 keys into 2^21 slots of
// 8-slot buckets).  Tried in its place: all 8 slots read before any
// compare-and-swap, 15 us; one-byte tags, eight to a word that is
// compare-and-swapped, 10 us (13 against 16 us at B = 16); four-bit tags, 15 us; slot pairs
// rotated by bucket against bank conflicts, no change.
__device__ __forceinline__ uint32_t lds_bucket_put(uint64_t* bk, uint32_t B, uint64_t k) {
  for (uint32_t q = 0; q < B; q += 2) {
    const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(bk + q);
    uint64_t v = x.x;
    if (v == kEmpty) v = lds_cas(bk + q, kEmpty, k);
    if (v == kEmpty) return 1;
    if (v == k) return 0;
    v = x.y;
    if (v == kEmpty) v = lds_cas(bk + q + 1, kEmpty, k);
    if (v == kEmpty) return 1;
    if (v == k) return 0;
  }
  return kTileMore;
}

struct TileLds {
  uint64_t slot[kTileSlots];
  uint32_t nnew;            // new keys of the block
};

// A tile's slots between the table and LDS (buckets are multiples of 8 slots).
__device__ __forceinline__ void tile_load(uint64_t* lds, const uint64_t* slots, uint32_t ns) {
  for (uint32_t i = threadIdx.x; i < ns / 2; i += kTileBlock)
    reinterpret_cast<ulonglong2*>(lds)[i] = reinterpret_cast<const ulonglong2*>(slots)[i];
}

__device__ __forceinline__ void tile_store(const uint64_t* lds, uint64_t* slots, uint32_t ns) {
  for (uint32_t i = threadIdx.x; i < ns / 2; i += kTileBlock)
    reinterpret_cast<ulonglong2*>(slots)[i] = reinterpret_cast<const ulonglong2*>(lds)[i];
}

// Insert every key of tile `tl` in LDS.  A group of run_lanes lanes serves a
// chunk's run; U runs per group are in flight together, and the first runs'
// bounds and keys are loaded with the tile.
template <uint32_t C>
__device__ __forceinline__ void tile_insert_keys(const TileJob& j, uint32_t tl, TileLds& l) {
  constexpr uint32_t U = 4;
  const uint32_t tid = threadIdx.x;
  const uint64_t first = (uint64_t)tl << j.shift;
  const uint64_t nslots = j.t.nrange * j.t.bucket_slots;
  const uint64_t left = nslots - first;
  const uint32_t ns = left < (1ull << j.shift) ? (uint32_t)left : 1u << j.shift;
  const uint32_t G = j.run_lanes;
  const uint32_t gl = tid & (G - 1);
  const uint32_t groups = kTileBlock / G;
  uint32_t e[U], z[U];
  uint64_t k[U];
  const auto bounds = [&](uint32_t c0) {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t c = c0 + u * groups;
      e[u] = z[u] = 0;
      if (c < j.chunks) {
        const uint16_t* off = j.off + (uint64_t)c * (j.tiles + 1) + tl;
        e[u] = off[0] + gl;
        z[u] = off[1];
      }
    }
  };
  const auto keys = [&](uint32_t c0) {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      k[u] = e[u] < z[u] ? j.skey[(uint64_t)(c0 + u * groups) * C + e[u]] : 0;
  };
  uint32_t c0 = tid / G;
  bounds(c0);
  if (tid == 0) l.nnew = 0;
  tile_load(l.slot, j.t.slots + first, ns);
  keys(c0);
  __syncthreads();
  uint32_t nnew = 0;
  for (;;) {
    bool more = false;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      if (e[u] < z[u]) {
        const uint32_t r = k[u] == kEmpty
                               ? sentinel_put(j.t)
                               : lds_bucket_put(l.slot + (tile_home(j.t, k[u]) - first), j.t.bucket_slots, k[u]);
        nnew += r == 1;
        j.sflag[(uint64_t)(c0 + u * groups) * C + e[u]] = (uint8_t)r;
        e[u] += G;
        more |= e[u] < z[u];
      }
    }
    if (!more) {
      c0 += U * groups;
      if (c0 >= j.chunks) break;
      bounds(c0);
    }
    keys(c0);
  }
  block_count(j.t.ctr->size, nnew, &l.nnew, tl);
  if (l.nnew) tile_store(l.slot, j.t.slots + first, ns);
}

// Tile of a block of the tile pass: consecutive tiles share lines of the run
// starts and of the sorted keys, so each XCD (blocks are dealt to the eight in
// turn) takes a contiguous share of them.
__device__ __forceinline__ uint32_t tile_of_block(uint32_t b, uint32_t tiles) {
  return (b & 7) * ((tiles + 7) / 8) + (b >> 3);
}

// ---- finish -------------------------------------------------------------------

template <uint32_t C>
struct TileFinishLds {
  uint64_t mkey[C];         // keys that go on at h_2
  uint16_t midx[C];         // and their places in the chunk
  uint8_t flag[C];
  uint32_t meet[kTileBlock / kWave][kMeetPlaces];
  uint32_t nmore;
  uint32_t nnew;
  uint32_t ncopy;
};

// Finish chunk `c`: flags back into batch order, and the rest of the keys
// marked kTileMore.
template <uint32_t C>
__device__ __forceinline__ void tile_finish_chunk(const TileJob& j, uint32_t c, TileFinishLds<C>& l) {
  constexpr uint32_t PER = C / kTileBlock;
  const uint32_t tid = threadIdx.x;
  const uint64_t base = (uint64_t)c * C;
  const uint32_t m = j.n - base < C ? (uint32_t)(j.n - base) : C;
  uint32_t f[PER], x[PER];
  uint64_t k[PER];
#pragma unroll
  for (uint32_t r = 0; r < PER; ++r) {
    const uint32_t i = r * kTileBlock + tid;
    f[r] = i < m ? j.sflag[base + i] : 0u;
    x[r] = i < m ? j.sidx[base + i] : 0u;
    k[r] = i < m ? j.skey[base + i] : 0u;
  }
  if (tid == 0) l.nmore = l.nnew = l.ncopy = 0;
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < PER; ++r) {
    const bool in = r * kTileBlock + tid < m;
    const bool more = in && f[r] == kTileMore;
    const bool copy = in && f[r] == kTileCopy;
    const uint64_t mm = ballot(more);
    uint32_t at = 0;
    if (mm && lane_id() == 0)
      at = __hip_atomic_fetch_add(&l.nmore, (uint32_t)__popcll(mm), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    at = shfl32(at, 0) + lanes_below(mm);
    if (more) {
      l.mkey[at] = k[r];
      l.midx[at] = (uint16_t)x[r];
    } else if (copy) {
      l.ncopy = 1;
    } else if (in) {
      l.flag[x[r]] = (uint8_t)f[r];
    }
  }
  __syncthreads();
  const uint32_t nmore = l.nmore;
  uint32_t nnew = 0;
  for (uint32_t e = tid; e < nmore; e += kTileBlock) {
    const uint64_t key = l.mkey[e];
    const uint32_t r = lane_put_from<false>(j.t, key, 0, hidx<false>(j.t, key, 0), j.t.bucket_slots,
                                            l.meet[tid / kWave]);
    nnew += r == 1;
    l.flag[l.midx[e]] = (uint8_t)r;
  }
  block_count(j.t.ctr->size, nnew, &l.nnew, c);      // a barrier: every flag but the copies' is in place
  if (!j.out) return;
  if (l.ncopy) {
    // a copy: present, unless the key could not be kept in the table (read
    // again, so that no register waits for this)
    for (uint32_t i = tid; i < m; i += kTileBlock)
      if (j.sflag[base + i] == kTileCopy)
        l.flag[j.sidx[base + i]] = l.flag[(uint16_t)j.skey[base + i]] == 2 ? 2 : 0;
    __syncthreads();
  }
  uint8_t* out = j.out + base;
  uint32_t done = 0;
  if ((reinterpret_cast<uintptr_t>(out) & 3) == 0) {
    done = m & ~3u;
    for (uint32_t i = 4 * tid; i < done; i += 4 * kTileBlock)
      *reinterpret_cast<uint32_t*>(out + i) = *reinterpret_cast<const uint32_t*>(l.flag + i);
  }
  for (uint32_t i = done + tid; i < m; i += kTileBlock) out[i] = l.flag[i];
}

// ---- small tables -------------------------------------------------------------
// A table that fits in one tile needs no partition: one block holds
// the whole table in LDS and runs every key's whole probe sequence there.

__device__ __forceinline__ uint32_t lds_find_or_put(const DevTable& t, uint64_t* lds, uint64_t k) {
  if (k == kEmpty) return sentinel_put(t);
  const uint32_t nseq = t.nhash + t.walk;
  uint64_t b = 0;
  for (uint32_t j = 0; j < nseq; ++j) {
    b = probe_bucket<false>(t, k, j, b);
    const uint32_t r = lds_bucket_put(lds + b * t.bucket_slots, t.bucket_slots, k);
    if (r != kTileMore) return r;
  }
  return stash_put(t, k);
}

__device__ __forceinline__ void tile_whole_table(const DevTable& t, const uint64_t* __restrict__ keys, uint64_t n,
                                                 uint8_t* __restrict__ out, TileLds& l) {
  const uint32_t tid = threadIdx.x;
  const uint32_t ns = (uint32_t)(t.nrange * t.bucket_slots);
  uint64_t k = tid < n ? keys[tid] : 0;      // goes out with the table's loads
  if (tid == 0) l.nnew = 0;
  tile_load(l.slot, t.slots, ns);
  __syncthreads();
  uint32_t nnew = 0;
  for (uint64_t i = tid; i < n; i += kTileBlock) {
    const uint64_t next = i + kTileBlock < n ? keys[i + kTileBlock] : 0;
    const uint32_t r = lds_find_or_put(t, l.slot, k);
    if (out) out[i] = (uint8_t)r;
    nnew += r == 1;
    k = next;
  }
  block_count(t.ctr->size, nnew, &l.nnew, 0);
  if (l.nnew) tile_store(l.slot, t.slots, ns);
}

}  // namespace ht
