// Breadth-first state-space exploration on the GPU with the hash table as the
// visited set (the use the tables are built for: GPUexplore keeps its
// explored states in one, Sec. 3.2).  Each level: the successors of the
// frontier are generated on the device and find-or-put into the table, and
// the states reported new become the next frontier.
//
// Model: P = 16 processes with 16 local states each, packed 4 bits per
// process into one 64-bit word; each local state has up to 4 local
// transitions; 4 synchronising actions each move two processes p, q at once
// (at most one edge per local state for each).  Successor order of one state:
// for p = 0..15 each local target in list order, then for each synchronising
// action the (p-edge, q-edge) pair when both exist; at most 68 successors.
//
// All bookkeeping is per group of 64 consecutive frontier states (one wave): a
// group's number of successors (or of new ones), and an exclusive scan of
// those.  Places within a group come from a wave scan of the lanes' counts, so
// no per-state counts or offsets are stored.
//
// Split levels (the batch interface of Sec. 5): a counting pass and the scan,
// then the level goes through in slices of consecutive groups: a slice's
// successors are written to one buffer in frontier order, find-or-put as one
// call, and the keys flagged new are appended to the next frontier in batch
// order (the selection of compact.hip).  A slice bounds the buffers to about
// half a GB whatever the level's size; a whole level at once took 12.2 GB for
// the 715 M successors of the 7-level workload's last level, and allocating
// memory that has been used before costs about 30 ms per GB (it is cleared
// first): an exploration whose kernels run 25 ms took 395 ms on one machine,
// 349 on another and 28 while there was unused memory.  The last level's
// new states are counted and not written: there is no level to read them.
//
// Fused levels (successor generation and hash table access in one kernel, as
// GPUexplore does, Sec. 3.2 and 7): a lane takes a frontier state, generates
// its successors in registers in the same order, and find-or-puts each with
// the one-lane bucket probe (Cuckoo: probes and places it, listing those whose
// candidates are all taken for an evict pass), recording in a 68-bit mask
// which of them were new; after the scan of the new counts a second pass
// regenerates the successors and writes the new ones.  The successor batch is
// never stored: a level moves the frontier, the masks and the new states.
#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "bucketed_dev.h"
#include "cuckoo_dev.h"
#include "runtime.h"

namespace ht {
hipError_t zero_words(uint32_t*, uint64_t, hipStream_t);
hipError_t scan_exclusive(const unsigned long long*, unsigned long long*, uint64_t, unsigned long long*,
                          unsigned long long*, uint32_t, hipStream_t);
hipError_t select_count(const uint8_t*, uint64_t, unsigned long long*, unsigned long long*, uint32_t, hipStream_t);
hipError_t select_write(const uint64_t*, const uint8_t*, uint64_t, uint64_t*, const unsigned long long*, uint32_t,
                        hipStream_t);
}  // namespace ht

using namespace ht;
using namespace ht_rt;

namespace {

struct BfsModelDev {
  uint8_t lcnt[16][16];
  uint8_t ltgt[16][16][4];
  uint8_t sp[4], sq[4];
  int8_t pe[4][16], qe[4][16];   // -1: no edge
};

__device__ __forceinline__ uint32_t local_of(uint64_t st, uint32_t p) { return (uint32_t)(st >> (4 * p)) & 15u; }

// The model's transitions in LDS, a row per process and local state: the four
// targets and their number in one 8-byte read.
struct ModelLds {
  uint2 row[16 * 16];
  int8_t act[2][4][16];
  uint8_t proc[2][4];
};

__device__ __forceinline__ void model_to_lds(const BfsModelDev& m, ModelLds& l) {
  for (uint32_t q = threadIdx.x; q < 256; q += kBlock) {
    const uint8_t* g = m.ltgt[q / 16][q % 16];
    l.row[q] = make_uint2(g[0] | (uint32_t)g[1] << 8 | (uint32_t)g[2] << 16 | (uint32_t)g[3] << 24,
                          m.lcnt[q / 16][q % 16]);
  }
  for (uint32_t q = threadIdx.x; q < 64; q += kBlock) {
    l.act[0][q / 16][q % 16] = m.pe[q / 16][q % 16];
    l.act[1][q / 16][q % 16] = m.qe[q / 16][q % 16];
    if (q < 4) {
      l.proc[0][q] = m.sp[q];
      l.proc[1][q] = m.sq[q];
    }
  }
  __syncthreads();
}

// Number of successors of `st`.
__device__ __forceinline__ uint32_t successor_count(const BfsModelDev& m, const ModelLds& l, uint64_t st) {
  uint32_t c = 0;
#pragma unroll
  for (uint32_t p = 0; p < 16; ++p) c += l.row[p * 16 + local_of(st, p)].y;
#pragma unroll
  for (uint32_t a = 0; a < 4; ++a)
    c += (l.act[0][a][local_of(st, m.sp[a])] >= 0 && l.act[1][a][local_of(st, m.sq[a])] >= 0) ? 1u : 0u;
  return c;
}

// Successors of each group of 64 frontier states.
__global__ __launch_bounds__(kBlock) void bfs_count_kernel(BfsModelDev m, const uint64_t* __restrict__ f, uint64_t nf,
                                                           unsigned long long* __restrict__ gcnt) {
  __shared__ ModelLds model;
  model_to_lds(m, model);
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i0 = (uint64_t)blockIdx.x * kBlock + (threadIdx.x & ~63u); i0 < nf; i0 += stride) {
    const uint64_t i = i0 + lane_id();
    const uint32_t incl = wave_inclusive32(i < nf ? successor_count(m, model, f[i]) : 0u);
    if (lane_id() == kWave - 1) gcnt[i0 / kWave] = incl;
  }
}

// Successors of `st` in model order; visit(succ) is called for each.
template <class F>
__device__ __forceinline__ void for_each_successor(const BfsModelDev& m, const ModelLds& l, uint64_t st, F&& visit) {
  for (uint32_t p = 0; p < 16; ++p) {
    const uint2 r = l.row[p * 16 + local_of(st, p)];
    const uint64_t cleared = st & ~(15ull << (4 * p));
    for (uint32_t k = 0; k < r.y; ++k) visit(cleared | ((uint64_t)((r.x >> (8 * k)) & 255u) << (4 * p)));
  }
  for (uint32_t a = 0; a < 4; ++a) {
    const uint32_t p = m.sp[a], q = m.sq[a];
    const int tp = l.act[0][a][local_of(st, p)], tq = l.act[1][a][local_of(st, q)];
    if (tp >= 0 && tq >= 0) {
      const uint64_t cleared = st & ~(15ull << (4 * p)) & ~(15ull << (4 * q));
      visit(cleared | ((uint64_t)tp << (4 * p)) | ((uint64_t)tq << (4 * q)));
    }
  }
}

// Successors of `st` in model order as for_each_successor, with the loops
// over processes and targets unrolled (constant shifts): visit(live, succ) is
// called 68 times.
template <class F>
__device__ __forceinline__ void unrolled_successors(const BfsModelDev& m, const ModelLds& l, uint64_t st, F&& visit) {
#pragma unroll
  for (uint32_t p = 0; p < 16; ++p) {
    const uint2 r = l.row[p * 16 + local_of(st, p)];
    const uint64_t cleared = st & ~(15ull << (4 * p));
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) visit(k < r.y, cleared | ((uint64_t)((r.x >> (8 * k)) & 255u) << (4 * p)));
  }
#pragma unroll
  for (uint32_t a = 0; a < 4; ++a) {
    const uint32_t p = m.sp[a], q = m.sq[a];
    const int tp = l.act[0][a][local_of(st, p)], tq = l.act[1][a][local_of(st, q)];
    const uint64_t cleared = st & ~(15ull << (4 * p)) & ~(15ull << (4 * q));
    visit(tp >= 0 && tq >= 0, cleared | ((uint64_t)tp << (4 * p)) | ((uint64_t)tq << (4 * q)));
  }
}

// Writing successors (all of them, or those a mask marks) at their scanned
// places, staged through LDS so that the stores coalesce: a block takes a tile
// of four groups of 64 states, whose outputs form one contiguous range; its
// waves in turn place their group's successors in the window, which the block
// then copies out in consecutive words.  A thread per state storing its own
// successors one after another wrote 8-byte words to 64 unrelated places per
// instruction: 7.7 ms for the 5.7 GB batch of the 7-level workload's last
// level.  What it costs is making the successors: with the transitions read
// from kernel arguments in loops, and windows that cut across the waves, all
// seven levels took 4.6 ms, with rows in LDS and a window per wave 1.45 (4.4
// TB/s).  The tiles cover groups g0 .. g1-1 of the frontier's nf states; goff
// (one entry more than there are groups) is the scan of the groups' counts,
// and out[0] receives the first output of group g0.
constexpr uint32_t kMostSuccessors = 16 * 4 + 4;

template <bool MASKED>
__device__ __forceinline__ void write_tiles(const BfsModelDev& m, const uint64_t* __restrict__ f, uint64_t nf,
                                            uint64_t g0, uint64_t g1, const unsigned long long* __restrict__ goff,
                                            const uint64_t* __restrict__ mask, uint64_t* __restrict__ out) {
  constexpr uint64_t kTileGroups = kBlock / kWave;
  __shared__ uint64_t win[kWave * kMostSuccessors];
  __shared__ ModelLds model;
  model_to_lds(m, model);
  const uint32_t tid = threadIdx.x;
  const uint64_t zero = goff[g0];
  for (uint64_t t0 = g0 + (uint64_t)blockIdx.x * kTileGroups; t0 < g1; t0 += (uint64_t)gridDim.x * kTileGroups) {
    const uint64_t g = t0 + tid / kWave;
    const uint64_t i = t0 * kWave + tid;
    const bool live = g < g1 && i < nf;
    const uint64_t st = live ? f[i] : 0ull;
    const uint64_t m0 = MASKED && live ? mask[2 * i] : ~0ull;
    const uint64_t m1 = MASKED && live ? mask[2 * i + 1] : ~0ull;
    const uint32_t c = !live ? 0u : MASKED ? (uint32_t)(__popcll(m0) + __popcll(m1)) : successor_count(m, model, st);
    const uint32_t mine = wave_inclusive32(c) - c;
    for (uint64_t q = t0; q < g1 && q < t0 + kTileGroups; ++q) {
      if (q == g && c) {
        uint32_t o = mine, k = 0;
        unrolled_successors(m, model, st, [&](bool is, uint64_t succ) {
          const bool take = is && (!MASKED || (((k < 64 ? (m0 >> k) : (m1 >> (k - 64))) & 1ull) != 0));
          if (take) win[o] = succ;
          o += take;
          k += is;
        });
      }
      __syncthreads();
      const uint64_t base = goff[q];
      const uint32_t nw = (uint32_t)(goff[q + 1] - base);
      uint64_t* const to = out + (base - zero);
      for (uint32_t j = tid; j < nw; j += kBlock) to[j] = win[j];
      __syncthreads();
    }
  }
}

// Where the slices of `per` groups begin in the scan of the groups' counts
// (ng + 1 entries), and the total: out[0 .. nslices].
__global__ __launch_bounds__(kBlock) void bfs_bounds_kernel(const unsigned long long* __restrict__ goff, uint64_t ng,
                                                            uint64_t per, uint64_t nslices,
                                                            unsigned long long* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t q = (uint64_t)blockIdx.x * kBlock + threadIdx.x; q <= nslices; q += stride)
    out[q] = goff[q < nslices ? q * per : ng];
}

// Split pass: every successor of groups g0 .. g1-1.
__global__ __launch_bounds__(kBlock) void bfs_write_kernel(BfsModelDev m, const uint64_t* __restrict__ f, uint64_t nf,
                                                           uint64_t g0, uint64_t g1,
                                                           const unsigned long long* __restrict__ goff,
                                                           uint64_t* __restrict__ out) {
  write_tiles<false>(m, f, nf, g0, g1, goff, nullptr, out);
}

// Fused pass: find-or-put of every successor of the frontier; per state the
// mask of new successors (bit k = successor k; two words; not written when
// mask is NULL), per group of 64 states their number, and the number of
// successors generated added to *generated.
__global__ __launch_bounds__(kBlock) HT_EIGHT_WAVES
void bfs_fused_kernel(BfsModelDev m, DevTable t, const uint64_t* __restrict__ f, uint64_t nf,
                      unsigned long long* __restrict__ gcnt, uint64_t* __restrict__ mask,
                      unsigned long long* __restrict__ generated) {
  __shared__ ModelLds model;
  model_to_lds(m, model);
  const uint64_t first = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  const int lane = lane_id();
  unsigned long long placed = 0, gen = 0;
  for (uint64_t i0 = first - lane; i0 < nf; i0 += stride) {
    const uint64_t i = i0 + lane;
    uint64_t m0 = 0, m1 = 0;
    uint32_t k = 0, nnew = 0;
    if (i < nf) {
      for_each_successor(m, model, f[i], [&](uint64_t succ) {
        const uint32_t r = lane_find_or_put<false, false>(t, succ, nullptr);
        if (r) {                   // 1 = stored, 2 = kept on the overflow list: new either way
          if (k < 64) m0 |= 1ull << k;
          else m1 |= 1ull << (k - 64);
          ++nnew;
        }
        placed += r == 1;
        ++k;
      });
      if (mask) {
        mask[2 * i] = m0;
        mask[2 * i + 1] = m1;
      }
    }
    gen += k;
    const uint32_t incl = wave_inclusive32(nnew);
    if (lane == kWave - 1) gcnt[i0 / kWave] = incl;
  }
  wave_count(t.ctr->size, placed, (uint32_t)(first / kWave));
  const unsigned long long g = wave_sum(gen);
  if (lane == 0 && g) add_agent(generated, g);
}

// Second fused pass: the successors marked new, at the scanned places.
__global__ __launch_bounds__(kBlock) void bfs_fused_write_kernel(BfsModelDev m, const uint64_t* __restrict__ f,
                                                                 uint64_t nf, uint64_t ngroups,
                                                                 const uint64_t* __restrict__ mask,
                                                                 const unsigned long long* __restrict__ goff,
                                                                 uint64_t* __restrict__ out) {
  write_tiles<true>(m, f, nf, 0, ngroups, goff, mask, out);
}

// Successors of one state, one per call, in model order (the same order as
// for_each_successor); lets a wave step through its lanes' successors
// together, so wave-wide votes stay converged.
struct SuccIter {
  uint64_t st;
  uint32_t p = 0, kk = 0, a = 0;
  __device__ __forceinline__ bool next(const ModelLds& l, uint64_t& succ) {
    while (p < 16) {
      const uint2 r = l.row[p * 16 + local_of(st, p)];
      if (kk < r.y) {
        succ = (st & ~(15ull << (4 * p))) | ((uint64_t)((r.x >> (8 * kk)) & 255u) << (4 * p));
        ++kk;
        return true;
      }
      ++p;
      kk = 0;
    }
    while (a < 4) {
      const uint32_t pp = l.proc[0][a], q = l.proc[1][a];
      const int tp = l.act[0][a][local_of(st, pp)], tq = l.act[1][a][local_of(st, q)];
      ++a;
      if (tp >= 0 && tq >= 0) {
        succ = (st & ~(15ull << (4 * pp)) & ~(15ull << (4 * q))) | ((uint64_t)tp << (4 * pp)) |
               ((uint64_t)tq << (4 * q));
        return true;
      }
    }
    return false;
  }
};

// Fused Cuckoo pass 1: a wave takes groups g0 .. g1-1 of 64 frontier states,
// one state per lane, and steps through their successors together; each
// successor is probed and placed as above, new ones marked in the state's mask
// (not kept when mask is NULL) and counted per group, and those with every
// candidate taken listed as (key, state << 7 | successor number) in the
// group's region of the scratch list, which starts at the group's first
// successor offset, counted from group g0's (a group never lists more keys
// than it has successors).
__global__ __launch_bounds__(kBlock) HT_EIGHT_WAVES
void bfs_cuckoo_probe_kernel(BfsModelDev m, DevTable t, const uint64_t* __restrict__ f, uint64_t nf, uint64_t g0,
                             uint64_t g1, const unsigned long long* __restrict__ soff, CuckooScratch s,
                             uint32_t* __restrict__ lcnt, unsigned long long* __restrict__ gnew,
                             uint64_t* __restrict__ mask) {
  __shared__ ModelLds model;
  model_to_lds(m, model);
  const int lane = lane_id();
  const uint64_t wave =
      __builtin_amdgcn_readfirstlane((uint32_t)(((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kWave));
  const uint64_t nwaves = (uint64_t)gridDim.x * (kBlock / kWave);
  const uint64_t zero = soff[g0];
  const uint32_t sc = t.ctr->stash_count;
  const uint32_t oc = t.ctr->overflow_count;
  unsigned long long placed = 0;
  for (uint64_t g = g0 + wave; g < g1; g += nwaves) {
    const uint64_t i = g * kWave + lane;
    const bool live = i < nf;
    SuccIter it{live ? f[i] : 0ull};
    const uint64_t begin = soff[g] - zero;
    uint64_t m0 = 0, m1 = 0;
    uint32_t k = 0, nnew = 0, nlist = 0;
    for (;;) {
      uint64_t succ = 0;
      const bool has = live && it.next(model, succ);
      if (!ballot(has)) break;
      const uint32_t r = cuckoo_probe_key(t, t.slots, succ, has, sc, oc);
      if (has && r == 1) {
        if (k < 64) m0 |= 1ull << k;
        else m1 |= 1ull << (k - 64);
        ++nnew;
      }
      const bool l = has && r == kListed;
      const uint64_t mm = ballot(l);
      if (l) {
        const uint64_t slot = begin + nlist + lanes_below(mm);
        s.wkey[slot] = succ;
        s.wmeta[slot] = (i << 7) | k;
      }
      nlist += (uint32_t)__popcll(mm);
      k += has ? 1u : 0u;
    }
    if (mask && live) {
      mask[2 * i] = m0;
      mask[2 * i + 1] = m1;
    }
    placed += nnew;
    const uint32_t incl = wave_inclusive32(nnew);
    if (lane == kWave - 1) {
      gnew[g] = incl;
      lcnt[g - g0] = nlist;
    }
  }
  wave_count(t.ctr->size, placed, (uint32_t)wave);
}

// Fused Cuckoo pass 2: the listed keys, deduplicated in the scratch set; each
// winner marks its successor new in the state's mask, is added to its group's
// count (the wave that serves a group is the only one to write it) and runs
// the eviction chain from h_1 (then the stash), as the single-table evict
// kernel does.  The scratch-set slot a winner took replaces its list entry's
// meta.
__global__ __launch_bounds__(kBlock) void bfs_cuckoo_evict_kernel(DevTable t, uint64_t g0, uint64_t g1,
                                                                  const unsigned long long* __restrict__ soff,
                                                                  CuckooScratch s, const uint32_t* __restrict__ lcnt,
                                                                  unsigned long long* __restrict__ gnew,
                                                                  uint64_t* __restrict__ mask) {
  const int lane = lane_id();
  const uint64_t wave =
      __builtin_amdgcn_readfirstlane((uint32_t)(((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kWave));
  const uint64_t nwaves = (uint64_t)gridDim.x * (kBlock / kWave);
  const uint64_t zero = soff[g0];
  unsigned long long nnew = 0, nevict = 0;
  for (uint64_t g = g0 + wave; g < g1; g += nwaves) {
    const uint64_t begin = soff[g] - zero;
    const uint32_t c = lcnt[g - g0];
    unsigned long long mine = 0;
    for (uint32_t e = lane; e < c; e += kWave) {
      const uint64_t k = s.wkey[begin + e];
      const uint64_t meta = s.wmeta[begin + e];
      uint64_t p = mix64(k ^ s.dset_seed) & s.dset_mask;
      bool winner = false;
      for (;;) {
        const uint64_t old = cas64(&s.dset[p], kEmpty, k);
        if (old == kEmpty) {
          winner = true;
          break;
        }
        if (old == k) break;
        p = (p + 1) & s.dset_mask;
      }
      s.wmeta[begin + e] = winner ? p : ~0ull;
      if (!winner) continue;
      const uint64_t i = meta >> 7;
      const uint32_t kb = (uint32_t)(meta & 127);
      if (mask)
        __hip_atomic_fetch_or(&mask[2 * i + (kb >> 6)], 1ull << (kb & 63), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
      uint64_t y = k;
      uint32_t steps = 0;
      const uint64_t h1 = hidx<false>(t, y, 0);
      const bool placed = (t.flags & kFlagLookahead) ? cuckoo_chain<false, true>(t, t.slots, t.nhash, y, h1, nevict, steps)
                                                      : cuckoo_chain<false, false>(t, t.slots, t.nhash, y, h1, nevict, steps);
      if (!placed) stash_put(t, y);
      ++mine;
    }
    if (c) {
      nnew += mine;
      mine = wave_sum(mine);
      if (lane == 0) gnew[g] += mine;
    }
  }
  wave_count(t.ctr->size, nnew, (uint32_t)wave);
  wave_count(t.ctr->evictions, nevict, (uint32_t)wave);
}

// Fused Cuckoo pass 3: empty the scratch-set slots the evict pass took.
__global__ __launch_bounds__(kBlock) void bfs_cuckoo_scrub_kernel(uint64_t g0, uint64_t g1,
                                                                  const unsigned long long* __restrict__ soff,
                                                                  CuckooScratch s, const uint32_t* __restrict__ lcnt) {
  const int lane = lane_id();
  const uint64_t wave =
      __builtin_amdgcn_readfirstlane((uint32_t)(((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kWave));
  const uint64_t nwaves = (uint64_t)gridDim.x * (kBlock / kWave);
  const uint64_t zero = soff[g0];
  for (uint64_t g = g0 + wave; g < g1; g += nwaves) {
    const uint64_t begin = soff[g] - zero;
    const uint32_t c = lcnt[g - g0];
    for (uint32_t e = lane; e < c; e += kWave) {
      const uint64_t p = s.wmeta[begin + e];
      if (p != ~0ull) s.dset[p] = kEmpty;
    }
  }
}

// Device buffer that only grows.
struct Buf {
  void* p = nullptr;
  size_t bytes = 0;
  // Room for `need` bytes; the first `keep` bytes of the old contents stay
  // (copied on stream s, which is waited for), also when there is no room.
  int ensure(size_t need, size_t keep = 0, hipStream_t s = nullptr) {
    if (need <= bytes) return HT_OK;
    if (!keep) drop();
    void* q = nullptr;
    if (hipMalloc(&q, need) != hipSuccess) {
      (void)hipGetLastError();
      return fail(HT_ENOMEM, "hipMalloc in breadth-first exploration failed");
    }
    if (keep) {
      hipError_t e = hipMemcpyAsync(q, p, keep, hipMemcpyDeviceToDevice, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (e != hipSuccess) {
        (void)hipFree(q);
        return hip_fail(e, "copy of an exploration buffer");
      }
    }
    drop();
    p = q;
    bytes = need;
    return HT_OK;
  }
  void drop() {
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
  }
  ~Buf() { drop(); }
};

}  // namespace

// Buffers of an exploration, kept with the table for its next one while they
// are small (kKeepBytes); given back with it, by a rebuild, and when an
// allocation for the table finds no room.
struct ht_explore_ws {
  int device = 0;
  Buf frontier, next, batch, flags, gcounts, goffsets, gnews, tmp, nsel, masks, lists, slices;
  size_t bytes() const {
    size_t n = 0;
    for (const Buf* b : {&frontier, &next, &batch, &flags, &gcounts, &goffsets, &gnews, &tmp, &nsel, &masks, &lists,
                         &slices})
      n += b->bytes;
    return n;
  }
};

void ht_rt::free_explore(ht_table* t) {
  delete t->explore;
  t->explore = nullptr;
}

namespace {

constexpr size_t kKeepBytes = 1ull << 30;

// The table's exploration buffers for one call: those it kept, if they lie on
// the current device, else new ones.  The call takes them from the table, and
// they go back to it afterwards when they are small and the call went well.
struct ExploreHold {
  ht_table* t;
  std::unique_ptr<ht_explore_ws> ws;
  bool keep = false;
  explicit ExploreHold(ht_table* table) : t(table), ws(table->explore) {
    t->explore = nullptr;
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (ws && ws->device == dev) return;
    ws.reset();
    ws.reset(new ht_explore_ws());
    ws->device = dev;
  }
  ~ExploreHold() {
    if (!keep || ws->bytes() > kKeepBytes) return;
    free_explore(t);
    t->explore = ws.release();
  }
};

// Device time of the spans of work between host round trips: pairs of events
// recorded on the stream, kept for the next level, destroyed on every return
// path.
struct Spans {
  std::vector<hipEvent_t> ev;
  size_t used = 0;
  hipError_t mark(hipStream_t s) {
    if (used == ev.size()) {
      ev.push_back(nullptr);
      const hipError_t rc = hipEventCreate(&ev.back());
      if (rc != hipSuccess) {
        ev.pop_back();
        return rc;
      }
    }
    return hipEventRecord(ev[used++], s);
  }
  // Sum in ms; the stream's work is done.  The next level starts over.
  double total() {
    double ms = 0.0;
    for (size_t i = 0; i + 1 < used; i += 2) {
      float x = 0.f;
      if (hipEventElapsedTime(&x, ev[i], ev[i + 1]) == hipSuccess) ms += (double)x;
    }
    used = 0;
    return ms;
  }
  ~Spans() {
    for (auto& x : ev) (void)hipEventDestroy(x);
  }
};

// Groups of 64 states per slice.  Split: 16384 groups have about 50 M
// successors (at most 71 M), half a GB of batch and flags.  The 7-level
// workload's split bucketed levels, device time and whole call: 4096 groups
// 28.4 and 31.1 ms, 8192 26.4 and 28.2, 16384 25.4 and 27.7, 32768 24.9 and
// 28.9 (its buffers no longer stay with the table), whole levels 24.3 and
// 28.1 while there is unused memory (349 to 395 after).  Fused Cuckoo: four groups
// for each wave of the probe grid (at most 2.3 GB of lists).  Its fused levels
// of a 6-level exploration: 5.25 ms a call at three turns of 8 blocks per
// compute unit, 5.04 at four; four turns of 6 blocks 5.20.
constexpr uint64_t kSplitGroups = 16384;
constexpr uint64_t kCuckooTurns = 4;

}  // namespace

static int explore(ht_table* t, const ht_bfs_model* model, uint64_t initial, uint32_t levels, uint32_t mode,
                   uint64_t* batch_sizes, uint64_t* new_counts, double* fop_ms, double* level_ms, hipStream_t s) {
  int rc = check_table(t);
  if (rc) return rc;
  if (!model) return fail(HT_EINVAL, "model is NULL");
  if (t->cfg.key_words > 1) return fail(HT_EINVAL, "the exploration packs states into single-word keys");
  if (mode != HT_BFS_SPLIT && mode != HT_BFS_FUSED) return fail(HT_EINVAL, "unknown exploration mode");
  const bool fused = mode == HT_BFS_FUSED;
  const bool ck = fused && t->cfg.kind == HT_CUCKOO;   // fused Cuckoo levels: count and scan first
  if (fused && is_scripted(t)) return fail(HT_EINVAL, "fused levels do not take scripted-hash tables");
  BfsModelDev m;
  static_assert(sizeof(BfsModelDev) == sizeof(ht_bfs_model), "model layout");
  std::memcpy(&m, model, sizeof(m));
  for (int a = 0; a < 4; ++a)
    if (m.sp[a] > 15 || m.sq[a] > 15) return fail(HT_EINVAL, "synchronising action names a process above 15");
  for (int p = 0; p < 16; ++p)
    for (int q = 0; q < 16; ++q)
      if (m.lcnt[p][q] > 4) return fail(HT_EINVAL, "more than 4 local transitions");
  ExploreHold hold(t);
  ht_explore_ws& ws = *hold.ws;
  Buf &frontier = ws.frontier, &next = ws.next, &batch = ws.batch, &flags = ws.flags, &gcounts = ws.gcounts,
      &goffsets = ws.goffsets, &gnews = ws.gnews, &tmp = ws.tmp, &nsel = ws.nsel, &masks = ws.masks, &lists = ws.lists,
      &slices = ws.slices;
  const uint32_t grid = max_blocks(t);
  rc = frontier.ensure(8);
  if (!rc) rc = nsel.ensure(8);
  if (!rc) rc = tmp.ensure((grid + 1) * 8ull);   // block totals of the scans and the selection
  if (rc) return rc;
  auto* wk = static_cast<unsigned long long*>(tmp.p);
  auto* ns = static_cast<unsigned long long*>(nsel.p);
  HT_HIP(hipMemcpyAsync(frontier.p, &initial, 8, hipMemcpyHostToDevice, s));
  rc = do_find_or_put(t, static_cast<uint64_t*>(frontier.p), 1, nullptr, s);
  if (rc) return rc;
  const DevTable dt = launch_view(t);
  uint64_t nf = 1;
  Spans all, fop;
  std::vector<unsigned long long> bounds;
  for (uint32_t L = 0; L < levels && nf && rc == HT_OK; ++L) {
    const bool last = L + 1 == levels;     // no next level: new states are counted, not written
    const uint64_t ng = (nf + kWave - 1) / kWave;
    rc = gcounts.ensure(ng * 8);
    if (!rc) rc = goffsets.ensure((ng + 1) * 8);
    if (!rc && fused && !last) rc = masks.ensure(nf * 16);
    if (!rc && ck) rc = gnews.ensure(ng * 8);
    if (rc) break;
    auto* gcnt = static_cast<unsigned long long*>(gcounts.p);
    auto* goff = static_cast<unsigned long long*>(goffsets.p);
    auto* fr = static_cast<const uint64_t*>(frontier.p);
    auto* mk = last ? nullptr : static_cast<uint64_t*>(masks.p);
    const uint32_t g1 = (uint32_t)std::min<uint64_t>((nf + kBlock - 1) / kBlock, grid);
    const uint32_t gsc = (uint32_t)std::min<uint64_t>((ng + 1023) / 1024, grid);
    uint64_t nb = 0, nnew = 0;
    // first span: successor counts (split, fused Cuckoo) or the fused bucketed pass, then a scan
    if (fused && !ck) HT_HIP(zero_words(reinterpret_cast<uint32_t*>(ns), 2, s));
    HT_HIP(all.mark(s));
    if (fused && !ck) {
      HT_HIP(fop.mark(s));
      // 3 blocks per compute unit: successors repeat among the states in flight,
      // and the fewer these are, the more copies meet in the caches (fused levels
      // of the 7-level workload: 17.8 ms at 2, 16.5 at 3, 17.2 at 4, 17.8 at 5,
      // 18.7 at 8; 6 levels 2.30 at 3, 2.35 at 5 and 8)
      const uint32_t gf = (uint32_t)std::min<uint64_t>((nf + kBlock - 1) / kBlock, t->cus * 3);
      hipLaunchKernelGGL(bfs_fused_kernel, dim3(gf), dim3(kBlock), 0, s, m, dt, fr, nf, gcnt, mk, ns);
      HT_HIP(hipGetLastError());
      HT_HIP(fop.mark(s));
    } else {
      hipLaunchKernelGGL(bfs_count_kernel, dim3(g1), dim3(kBlock), 0, s, m, fr, nf, gcnt);
      HT_HIP(hipGetLastError());
    }
    HT_HIP(scan_exclusive(gcnt, goff, ng, goff + ng, wk, gsc, s));
    HT_HIP(all.mark(s));
    if (fused && !ck) {
      unsigned long long got[2] = {0, 0};
      HT_HIP(hipMemcpyAsync(&got[0], goff + ng, 8, hipMemcpyDeviceToHost, s));
      HT_HIP(hipMemcpyAsync(&got[1], ns, 8, hipMemcpyDeviceToHost, s));
      HT_HIP(hipStreamSynchronize(s));
      nnew = got[0];
      nb = got[1];
    } else {
      // where each slice's successors begin: slice q is groups q * per ...
      const uint64_t per = ck ? (uint64_t)grid * (kBlock / kWave) * kCuckooTurns : kSplitGroups;
      const uint64_t nslices = (ng + per - 1) / per;
      bounds.resize(nslices + 1);
      rc = slices.ensure((nslices + 1) * 8);
      if (rc) break;
      auto* sl = static_cast<unsigned long long*>(slices.p);
      const uint32_t gb = (uint32_t)std::min<uint64_t>(nslices / kBlock + 1, grid);
      hipLaunchKernelGGL(bfs_bounds_kernel, dim3(gb), dim3(kBlock), 0, s, goff, ng, per, nslices, sl);
      HT_HIP(hipGetLastError());
      // (a strided copy to host memory had not arrived after the wait when a
      // profiler's interception was in place)
      HT_HIP(hipMemcpyAsync(bounds.data(), sl, (nslices + 1) * 8, hipMemcpyDeviceToHost, s));
      HT_HIP(hipStreamSynchronize(s));
      nb = bounds[nslices];
      uint64_t most = 1;
      for (uint64_t q = 0; q < nslices; ++q) most = std::max<uint64_t>(most, bounds[q + 1] - bounds[q]);
      rc = reserve_scratch(t, most);   // the find-or-put's scratch for a slice, outside the timed spans
      if (!rc && ck) rc = lists.ensure(std::min(per, ng) * 4);
      if (!rc && !ck) rc = batch.ensure(most * 8);
      if (!rc && !ck) rc = flags.ensure(most);
      if (!rc && !ck) rc = nsel.ensure(nslices * 8);
      if (rc) break;
      ns = static_cast<unsigned long long*>(nsel.p);
      auto* bt = static_cast<uint64_t*>(batch.p);
      auto* fl = static_cast<uint8_t*>(flags.p);
      auto* lc = static_cast<uint32_t*>(lists.p);
      auto* gn = static_cast<unsigned long long*>(gnews.p);
      if (ck) HT_HIP(all.mark(s));
      for (uint64_t q = 0; q < nslices && rc == HT_OK; ++q) {
        const uint64_t n = bounds[q + 1] - bounds[q];
        const uint64_t a = q * per, z = std::min(ng, a + per);
        if (ck) {
          // probe and place, evict, scrub, at 8 blocks per compute unit (fused
          // levels of the 7-level workload: 29.6 ms at 4, 28.8 at 6, 28.6 at 8)
          const CuckooScratch sc = scratch_view(t, std::max<uint64_t>(n, 1));
          const uint32_t g2 = (uint32_t)std::min<uint64_t>((z - a + 3) / 4, grid);
          HT_HIP(fop.mark(s));
          hipLaunchKernelGGL(bfs_cuckoo_probe_kernel, dim3(g2), dim3(kBlock), 0, s, m, dt, fr, nf, a, z, goff, sc, lc,
                             gn, mk);
          HT_HIP(hipGetLastError());
          hipLaunchKernelGGL(bfs_cuckoo_evict_kernel, dim3(g2), dim3(kBlock), 0, s, dt, a, z, goff, sc, lc, gn, mk);
          HT_HIP(hipGetLastError());
          hipLaunchKernelGGL(bfs_cuckoo_scrub_kernel, dim3(g2), dim3(kBlock), 0, s, a, z, goff, sc, lc);
          HT_HIP(hipGetLastError());
          HT_HIP(fop.mark(s));
          continue;
        }
        // split: write the slice's batch, find-or-put it, select the new keys
        if (!n) {                        // no state of the slice has a successor
          HT_HIP(zero_words(reinterpret_cast<uint32_t*>(ns + q), 2, s));
          continue;
        }
        const uint32_t gw = (uint32_t)std::min<uint64_t>((z - a + kBlock / kWave - 1) / (kBlock / kWave), grid);
        HT_HIP(all.mark(s));
        hipLaunchKernelGGL(bfs_write_kernel, dim3(gw), dim3(kBlock), 0, s, m, fr, nf, a, z, goff, bt);
        HT_HIP(hipGetLastError());
        HT_HIP(fop.mark(s));
        rc = do_find_or_put(t, bt, n, fl, s, FopMode{nullptr, true, true});
        if (rc) break;
        HT_HIP(fop.mark(s));
        const uint32_t gs = (uint32_t)std::min<uint64_t>((n + 4095) / 4096, grid);
        HT_HIP(select_count(fl, n, ns + q, wk, gs, s));
        HT_HIP(all.mark(s));
        if (!last) {
          // the next frontier's room grows with the new states found
          unsigned long long got = 0;
          HT_HIP(hipMemcpyAsync(&got, ns + q, 8, hipMemcpyDeviceToHost, s));
          HT_HIP(hipStreamSynchronize(s));
          if ((nnew + got) * 8 > next.bytes) {
            // what the slices so far give for the whole level, and a tenth
            // more; where there is no room for that, what there is
            const uint64_t guess = (uint64_t)((double)(nnew + got) / (double)(q + 1) * (double)nslices * 1.1);
            rc = next.ensure(std::max<uint64_t>(guess, nnew + got) * 8, nnew * 8, s);
            if (rc == HT_ENOMEM) rc = next.ensure((nnew + got) * 8, nnew * 8, s);
            if (rc) break;
          }
          HT_HIP(all.mark(s));
          HT_HIP(select_write(bt, fl, n, static_cast<uint64_t*>(next.p) + nnew, wk, gs, s));
          HT_HIP(all.mark(s));
          nnew += got;
        }
      }
      if (rc) break;
      if (ck) {
        HT_HIP(scan_exclusive(gn, goff, ng, goff + ng, wk, gsc, s));
        HT_HIP(all.mark(s));
        unsigned long long got = 0;
        HT_HIP(hipMemcpyAsync(&got, goff + ng, 8, hipMemcpyDeviceToHost, s));
        HT_HIP(hipStreamSynchronize(s));
        nnew = got;
      } else if (last) {
        bounds.resize(nslices);
        HT_HIP(hipMemcpyAsync(bounds.data(), ns, nslices * 8, hipMemcpyDeviceToHost, s));
        HT_HIP(hipStreamSynchronize(s));
        for (auto x : bounds) nnew += x;
      }
    }
    if (fused && !last) {
      // last span: the new states written at their scanned places
      rc = next.ensure(std::max<uint64_t>(nnew, 1) * 8);
      if (rc) break;
      HT_HIP(all.mark(s));
      hipLaunchKernelGGL(bfs_fused_write_kernel, dim3(g1), dim3(kBlock), 0, s, m, fr, nf, ng, mk, goff,
                         static_cast<uint64_t*>(next.p));
      HT_HIP(hipGetLastError());
      HT_HIP(all.mark(s));
    }
    HT_HIP(hipStreamSynchronize(s));
    if (fused) t->puts += nb;
    const double lms = all.total(), fms = fop.total();
    if (fop_ms) fop_ms[L] = fms;
    if (level_ms) level_ms[L] = lms;
    if (batch_sizes) batch_sizes[L] = nb;
    if (new_counts) new_counts[L] = nnew;
    std::swap(frontier.p, next.p);
    std::swap(frontier.bytes, next.bytes);
    nf = nnew;
  }
  const hipError_t end = hipStreamSynchronize(s);
  hold.keep = rc == HT_OK && end == hipSuccess;
  return rc;
}

extern "C" int ht_bfs_explore_ex(ht_table* t, const ht_bfs_model* model, uint64_t initial, uint32_t levels,
                                 uint32_t mode, uint64_t* batch_sizes, uint64_t* new_counts, double* fop_ms,
                                 double* level_ms, hipStream_t s) {
  try {
    return explore(t, model, initial, levels, mode, batch_sizes, new_counts, fop_ms, level_ms, s);
  } catch (const std::bad_alloc&) {
    return fail(HT_ENOMEM, "host memory for the breadth-first exploration");
  }
}

extern "C" int ht_bfs_explore(ht_table* t, const ht_bfs_model* model, uint64_t initial, uint32_t levels,
                              uint64_t* batch_sizes, uint64_t* new_counts, double* fop_ms, hipStream_t s) {
  return ht_bfs_explore_ex(t, model, initial, levels, HT_BFS_SPLIT, batch_sizes, new_counts, fop_ms, nullptr, s);
}
