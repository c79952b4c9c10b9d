// Host launchers of the tiled find-or-put (device code: tile_dev.h).
#include "tile.h"

#include "tile_dev.h"

namespace ht {

template <uint32_t C>
__global__ __launch_bounds__(kTileBlock, C == 4096 ? 8 : 4) void tile_partition_kernel(TileJob j) {
  __shared__ TilePartLds<C> l;
  tile_partition_chunk<C>(j, blockIdx.x, l);
}

template <uint32_t C>
__global__ __launch_bounds__(kTileBlock) void tile_insert_kernel(TileJob j) {
  __shared__ TileLds l;
  const uint32_t tl = tile_of_block(blockIdx.x, j.tiles);
  if (tl < j.tiles) tile_insert_keys<C>(j, tl, l);
}

template <uint32_t C>
__global__ __launch_bounds__(kTileBlock) HT_EIGHT_WAVES
void tile_finish_kernel(TileJob j) {
  __shared__ TileFinishLds<C> l;
  tile_finish_chunk<C>(j, blockIdx.x, l);
}

__global__ __launch_bounds__(kTileBlock) HT_EIGHT_WAVES
void tile_whole_kernel(DevTable t, const uint64_t* __restrict__ keys, uint64_t n, uint8_t* __restrict__ out) {
  __shared__ TileLds l;
  tile_whole_table(t, keys, n, out, l);
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  return ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32) |
         __builtin_amdgcn_readfirstlane((uint32_t)x);
}

__global__ __launch_bounds__(kTileBlock, 8) void tile_multi_partition_kernel(const TileJob* __restrict__ jobs,
                                                                             const uint64_t* __restrict__ items) {
  __shared__ TilePartLds<4096> l;
  const uint64_t it = uniform64(items[blockIdx.x]);
  tile_partition_chunk<4096>(jobs[it >> 32], (uint32_t)it, l);
}

__global__ __launch_bounds__(kTileBlock) HT_EIGHT_WAVES
void tile_multi_insert_kernel(const TileJob* __restrict__ jobs, const uint64_t* __restrict__ items) {
  __shared__ TileLds l;
  const uint64_t it = uniform64(items[blockIdx.x]);
  const TileJob& j = jobs[it >> 32];
  if (j.tiles) tile_insert_keys<4096>(j, (uint32_t)it, l);
  else tile_whole_table(j.t, j.keys, j.n, j.out, l);
}

__global__ __launch_bounds__(kTileBlock) HT_EIGHT_WAVES
void tile_multi_finish_kernel(const TileJob* __restrict__ jobs, const uint64_t* __restrict__ items) {
  __shared__ TileFinishLds<4096> l;
  const uint64_t it = uniform64(items[blockIdx.x]);
  tile_finish_chunk<4096>(jobs[it >> 32], (uint32_t)it, l);
}

hipError_t tile_multi(const TileJob* jobs, const uint64_t* chunks, uint32_t nchunks, const uint64_t* tiles,
                      uint32_t ntiles, hipStream_t st) {
  const dim3 b(kTileBlock);
  if (nchunks) hipLaunchKernelGGL(tile_multi_partition_kernel, dim3(nchunks), b, 0, st, jobs, chunks);
  if (ntiles) hipLaunchKernelGGL(tile_multi_insert_kernel, dim3(ntiles), b, 0, st, jobs, tiles);
  if (nchunks) hipLaunchKernelGGL(tile_multi_finish_kernel, dim3(nchunks), b, 0, st, jobs, chunks);
  return hipGetLastError();
}

static size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// Tiles: 8192 slots, down to 2048 while that leaves fewer than 512 of them (a
// block each, two to a compute unit).  Chunks: 4096 keys, 8192 from 2^21 keys
// on, where runs get short (2^22 keys into 2^23 slots, the three passes: 120
// us with 4096, 104 with 8192; 2^20 keys: 37 and 40, half the blocks).  Lanes
// per run: about a run's length.
TileShape tile_shape(uint64_t nslots, uint64_t n, uint32_t min_tiles, uint32_t chunk) {
  TileShape s{};
  s.shift = 13;
  while (s.shift > 11 && (nslots >> s.shift) < min_tiles) --s.shift;
  s.tiles = (uint32_t)((nslots + (1ull << s.shift) - 1) >> s.shift);
  s.chunk = chunk ? chunk : n >= kTileLongChunks ? 8192 : 4096;
  s.chunks = (uint32_t)((n + s.chunk - 1) / s.chunk);
  const uint64_t len = s.chunk / (s.tiles ? s.tiles : 1);
  s.run_lanes = 1;
  while (s.run_lanes < 64 && s.run_lanes < len) s.run_lanes <<= 1;
  const uint64_t keys = (uint64_t)s.chunks * s.chunk;
  s.bytes = up256(keys * 8) + up256(keys * 2) + up256(keys) + up256((uint64_t)s.chunks * (s.tiles + 1) * 2);
  return s;
}

TileJob tile_job(const DevTable& t, const uint64_t* keys, uint64_t n, uint8_t* out, const TileShape& s, void* ws) {
  TileJob j{};
  j.t = t;
  j.keys = keys;
  j.out = out;
  j.n = n;
  const uint64_t room = (uint64_t)s.chunks * s.chunk;
  char* c = static_cast<char*>(ws);
  const auto take = [&](size_t b) {
    char* p = c;
    c += up256(b);
    return p;
  };
  j.skey = reinterpret_cast<uint64_t*>(take(room * 8));
  j.sidx = reinterpret_cast<uint16_t*>(take(room * 2));
  j.sflag = reinterpret_cast<uint8_t*>(take(room));
  j.off = reinterpret_cast<uint16_t*>(take((uint64_t)s.chunks * (s.tiles + 1) * 2));
  j.chunks = s.chunks;
  j.tiles = s.tiles;
  j.shift = s.shift;
  j.run_lanes = s.run_lanes;
  j.run_most = 2 * (s.chunk / (s.tiles ? s.tiles : 1)) + 16;
  return j;
}

#define HT_TILE(KERNEL, GRID)                                                             \
  do {                                                                                    \
    if (s.tiles > kTileMax) return hipErrorInvalidValue;                                  \
    if (s.chunk == 4096)                                                                  \
      hipLaunchKernelGGL((KERNEL<4096>), dim3(GRID), dim3(kTileBlock), 0, st, j);         \
    else if (s.chunk == 8192)                                                             \
      hipLaunchKernelGGL((KERNEL<8192>), dim3(GRID), dim3(kTileBlock), 0, st, j);         \
    else                                                                                  \
      return hipErrorInvalidValue;                                                        \
    return hipGetLastError();                                                             \
  } while (0)

hipError_t tile_partition(const TileJob& j, const TileShape& s, hipStream_t st) {
  HT_TILE(tile_partition_kernel, s.chunks);
}

hipError_t tile_insert(const TileJob& j, const TileShape& s, hipStream_t st) {
  HT_TILE(tile_insert_kernel, (s.tiles + 7) / 8 * 8);
}

hipError_t tile_finish(const TileJob& j, const TileShape& s, hipStream_t st) { HT_TILE(tile_finish_kernel, s.chunks); }

hipError_t tile_whole(const DevTable& t, const uint64_t* keys, uint64_t n, uint8_t* out, hipStream_t st) {
  if (t.nrange * t.bucket_slots > kTileSlots) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tile_whole_kernel, dim3(1), dim3(kTileBlock), 0, st, t, keys, n, out);
  return hipGetLastError();
}

}  // namespace ht
