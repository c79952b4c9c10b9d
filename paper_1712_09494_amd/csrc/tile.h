// Tiled find-or-put: shared declarations.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ht_device.h"

namespace ht {

constexpr uint32_t kTileSlots = 8192;       // most slots of a tile: 64 KiB of LDS, two blocks per compute unit
constexpr uint32_t kTileMax = 4096;         // most tiles of a table (the partition's LDS counters)

// One bucketed table's tiled find-or-put.
struct TileJob {
  DevTable t;
  const uint64_t* keys;
  uint8_t* out;             // may be NULL
  uint64_t n;
  uint64_t* skey;           // keys, each chunk sorted by tile
  uint16_t* sidx;           // their places within the chunk
  uint8_t* sflag;           // their flags
  uint16_t* off;            // chunks * (tiles + 1): start of each tile's run in the chunk
  uint32_t chunks;
  uint32_t tiles;
  uint32_t shift;           // log2 of the slots of a tile
  uint32_t run_lanes;       // lanes that serve one run (a power of two)
  uint32_t run_most;        // longest run that keys without copies make
};

// An item of a many-table launch: a chunk or a tile of a job (tiles == 0: the
// whole table by one block).
__host__ __device__ inline uint64_t tile_item(uint32_t job, uint32_t part) { return ((uint64_t)job << 32) | part; }

// Shape of a tiled find-or-put of n keys into a table of nslots slots, and
// the workspace it needs.
struct TileShape {
  uint32_t tiles, chunks, chunk, shift, run_lanes;
  size_t bytes;
};

constexpr uint64_t kTileLongChunks = 1ull << 21;   // chunks of 8192 keys from so many keys on

// `min_tiles`: tiles are made smaller (to 2048 slots) while there are fewer;
// `chunk`: 4096 or 8192 keys, 0 to choose by n.
TileShape tile_shape(uint64_t nslots, uint64_t n, uint32_t min_tiles = 512, uint32_t chunk = 0);
// The job of a call, its workspace `ws` holding shape.bytes.
TileJob tile_job(const DevTable& t, const uint64_t* keys, uint64_t n, uint8_t* out, const TileShape& s, void* ws);

// The three passes.
hipError_t tile_partition(const TileJob& j, const TileShape& s, hipStream_t st);
hipError_t tile_insert(const TileJob& j, const TileShape& s, hipStream_t st);
hipError_t tile_finish(const TileJob& j, const TileShape& s, hipStream_t st);
// One block, the whole table in LDS (at most kTileSlots slots).
hipError_t tile_whole(const DevTable& t, const uint64_t* keys, uint64_t n, uint8_t* out, hipStream_t st);

// The same for many tables (every job with chunks of 4096 keys): `chunks` are
// the (job, chunk) items of the partition and finish passes, `tiles` the (job,
// tile) items of the tile pass, in device memory.
hipError_t tile_multi(const TileJob* jobs, const uint64_t* chunks, uint32_t nchunks, const uint64_t* tiles,
                      uint32_t ntiles, hipStream_t st);

}  // namespace ht
