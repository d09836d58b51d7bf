// Launch wrappers for the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "slices.hpp"
#include "tiles.hpp"

namespace caramel {

// Cache policy of a launch's 128-bit loads and stores.
//  kStream   `nt` both ways
//  kThrough  `nt` loads, `sc1 nt` stores: a line is written through the XCD's L2 at once instead of
//            leaving it at some later eviction, so the writes reach HBM in the long contiguous runs
//            they were issued in.  In-place update of 8 x 512 MiB (16 x 96 MiB), same loads: plain
//            stores 68.0 (70.1), `nt` 73.6 (74.1), `sc1 nt` 76.5 (77.5) % of 8 TB/s.
enum Policy { kPlain = 0, kStream = 1, kThrough = 2 };

struct ReduceArgs {
  const ReduceTile* tiles;  // device
  const uint64_t* rows;     // device: (n_rows x W) base pointers
  uint32_t begin, count;    // tile range
  uint32_t world;
  bool bf16;
  Policy policy;
  bool tree;          // add as a balanced pairwise tree (halving-doubling) instead of a chain
  uint32_t unroll;    // vectors in flight per lane and worker: 1, 2 or 4 (0 = choose from W)
  uint32_t max_grid;  // 0 = one workgroup per tile
  uint32_t block;     // lanes per workgroup: 256, 512 or 1024
  uint32_t stream_major;  // 0: a launch over small tiles, fetch all workers at once; else: walk the
                          // workers one by one with (up to) that many vectors per lane; 8 exists for
                          // fp32 chains and fp32 trees over 2 and 4 workers, everything else gets 4
};

struct SliceArgs {
  const uint32_t* at;     // device (SliceTable)
  const uint32_t* bytes;  // device
  uint64_t base;
  uint32_t groups;        // workgroups
  uint32_t lanes, vecs;   // SliceShape
  uint32_t world;
  bool bf16;
  Policy policy;          // kStream or kThrough
  bool tree;
};

struct CopyArgs {
  const CopyTile* tiles;  // device
  const uint64_t* rows;   // device
  uint32_t begin, count;
  uint32_t world;
  uint32_t fused_row;
  bool bf16;
  bool unpack;  // false: tensors -> fused buffers; true: fused buffers -> tensors
  Policy policy;  // kStream for copies too large to stay in the caches, else kPlain
};

// Ring reduce-scatter arithmetic + 1/W scaling + all-gather for a range of tiles.
hipError_t launch_ring_reduce(const ReduceArgs& a, hipStream_t stream);
// The same for a job that was cut into slices.
hipError_t launch_slices(const SliceArgs& a, hipStream_t stream);
// Writes the tables `at` and `bytes` (SliceTable) from the pieces and the (n_tensors + 1) x W base addresses; all in
// device memory.
hipError_t launch_slice_table(const SliceTable& t, const SlicePiece* pieces, const uint64_t* rows, uint32_t* at,
                              uint32_t* bytes, hipStream_t stream);
// Segmented gather (pack) or scatter (unpack) driven by the copy-tile table.
hipError_t launch_copy(const CopyArgs& a, hipStream_t stream);

}  // namespace caramel
