// Descriptor tables that drive the kernels.  Built on the host from a HostPlan, uploaded at
// bind time.  All offsets are in 16-byte vectors relative to a "pointer row": row t < n_tensors
// is tensor t (one base pointer per worker), row n_tensors is the fused workspace.
#pragma once

#include <cstdint>
#include <vector>

#include "plan.hpp"

namespace caramel {

// One workgroup's share of the ring reduction: a piece of one row that lies inside one ring
// segment, or straddles boundaries between consecutive ones.  Inside a segment the chain of
// workers is the same for every lane; the sums of the next segment start one worker later.
constexpr uint32_t kMaxSplits = 4;  // boundaries a tile can hold
struct ReduceTile {
  uint32_t row;      // pointer row
  uint32_t first;    // worker whose value is read first: (segment + 1) mod W for the ring, else 0
  uint32_t vec_off;  // offset of the piece inside the row, in 16-byte vectors
  uint32_t n_elems;  // elements in the piece; only a piece that ends a tensor may be ragged
  uint32_t split;    // 0, or the number of elements that belong to the first of several segments (a
                     // multiple of the vector size): the sums of the elements from `split` on
                     // start at worker first + 1 (mod W)
  uint32_t more[kMaxSplits - 1];  // further boundaries likewise, ascending, 0 when there are no more:
                                  // the sums of the elements from more[i] on start at first + i + 2
};

// One workgroup's share of pack / unpack: a run of one batch member.
struct CopyTile {
  uint32_t row;        // tensor row
  uint32_t t_vec_off;  // offset inside the tensor, in vectors
  uint32_t f_vec_off;  // offset inside a replica's fused buffer, in vectors
  uint32_t n_elems;    // elements to copy
  uint32_t n_zero;     // padding elements that follow in the fused buffer (pack writes +0.0)
  uint32_t pad_[3];
};

struct Range {
  uint32_t begin = 0, count = 0;
};

// A run is a maximal contiguous piece of one row (a tensor, or the fused buffer) that belongs to
// one unit: a whole chunk, a whole member of a batch unit reduced in place, or a batch unit's
// region of the fused buffer.  It consists of one part per ring segment it crosses.  Runs are
// cut into tiles along aligned blocks of memory, whatever the segment boundaries; a tile that
// contains boundaries carries their positions (`split`, `more`), and where a tile would contain more
// than `max_splits` of them, it ends at the next.  Long runs are cut into long tiles, for 1024-lane
// workgroups that walk the replicas one after the other; the rest into small tiles, for 256-lane
// workgroups that fetch all replicas at once.
struct TileShape {
  uint32_t long_vecs = 0;              // vectors per long tile; 0 (options only) = chosen at bind: 2048, 4096 or 8192
  uint32_t small_vecs = 256;           // vectors per small tile
  uint64_t long_run_bytes = 0;         // a run of at least this many bytes per replica is long; 0 (options only) = chosen at bind
  uint32_t copy_vecs = 1024;           // vectors per copy tile: one per lane of the copy kernel's workgroup
  // Where every replica of a run has the same address modulo the tile size, the first tile of
  // the run is shortened so that all later ones start on multiples of the tile size in memory
  // (bit 0: small tiles, bit 1: long tiles).
  uint32_t align_tiles = 3;
  bool split_tiles = false;  // tiles may straddle segment boundaries (set at bind if the kernel handles them)
  uint32_t max_splits = 1;   // boundaries a long tile may hold then, at most kMaxSplits and world - 1
  uint32_t small_splits = 1; // ... and a small tile
  // The last `tail_tiles` long tiles of every stream are cut into pieces of `tail_vecs` vectors:
  // when a launch runs out of tiles the workgroups still at work finish at different times, and
  // with short pieces at the end that drain is short.  Over 104 calls of 66 MiB to 10 GB 0, 32, 128 and
  // 256 are on average 0.5, 0.4, 0.8 and 3.6 % slower than 64, and each of them faster in some (0: by up
  // to 3 %, where whole rounds of workgroups come out even).
  uint32_t tail_tiles = 64;
  uint32_t tail_vecs = 1024;
};

enum { kLong = 0, kSmall = 1 };


struct UnitTiles {
  Range tiles[2];                // [class] range in the table
  uint64_t elems[2] = {0, 0};    // [class] elements covered
};

struct TileTables {
  // Both reduce tables are ordered class by class, stream by stream, unit by unit: the long
  // tiles of the units of stream 0, of stream 1, then the small tiles likewise.  So the tiles of
  // one class of consecutive units of a stream are adjacent.
  std::vector<ReduceTile> staged;  // batch units on the fused row, chunk units on tensor rows
  std::vector<ReduceTile> direct;  // batch units addressed through their member tensors
  std::vector<CopyTile> copy;      // stream by stream, unit by unit
  std::vector<uint32_t> order[2];  // [stream] -> its units, in plan order
  std::vector<UnitTiles> staged_unit, direct_unit;
  std::vector<Range> copy_unit;
  Range copy_stream[2];            // copy tiles of all batch units of a stream
};

// Whether the kernel that launch_ring_reduce picks for the long (stream_major != 0) or small tiles of
// this world size handles tiles that straddle segment boundaries (ReduceTile::split != 0).  The tile
// tables must hold none otherwise.
bool reduce_handles_split_tiles(uint32_t world, bool long_tiles);
// Fills in what the options leave to the library: tile sizes, which runs are long, where tiles may hold
// boundaries.  `split_tiles`, `stream_major` and `block` are the options of those names; `few_tiles`: the
// tables must stay small, even where that is not the fastest.
void choose_shape(const HostPlan& p, bool split_tiles, uint32_t stream_major, uint32_t block, bool few_tiles,
                  TileShape& ts);

// `row_addr`, if given, holds (n_tensors + 1) x W base addresses, row-major (the last row is
// the fused workspace; zeros if there is none): needed to cut tiles on aligned blocks.
void build_tiles(const HostPlan& p, const TileShape& ts, TileTables& out, const uint64_t* row_addr = nullptr);

}  // namespace caramel
