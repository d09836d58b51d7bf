// Slices: the work of a small job cut for workgroups that each get an equal share of it, whatever the runs.
#pragma once

#include <cstdint>
#include <vector>

#include "plan.hpp"

namespace caramel {

constexpr uint32_t kSliceBytes = 1024;  // one 16-byte vector per lane of a wavefront
constexpr uint32_t kComputeUnits = 256;

// A slice is a piece of at most kSliceBytes of one run, inside one ring segment: one order of workers for
// every lane.  A wavefront takes `vecs` of them, one vector per lane and slice, and a workgroup a stretch of
// slices that are neighbours in unit order, laid out row by row over its wavefronts.
//
// A wavefront's part of the tables, wavefronts in grid order:
//   at     W x vecs places: for step k the `vecs` slices in the worker that is added k-th, in 16-byte vectors from
//          `base` (half the bytes of addresses: what a call's first lookups wait for)
//   bytes  vecs lengths, rounded up to a whole dword (0: no slice), then a word whose bit u says that slice
//          u ends in the middle of its last dword (an odd number of bf16 values)
//
// The GPU writes them (launch_slice_table), from the pieces below: a bind uploads 20 bytes for each part of a run
// that lies in one segment, not 4 for every slice in every worker.

// A part of a row (tensor) inside one ring segment.
struct SlicePiece {
  uint32_t first_slice;  // slices of all pieces before it
  uint32_t row;
  uint32_t at;           // start, in 16-byte vectors from the start of the row
  uint32_t bytes;
  uint16_t phase;        // position of the row's start inside an aligned block of kSliceBytes: the same in
                         // every replica, or that of most
  uint16_t first;        // worker that is added first
};

// Slices end on multiples of kSliceBytes in memory, but a piece that one wavefront holds is one slice (tensors of 520
// bytes, half of them across such a multiple, ring over 8 workers, us, tiles / cut / whole: 6000 14.1 / 14.3 / 13.1, 15000
// 29.1 / 34.7 / 31.7).
constexpr uint32_t slices_of(const SlicePiece& c) {
  if (c.bytes <= kSliceBytes) return 1;
  const uint64_t start = uint64_t(c.at) * 16 + c.phase;
  return uint32_t((start + c.bytes + kSliceBytes - 1) / kSliceBytes - start / kSliceBytes);
}

struct SliceTable {
  uint32_t lanes = 0, vecs = 0, groups = 0;
  uint32_t share = 0;  // slices per workgroup
  uint32_t world = 0;
  uint32_t slices = 0, pieces = 0;
  uint64_t base = 0;  // the lowest address of any tensor
  constexpr uint32_t waves() const { return groups * (lanes / 64); }
  // words of the two tables (sixteen more: the kernel for one slice per wavefront looks eight workers up at a time)
  constexpr size_t at_words() const { return size_t(waves()) * vecs * world + 16; }
  constexpr size_t bytes_words() const { return size_t(waves()) * (vecs + 1); }
};

// Slice u of a wavefront: writes its places for the steps [k0, k1) to at[k0 * vecs], ... and returns its length in
// bytes (0: there is none, and all places are 0).
constexpr uint32_t place_slice(const SliceTable& t, const SlicePiece* pieces, const uint64_t* row_addr, uint32_t wave,
                               uint32_t u, uint32_t k0, uint32_t k1, uint32_t* at) {
  const uint32_t waves = t.lanes / 64, r = u * waves + wave % waves;
  const uint64_t i = uint64_t(wave / waves) * t.share + r;
  if (r >= t.share || i >= t.slices) {
    for (uint32_t k = k0; k < k1; ++k) at[size_t(k) * t.vecs] = 0;
    return 0;
  }
  // the last piece that starts at or before slice i
  uint32_t lo = 0, hi = t.pieces;
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if (pieces[mid].first_slice <= i) lo = mid;
    else hi = mid;
  }
  const SlicePiece& c = pieces[lo];
  const uint64_t start = uint64_t(c.at) * 16 + c.phase, block = (start / kSliceBytes + (i - c.first_slice)) * kSliceBytes;
  const bool whole = c.bytes <= kSliceBytes;
  const uint64_t begin = block > start ? block : start;
  const uint64_t end = !whole && block + kSliceBytes < start + c.bytes ? block + kSliceBytes : start + c.bytes;
  for (uint32_t k = k0; k < k1; ++k) {
    const uint32_t w = (c.first + k) % t.world;
    at[size_t(k) * t.vecs] = uint32_t((row_addr[size_t(c.row) * t.world + w] - t.base + begin - c.phase) / 16);
  }
  return uint32_t(end - begin);
}

struct SliceShape {
  uint32_t lanes = 0, vecs = 0;  // 0: the job has tiles instead
  uint32_t share = 0;            // slices per workgroup
  bool through = true;           // stores are written through the caches
};

// The kernels there are: choose_slices returns no other shapes, and each of these for some job.
//   ROUND(bf16, through, vecs, lanes)   chains, several slices per wavefront
//   ONE(bf16, through, world)           chains, one slice per wavefront; world 0: any other (listed last)
//   TREE_ROUND(world, bf16, vecs)       halving-doubling in one round of 256 lanes, not through
//   TREE_ONE(world, bf16, through)      halving-doubling, one slice per wavefront
#define CARAMEL_ROUNDS_256(ROUND, BF16) \
  ROUND(BF16, false, 4, 256) ROUND(BF16, false, 6, 256) ROUND(BF16, false, 8, 256) ROUND(BF16, false, 10, 256) \
  ROUND(BF16, false, 12, 256) ROUND(BF16, false, 14, 256) ROUND(BF16, false, 16, 256) ROUND(BF16, true, 6, 256) \
  ROUND(BF16, true, 8, 256) ROUND(BF16, true, 10, 256) ROUND(BF16, true, 12, 256) ROUND(BF16, true, 14, 256) \
  ROUND(BF16, true, 16, 256)
#define CARAMEL_ONES(ONE, BF16, THROUGH) \
  ONE(BF16, THROUGH, 2) ONE(BF16, THROUGH, 3) ONE(BF16, THROUGH, 4) ONE(BF16, THROUGH, 8) ONE(BF16, THROUGH, 0)
#define CARAMEL_TREE_ROUNDS_8(TREE_ROUND, W, BF16) \
  TREE_ROUND(W, BF16, 2) TREE_ROUND(W, BF16, 4) TREE_ROUND(W, BF16, 6) TREE_ROUND(W, BF16, 8)
#define CARAMEL_SLICE_KERNELS(ROUND, ONE, TREE_ROUND, TREE_ONE) \
  ONE(false, false, 16) ONE(true, false, 16) ONE(true, true, 16) \
  CARAMEL_ONES(ONE, false, false) CARAMEL_ONES(ONE, true, false) CARAMEL_ONES(ONE, false, true) \
  CARAMEL_ONES(ONE, true, true) \
  CARAMEL_ROUNDS_256(ROUND, false) ROUND(false, false, 18, 256) ROUND(false, false, 20, 256) \
  ROUND(false, true, 18, 256) ROUND(false, true, 20, 256) CARAMEL_ROUNDS_256(ROUND, true) \
  ROUND(false, true, 14, 512) ROUND(false, true, 16, 512) ROUND(false, true, 18, 512) ROUND(false, true, 20, 512) \
  ROUND(false, true, 5, 1024) ROUND(false, true, 6, 1024) ROUND(false, true, 7, 1024) ROUND(false, true, 8, 1024) \
  ROUND(true, true, 4, 1024) ROUND(true, true, 5, 1024) ROUND(true, true, 6, 1024) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 2, false) TREE_ROUND(2, false, 12) TREE_ROUND(2, false, 16) TREE_ROUND(2, false, 20) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 4, false) TREE_ROUND(4, false, 12) TREE_ROUND(4, false, 16) TREE_ROUND(4, false, 20) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 8, false) TREE_ROUND(8, false, 12) TREE_ROUND(8, false, 16) TREE_ROUND(8, false, 18) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 16, false) TREE_ROUND(16, false, 12) TREE_ROUND(16, false, 14) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 32, false) TREE_ROUND(32, false, 12) TREE_ROUND(32, false, 14) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 64, false) TREE_ROUND(64, false, 12) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 2, true) TREE_ROUND(2, true, 12) TREE_ROUND(2, true, 16) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 4, true) TREE_ROUND(4, true, 12) TREE_ROUND(4, true, 16) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 8, true) TREE_ROUND(8, true, 12) TREE_ROUND(8, true, 14) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 16, true) TREE_ROUND(16, true, 10) \
  CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 32, true) CARAMEL_TREE_ROUNDS_8(TREE_ROUND, 64, true) \
  TREE_ONE(2, false, false) TREE_ONE(4, false, false) TREE_ONE(8, false, false) TREE_ONE(16, false, false) \
  TREE_ONE(32, false, false) TREE_ONE(64, false, false) TREE_ONE(2, true, false) TREE_ONE(4, true, false) \
  TREE_ONE(8, true, false) TREE_ONE(16, true, false) TREE_ONE(32, true, false) TREE_ONE(64, true, false) \
  TREE_ONE(2, false, true) TREE_ONE(4, false, true) TREE_ONE(8, false, true) TREE_ONE(16, false, true) \
  TREE_ONE(2, true, true) TREE_ONE(4, true, true) TREE_ONE(8, true, true) TREE_ONE(16, true, true)

// Whether choose_slices could ever cut this plan into slices.
bool may_have_slices(const HostPlan& p);
// The pieces of the plan's units, batches in place; `row_addr`: (n_tensors + 1) x W base addresses.  Returns how many
// slices they come to.
uint64_t slice_pieces(const HostPlan& p, const uint64_t* row_addr, std::vector<SlicePiece>& out);
SliceShape choose_slices(const HostPlan& p, uint64_t n_slices, uint64_t n_pieces);
// No workgroups if some tensors lie too far apart (64 GiB) for the table.
SliceTable slice_table(const HostPlan& p, const SliceShape& shape, uint64_t n_slices, uint64_t n_pieces,
                       const uint64_t* row_addr);

}  // namespace caramel
