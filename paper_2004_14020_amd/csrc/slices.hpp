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
  // slices end on multiples of kSliceBytes in memory
  const uint64_t start = uint64_t(c.at) * 16 + c.phase, block = (start / kSliceBytes + (i - c.first_slice)) * kSliceBytes;
  const uint64_t begin = block > start ? block : start;
  const uint64_t end = block + kSliceBytes < start + c.bytes ? block + kSliceBytes : start + c.bytes;
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
