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
//          `base` (half the bytes of addresses: what a call's first lookups wait for, and what a bind uploads)
//   bytes  vecs lengths, rounded up to a whole dword (0: no slice), then a word whose bit u says that slice
//          u ends in the middle of its last dword (an odd number of bf16 values)
struct SliceTable {
  uint32_t lanes = 0, vecs = 0, groups = 0;
  uint64_t base = 0;  // the lowest address of any tensor
  std::vector<uint32_t> at, bytes;
};

struct SliceShape {
  uint32_t lanes = 0, vecs = 0;  // 0: the job has tiles instead
  uint32_t share = 0;            // slices per workgroup
  bool through = true;           // stores are written through the caches
};

// Whether choose_slices could ever cut this plan into slices.
bool may_have_slices(const HostPlan& p);
// Number of slices of the plan's units, batches in place; `row_addr`: (n_tensors + 1) x W base addresses.
uint64_t count_slices(const HostPlan& p, const uint64_t* row_addr);
SliceShape choose_slices(const HostPlan& p, uint64_t n_slices);
// Leaves `out` without workgroups if some tensors lie too far apart (64 GiB) for the table.
void build_slices(const HostPlan& p, const SliceShape& shape, const uint64_t* row_addr, SliceTable& out);

}  // namespace caramel
