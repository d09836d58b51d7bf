#include "slices.hpp"

#include <algorithm>

namespace caramel {
namespace {

// Calls f(row, first worker, byte offset in the row, bytes) for every slice, in unit order.  Slices end on
// multiples of kSliceBytes in memory, in most replicas if they lie differently.
template <typename F>
void for_each_slice(const HostPlan& p, const uint64_t* row_addr, F&& f) {
  const uint32_t W = p.cfg.world;
  const uint64_t es = p.elem_size();
  uint32_t phase_row = ~0u;
  uint64_t phase = 0;  // position of row `phase_row` inside a block of kSliceBytes
  auto common_phase = [&](uint32_t row) {
    if (row == phase_row) return phase;
    const uint64_t* a = row_addr + size_t(row) * W;
    uint32_t best = 0;
    for (uint32_t w = 0; w < W && 2 * best < W; ++w) {
      const uint64_t mine = a[w] % kSliceBytes;
      uint32_t n = 0;
      for (uint32_t x = 0; x < W; ++x) n += a[x] % kSliceBytes == mine;
      if (n > best) best = n, phase = mine;
    }
    phase_row = row;
    return phase;
  };
  auto cut = [&](uint32_t row, uint64_t row_elem, uint64_t n, uint32_t first) {
    const uint64_t ph = common_phase(row), end = (row_elem + n) * es;
    for (uint64_t at = row_elem * es; at < end;) {
      const uint64_t len = std::min(kSliceBytes - (ph + at) % kSliceBytes, end - at);
      f(row, first, at, uint32_t(len));
      at += len;
    }
  };
  for (uint32_t ui = 0; ui < p.units.size(); ++ui) {
    const caramel_unit& u = p.units[ui];
    const uint64_t* seg = p.segments(ui);
    const caramel_entry* ent = &p.entries[u.first_entry];
    // [lo, hi) in unit positions, starting at element `row_elem` of `row`.  Ring: the sums of segment c
    // start at worker c + 1; shuffle adds from worker 0 everywhere.
    auto add = [&](uint32_t row, uint64_t row_elem, uint64_t lo, uint64_t hi) {
      if (p.cfg.pattern != CARAMEL_PATTERN_RING) return cut(row, row_elem, hi - lo, 0);
      for (uint32_t c = 0; c < W; ++c) {
        const uint64_t a = std::max(lo, seg[c]), b = std::min(hi, seg[c + 1]);
        if (a < b) cut(row, row_elem + (a - lo), b - a, (c + 1) % W);
      }
    };
    if (u.kind == CARAMEL_KIND_CHUNK) {
      add(ent[0].tensor, ent[0].tensor_off, 0, u.elems);
    } else {
      for (uint32_t k = 0; k < u.n_entries; ++k)
        add(ent[k].tensor, ent[k].tensor_off, ent[k].unit_off, ent[k].unit_off + ent[k].elems);
    }
  }
}

}  // namespace

bool may_have_slices(const HostPlan& p) {
  return !(p.cfg.pattern == CARAMEL_PATTERN_HALVING_DOUBLING && p.cfg.world > 1) &&
         p.replica_elems * p.elem_size() < (uint64_t(32) << 20);
}

uint64_t count_slices(const HostPlan& p, const uint64_t* row_addr) {
  uint64_t n = 0;
  for_each_slice(p, row_addr, [&](uint32_t, uint32_t, uint64_t, uint32_t) { ++n; });
  return n;
}

// Measured on MI355X, microseconds, tiles / slices, data not in the last-level cache where they fit no more.
//  * One round: if all slices fit the registers of 256 workgroups at a time, every compute unit reads its whole
//    share, worker by worker, and then writes it, all of them at the same time: reads and writes hardly
//    mix at the memory.  Workgroups of 256 lanes hold 20 vectors per lane in fp32, 16 in bf16 (8 workers fp32:
//    4 MiB per replica 14.6 / 12.2, 12 MiB 38.9 / 34.6, 16 MiB 52.3 / 46.3; 16 workers 16 MiB 109 / 94; 2 workers
//    16 MiB 14.0 / 12.0; 8 workers bf16 12 MiB 39.4 / 36.4).  The fewer, longer stretches of memory win over
//    the last compute units: vectors are dealt out so that about 210 of them have work (12 MiB: 34.6 over 195, 35.2
//    over 223; with all in 256 lanes x 12, which takes two rounds, 43.6).
//  * Below some 2300 slices workgroups of one vector per lane, whose values all workers send at once, are
//    over sooner (8 workers 2 MiB 8.4 / 7.1, four vectors 7.5; 3 MiB 11.6 / 9.8, one vector 11.1); up to 4
//    workers there are fewer steps to wait for (4 workers bf16 2.7 MiB 5.7, one vector 5.6, four 5.8).
//  * Above one round of 256 lanes, fp32: from 16 workers on one round of 512 lanes (24 workers 26 MiB 247 / 238, 32
//    workers 31 MiB 414 / 375); 8 to 15 workers 1024 lanes in equal shares (8 workers 31 MiB 100 / 90, 12 workers
//    144 / 136), but where that comes to seven vectors per lane again 512 lanes (12 workers 27 MiB 122.5 / 125.4,
//    with 512 lanes 122).  Up to 7 workers, and with bf16 but for 9 to 24 workers, one vector per lane
//    in many rounds (5 workers 31 MiB 59 / 58, 1024 lanes 56 but 49.8 / 46.9 at 26; 8 workers bf16 98 / 92, 1024
//    lanes 96; 12 workers bf16 143 / 139, one vector 142.5).  One worker has tiles there (26 MiB 11.5 / 13.0).
SliceShape choose_slices(const HostPlan& p, uint64_t n) {
  const uint32_t W = p.cfg.world;
  // (the table of a job of very many tiny tensors would outgrow them)
  if (!may_have_slices(p) || n == 0 || n * W > (1u << 23)) return {};
  const bool bf16 = p.cfg.dtype == CARAMEL_BF16;
  const uint32_t most = bf16 ? 16 : 20;  // vectors per lane that fit the registers
  auto even = [](uint64_t v, uint32_t lo, uint32_t hi) { return std::clamp(uint32_t((v + 1) / 2 * 2), lo, hi); };
  SliceShape s{256, 1, 4};
  if (n <= (W <= 4 ? 3328u : 2304u)) return s;
  if (n <= uint64_t(4) * most * kComputeUnits) {
    s.vecs = even((n + 849) / 850, 4, most);
    s.share = 4 * s.vecs;
  } else if (W == 1) {
    return {};
  } else if (!bf16 && (W >= 16 || (W >= 8 && (n + 4095) / 4096 == 7)) && n <= uint64_t(8) * most * kComputeUnits) {
    s.lanes = 512;
    s.vecs = even((n + 1549) / 1550, 14, most);
    s.share = 8 * s.vecs;
  } else if (bf16 ? W > 8 && W <= 24 : W >= 8) {
    const uint64_t full = 16 * (bf16 ? 6 : 8) * kComputeUnits, rounds = (n + full - 1) / full;
    s.lanes = 1024;
    s.share = uint32_t((n + rounds * kComputeUnits - 1) / (rounds * kComputeUnits));
    s.vecs = std::max<uint32_t>(bf16 ? 4 : 5, (s.share + 15) / 16);
  }
  return s;
}

void build_slices(const HostPlan& p, const SliceShape& shape, const uint64_t* row_addr, SliceTable& out) {
  out = SliceTable{};
  if (!shape.vecs) return;
  const uint32_t W = p.cfg.world, V = shape.vecs, waves = shape.lanes / 64;
  const uint64_t n = count_slices(p, row_addr);
  out.lanes = shape.lanes;
  out.vecs = V;
  out.groups = uint32_t((n + shape.share - 1) / shape.share);
  // (sixteen more addresses: the kernel for one slice per wavefront looks eight workers up at a time)
  out.addr.assign(size_t(out.groups) * waves * V * W + 16, 0);
  out.bytes.assign(size_t(out.groups) * waves * (V + 1), 0);
  uint64_t i = 0;
  for_each_slice(p, row_addr, [&](uint32_t row, uint32_t first, uint64_t at, uint32_t len) {
    const uint32_t r = uint32_t(i % shape.share), u = r / waves;
    const size_t wave = size_t(i / shape.share) * waves + r % waves;
    out.bytes[wave * (V + 1) + u] = (len + 3) & ~3u;
    if (len & 3u) out.bytes[wave * (V + 1) + V] |= 1u << u;
    for (uint32_t k = 0; k < W; ++k)
      out.addr[(wave * W + k) * V + u] = row_addr[size_t(row) * W + (first + k) % W] + at;
    ++i;
  });
}

}  // namespace caramel
