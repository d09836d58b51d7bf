#include "slices.hpp"

#include <algorithm>

namespace caramel {
namespace {

// Position of a row's start inside an aligned block of kSliceBytes: the same in every replica, or that of most.
uint64_t common_phase(const uint64_t* row_addr, uint32_t row, uint32_t W) {
  const uint64_t* a = row_addr + size_t(row) * W;
  uint64_t phase = 0;
  uint32_t best = 0;
  for (uint32_t w = 0; w < W && 2 * best < W; ++w) {
    const uint64_t mine = a[w] % kSliceBytes;
    uint32_t n = 0;
    for (uint32_t x = 0; x < W; ++x) n += a[x] % kSliceBytes == mine;
    if (n > best) best = n, phase = mine;
  }
  return phase;
}

}  // namespace

uint64_t slice_pieces(const HostPlan& p, const uint64_t* row_addr, std::vector<SlicePiece>& out) {
  out.clear();
  const uint32_t W = p.cfg.world;
  const uint64_t es = p.elem_size();
  uint64_t n = 0, phase = 0;
  uint32_t phase_row = ~0u;
  // `elems` of `row` from element `row_elem` on, added from worker `first` on
  auto cut = [&](uint32_t row, uint64_t row_elem, uint64_t elems, uint32_t first) {
    if (row != phase_row) phase = common_phase(row_addr, row, W), phase_row = row;
    const uint64_t at = row_elem * es, end = at + elems * es;
    out.push_back(SlicePiece{uint32_t(n), row, uint32_t(at / 16), uint32_t(end - at), uint16_t(phase), uint16_t(first)});
    n += slices_of(out.back());
  };
  for (uint32_t ui = 0; ui < p.units.size(); ++ui) {
    const caramel_unit& u = p.units[ui];
    const uint64_t* seg = p.segments(ui);
    const caramel_entry* ent = &p.entries[u.first_entry];
    // [lo, hi) in unit positions, starting at element `row_elem` of `row`.  Ring: the sums of segment c
    // start at worker c + 1; the other patterns read from worker 0 everywhere.
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
  return n;
}

// Up to 32 MiB per replica slices are the better cut but for the shapes that choose_slices leaves out.  Few workers
// have them longer: their walks over long tiles are short, and a tile that is left over at the end, or at a segment
// boundary, weighs as much as elsewhere (us, tiles / slices, fp32 ring unless said otherwise: 2 workers 90 MiB 69.5 /
// 61.0, 110 MiB 80.2 / 75.0, bf16 75.0 / 73.8, but 190 MiB 125.4 / 126.6; 4 workers 42 MiB 61.3 / 59.5, bf16 56 MiB
// 81.0 / 83.4; 6 workers 48 MiB 106.2 / 101.5, 65 MiB 137.6 / 141.0; 8 workers 33 MiB 109 / 103, 37 MiB 118.5 / 112.1,
// but shuffle 38 MiB 108.9 / 116.3; 12 workers 37 MiB 166.5 / 167.6; halving-doubling over 4 42 MiB 63.1 / 60.4, over
// 8 33 MiB 96.4 / 98.9).
bool may_have_slices(const HostPlan& p) {
  const uint32_t W = p.cfg.world;
  const bool tree = p.cfg.pattern == CARAMEL_PATTERN_HALVING_DOUBLING;
  const uint64_t mib = W == 2 ? 112 : (W > 2 && W <= (tree ? 4u : 6u) ? 48 : (!tree && (W == 7 || W == 8) ? 36 : 32));
  return p.replica_elems * p.elem_size() < mib << 20;
}

// Longest mean length of the pieces with which a job above 32 MiB per replica has slices: what they save are tiles that
// are left over at the ends of pieces.  Tiles = 1, three placements of the replicas each: shuffle over 8 workers, 33 to 35.5
// MiB: pieces of 170 KiB (200 tensors) 0.93 to 0.97, 450 KiB (60 tensors) 0.97 to 1.06, 3 to 4.5 MiB (four tensors and one)
// 0.99 to 1.09; rings over 8, which have eight times the pieces: 90 KiB 0.90 to 0.93, 430 KiB 0.94 to 1.00, 540 KiB (one
// tensor) 0.92 to 1.03, 568 KiB 0.99 to 1.05.  7 workers: 3 MiB 0.95 to 1.03, 4.3 MiB 1.00 to 1.03.  2 workers in bf16 from 90
// MiB on: 1 MiB 0.90 to 0.97, 4 MiB 0.98 to 1.01, 6 to 8 MiB 0.97 to 1.03, 11 to 14 MiB 1.00 to 1.04; in fp32 at most 1.00.
// 3 to 6 workers: 4 to 6 MiB 0.96 to 1.02.
static uint64_t longest_mean_piece(const HostPlan& p) {
  const uint32_t W = p.cfg.world;
  if (W == 8) return (p.cfg.pattern == CARAMEL_PATTERN_RING ? 560 : 448) << 10;
  if (W == 7) return 4 << 20;
  return W == 2 && p.cfg.dtype == CARAMEL_BF16 ? 5 << 20 : ~uint64_t(0);
}

// Measured on MI355X, microseconds, tiles / slices, data not in the last-level cache where they fit no more.
//  * One round: if all slices fit the registers of 256 workgroups at a time, every compute unit reads its whole
//    share, worker by worker, and then writes it, all of them at the same time: reads and writes hardly
//    mix at the memory (8 workers fp32 4 MiB per replica 14.6 / 11.6, 12 MiB 38.9 / 34.2, 16 MiB 51.2 / 47.1; 16
//    workers 16 MiB 107 / 96; 2 workers 16 MiB 14.0 / 11.7; 8 workers bf16 12 MiB 41.2 / 34.6; halving-doubling, 8
//    workers 13.5 MiB 46.0 / 36.8, 64 workers 3 MiB 85 / 70).  From some 8 MiB on the fewer, longer stretches of
//    memory win over the last compute units: vectors are dealt out so that about 210 of them have work (12 MiB:
//    34.6 over 195, 35.2 over 223; with all in 256 lanes x 12, which takes two rounds, 43.6); below, the work is
//    spread over as many as there are (4 workers 3.3 MiB 5.7 over 215, 6.1 over 143).
//  * Below some 2000 slices workgroups of one vector per lane, whose values all workers send at once, are
//    over sooner (8 workers 1.2 MiB 6.0, two vectors 6.1, four 6.6; 2.1 MiB 8.2, four 7.5).  Up to 4 workers there
//    are fewer steps to wait for (4 workers 2.2 MiB 5.2, four vectors 5.3; 2.7 MiB 5.5 / 5.3).  Trees, which take
//    the workers by pairs, have two vectors from 1000 slices on (16 workers 1.5 MiB 11.4, two vectors 9.7).
//  * Many tensors of a few hundred bytes: slices are short, and what counts is how many of them are on their way.  One
//    per wavefront where otherwise four would take turns (ring, tiles / four / one: 16 workers 2500 tensors of 64 bytes
//    6.45 / 8.54 / 5.91, 3000 of 256 7.7 / 8.9 / 7.1, 8 workers 5.3 / 5.4 / 4.2; 6000, eight vectors: 8 workers 8.2 / 6.5,
//    16 12.6 / 11.4), and beyond one round, with up to 15 fp32 workers up to 700 bytes a slice (8 workers 15000 of
//    1200 bytes 60.8 / 1024 lanes 61.9 / 56.9, 16 workers 60000 of 64 86.4 / 512 lanes 84.4 / 67.3).
//  * Stores: what one round writes is left to the last-level cache, where it fits (8 workers 4 MiB 12.6 written
//    through, 11.6; 2 workers 12 MiB 9.2 / 8.8; called one at a time 8 x 15 MB 56.0 / 53.0; 32 workers 12 MiB, 384
//    MiB in all, 142 / 144).  Longer jobs write while others read, and are better off through (4 workers 30
//    MiB 43.8 / 44.9, 8 workers 87.4 / 90.1), but for up to 64 MiB in all: where those are still in the caches, writing
//    through made them slower than tiles (2 workers bf16 17 MiB, called over and over on the same memory 11.4 tiles /
//    13.6 through / 11.8, with others in between 14.6 / 13.6 / 14.3; 31 MiB 21.7 / 22.6 / 21.4 and 23.5 / 22.3 / 22.9).
//  * Above one round of 256 lanes, fp32 chains: from 16 workers on one round of 512 lanes (24 workers 26 MiB 247 /
//    238, 32 workers 31 MiB 414 / 375); 8 to 15 workers 1024 lanes in equal shares (8 workers 31 MiB 100 / 90, 12
//    workers 144 / 136), but where that comes to seven vectors per lane again 512 lanes (12 workers 27 MiB
//    122.5 / 125.4, with 512 lanes 122), and rings one vector per lane where the last row of slices would be nearly
//    empty, over 9 workers also where the sixth is not full (tiles / 1024 lanes / one vector: 20 MiB 8 workers 62.7 / 62.9
//    / 60.4, 9 68.9 / 70.8 / 67.4, 12 92.0 / 93.3 / 92.0; 23 MiB 9 workers 77.9 / 78.3 / 77.0; 27.7 MiB 14 workers 148.7 /
//    154.4 / 147.5; shuffle over 12 and more of 20 MiB 1024 lanes 1 to 5 % faster).  bf16 chains over 12 to 24 workers from
//    20 MiB on likewise (12 workers 143 / 139, one vector 142.5).  Up to 7 workers, and with bf16 otherwise, one vector per
//    lane in many rounds (5 workers 31 MiB 59 / 58, 1024 lanes 56 but 49.8 / 46.9 at 26; bf16: 8 workers 98 / 92, 1024
//    lanes 96; 9 workers 31.5 MiB 107.9 / 103.6, 107.3; 10 118.4 / 117.0, 127.9; 11 20.3 MiB 85.4 / 84.2, 85.4), and so for
//    trees (8 workers 25 MiB 79.9 / 75.3, 16 workers 170 / 158, bf16 165 / 153).  One worker has tiles there (26 MiB 11.5 /
//    13.0), and so have 12 to 15 workers in bf16 where a second round of 1024 lanes would be nearly empty (12 workers 24 MiB
//    108 / 111), halving-doubling over 64 in fp32 (16 MiB 440 / 447), and over 32 and 64 if pieces are long (one large
//    tensor 2 to 5 % slower: 32 workers 31 MiB 411.8 / 422.5, 64 in bf16 15 MiB 418 / 435; 60 tensors 3 % faster to 1 % slower,
//    200 and more, pieces of 150 KiB and less, 0 to 4 % faster, 20000 11 %).
SliceShape choose_slices(const HostPlan& p, uint64_t n, uint64_t n_pieces) {
  const uint32_t W = p.cfg.world;
  const uint64_t replica_bytes = p.replica_elems * p.elem_size();
  // (the table of a job of very many tiny tensors would outgrow them)
  if (!may_have_slices(p) || n == 0 || n * W > (1u << 23)) return {};
  if (replica_bytes >= (uint64_t(32) << 20) && replica_bytes / n_pieces > longest_mean_piece(p)) return {};
  const bool bf16 = p.cfg.dtype == CARAMEL_BF16;
  const bool tree = p.cfg.pattern == CARAMEL_PATTERN_HALVING_DOUBLING && W > 1;
  // vectors per lane that fit the registers: two buffers and the sum, or four buffers and a sum for every level
  const uint32_t most = !tree ? (bf16 ? 16 : 20)
                              : (bf16 ? (W <= 4 ? 16 : (W == 8 ? 14 : (W == 16 ? 10 : 8)))
                                      : (W <= 4 ? 20 : (W == 8 ? 18 : (W <= 32 ? 14 : 12))));
  auto up = [](uint64_t v, uint32_t step) { return uint32_t((v + step - 1) / step * step); };
  SliceShape s{256, 1, 4, W * replica_bytes > (uint64_t(256) << 20)};
  if (n <= (tree ? 1024u : (W <= 4 ? 2560u : 2048u))) return s;
  const uint64_t whole = uint64_t(4) * most * kComputeUnits;  // slices of one round of 256 lanes
  const bool one_round = n <= whole, large = W * replica_bytes > (uint64_t(64) << 20);
  const uint32_t shortest = one_round ? (n <= 4096 ? 320 : 0) : (!bf16 && W >= 8 && W < 16 ? 700 : 320);
  if (replica_bytes < n * shortest) {
    s.through = large && !(tree && W >= 32);
    return s;
  }
  if (one_round) {
    const uint64_t each = n <= 8192 ? 4 * kComputeUnits : 850;
    s.vecs = std::min(most, up((n + each - 1) / each, tree && n > 8192 ? 4 : 2));
    if (!tree) s.vecs = std::max(s.vecs, 4u);
    if (tree) s.through = false;
    s.share = 4 * s.vecs;
    return s;
  }
  const bool long_pieces = replica_bytes / n_pieces > (192 << 10) || (W == 64 && !bf16);
  if (W == 1 || (tree && W >= 32 && long_pieces) || (bf16 && W >= 12 && W < 16 && n > 24576 && n <= 28672)) return {};
  s.through = large && !(tree && W >= 32);
  if (tree || replica_bytes >= (uint64_t(32) << 20)) return s;
  if (!bf16 && (W >= 16 || (W >= 8 && (n + 4095) / 4096 == 7)) && n <= uint64_t(8) * most * kComputeUnits) {
    s.lanes = 512;
    s.through = true;
    s.vecs = std::clamp(up((n + 1549) / 1550, 2), 14u, most);
    s.share = 8 * s.vecs;
  } else if (bf16 ? W >= 12 && W <= 24 && n > 20480 : W >= 8) {
    const uint64_t full = 16 * (bf16 ? 6 : 8) * kComputeUnits, rounds = (n + full - 1) / full;
    const uint32_t share = uint32_t((n + rounds * kComputeUnits - 1) / (rounds * kComputeUnits));
    if (p.cfg.pattern == CARAMEL_PATTERN_RING && ((share - 1) % 16 < 2 || (W == 9 && n <= 24576))) return s;
    s.lanes = 1024;
    s.through = true;
    s.share = share;
    s.vecs = std::max<uint32_t>(bf16 ? 4 : 5, (s.share + 15) / 16);
  }
  return s;
}

SliceTable slice_table(const HostPlan& p, const SliceShape& shape, uint64_t n_slices, uint64_t n_pieces,
                       const uint64_t* row_addr) {
  SliceTable t;
  if (!shape.vecs) return t;
  const uint32_t W = p.cfg.world;
  uint64_t lo = ~uint64_t(0), hi = 0;
  for (size_t r = 0; r < p.tensor_elems.size(); ++r)
    for (uint32_t w = 0; w < W; ++w) {
      const uint64_t a = row_addr[r * W + w];
      lo = std::min(lo, a);
      hi = std::max(hi, a + p.tensor_elems[r] * p.elem_size());
    }
  if ((hi - lo) >> 36) return t;
  t.lanes = shape.lanes;
  t.vecs = shape.vecs;
  t.share = shape.share;
  t.groups = uint32_t((n_slices + shape.share - 1) / shape.share);
  t.world = W;
  t.slices = uint32_t(n_slices);
  t.pieces = uint32_t(n_pieces);
  t.base = lo;
  return t;
}

}  // namespace caramel
