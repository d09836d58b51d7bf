#include "tiles.hpp"

#include <algorithm>

namespace caramel {
namespace {

// One ring segment's part of a run.
struct Part {
  uint32_t first;  // worker whose value is read first
  uint64_t n;      // elements
};

struct Run {
  uint32_t row;
  uint64_t row_elem;  // start inside the row, in elements
  uint64_t n;         // length = sum of the parts
  std::vector<Part> parts;
};

// The i-th boundary inside a tile.
uint32_t& boundary(ReduceTile& t, uint32_t i) { return i == 0 ? t.split : t.more[i - 1]; }
uint32_t boundary(const ReduceTile& t, uint32_t i) { return i == 0 ? t.split : t.more[i - 1]; }

// The tile [at, at + len) of a run: first worker and boundaries (cut_run sees to it that there are
// at most kMaxSplits of them).
ReduceTile make_tile(const Run& r, uint64_t at, uint64_t len, uint64_t vec_elems) {
  ReduceTile t{};
  t.row = r.row;
  t.vec_off = uint32_t((r.row_elem + at) / vec_elems);
  t.n_elems = uint32_t(len);
  uint64_t part_begin = 0;
  uint32_t inside = 0;
  for (const Part& pt : r.parts) {
    const uint64_t part_end = part_begin + pt.n;
    if (part_begin <= at && at < part_end) t.first = pt.first;
    if (part_begin > at && part_begin < at + len) boundary(t, inside++) = uint32_t(part_begin - at);
    part_begin = part_end;
  }
  return t;
}

// Cut a run into tiles of `tile_elems`.  `phase_elems` is the position of the run's start
// inside a tile-sized block of memory (0 if unknown or not to be used): the first tile is
// shortened so that every later tile starts on a multiple of the tile size in memory.  A tile
// ends early at the part boundary that it would contain in excess of `max_splits`.  `phases`
// receives for every tile the position of its start inside such a block.
void cut_run(std::vector<ReduceTile>& out, const Run& r, uint64_t vec_elems, uint64_t tile_elems,
             uint64_t phase_elems, uint32_t max_splits, uint32_t world, std::vector<uint64_t>& phases) {
  std::vector<uint64_t> bounds;  // ends of the parts, relative to the run
  uint64_t acc = 0;
  for (const Part& pt : r.parts) bounds.push_back(acc += pt.n);
  uint64_t phase = phase_elems % tile_elems;
  for (uint64_t at = 0; at < r.n;) {
    uint64_t len = std::min(tile_elems - phase, r.n - at);
    // the parts end after `at`: the tile may run past the end of one if the sums of the next
    // part start exactly one worker later (what the kernels assume of a boundary inside a tile)
    const auto lo = std::upper_bound(bounds.begin(), bounds.end(), at);
    size_t part = size_t(lo - bounds.begin()), allowed = 0;
    while (allowed < max_splits && part + 1 < r.parts.size() &&
           r.parts[part + 1].first == (r.parts[part].first + 1) % world)
      ++allowed, ++part;
    if (size_t(bounds.end() - lo) > allowed && lo[allowed] < at + len) len = lo[allowed] - at;
    out.push_back(make_tile(r, at, len, vec_elems));
    phases.push_back(phase);
    at += len;
    phase = (phase + len) % tile_elems;
  }
}

// Cut the last `n_tail` tiles of tiles[begin..] into pieces of at most `piece_elems` elements
// (pieces of a tile stay where the tile was, in order) and move the tile ranges of the units
// along.  phases[i - begin] is the position of tile i's start inside a tile-sized block of
// memory; if the piece size divides the tile size, pieces are cut on multiples of the piece size
// in memory (the first piece of a tile that starts inside such a block is shortened).
void split_tail(std::vector<ReduceTile>& tiles, size_t begin, const std::vector<uint64_t>& phases, uint32_t n_tail,
                uint64_t piece_elems, bool align_pieces, uint64_t vec_elems, uint32_t world,
                std::vector<UnitTiles>& per_unit, const std::vector<uint32_t>& units) {
  const size_t n = tiles.size() - begin;
  if (n == 0) return;
  const size_t first = begin + (n > n_tail ? n - n_tail : 0);
  std::vector<ReduceTile> cut;
  std::vector<uint32_t> grew(tiles.size() - first, 0);  // pieces added per original tile
  for (size_t i = first; i < tiles.size(); ++i) {
    const ReduceTile& t = tiles[i];
    uint32_t pieces = 0;
    const uint64_t ph = align_pieces ? phases[i - begin] % piece_elems : 0;
    uint64_t len = ph ? piece_elems - ph : piece_elems;
    for (uint64_t at = 0; at < t.n_elems; at += len, len = piece_elems, ++pieces) {
      ReduceTile q = t;
      q.vec_off = uint32_t(t.vec_off + at / vec_elems);
      q.n_elems = uint32_t(std::min<uint64_t>(len, t.n_elems - at));
      // where the piece lies relative to the tile's segment boundaries
      q.split = 0;
      for (uint32_t& m : q.more) m = 0;
      uint32_t inside = 0;
      for (uint32_t k = 0; k < kMaxSplits && boundary(t, k); ++k) {
        const uint32_t bd = boundary(t, k);
        if (bd <= at) q.first = (t.first + k + 1) % world;
        else if (bd < at + q.n_elems) boundary(q, inside++) = uint32_t(bd - at);
      }
      cut.push_back(q);
    }
    grew[i - first] = pieces - 1;
  }
  // unit ranges: a unit's begin moves by the pieces added before it, its count by those inside
  for (uint32_t u : units) {
    Range& r = per_unit[u].tiles[kLong];
    uint32_t before = 0, inside = 0;
    for (size_t i = first; i < tiles.size(); ++i) {
      if (i < r.begin) before += grew[i - first];
      else if (i < size_t(r.begin) + r.count) inside += grew[i - first];
    }
    r.begin += before;
    r.count += inside;
  }
  tiles.resize(first);
  tiles.insert(tiles.end(), cut.begin(), cut.end());
}

}  // namespace

// the rolled walk does, and that of three workers; the unrolled ones for 1, 2, 4 and 8 workers and the
// kernel for the small tiles of these and of 16 do not
bool reduce_handles_split_tiles(uint32_t world, bool long_tiles) {
  return world > 2 && world != 4 && world != 8 && (world != 16 || long_tiles);
}

void choose_shape(const HostPlan& p, bool split_tiles, uint32_t stream_major, uint32_t block, bool few_tiles,
                  TileShape& ts) {
  const caramel_config& c = p.cfg;
  // Shapes left to the library (option value 0) follow the size of the job, measured on MI355X:
  //  * a replica of less than 32 MiB is done before long tiles pay off (a 1024-lane workgroup
  //    walks its tile one replica after the other): every run is cut into small tiles, whose
  //    workgroups fetch all replicas at once (small against long tiles, fp32: 2 x 16 MiB 13.6 / 14.0 us, 2 x
  //    33 25.0 / 25.2, 4 x 24 36.6 / 37.8, 4 x 33 50.0 / 49.1, 8 x 24 76.6 / 78.3, 8 x 33 104.5 / 104.1, 8 x
  //    48 155 / 145; 16 workers cross earlier, 8 MiB 54.0 / 69.3, 16 MiB 110 / 104);
  //  * fp32 chains keep eight vectors per lane in registers, so their long tiles can be 128 KiB,
  //    which stream best, but are few (256 workgroups run at a time, and the last round is felt).
  //    2, 4 and 8 workers take them from 64 MiB per replica on, two rounds (VGG-16, 528 MiB: 1438 ->
  //    1396 us, ResNet-50, 98 MiB: 275.3 -> 272.5).  From 5 workers on, where a tile with a boundary
  //    costs a step more, the others take them from 192 MiB on (16 workers, VGG-16: 2893 -> 2807,
  //    ResNet-v2-152, 230 MiB: 1330 -> 1316, but Inception-v3, 91 MiB: 506 -> 521; 12 workers, VGG-16:
  //    2138 -> 2115, ResNet-50: 415 either way; 5 to 7, 24 and 48 workers: from 1.7 % slower, 200 MiB, to
  //    1.7 % faster, 300 MiB).  1 and 3 workers never: VGG-16 with 3 519.8 us in 128 KiB tiles and 517.4
  //    in 64 (536.8 / 528.9 where every replica lies at another offset), one worker, 200 MiB, 67.4 / 66.6.
  //    Everything else 64 KiB.
  ts.tail_vecs = block;  // one vector per lane: a piece is fetched from all replicas at once
  //  * tiles may straddle segment boundaries where the kernel sums the parts in their own orders.
  //    Every boundary costs a step of the walk and saves a partial tile.  Up to 8 workers a step is
  //    dear and segments are long: none for 2, 4 and 8, whose walk without boundaries is unrolled
  //    (ResNet-50, 8 workers: 272 us without, 277 with one; VGG-16 1396 / 1395), one for the others
  //    (VGG-16, 6 workers: 1082 / 1060).  16 workers: one (Inception-v3 517 / 506, VGG-16 2795 /
  //    2807).  From 24 workers on, where the segments of a unit of a few MiB are not much longer than a
  //    tile or shorter (4 MiB over 48 workers: 85 KiB), up to four (ResNet-50 bf16, 32
  //    workers: 607 without, 579 with one, 561 with four; Inception-v3, 48 workers: 1802, 1612, 1534;
  //    ResNet-50, 24 workers: 869, 831, 826).
  ts.small_splits = reduce_handles_split_tiles(c.world, false) ? 1 : 0;
  ts.max_splits = !reduce_handles_split_tiles(c.world, stream_major != 0) ? 0 : (c.world >= 24 ? 4 : 1);
  ts.split_tiles = split_tiles && c.pattern == CARAMEL_PATTERN_RING && (ts.small_splits || ts.max_splits);
  const uint64_t replica_bytes = p.replica_elems * p.elem_size();
  //  * halving-doubling over 32 and 64 workers in bf16 has no walk (the partial sums leave room for too
  //    short bursts): small tiles throughout (32 x 33 MiB 449 -> 433 us), unless there must be few; and
  //    so in fp32 if the option leaves the walk no more than two vectors (32 x 50 MiB 685 -> 664)
  const bool tree = c.pattern == CARAMEL_PATTERN_HALVING_DOUBLING;
  const bool bf16_tree = tree && c.dtype == CARAMEL_BF16;
  const bool no_walk = tree && c.world >= 32 && (bf16_tree || stream_major < 4);
  if (ts.long_run_bytes == 0)
    ts.long_run_bytes = replica_bytes < (32u << 20) || (no_walk && !few_tiles) ? ~uint64_t(0) : 16u << 10;
  if (ts.long_vecs == 0) {
    // The tree holds eight vectors with 2 and 4 workers only (VGG-16, 4 workers: 713 -> 704 us; 8
    // workers, with sums in LDS: 1408 -> 1430).
    const bool few = c.world == 2 || c.world == 4 || c.world == 8;
    const bool wide = c.dtype == CARAMEL_F32 && !(tree && c.world > 4) && stream_major >= 8 && block == 1024 &&
                      (few || few_tiles || c.world > 4) && replica_bytes >= (uint64_t(few ? 64 : 192) << 20);
    // a bf16 tree keeps four vectors per lane: workgroups of 512 lanes or fewer get tiles of 32 KiB (512
    // lanes, 8 x 60 MiB 202 -> 194 us, 2 x 60 MiB 48.9 -> 45.4), and so do shorter walks
    const bool narrow = bf16_tree && (c.world >= 32 || ((block < 1024 || stream_major < 4) && !few_tiles));
    ts.long_vecs = wide ? 8192 : (narrow ? 2048 : 4096);
  }
}

void build_tiles(const HostPlan& p, const TileShape& ts, TileTables& out, const uint64_t* row_addr) {
  out = TileTables{};
  const uint32_t W = p.cfg.world;
  const uint64_t es = p.elem_size();
  const uint64_t ve = 16 / es;  // elements per 16-byte vector
  const uint64_t copy_elems = uint64_t(ts.copy_vecs) * ve;
  const uint32_t fused_row = uint32_t(p.tensor_elems.size());
  const size_t nu = p.units.size();
  out.staged_unit.resize(nu);
  out.direct_unit.resize(nu);
  out.copy_unit.resize(nu);
  for (uint32_t ui = 0; ui < nu; ++ui) out.order[p.units[ui].stream].push_back(ui);

  // Position of a row's element inside an aligned block of `block_elems` elements of memory.
  // Normally it is the same in every replica (tensors at the same offsets of equally aligned
  // arenas); if not, the position most replicas share is taken (the first such, for a tie), so
  // that as many replicas as possible see aligned tiles.  Without addresses: 0.
  std::vector<uint64_t> ph(W);
  auto common_phase = [&](uint32_t row, uint64_t elem, uint64_t block_elems) -> uint64_t {
    if (!row_addr) return 0;
    const uint64_t block_b = block_elems * es;
    for (uint32_t w = 0; w < W; ++w) ph[w] = (row_addr[size_t(row) * W + w] + elem * es) % block_b;
    uint64_t best = ph[0];
    uint32_t best_n = 0;
    for (uint32_t w = 0; w < W; ++w) {
      uint32_t n = 0;
      for (uint32_t x = 0; x < W; ++x) n += ph[x] == ph[w];
      if (n > best_n) best = ph[w], best_n = n;
    }
    return best / es;
  };

  // The runs of a unit in one table, in memory order: a chunk, the unit's region of the fused
  // buffer, or (batch unit reduced in place) each member; every run with its part per segment.
  // Without split tiles a run ends where the first worker changes.
  std::vector<Run> runs;
  auto unit_runs = [&](uint32_t ui, bool direct) {
    runs.clear();
    const caramel_unit& u = p.units[ui];
    const uint64_t* seg = p.segments(ui);
    const caramel_entry* ent = &p.entries[u.first_entry];
    // ring: the chain of segment c starts at worker c+1; the other patterns add in an order
    // that does not depend on the segment and read the workers from 0
    auto first_of = [&](uint32_t c) { return p.cfg.pattern == CARAMEL_PATTERN_RING ? (c + 1) % W : 0u; };
    // [lo, hi) in unit positions, starting at element `row_elem` of `row`
    auto add_run = [&](uint32_t row, uint64_t row_elem, uint64_t lo, uint64_t hi) {
      Run r{row, row_elem, hi - lo, {}};
      for (uint32_t c = 0; c < W; ++c) {
        const uint64_t a = std::max(lo, seg[c]), b = std::min(hi, seg[c + 1]);
        if (a >= b) continue;
        // equal first workers need no boundary between them
        if (!r.parts.empty() && r.parts.back().first == first_of(c)) r.parts.back().n += b - a;
        else r.parts.push_back({first_of(c), b - a});
      }
      if (!r.n) return;
      if (ts.split_tiles) {
        runs.push_back(std::move(r));
        return;
      }
      // tiles that end at segment boundaries: every part is a run of its own
      uint64_t at = 0;
      for (const Part& pt : r.parts) {
        runs.push_back(Run{row, row_elem + at, pt.n, {pt}});
        at += pt.n;
      }
    };
    if (u.kind == CARAMEL_KIND_CHUNK) {
      add_run(ent[0].tensor, ent[0].tensor_off, 0, u.elems);
    } else if (!direct) {
      add_run(fused_row, u.fused_off, 0, u.elems);
    } else {
      for (uint32_t k = 0; k < u.n_entries; ++k)
        add_run(ent[k].tensor, ent[k].tensor_off, ent[k].unit_off, ent[k].unit_off + ent[k].elems);
    }
  };

  for (int table = 0; table < 2; ++table) {
    const bool direct = table == 1;
    std::vector<ReduceTile>& tiles = direct ? out.direct : out.staged;
    std::vector<UnitTiles>& per_unit = direct ? out.direct_unit : out.staged_unit;
    for (int cls = 0; cls < 2; ++cls) {
      const uint64_t tile_elems = uint64_t(cls == kLong ? ts.long_vecs : ts.small_vecs) * ve;
      const bool align = (ts.align_tiles & (cls == kSmall ? 1u : 2u)) != 0;
      const uint32_t wanted = ts.split_tiles ? (cls == kSmall ? ts.small_splits : ts.max_splits) : 0;
      const uint32_t splits = std::min(wanted, std::min(kMaxSplits, W - 1));
      for (uint32_t s = 0; s < p.cfg.num_streams; ++s) {
        const size_t stream_begin = tiles.size();
        std::vector<uint64_t> phases;
        for (uint32_t ui : out.order[s]) {
          unit_runs(ui, direct);
          UnitTiles& ut = per_unit[ui];
          ut.tiles[cls].begin = uint32_t(tiles.size());
          for (const Run& r : runs) {
            if ((r.n * es >= ts.long_run_bytes) != (cls == kLong)) continue;
            cut_run(tiles, r, ve, tile_elems, align ? common_phase(r.row, r.row_elem, tile_elems) : 0,
                    splits, W, phases);
            ut.elems[cls] += r.n;
          }
          ut.tiles[cls].count = uint32_t(tiles.size()) - ut.tiles[cls].begin;
        }
        if (cls == kLong && ts.tail_tiles && ts.tail_vecs && ts.tail_vecs < ts.long_vecs)
          split_tail(tiles, stream_begin, phases, ts.tail_tiles, uint64_t(ts.tail_vecs) * ve,
                     align && ts.long_vecs % ts.tail_vecs == 0, ve, W, per_unit, out.order[s]);
      }
    }
  }

  for (uint32_t s = 0; s < p.cfg.num_streams; ++s) {
    out.copy_stream[s].begin = uint32_t(out.copy.size());
    for (uint32_t ui : out.order[s]) {
      const caramel_unit& u = p.units[ui];
      out.copy_unit[ui].begin = uint32_t(out.copy.size());
      if (u.kind == CARAMEL_KIND_BATCH) {
        const caramel_entry* ent = &p.entries[u.first_entry];
        for (uint32_t k = 0; k < u.n_entries; ++k) {
          const caramel_entry& e = ent[k];
          const uint64_t next = (k + 1 < u.n_entries) ? ent[k + 1].unit_off : u.elems;
          for (uint64_t at = 0; at < e.elems; at += copy_elems) {
            CopyTile t{};
            t.row = e.tensor;
            t.t_vec_off = uint32_t((e.tensor_off + at) / ve);
            t.f_vec_off = uint32_t((u.fused_off + e.unit_off + at) / ve);
            t.n_elems = uint32_t(std::min(copy_elems, e.elems - at));
            t.n_zero = (at + copy_elems >= e.elems) ? uint32_t(next - (e.unit_off + e.elems)) : 0;
            out.copy.push_back(t);
          }
        }
      }
      out.copy_unit[ui].count = uint32_t(out.copy.size()) - out.copy_unit[ui].begin;
    }
    out.copy_stream[s].count = uint32_t(out.copy.size()) - out.copy_stream[s].begin;
  }
}

}  // namespace caramel
