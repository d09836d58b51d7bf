// Host-only check of the slice tables, built with AddressSanitizer and UBSan: slices cover every element
// of every tensor exactly once and nothing else, each stays inside its tensor and inside one aligned block
// of kSliceBytes in the replicas that share a position, and every element is added in the order of workers that
// the tile tables (the general path) give it.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <set>
#include <string>
#include <vector>

#include "plan.hpp"
#include "slices.hpp"
#include "tiles.hpp"

using namespace caramel;

#define CHECK(c)                                                \
  do {                                                          \
    if (!(c)) {                                                 \
      std::printf("FAIL %s:%d  %s\n", __FILE__, __LINE__, #c);  \
      std::exit(1);                                             \
    }                                                           \
  } while (0)

static std::map<std::string, int> shapes;

static void check(const HostPlan& p, const SliceShape& shape, const std::vector<uint64_t>& rows, bool alike) {
  const uint32_t W = p.cfg.world, V = shape.vecs, waves = shape.lanes / 64;
  const uint64_t es = p.elem_size();
  // the general path: first worker of every element
  TileShape ts;
  ts.long_vecs = 4096;
  ts.long_run_bytes = ~uint64_t(0);
  TileTables tt;
  build_tiles(p, ts, tt, rows.data());
  std::vector<std::vector<uint8_t>> first(p.tensor_elems.size()), seen(p.tensor_elems.size());
  for (size_t t = 0; t < first.size(); ++t) first[t].assign(p.tensor_elems[t], 255), seen[t].assign(p.tensor_elems[t], 0);
  for (const ReduceTile& t : tt.direct)
    for (uint32_t k = 0; k < t.n_elems; ++k) first[t.row][t.vec_off * (16 / es) + k] = uint8_t(t.first);

  std::vector<SlicePiece> pieces;
  const uint64_t n = slice_pieces(p, rows.data(), pieces);
  const SliceTable t = slice_table(p, shape, n, pieces.size(), rows.data());
  CHECK(t.lanes == shape.lanes && t.vecs == V && shape.share <= waves * V);
  CHECK(t.at_words() == size_t(t.groups) * waves * V * W + 16 && t.bytes_words() == size_t(t.groups) * waves * (V + 1));
  std::map<std::pair<size_t, uint64_t>, uint64_t> piece_bytes;  // by tensor and place
  for (const SlicePiece& c : pieces) piece_bytes[{c.row, uint64_t(c.at) * 16}] = c.bytes;
  // as k_slice_table does, a lane per slice and up to 16 steps
  struct {
    uint64_t base;
    uint32_t groups;
    std::vector<uint32_t> at, bytes;
  } st{t.base, t.groups, std::vector<uint32_t>(t.at_words()), std::vector<uint32_t>(t.bytes_words())};
  for (uint32_t wave = 0; wave < t.waves(); ++wave)
    for (uint32_t u = 0; u < V; ++u) {
      uint32_t len = 0;
      for (uint32_t k = 0; k < W; k += 16)
        len = place_slice(t, pieces.data(), rows.data(), wave, u, k, std::min(k + 16, W), &st.at[size_t(wave) * W * V + u]);
      st.bytes[size_t(wave) * (V + 1) + u] = (len + 3) & ~3u;
      if (len & 3u) st.bytes[size_t(wave) * (V + 1) + V] |= 1u << u;
    }
  std::map<uint64_t, size_t> at;  // worker 0's tensors by address
  for (size_t t = 0; t < first.size(); ++t) at[rows[t * W]] = t;
  uint64_t slices = 0;
  for (size_t wave = 0; wave < size_t(st.groups) * waves; ++wave) {
    const uint32_t odd = st.bytes[wave * (V + 1) + V];
    CHECK(odd >> V == 0);
    for (uint32_t u = 0; u < V; ++u) {
      const uint32_t bytes = st.bytes[wave * (V + 1) + u], whole = bytes - 2 * (odd >> u & 1);
      CHECK(bytes % 4 == 0 && bytes <= kSliceBytes && (bytes || !(odd >> u & 1)));
      auto address = [&](uint32_t k) { return st.base + uint64_t(st.at[(wave * W + k) * V + u]) * 16; };
      if (!bytes) {
        for (uint32_t k = 0; k < W; ++k) CHECK(address(k) == st.base);
        continue;
      }
      ++slices;
      // which step reads worker 0, hence which tensor and place
      size_t tensor = first.size();
      uint64_t off = 0;
      uint32_t step = W;
      for (uint32_t k = 0; k < W && step == W; ++k) {
        auto it = at.upper_bound(address(k));
        if (it == at.begin()) continue;
        --it;
        const uint64_t d = address(k) - it->first;
        if (d < p.tensor_elems[it->second] * es) tensor = it->second, off = d, step = k;
      }
      CHECK(step < W && off % 16 == 0 && off + whole <= p.tensor_elems[tensor] * es);
      const uint32_t f = (W - step) % W;
      for (uint32_t k = 0; k < W; ++k) CHECK(address(k) == rows[tensor * W + (f + k) % W] + off);
      // inside one aligned block, or a whole piece
      if (alike && address(0) / kSliceBytes != (address(0) + whole - 1) / kSliceBytes) {
        const auto c = piece_bytes.find(std::make_pair(tensor, off));
        CHECK(c != piece_bytes.end() && c->second == whole);
      }
      for (uint64_t e = off / es; e < (off + whole) / es; ++e) {
        CHECK(!seen[tensor][e] && first[tensor][e] == f);
        seen[tensor][e] = 1;
      }
    }
  }
  CHECK(slices == n);
  // what the host works out and a bind sends: at most two pieces per tensor and segment or chunk, however long
  uint64_t parts = 0;
  for (size_t u = 0; u < p.units.size(); ++u) parts += p.units[u].n_entries + W;
  CHECK(pieces.size() <= parts);
  for (const auto& s : seen)
    for (uint8_t x : s) CHECK(x == 1);
}

// The shape of a job of n slices of so many bytes on average, as "lanes x vecs", "tiles" if it has none.
static std::string shape_of(uint32_t world, uint32_t dtype, uint32_t pattern, uint64_t n, uint64_t pieces = 1000,
                            uint64_t slice_bytes = kSliceBytes) {
  HostPlan p;
  p.cfg.world = world;
  p.cfg.dtype = dtype;
  p.cfg.pattern = pattern;
  p.replica_elems = n * slice_bytes / p.elem_size();
  const SliceShape s = choose_slices(p, n, pieces);
  return s.vecs ? std::to_string(s.lanes) + " x " + std::to_string(s.vecs) : "tiles";
}

static bool through(uint32_t world, uint32_t dtype, uint32_t pattern, uint64_t n) {
  HostPlan p;
  p.cfg.world = world;
  p.cfg.dtype = dtype;
  p.cfg.pattern = pattern;
  p.replica_elems = n * kSliceBytes / p.elem_size();
  return choose_slices(p, n, 1000).through;
}

// Lines at which sweeps have found the other side to be slower.
static void lines() {
  const uint32_t ring = CARAMEL_PATTERN_RING, shuffle = CARAMEL_PATTERN_SHUFFLE, f32 = CARAMEL_F32, bf16 = CARAMEL_BF16;
  for (uint32_t pattern : {ring, shuffle})
    for (uint32_t W = 8; W < 16; ++W) {
      CHECK(shape_of(W, f32, pattern, 20480) == "256 x 20");
      for (uint64_t n : {20481, 20992}) CHECK(shape_of(W, f32, pattern, n) == (pattern == ring ? "256 x 1" : "1024 x 6"));
      for (uint64_t n : {20993, 24576})
        CHECK(shape_of(W, f32, pattern, n) == (pattern == ring && W == 9 ? "256 x 1" : "1024 x 6"));
      CHECK(shape_of(W, f32, pattern, 24577) == "512 x 16");
      for (uint64_t n : {28673, 29184}) CHECK(shape_of(W, f32, pattern, n) == (pattern == ring ? "256 x 1" : "1024 x 8"));
      CHECK(shape_of(W, f32, pattern, 29185) == "1024 x 8");
    }
  for (uint32_t W = 9; W < 16; ++W) {
    for (uint64_t n : {20481, 24577, 32767}) CHECK((shape_of(W, bf16, shuffle, n) == "256 x 1") == (W < 12));
    CHECK((shape_of(W, bf16, ring, 26000) == "tiles") == (W >= 12));
  }
  CHECK(shape_of(12, bf16, ring, 20992) == "256 x 1" && shape_of(12, bf16, ring, 20993) == "1024 x 6");
  CHECK(shape_of(24, bf16, ring, 33000, 1000, 900) == "256 x 1" && shape_of(24, bf16, shuffle, 33000, 1000, 900) == "1024 x 5");
  // vectors per lane of one round of a tree over 32 and 64 workers, and what lies beyond
  const uint32_t hd = CARAMEL_PATTERN_HALVING_DOUBLING, most[2][2] = {{14, 12}, {8, 8}};
  for (uint32_t dtype : {f32, bf16})
    for (uint32_t W : {32u, 64u}) {
      const uint32_t v = most[dtype == bf16][W == 64];
      CHECK(shape_of(W, dtype, hd, v * 1024) == "256 x " + std::to_string(v));
      for (uint64_t n : {uint64_t(v * 1024 + 1), uint64_t(32767)}) {
        CHECK(shape_of(W, dtype, hd, n, n / 200) == "tiles");
        CHECK(shape_of(W, dtype, hd, n, n / 180) == (W == 64 && dtype == f32 ? "tiles" : "256 x 1"));
      }
    }
  // from 32 MiB on, long pieces
  const struct {
    uint32_t world, dtype, pattern, mib, most_kib;
  } long_jobs[] = {{8, f32, shuffle, 35, 448},   {8, bf16, shuffle, 35, 448},  {8, f32, ring, 35, 560},
                   {8, bf16, ring, 35, 560},     {7, f32, shuffle, 35, 4096},  {7, bf16, ring, 35, 4096},
                   {2, bf16, shuffle, 105, 5120}, {2, bf16, ring, 105, 5120},  {2, bf16, hd, 105, 5120}};
  for (const auto& j : long_jobs) {
    const uint64_t n = uint64_t(j.mib) << 10, line = n / j.most_kib;
    CHECK(shape_of(j.world, j.dtype, j.pattern, n, line + 1) == "256 x 1");
    CHECK(shape_of(j.world, j.dtype, j.pattern, n, line - 1) == "tiles");
    CHECK(shape_of(j.world, j.dtype, j.pattern, 32767, 1) != "tiles");
  }
  for (uint32_t W = 3; W <= 6; ++W) CHECK(shape_of(W, f32, shuffle, 47 << 10, 1) == "256 x 1");
  // many short slices
  for (uint32_t dtype : {f32, bf16})
    for (uint32_t pattern : {ring, shuffle, hd}) {
      CHECK(shape_of(16, dtype, pattern, 4096, 4096, 319) == "256 x 1" && shape_of(16, dtype, pattern, 4096, 4096, 320) == "256 x 4");
      CHECK(shape_of(16, dtype, pattern, 4097, 4097, 64) == "256 x 6");
      CHECK(shape_of(16, dtype, pattern, 30000, 30000, 319) == "256 x 1");
    }
  CHECK(shape_of(16, f32, ring, 30000, 30000, 320) == "512 x 20" && shape_of(8, f32, shuffle, 30000, 30000, 699) == "256 x 1");
  CHECK(shape_of(8, f32, shuffle, 30000, 30000, 700) == "1024 x 8");
  // many rounds: written through from 64 MiB in all on
  for (uint32_t pattern : {ring, shuffle, hd})
    for (uint32_t dtype : {f32, bf16})
      for (uint64_t n : {uint64_t(20481), uint64_t(32768)}) CHECK(!through(2, dtype, pattern, n) && through(2, dtype, pattern, 32769));
  CHECK(!through(3, bf16, ring, 21845) && through(3, bf16, ring, 21846) && through(5, f32, ring, 20481));
  CHECK(shape_of(2, f32, shuffle, 111 << 10, 1) == "256 x 1");
}

// The kernel that launch_slices takes for a job, and with `all` every one there is.
static const char* kernel_of(uint32_t world, bool bf16, bool tree, const SliceShape& s, std::set<std::string>* all = nullptr) {
  const char* found = nullptr;
  auto match = [&](bool yes, const char* name) {
    if (all) CHECK(all->insert(name).second);
    if (yes && !found) found = name;
  };
  const bool one = s.vecs == 1 && s.lanes == 256;
#define ROUND(BF, TH, N, L) \
  match(!tree && bf16 == BF && s.through == TH && s.vecs == N && s.lanes == L, "slices " #BF " " #TH " " #N " " #L);
#define ONE(BF, TH, CW) match(!tree && one && bf16 == BF && s.through == TH && (CW == 0 || world == CW), "slice " #BF " " #TH " " #CW);
#define TREE_ROUND(W, BF, N) \
  match(tree && world == W && bf16 == BF && !s.through && s.vecs == N && s.lanes == 256, "tree_slices " #W " " #BF " " #N);
#define TREE_ONE(W, BF, TH) match(tree && one && world == W && bf16 == BF && s.through == TH, "tree_slice " #W " " #BF " " #TH);
  CARAMEL_SLICE_KERNELS(ROUND, ONE, TREE_ROUND, TREE_ONE)
  return found;
}

// Every shape that can be chosen has a kernel and fits what it assumes, and every kernel is chosen for some job.
static void kernels() {
  std::set<std::string> all, used;
  kernel_of(0, false, false, SliceShape{}, &all);
  for (uint32_t world = 1; world <= CARAMEL_MAX_WORLD; ++world)
    for (uint32_t dtype : {uint32_t(CARAMEL_F32), uint32_t(CARAMEL_BF16)})
      for (uint32_t pattern : {CARAMEL_PATTERN_RING, CARAMEL_PATTERN_SHUFFLE, CARAMEL_PATTERN_HALVING_DOUBLING}) {
        if (pattern == CARAMEL_PATTERN_HALVING_DOUBLING && (world & (world - 1))) continue;
        const bool tree = pattern == CARAMEL_PATTERN_HALVING_DOUBLING && world > 1;
        for (uint64_t n = 1; n < 150000; n += n < 70000 ? 61 : 997)
          for (uint64_t filled : {1024, 701, 400, 200}) {  // bytes of a slice on average
            HostPlan p;
            p.cfg.world = world;
            p.cfg.dtype = dtype;
            p.cfg.pattern = pattern;
            p.replica_elems = n * filled / p.elem_size();
            const SliceShape s = choose_slices(p, n, 1 + n / 64);
            if (!s.vecs) continue;
            const char* k = kernel_of(world, dtype == CARAMEL_BF16, tree, s);
            CHECK(k);
            CHECK(s.share && s.share <= s.lanes / 64 * s.vecs && s.vecs <= 32);
            used.insert(k);
          }
      }
  for (const std::string& k : all)
    if (!used.count(k)) std::printf("never chosen: %s\n", k.c_str());
  CHECK(used == all);
}

int main() {
  lines();
  kernels();
  std::mt19937_64 rng(11);
  auto pick = [&](std::initializer_list<uint64_t> xs) { return *(xs.begin() + rng() % xs.size()); };
  for (int it = 0; it < 260; ++it) {
    caramel_config cfg{};
    cfg.world = uint32_t(pick({1, 2, 3, 4, 8, 12, 16, 33, 64}));
    cfg.dtype = uint32_t(rng() % 2);
    cfg.align_bytes = uint32_t(pick({16, 16, 64, 256}));
    cfg.batch_threshold_bytes = pick({0, 1024, 65536, 1 << 20});
    cfg.split_mode = uint32_t(pick({CARAMEL_SPLIT_NONE, CARAMEL_SPLIT_FIXED, CARAMEL_SPLIT_ADAPTIVE}));
    cfg.split_bytes = pick({4096, 102400, 1 << 20});
    cfg.max_depth = 8;
    cfg.num_streams = uint32_t(pick({1, 2}));
    cfg.pattern = uint32_t(pick({CARAMEL_PATTERN_RING, CARAMEL_PATTERN_RING, CARAMEL_PATTERN_SHUFFLE, CARAMEL_PATTERN_HALVING_DOUBLING}));
    if (cfg.pattern == CARAMEL_PATTERN_HALVING_DOUBLING && (cfg.world & (cfg.world - 1))) cfg.world = 16;
    const bool wide = it % 20 == 3, large = it % 13 == 0;  // one round of 256 lanes; more than that, fp32 chains
    std::vector<uint64_t> elems(1 + rng() % (large ? 3 : 40));
    for (uint64_t& e : elems) e = large ? 700001 + rng() % 2000000 : pick({1, 2, 3, 17, 100, 257, 1000, 4099, 16384, 70001});
    if (wide) {
      cfg.world = uint32_t(pick({10, 12, 16, 24}));
      cfg.dtype = CARAMEL_F32;
      if (cfg.pattern == CARAMEL_PATTERN_HALVING_DOUBLING) cfg.pattern = CARAMEL_PATTERN_RING;
      elems.assign({5600001 + rng() % 1000000, 17, 1 + rng() % 1000000});  // 21 to 30 MiB
    }
    HostPlan p;
    std::string why;
    CHECK(build_host_plan(cfg, elems.data(), uint32_t(elems.size()), nullptr, 0.0, 0.0, p, why) == CARAMEL_OK);
    const bool alike = rng() % 2;
    std::vector<uint64_t> rows((elems.size() + 1) * cfg.world, 0);
    for (size_t t = 0; t < elems.size(); ++t) {
      const uint64_t common = rng() % 4096;
      for (uint32_t w = 0; w < cfg.world; ++w)
        rows[t * cfg.world + w] = (uint64_t(1) << 46) + (uint64_t(w) << 29) + (uint64_t(t) << (wide ? 25 : (large ? 24 : 21))) + (alike ? common : rng() % 4096) * cfg.align_bytes;
    }
    if (it % 20 == 1 && rows.size() > 2 * cfg.world) {  // out of the table's reach
      std::vector<uint64_t> far = rows;
      far[0] += uint64_t(1) << 37;
      std::vector<SlicePiece> pieces;
      const uint64_t n = slice_pieces(p, far.data(), pieces);
      CHECK(slice_table(p, SliceShape{256, 1, 4}, n, pieces.size(), far.data()).groups == 0);
    }
    std::vector<SlicePiece> pieces;
    const uint64_t n = slice_pieces(p, rows.data(), pieces);
    const SliceShape own = choose_slices(p, n, pieces.size());
    if (own.vecs) {
      CHECK(own.share && own.share <= own.lanes / 64 * own.vecs);
      ++shapes[std::to_string(own.lanes) + (own.vecs == 1 ? " x 1" : " x n")];
      check(p, own, rows, alike);
    }
    const uint32_t lanes = uint32_t(pick({256, 512, 1024})), vecs = uint32_t(pick({1, 4, 5, 20}));
    check(p, SliceShape{lanes, vecs, uint32_t(1 + rng() % (lanes / 64 * vecs))}, rows, alike);
  }
  CHECK(shapes["256 x 1"] && shapes["256 x n"] && shapes["512 x n"] && shapes["1024 x n"]);
  std::printf("slices_check ok\n");
  return 0;
}
