// Host-only check of tiles that hold several segment boundaries, built with AddressSanitizer and
// UBSan: for every element of every tile the worker its sum starts at is the one its segment gives,
// tiles cover every element exactly once, and no tile holds more boundaries than it may.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>
#include <vector>

#include "plan.hpp"
#include "tiles.hpp"

using namespace caramel;

#define CHECK(c)                                                \
  do {                                                          \
    if (!(c)) {                                                 \
      std::printf("FAIL %s:%d  %s\n", __FILE__, __LINE__, #c);  \
      std::exit(1);                                             \
    }                                                           \
  } while (0)

int main() {
  std::mt19937_64 rng(7);
  uint32_t most = 0;
  for (int it = 0; it < 400; ++it) {
    auto pick = [&](std::initializer_list<uint64_t> xs) { return *(xs.begin() + rng() % xs.size()); };
    caramel_config cfg{};
    cfg.world = uint32_t(pick({2, 3, 5, 16, 24, 33, 48, 64}));
    cfg.dtype = uint32_t(rng() % 2);
    cfg.align_bytes = 16;
    cfg.batch_threshold_bytes = pick({0, 0, 1024, 65536});
    cfg.split_mode = CARAMEL_SPLIT_NONE;
    cfg.max_depth = 1;
    cfg.num_streams = 1;
    cfg.pattern = CARAMEL_PATTERN_RING;
    std::vector<uint64_t> elems(1 + rng() % 6);
    for (uint64_t& e : elems) e = pick({1, 17, 100, 1000, 4099, 16384, 70001});
    HostPlan p;
    std::string why;
    CHECK(build_host_plan(cfg, elems.data(), uint32_t(elems.size()), nullptr, 0.0, 0.0, p, why) == CARAMEL_OK);
    TileShape ts;
    ts.long_vecs = uint32_t(pick({64, 256, 1024}));
    ts.small_vecs = 64;
    ts.long_run_bytes = pick({0, 0, 4096});
    ts.tail_tiles = uint32_t(pick({0, 3, 1000}));
    ts.tail_vecs = 16;
    ts.split_tiles = true;
    ts.max_splits = uint32_t(1 + rng() % kMaxSplits);
    ts.small_splits = uint32_t(rng() % 2);
    TileTables tt;
    build_tiles(p, ts, tt);
    const uint64_t ve = 16 / p.elem_size();
    std::vector<std::vector<uint8_t>> seen(elems.size());
    for (size_t t = 0; t < elems.size(); ++t) seen[t].assign(elems[t], 0);
    for (uint32_t u = 0; u < p.units.size(); ++u) {
      const caramel_unit& un = p.units[u];
      for (int cls = 0; cls < 2; ++cls) {
        const Range r = tt.direct_unit[u].tiles[cls];
        for (uint32_t i = r.begin; i < r.begin + r.count; ++i) {
          const ReduceTile& t = tt.direct[i];
          const uint32_t b[kMaxSplits] = {t.split, t.more[0], t.more[1], t.more[2]};
          uint32_t n = 0;
          while (n < kMaxSplits && b[n]) {
            CHECK(b[n] % ve == 0 && b[n] < t.n_elems && (n == 0 || b[n] > b[n - 1]));
            ++n;
          }
          for (uint32_t k = n; k < kMaxSplits; ++k) CHECK(b[k] == 0);
          CHECK(n <= (cls == kLong ? ts.max_splits : ts.small_splits) && n < cfg.world);
          most = std::max(most, n);
          uint64_t unit_pos = ~0ull;
          for (uint32_t k = 0; k < un.n_entries; ++k) {
            const caramel_entry& e = p.entries[un.first_entry + k];
            if (e.tensor == t.row) unit_pos = (un.kind == CARAMEL_KIND_CHUNK ? 0 : e.unit_off) + t.vec_off * ve - e.tensor_off;
          }
          CHECK(unit_pos != ~0ull);
          uint32_t c = 0, s = 0;
          for (uint64_t k = 0; k < t.n_elems; ++k) {
            while (p.segments(u)[c + 1] <= unit_pos + k) ++c;
            while (s < n && b[s] <= k) ++s;
            CHECK((t.first + s) % cfg.world == (c + 1) % cfg.world);
            uint8_t& x = seen[t.row][t.vec_off * ve + k];
            CHECK(x == 0);
            x = 1;
          }
        }
      }
    }
    for (const auto& s : seen)
      for (uint8_t x : s) CHECK(x == 1);
  }
  CHECK(most == kMaxSplits);
  std::printf("splits_check ok\n");
  return 0;
}
