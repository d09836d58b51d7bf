// Prints the tile shape that the library chooses: world dtype pattern replica_bytes block few_tiles stream_major -> one line.
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "plan.hpp"
#include "tiles.hpp"

using namespace caramel;

int main(int argc, char** argv) {
  if (argc != 8) return 2;
  caramel_config cfg{};
  cfg.world = uint32_t(std::atoi(argv[1]));
  cfg.dtype = uint32_t(std::atoi(argv[2]));
  cfg.pattern = uint32_t(std::atoi(argv[3]));
  cfg.align_bytes = 16;
  cfg.split_mode = CARAMEL_SPLIT_NONE;
  cfg.max_depth = 1;
  cfg.num_streams = 1;
  const uint64_t elems = std::strtoull(argv[4], nullptr, 10) / (cfg.dtype == CARAMEL_F32 ? 4 : 2);
  HostPlan p;
  std::string why;
  if (build_host_plan(cfg, &elems, 1, nullptr, 0.0, 0.0, p, why) != CARAMEL_OK) return 3;
  TileShape ts;
  choose_shape(p, true, uint32_t(std::atoi(argv[7])), uint32_t(std::atoi(argv[5])), std::atoi(argv[6]) != 0, ts);
  const bool long_tiles = ts.long_run_bytes != ~uint64_t(0);
  std::printf("%u %u %u\n", long_tiles ? ts.long_vecs : 0, ts.split_tiles ? ts.max_splits : 0,
              ts.split_tiles ? ts.small_splits : 0);
  return 0;
}
