// Tile GEMM instances: 256x256 tiles (large row counts). The kernel is in gemm_tile.h.
#include "gemm_tile.h"

namespace ps {
PS_TILE_INSTANCES_256(PS_TILE_INSTANTIATE)
}  // namespace ps
