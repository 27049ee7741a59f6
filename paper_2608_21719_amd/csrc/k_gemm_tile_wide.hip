// Tile GEMM instances: 192x256 and 128x256 tiles. The kernel is in gemm_tile.h.
#include "gemm_tile.h"

namespace ps {
PS_TILE_INSTANCES_WIDE(PS_TILE_INSTANTIATE)
}  // namespace ps
