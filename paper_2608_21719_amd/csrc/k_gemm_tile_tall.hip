// Tile GEMM instances: 256x128 and 192x128 tiles. The kernel is in gemm_tile.h.
#include "gemm_tile.h"

namespace ps {
PS_TILE_INSTANCES_TALL(PS_TILE_INSTANTIATE)
}  // namespace ps
