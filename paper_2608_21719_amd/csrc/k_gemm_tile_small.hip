// Tile GEMM instances: 128x128, 128x64 and 64x64 tiles (few rows). The kernel is in gemm_tile.h.
#include "gemm_tile.h"

namespace ps {
PS_TILE_INSTANCES_SMALL(PS_TILE_INSTANTIATE)
}  // namespace ps
