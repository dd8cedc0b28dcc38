// mg_tile_f32_2.hip -- the region-tile legs of 2 sweeps per leg in FP32 (compiled apart to build in parallel).
#include "mg_tile.inl"

namespace mg {
MG_TILE_INST(float, 2)
}  // namespace mg
