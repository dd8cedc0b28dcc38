// mg_tile_f32_1.hip -- the region-tile legs of 1 sweep per leg in FP32 (compiled apart to build in parallel).
#include "mg_tile.inl"

namespace mg {
MG_TILE_INST(float, 1)
}  // namespace mg
