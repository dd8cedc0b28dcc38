// mg_tile_f64_1.hip -- the region-tile legs of 1 sweep per leg in FP64 (compiled apart to build in parallel).
#include "mg_tile.inl"

namespace mg {
MG_TILE_INST(double, 1)
}  // namespace mg
