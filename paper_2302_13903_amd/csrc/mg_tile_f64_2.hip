// mg_tile_f64_2.hip -- the region-tile legs of 2 sweeps per leg in FP64 (compiled apart to build in parallel).
#include "mg_tile.inl"

namespace mg {
MG_TILE_INST(double, 2)
}  // namespace mg
