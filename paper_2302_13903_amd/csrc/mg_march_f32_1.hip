// mg_march_f32_1.hip -- the streaming passes of 1 sweep per leg in FP32 (compiled apart to build in parallel).
#define MG_MARCH_T float
#define MG_MARCH_NS 1
#include "mg_march.inl"
