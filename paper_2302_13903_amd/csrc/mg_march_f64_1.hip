// mg_march_f64_1.hip -- the streaming passes of 1 sweep per leg in FP64 (compiled apart to build in parallel).
#define MG_MARCH_T double
#define MG_MARCH_FAS   // the Full Approximation Scheme runs in FP64
#define MG_MARCH_NS 1
#include "mg_march.inl"
