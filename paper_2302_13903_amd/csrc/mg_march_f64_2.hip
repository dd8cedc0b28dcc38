// mg_march_f64_2.hip -- the streaming passes of 2 sweeps per leg in FP64 (compiled apart to build in parallel).
#define MG_MARCH_T double
#define MG_MARCH_FAS   // the Full Approximation Scheme runs in FP64
#define MG_MARCH_NS 2
#include "mg_march.inl"
