// The pair solver's variants that keep the consumers' coordinates in LDS.
#define NNSEMD_PAIR_COORDS_TU 1
#include "pair_solver.hip"
