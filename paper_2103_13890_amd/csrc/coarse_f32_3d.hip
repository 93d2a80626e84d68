// Coarse solver, FP32 3D levels.
#define COARSE_T float
#define COARSE_DIM 3
#include "coarse.inc"
