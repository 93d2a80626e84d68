// Coarse solver, FP32 2D levels.
#define COARSE_T float
#define COARSE_DIM 2
#include "coarse.inc"
