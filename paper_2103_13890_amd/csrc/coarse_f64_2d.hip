// Coarse solver, FP64 2D levels.
#define COARSE_T double
#define COARSE_DIM 2
#include "coarse.inc"
