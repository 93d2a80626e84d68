// Coarse solver, FP64 3D levels.
#define COARSE_T double
#define COARSE_DIM 3
#include "coarse.inc"
