// Stencil launchers: JFNK_BRATU, F64 levels and the outer FP64 operator.
#define JFNK_T double
#define JFNK_KIND_ID JFNK_BRATU
#define JFNK_JV_MIXED Ops::jv<float>
#include "ops_stencil.inc"
