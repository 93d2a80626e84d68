// Stencil launchers: JFNK_PLAP, F64 levels and the outer FP64 operator.
#define JFNK_T double
#define JFNK_KIND_ID JFNK_PLAP
#define JFNK_JV_MIXED Ops::jv<float>
#include "ops_stencil.inc"
