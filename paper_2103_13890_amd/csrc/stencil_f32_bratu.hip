// Stencil launchers: JFNK_BRATU, F32 levels.
#define JFNK_T float
#define JFNK_KIND_ID JFNK_BRATU
#define JFNK_JV_MIXED nullptr
#include "ops_stencil.inc"
