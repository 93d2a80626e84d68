// Stencil launchers: JFNK_INVCOEF, F32 levels.
#define JFNK_T float
#define JFNK_KIND_ID JFNK_INVCOEF
#define JFNK_JV_MIXED nullptr
#include "ops_stencil.inc"
