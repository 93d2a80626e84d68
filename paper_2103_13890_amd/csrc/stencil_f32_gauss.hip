// Stencil launchers: JFNK_PLAP_GAUSS, F32 levels.
#define JFNK_T float
#define JFNK_KIND_ID JFNK_PLAP_GAUSS
#define JFNK_JV_MIXED nullptr
#include "ops_stencil.inc"
