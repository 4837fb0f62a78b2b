#define G355_TU_ES 1
#define G355_TU_NAME sliced_fp8
#include "sliced.inc"
