#define G355_TU_ES 1
#define G355_TU_NAME chained_fp8
#include "chained.inc"
