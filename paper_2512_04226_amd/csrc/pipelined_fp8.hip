#define G355_TU_ES 1
#define G355_TU_NAME pipelined_fp8
#include "pipelined.inc"
