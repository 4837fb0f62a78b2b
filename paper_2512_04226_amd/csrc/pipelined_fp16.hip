#define G355_TU_ES 2
#define G355_TU_FT 1
#define G355_TU_NAME pipelined_fp16
#include "pipelined.inc"
