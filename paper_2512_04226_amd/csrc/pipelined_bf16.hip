#define G355_TU_ES 2
#define G355_TU_NAME pipelined_bf16
#include "pipelined.inc"
