#define G355_TU_ES 2
#define G355_TU_NAME chained_bf16
#include "chained.inc"
