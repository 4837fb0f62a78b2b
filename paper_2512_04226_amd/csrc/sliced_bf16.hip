#define G355_TU_ES 2
#define G355_TU_NAME sliced_bf16
#include "sliced.inc"
