#define G355_TU_ES 2
#define G355_TU_FT 1
#define G355_TU_NAME sliced_fp16
#include "sliced.inc"
