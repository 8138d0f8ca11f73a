// Strip-walk detection kernels for bf16 FOP storage, 8 bins per lane,
// H = 1..4.
#define HS_WALK_T bf16_t
#define HS_WALK_NAME bf16
#define HS_WALK_V 8
#define HS_WALK_GROUP 0
#include "hs_walk_inst.h"
