// The bidir kernels for fp32 elements: the same source as the bfloat16 build, compiled with the
// element type switched (see device_common.h).
#define COTTN_ELEM_F32
#include "bidir_bf16.hip"
