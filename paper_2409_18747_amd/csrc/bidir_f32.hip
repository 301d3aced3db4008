// The bidirectional kernels for fp32 elements: the same source as the bfloat16 build, compiled with the
// element type switched (see device_common.h), and before it once more as the functions of whole products that a
// workgroup turns to whose values the parts cannot carry.
#define COTTN_ELEM_F32
#define COTTN_F32_WHOLE
#define COTTN_REDO
#include "bidir_bf16.hip"
#undef COTTN_F32_WHOLE
#undef COTTN_REDO
#include "bidir_bf16.hip"
