// The causal forward kernels for fp32 elements on the fp32 matrix instruction: the shapes for which
// operands in three bfloat16 parts take too much of the LDS (device_common.h: SPLIT3).
#define COTTN_ELEM_F32
#define COTTN_F32_WHOLE
#include "fwd_causal_bf16.hip"
