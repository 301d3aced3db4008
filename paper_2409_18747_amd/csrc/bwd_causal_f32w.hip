// The causal backward kernels for fp32 elements on the fp32 matrix instruction, where that is better than
// operands in three bfloat16 parts (device_common.h: SPLIT3).
#define COTTN_ELEM_F32
#define COTTN_F32_WHOLE
#include "bwd_causal_bf16.hip"
