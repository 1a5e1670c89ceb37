// The second projection's kernels of the grouped GEMM.
#define GG_SECOND_PROJECTION
#include "moe_ffn_grouped.hip"
