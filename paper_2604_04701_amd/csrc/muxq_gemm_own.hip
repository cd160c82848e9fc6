// The persistent GEMM's kernels for Aux codes on a scale of their own (see MUXQ_GEMM_PART in muxq_gemm.hip).
#define MUXQ_GEMM_PART 1
#include "muxq_gemm.hip"
