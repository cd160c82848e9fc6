// The persistent GEMM's kernels with the GELU fused in (see MUXQ_GEMM_PART in muxq_gemm.hip).
#define MUXQ_GEMM_PART 2
#include "muxq_gemm.hip"
