// The persistent GEMM's kernels for the accumulator export, rows of Y far apart and codes without a zero point
// (see MUXQ_GEMM_PART in muxq_gemm.hip).
#define MUXQ_GEMM_PART 3
#include "muxq_gemm.hip"
