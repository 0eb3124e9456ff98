// Part 1 of the grouped GEMMs: the gate/up GEMM that keeps the SwiGLU derivatives.
#define FEPLB_GEMM_PART 1
#include "ffn_gemm.hip"
