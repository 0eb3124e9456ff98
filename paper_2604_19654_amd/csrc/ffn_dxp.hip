// Part 3 of the grouped GEMMs: the plain GEMM on [N,K] weights.
#define FEPLB_GEMM_PART 3
#include "ffn_gemm.hip"
