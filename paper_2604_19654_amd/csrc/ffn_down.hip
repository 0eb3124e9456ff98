// Part 2 of the grouped GEMMs: the plain GEMM on [K,N] weights.
#define FEPLB_GEMM_PART 2
#include "ffn_gemm.hip"
