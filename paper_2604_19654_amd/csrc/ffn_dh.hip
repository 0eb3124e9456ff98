// Part 4 of the grouped GEMMs: the input gradient through the SwiGLU product.
#define FEPLB_GEMM_PART 4
#include "ffn_gemm.hip"
