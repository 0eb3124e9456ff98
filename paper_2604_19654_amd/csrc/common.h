// Shared host-side helpers of the library: error reporting and argument checks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include "feplb.h"

namespace feplb {

void set_error(const char* fmt, ...);

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

namespace dev {
struct WeightTable;
}
// one grouped GEMM over the ragged rows of groups [g_begin, g_begin + ng) (ffn_gemm.hip)
struct GroupedGemm {
  const void* A;                    // rows, bf16, row stride lda
  int lda;
  const int* row_src;               // gate/up only: row r is A[row_src[r] / src_k, :], or null
  int n_src_rows, src_k;
  const int* offsets;
  int g_begin, ng, R_cap;
  int K, N;                         // contraction length and output columns (gate/up: of one matrix)
  const dev::WeightTable* weights;  // row-major [K,N] matrices, row stride ldw; with w_nk row-major [N,K] ones
  int ldw;
  bool w_nk;                        // plain, dswiglu
  int k_split;                      // w_nk: k from here on lies in the tables' second matrix; K if there is none
  void* out;
  int ldo;
  void* aux;                        // gate/up: receives the derivatives p | q, or null; dswiglu: p | q in, da | db out
  int ld_aux;
};
hipError_t launch_gate_up(const GroupedGemm& a, hipStream_t s);
hipError_t launch_gate_up_keeping(const GroupedGemm& a, hipStream_t s);             // with aux
hipError_t launch_plain_gemm(const GroupedGemm& a, bool out_bf16, hipStream_t s);
hipError_t launch_plain_gemm_nk(const GroupedGemm& a, bool out_bf16, hipStream_t s);   // with w_nk
hipError_t launch_dswiglu(const GroupedGemm& a, hipStream_t s);
int gemm_tile_rows(const GroupedGemm& a, bool gate_up);   // rows of a tile of the shape that these pick
int gemm_tall_rows(const GroupedGemm& a, bool gate_up, bool save, bool out_bf16, const int* offsets);   // of a launch in tall tiles, else 0

// The GEMMs address the rows of a tile as 32-bit byte offsets from its first row: can `rows` rows of `ld` bf16 be?
inline bool rows_fit_32_bits(int64_t rows, int64_t ld) { return rows * ld * 2 <= 0xffffffffll; }

// backward-pass launchers (ffn_backward.hip), used by feplb_grouped_ffn_backward
hipError_t launch_wgrad(const void* P, int ldp, int M, const void* Q, int ldq, int N, const int* offsets,
                        int g_begin, int n_groups, int R_cap, void* const* c0, void* const* c1,
                        int n_split, int ldc, bool accumulate, hipStream_t s);
int wgrad_tile_rows(int R_cap, int n_groups, int M, int N);
hipError_t launch_transpose(const void* const* src, int g_begin, int n_groups, int rows, int cols, void* dst,
                            size_t group_stride, hipStream_t s);

}  // namespace feplb

#define FEPLB_FAIL(code, ...)        \
  do {                               \
    feplb::set_error(__VA_ARGS__);   \
    return (code);                   \
  } while (0)

#define FEPLB_REQUIRE(cond, code, ...) \
  do {                                 \
    if (!(cond)) FEPLB_FAIL(code, __VA_ARGS__); \
  } while (0)

#define FEPLB_HIP(expr)                                                         \
  do {                                                                          \
    hipError_t e__ = (expr);                                                    \
    if (e__ != hipSuccess)                                                      \
      FEPLB_FAIL(FEPLB_EHIP, "%s: %s", #expr, hipGetErrorString(e__));          \
  } while (0)

#define FEPLB_LAUNCH_CHECK(name)                                                \
  do {                                                                          \
    hipError_t e__ = hipGetLastError();                                         \
    if (e__ != hipSuccess)                                                      \
      FEPLB_FAIL(FEPLB_EHIP, "launch of %s: %s", name, hipGetErrorString(e__)); \
  } while (0)
