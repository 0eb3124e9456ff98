// Backward-pass kernels of the grouped expert FFN that have no forward counterpart (paper
// Section 3.2 reports the layer's backward time beside the forward one):
//
//   weight gradients   C[g] = P_g^T Q_g, the sum over the rows of group g of outer products of a
//                      row of P with the same row of Q.  dW_down = H^T dYp, and
//                      [dW_gate | dW_up] = Xp^T [da | db].  The contraction runs over the ragged
//                      row range of the group, the output has the fixed shape of the weights.
//   transposes         W [r,c] -> W^T [c,r] (bf16), for a caller that hands the input-gradient GEMMs
//                      transposed copies instead of the weights.
//
// The weight gradients run on the forward GEMMs' main loop (panel_gemm.h) with the contraction index along
// the rows of both operands, 64 rows per step.  The loads are buffer loads whose descriptor covers the rows of
// the group that are left: the hardware returns zeros for rows past the group's end, so a ragged end needs neither
// masks nor padding and nothing outside the group is read.
#include <type_traits>
#include "common.h"
#include "panel_gemm.h"

namespace {
using namespace feplb::dev;

struct OutTable {
  void* c0[FEPLB_MAX_GROUPS];   // output matrix for columns [0, n_split)
  void* c1[FEPLB_MAX_GROUPS];   // output matrix for columns [n_split, 2 n_split), or unused
};

// The group (relative to g_begin) with the rank-th most rows, ties by group index; wave-uniform.  The grid walks the
// groups in this order: a tile's run time is proportional to its group's row count and workgroups start in grid
// order, so the long tiles go first and the last compute units to finish are busy with short ones (empty groups, which
// only write zeros, last).  A radix selection over the bits of the row counts, two groups per lane: every wave finds its
// group without a table and without a launch to sort one.
__device__ __forceinline__ int group_of_rank(const int* __restrict__ offsets, int g_begin, int ng, int R_cap, int rank) {
  const int lane = threadIdx.x % 64;
  auto rows_of = [&](int i) {
    if (i >= ng) return 0;
    const int lo = min(offsets[g_begin + i], R_cap);
    return max(min(offsets[g_begin + i + 1], R_cap), lo) - lo;
  };
  const int r0 = rows_of(lane), r1 = ng > 64 ? rows_of(64 + lane) : 0;
  uint64_t c0 = __ballot(lane < ng), c1 = __ballot(64 + lane < ng);   // the groups still in question
  for (int bit = 31 - __clz(R_cap | 1); bit >= 0; --bit) {
    const uint64_t s0 = __ballot((r0 >> bit) & 1) & c0, s1 = __ballot((r1 >> bit) & 1) & c1;
    const int n = __popcll(s0) + __popcll(s1);
    if (rank < n) {
      c0 = s0;
      c1 = s1;
    } else {
      rank -= n;
      c0 &= ~s0;
      c1 &= ~s1;
    }
  }
  const int n0 = __popcll(c0);
  const uint64_t c = rank < n0 ? c0 : c1;
  const int want = rank < n0 ? rank : rank - n0;
  const int before = __popcll(c & ((1ull << lane) - 1));
  const uint64_t hit = __ballot(((c >> lane) & 1) && before == want);
  return (rank < n0 ? 0 : 64) + __ffsll((unsigned long long)hit) - 1;
}

// 16-byte-per-lane buffer load into LDS, as load_to_lds_16; lanes at or past `bytes` from base bring zeros.  `bytes` is what
// keeps rows past the group's end out, and the compiler computes it with vector instructions and a readfirstlane right
// ahead of the load: the 5 wait states that the descriptor then needs stand here (s_mov_b32 counts as 1, s_nop 3 as 4).
// With fewer the load could still see the bound of an earlier step.
__device__ __forceinline__ void bounded_load_to_lds_16(const char* base, uint32_t bytes, uint32_t lane_off, uint32_t lds_base) {
  const uint64_t v = (uint64_t)(uintptr_t)base;
  const u32x4 rsrc = {(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v), (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) & 0xffffu,
                      (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00020000u};
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(lane_off), "s"(rsrc), "s"(lds_base)
               : "memory", "m0");
}

template <bool ACCUMULATE, int WR, int MI, int NJ, int DA, int DB, int OCC>
__global__ __launch_bounds__(128 * WR, OCC) void wgrad_gemm_kernel(
    const uint16_t* __restrict__ P, int ldp, const uint16_t* __restrict__ Q, int ldq,
    const int* __restrict__ offsets, int g_begin, int n_groups, int R_cap, int m_tiles, int n_tiles, int band, int n_split,
    OutTable out, int ldc) {
  using Core = PanelGemm<WR, MI, NJ, DA, DB, true, true>;
  __shared__ __attribute__((aligned(1024))) char lds[Core::LDS_BYTES];

  // ---- block -> (group, tile): every group has the same tile grid, walked in bands of `band` tiles of P's columns
  const int per_group = m_tiles * n_tiles;
  const int idx = tile_of_block<32 * Core::BLOCKS_PER_CU>(blockIdx.x, per_group * n_groups);
  if (idx < 0) return;
  const int slot = idx / per_group, in_group = idx - slot * per_group;
  const int b0 = in_group / (band * n_tiles) * band;
  const int in_band = in_group - b0 * n_tiles;
  const int height = min(band, m_tiles - b0);
  const int nt = in_band / height, mt = b0 + in_band % height;
  const int g = g_begin + group_of_rank(offsets, g_begin, n_groups, R_cap, slot);
  const int lo = __builtin_amdgcn_readfirstlane(min(offsets[g], R_cap));
  const int hi = __builtin_amdgcn_readfirstlane(max(min(offsets[g + 1], R_cap), lo));
  if (ACCUMULATE && hi == lo) return;   // nothing to add for an empty group

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int wm = wave / 2, wn = wave % 2;

  // ---- loads: each operand keeps a running pointer to its next 64 rows and the number of rows left there
  constexpr int NBA = Core::BM / 64;
  const uint32_t p_row = (uint32_t)ldp * 2, q_row = (uint32_t)ldq * 2;
  uint32_t p_goff[Core::LA], q_goff[Core::LB];
#pragma unroll
  for (int i = 0; i < Core::LA; ++i) {
    const int li = wave * Core::LA + i;
    p_goff[i] = (uint32_t)Core::template cols_row<NBA>(li, lane) * p_row + Core::template cols_chunk<NBA>(li, lane) * 16;
  }
#pragma unroll
  for (int i = 0; i < Core::LB; ++i) {
    const int li = wave * Core::LB + i;
    q_goff[i] = (uint32_t)Core::template cols_row<NJ>(li, lane) * q_row + Core::template cols_chunk<NJ>(li, lane) * 16;
  }
  const char* p_ptr = wave_uniform(P + (size_t)lo * ldp + (size_t)mt * Core::BM);
  const char* q_ptr = wave_uniform(Q + (size_t)lo * ldq + (size_t)nt * Core::BN);
  int p_left = hi - lo, q_left = hi - lo;
  auto issue_p = [&](uint32_t stage, int, int i) {
    bounded_load_to_lds_16(p_ptr, (uint32_t)min(p_left, 64) * p_row, p_goff[i], stage + (wave * Core::LA + i) * 1024);
    if (i == Core::LA - 1) {
      p_ptr += 64 * (size_t)p_row;
      p_left = max(p_left - 64, 0);
    }
  };
  auto issue_q = [&](uint32_t stage, int u, int i) {
    const int half = u & 1;
    bounded_load_to_lds_16(q_ptr + half * (Core::HW * 2), (uint32_t)min(q_left, 64) * q_row, q_goff[i], stage + (wave * Core::LB + i) * 1024);
    if (half == 1 && i == Core::LB - 1) {
      q_ptr += 64 * (size_t)q_row;
      q_left = max(q_left - 64, 0);
    }
  };

  typename Core::FragA fa;
  typename Core::FragB fb;
  fa.init(wm * 32, lane);
  fb.init(wn * 32 * NJ, lane);
  f32x4 acc[2][2 * MI][2 * NJ];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf)
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
      for (int j = 0; j < 2 * NJ; ++j) acc[hf][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (hi > lo) Core::template run<MI>(lds, 2 * ((hi - lo + 63) / 64), fa, fb, issue_p, issue_q, acc);

  // ---- epilogue, as the forward kernel's: each wave passes 32 rows x 32 NJ columns at a time through an LDS region of
  // its own, so that every store (and load, where the product is added) covers whole lines
  constexpr int COLS = 32 * NJ;
  constexpr int ROW_BYTES = COLS * 4;
  constexpr int CH = ROW_BYTES / 16;
  constexpr int RPI = 64 / CH;
  constexpr int LINES = 32 / RPI;
  constexpr int SWZ_DIV = ROW_BYTES >= 256 ? 1 : 256 / ROW_BYTES;
  static_assert(32 * ROW_BYTES <= Core::LDS_BYTES / (2 * WR), "staging region");
  auto swz = [&](int r) { return (r / SWZ_DIV) & (CH - 1); };
  char* const ep = lds + wave * (Core::LDS_BYTES / (2 * WR));
  const int rd_row = lane / CH, rd_chunk = lane % CH;
  int ncol0 = nt * Core::BN;
  char* cbase = (char*)out.c0[g];
  if (ncol0 >= n_split) {
    ncol0 -= n_split;
    cbase = (char*)out.c1[g];
  }
  const size_t row_bytes = (size_t)ldc * 4;
  char* const out_wave = cbase + (size_t)(mt * Core::BM + wm * 32 + rd_row) * row_bytes + (size_t)(ncol0 + wn * COLS) * 4 + rd_chunk * 16;
  auto line = [&](int pass, int j) {
    return (f32x4*)(out_wave + (size_t)(pass / 2 * 32 * WR + j * RPI) * row_bytes + (pass % 2) * Core::HW * 4);
  };
  f32x4 old[2][LINES];
  auto fetch = [&](int pass) {
#pragma unroll
    for (int j = 0; j < LINES; ++j) old[pass % 2][j] = __builtin_nontemporal_load(line(pass, j));
  };
  if (ACCUMULATE) fetch(0);
#pragma unroll
  for (int pass = 0; pass < 2 * MI; ++pass) {
    if (ACCUMULATE && pass + 1 < 2 * MI) fetch(pass + 1);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2 * NJ; ++j) {
        const int r = i * 16 + lane % 16, chunk = j * 4 + lane / 16;
        *(f32x4*)(ep + r * ROW_BYTES + ((chunk ^ swz(r)) << 4)) = acc[pass % 2][2 * (pass / 2) + i][j];
      }
#pragma unroll
    for (int j = 0; j < LINES; ++j) {
      const int r = j * RPI + rd_row;
      f32x4 v = *(const f32x4*)(ep + r * ROW_BYTES + ((rd_chunk ^ swz(r)) << 4));
      if (ACCUMULATE) v += old[pass % 2][j];
      __builtin_nontemporal_store(v, line(pass, j));
    }
  }
}

// Tile shape by estimated time, as for the forward GEMMs: a round of tiles takes `start`, most of it the write of the fp32
// tile, plus k times the measured cost per k.  Two workgroups per CU (128 x 256) write one tile while they multiply for the
// other: the better shape up to about 1500 rows per group.  16 groups of 512 rows, d = 4096, f = 1536: 418 us (256 x 256),
// 363 (128 x 256), 569 (64 x 128); 32 groups of 2500 rows, d = 7168, f = 2048: 5.73, 6.03, 10.0 ms; one group of 8192
// rows, d = 2048, f = 1024, which leaves CUs idle: 291, 190, 137 us (the costs below were fitted with MFMAs 32x32x16, where these were 413, 383,
// 558; 5.97, 6.20, 10.1; 259, 175, 148).  (256 x 256 tiles of four
// wavefronts with masked 32-row windows, before all of these: 516 us, 7.04 ms, 356 us; adding to the gradients 1175 us and 9.51 ms against
// 501 us and 6.30 ms now, that are requested a pass ahead.)
struct WgradShape {
  int bm, bn, per_cu;
  double start, round[2];   // us; us per 1000 rows
};
constexpr WgradShape WGRAD_SHAPES[3] = {{256, 256, 1, 12.0, {23.6, 0.}}, {128, 256, 2, 7.8, {10.6, 26.4}}, {64, 128, 2, 2.5, {5.8, 11.9}}};

int pick_wgrad_shape(int R_cap, int ng, int M, int N) {
  int best = 0;
  double best_us = 0.;
  for (int i = 0; i < 3; ++i) {
    const WgradShape& s = WGRAD_SHAPES[i];
    const long tiles = (long)ng * (M / s.bm) * (N / s.bn), round = 256 * s.per_cu;
    const long full = tiles / round, rest = tiles % round;
    const double k = 1e-3 * R_cap / ng;
    const double tail = rest == 0 ? 0. : s.start + k * s.round[rest > 256 ? 1 : 0];
    const double us = full * (s.start + k * s.round[s.per_cu - 1]) + tail;
    if (i == 0 || us < best_us) {
      best = i;
      best_us = us;
    }
  }
  return best;
}

template <bool ACCUMULATE, int WR, int MI, int NJ, int DA, int DB, int OCC>
hipError_t launch_wgrad_shape(const void* P, int ldp, int M, const void* Q, int ldq, int N, const int* offsets, int g_begin,
                              int n_groups, int R_cap, const OutTable& tab, int n_split, int ldc, hipStream_t s) {
  using Core = PanelGemm<WR, MI, NJ, DA, DB, true, true>;
  const int m_tiles = M / Core::BM, n_tiles = N / Core::BN;
  const int band = Core::BM == 256 ? 8 : 16;
  hipLaunchKernelGGL((wgrad_gemm_kernel<ACCUMULATE, WR, MI, NJ, DA, DB, OCC>), dim3(blocks_for_tiles((long)m_tiles * n_tiles * n_groups)),
                     dim3(128 * WR), 0, s, (const uint16_t*)P, ldp, (const uint16_t*)Q, ldq, offsets, g_begin, n_groups, R_cap,
                     m_tiles, n_tiles, band, n_split, tab, ldc);
  return hipGetLastError();
}

// W [rows, cols] -> W^T [cols, rows], bf16, one 64 x 64 tile per block; z picks the group
constexpr int TT = 64;
__global__ __launch_bounds__(256) void transpose_bf16_kernel(WeightTable src, int g_begin, int rows, int cols,
                                                              uint16_t* __restrict__ dst0, size_t dst_group_stride) {
  __shared__ uint16_t tile[TT][TT + 2];
  const int g = g_begin + blockIdx.z;
  const uint16_t* __restrict__ W = (const uint16_t*)src.w0[g];
  uint16_t* __restrict__ WT = dst0 + (size_t)blockIdx.z * dst_group_stride;
  const int r0 = blockIdx.y * TT, c0 = blockIdx.x * TT;
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = t + i * 256;           // 512 pieces of 8 elements
    const int r = idx / 8, c8 = (idx % 8) * 8;
    const u32x4 v = __builtin_nontemporal_load((const u32x4*)(W + (size_t)(r0 + r) * cols + c0 + c8));
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile[r][c8 + 2 * e] = (uint16_t)(w[e] & 0xffffu);
      tile[r][c8 + 2 * e + 1] = (uint16_t)(w[e] >> 16);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = t + i * 256;
    const int c = idx / 8, r8 = (idx % 8) * 8;   // output row c (a column of W), 8 consecutive rows of W
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = (uint32_t)tile[r8 + 2 * e][c] | ((uint32_t)tile[r8 + 2 * e + 1][c] << 16);
    const u32x4 o = {w[0], w[1], w[2], w[3]};
    __builtin_nontemporal_store(o, (u32x4*)(WT + (size_t)(c0 + c) * rows + r0 + r8));
  }
}

}  // namespace

namespace feplb {

// C[g] = P_g^T Q_g for g in [g_begin, g_begin + n_groups): P [R_cap, ldp] columns [0, M),
// Q [R_cap, ldq] columns [0, N); output fp32 row-major with row stride ldc; columns of the
// product at or past n_split go to c1[g] (shifted by n_split).  M, N, n_split multiples of 256.
// accumulate: the product is added to what the output matrices hold (an empty group's are left
// alone) instead of replacing it.
hipError_t launch_wgrad(const void* P, int ldp, int M, const void* Q, int ldq, int N, const int* offsets, int g_begin,
                        int n_groups, int R_cap, void* const* c0, void* const* c1, int n_split, int ldc, bool accumulate,
                        hipStream_t s) {
  OutTable tab{};
  for (int i = 0; i < n_groups; ++i) {
    tab.c0[g_begin + i] = c0[g_begin + i];
    tab.c1[g_begin + i] = c1 ? c1[g_begin + i] : nullptr;
  }
  auto run = [&](auto acc) {
    constexpr bool A = decltype(acc)::value;
    switch (pick_wgrad_shape(R_cap, n_groups, M, N)) {
      case 0: return launch_wgrad_shape<A, 4, 2, 2, 3, 3, 2>(P, ldp, M, Q, ldq, N, offsets, g_begin, n_groups, R_cap, tab, n_split, ldc, s);
      case 1: return launch_wgrad_shape<A, 2, 2, 2, 2, 3, 2>(P, ldp, M, Q, ldq, N, offsets, g_begin, n_groups, R_cap, tab, n_split, ldc, s);
      default: return launch_wgrad_shape<A, 2, 1, 1, 3, 6, 2>(P, ldp, M, Q, ldq, N, offsets, g_begin, n_groups, R_cap, tab, n_split, ldc, s);
    }
  };
  return accumulate ? run(std::true_type{}) : run(std::false_type{});
}

int wgrad_tile_rows(int R_cap, int n_groups, int M, int N) { return WGRAD_SHAPES[pick_wgrad_shape(R_cap, n_groups, M, N)].bm; }

// dst + i * group_stride (elements) receives the transpose of src[g_begin + i] ([rows, cols] bf16)
hipError_t launch_transpose(const void* const* src, int g_begin, int n_groups, int rows, int cols, void* dst,
                            size_t group_stride, hipStream_t s) {
  WeightTable tab{};
  for (int i = 0; i < n_groups; ++i) tab.w0[g_begin + i] = src[g_begin + i];
  hipLaunchKernelGGL(transpose_bf16_kernel, dim3(cols / TT, rows / TT, n_groups), dim3(256), 0, s, tab, g_begin,
                     rows, cols, (uint16_t*)dst, group_stride);
  return hipGetLastError();
}

}  // namespace feplb
