// The grouped GEMM kernel: for every row r of a group g with rows in [offsets[g], offsets[g+1])
//   MODE 0  gate/up:  H[r,:] = bf16( silu(x_r Wg[g]) * (x_r Wu[g]) ); with SAVE also the two derivatives p, q of that
//           product with respect to its factors' products, bf16, in columns [0,N) and [N,2N) of `aux`
//   MODE 1  plain:    out[r,:] = a_r W[g], fp32 or bf16
//   MODE 2  dswiglu:  dH = a_r W[g], times the derivatives in `aux`: da = dH p | db = dH q, bf16, written over them
// One launch covers a whole range of ragged groups; a workgroup finds its tile from offsets[] (device memory), so the
// host never needs the number of rows: the grid covers an upper bound and surplus workgroups leave at once.
// panel_gemm.h holds the main loop and the mapping of workgroups to tiles, tall_gemm.h the loop for tall tiles.
//
// Three tile shapes (rows x weight columns; for gate/up half of the columns are gate, half the matching up columns):
//   256 x 256, 8 wavefronts, one workgroup per CU: the least operand traffic per flop, for shapes with several rounds
//              of tiles per CU.  Two waves per SIMD cover each other's latencies, so a ragged tile may skip the MFMAs
//              of its empty 32-row blocks (wave-uniform choice of a loop variant), which one wave per SIMD could not.
//   128 x 256, 4 wavefronts, two workgroups per CU: one's prologue and epilogue hide behind the other's loop and half
//              the rows are lost to rounding a group up, but operand traffic in LDS is 1.1x its bandwidth at full MFMA rate.
//   64 x 128,  4 wavefronts, two workgroups per CU with deep rings: for launches that would leave most CUs idle otherwise.
// and tall tiles, up to 320 x 256, 4 wavefronts, one workgroup per CU, whose height every launch finds from its groups' rows: where another
// height fills the rounds better, and for gate/up with many rounds of tiles (use_tall below).
// 256 weight columns x 64 k of LDS-DMA loads in flight per CU also stream weights well: 16 groups of 8 rows, d = 4096,
// f = 1536 (400 MB of gate/up weights): 109 -> 77 us, 5.2 TB/s.
// The weights are row-major [K,N] (B_TR: the MFMA operand needs 8 consecutive k of one column, which the transposing LDS
// read delivers), or row-major [N,K] for the products with W^T of the backward pass, read like the rows of A.  [N,K]
// weights may be two matrices that share k: w0 holds the first k_split of it, w1 the rest (dXp = [da | db] [Wg | Wu]^T).
// The result's bits do not depend on the shape: every element is one chain of MFMAs 16x16x32 over ascending k.
#include "common.h"
#include "tall_gemm.h"

namespace {
using namespace feplb::dev;

// 256 x 256 tiles that are left after whole rounds on the 256 CUs cost a round however few they are.  Up to 64 of them are
// computed as quarters, 128 x 128 by the same eight wavefronts with rings of their own size: four times as many
// workgroups for half of a round's time (a quarter moves half of the operand bytes of a tile, and they bound it).  More would take two
// such rounds, and halves of 128 x 256 take 0.8 of a whole tile's time.  T = 8192, 20396 rows in 8 groups, d = 4096, f = 1536, whose
// gate/up is 4 rounds and 8 tiles: 766 -> 728 us a layer step; 298 drawn forward steps 1.01x on average, up to 1.75x.
constexpr int QUARTERS_MAX = 64;
constexpr int HALVES_MAX = 128;   // tall tiles: from 65 left-over ones on halves of 128 columns, 0.6 of a whole tile's time

struct Tile {
  int g, row0, rows, nt;   // group, first row, number of rows, column
};

// a tall tile's main loop, `blocks` <= ME row blocks per wave
template <class Core, int ME, class IA, class IB, class Acc>
__device__ __forceinline__ void run_blocks(int blocks, char* lds, int U, const typename Core::FragA& fa, const typename Core::FragB& fb, IA& issue_a,
                                           IB& issue_b, Acc& acc) {
  if constexpr (ME > 1) {
    if (blocks < ME) return run_blocks<Core, ME - 1>(blocks, lds, U, fa, fb, issue_a, issue_b, acc);
  }
  Core::template run<ME>(lds, U, fa, fb, issue_a, issue_b, acc);
}

// one tile of the output, by panel_gemm.h's loop or (TALL, two wave rows) tall_gemm.h's
template <int MODE, bool OUT_BF16, bool SAVE, bool B_TR, int WR, int MI, int NJ, int DA, int DB, bool TALL = false>
__device__ __forceinline__ void panel_tile(
    char* lds, const Tile& tile, const uint16_t* __restrict__ A, int lda, const int* __restrict__ row_src, int n_src_rows, int src_k, int K,
    const WeightTable& wt, int ldw, int k_split, void* __restrict__ out, int ldo, void* aux, int ld_aux) {
  using Core = std::conditional_t<TALL, TallGemm<MI, NJ, DA, DB, B_TR>, PanelGemm<WR, MI, NJ, DA, DB, false, B_TR>>;
  const int g = tile.g, row0 = tile.row0, rows = tile.rows, nt = tile.nt;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int wm = wave / 2, wn = wave % 2;
  const int KT = K / 64;

  // ---- loads
  // a tall tile asks for the rows it has only: its loads go to the waves in turn
  auto a_load = [&](int i) { return TALL ? i * 2 * WR + wave : wave * Core::LA + i; };
  uint32_t a_goff[Core::LA];
  const bool gather = MODE == 0 && row_src != nullptr;
#pragma unroll
  for (int i = 0; i < Core::LA; ++i) {
    const int li = a_load(i);
    int row = min(Core::rows_row(li, lane), rows - 1);
    if (gather) row = min(max(row_src[row0 + row] / src_k, 0), n_src_rows - 1);
    a_goff[i] = ((uint32_t)row * (uint32_t)lda + Core::rows_chunk(li, lane) * 8) * 2;
  }
  const char* a_ptr = wave_uniform(gather ? A : A + (size_t)row0 * lda);
  // the requests come in order, so each operand keeps one running scalar pointer; it stays on the last tile for
  // requests past the end
  auto issue_a = [&](uint32_t stage, int t, int i, int la = Core::LA) {
    load_to_lds_16(a_ptr, a_goff[i], stage + a_load(i) * 1024);
    if (i == la - 1) a_ptr += t < KT - 1 ? 128 : 0;
  };
  uint32_t b_goff[Core::LB];
  const char *b_ptr0, *b_ptr1;
  const size_t ldw_bytes = (size_t)ldw * 2;
#pragma unroll
  for (int i = 0; i < Core::LB; ++i) {
    const int li = wave * Core::LB + i;
    b_goff[i] = B_TR ? (uint32_t)Core::template cols_row<NJ>(li, lane) * (uint32_t)ldw_bytes + Core::template cols_chunk<NJ>(li, lane) * 16
                     : (uint32_t)Core::rows_row(li, lane) * (uint32_t)ldw_bytes + Core::rows_chunk(li, lane) * 16;
  }
  if (MODE == 0) {
    b_ptr0 = wave_uniform((const uint16_t*)wt.w0[g] + (size_t)nt * Core::HW);
    b_ptr1 = wave_uniform((const uint16_t*)wt.w1[g] + (size_t)nt * Core::HW);
  } else {
    const size_t col_bytes = B_TR ? 2 : ldw_bytes;
    b_ptr0 = wave_uniform((const char*)wt.w0[g] + nt * Core::BN * col_bytes);
    b_ptr1 = b_ptr0 + Core::HW * col_bytes;
  }
  const size_t b_step = B_TR ? 64 * ldw_bytes : 128;
  const int t_split = B_TR ? KT : k_split / 64;
  const ptrdiff_t b_jump = !B_TR && t_split < KT   // from the last k tile of w0 to the first of w1
                               ? wave_uniform(wt.w1[g]) - wave_uniform(wt.w0[g]) - (ptrdiff_t)(t_split - 1) * 128 : 0;
  auto issue_b = [&](uint32_t stage, int u, int i) {
    const int t = u >> 1, half = u & 1;
    const char*& ptr = half ? b_ptr1 : b_ptr0;
    load_to_lds_16(ptr, b_goff[i], stage + (wave * Core::LB + i) * 1024);
    if (i == Core::LB - 1) {
      if (B_TR)
        ptr += t < KT - 1 ? b_step : 0;
      else
        ptr += t >= KT - 1 ? 0 : t == t_split - 1 ? b_jump : 128;
    }
  };

  typename Core::FragA fa;
  typename Core::FragB fb;
  fa.init(wm * 32, lane);
  fb.init(wn * 32 * NJ, lane);
  f32x4 acc[2][2 * MI][2 * NJ];
  if constexpr (TALL) {
    run_blocks<Core, MI>((rows + 32 * WR - 1) / (32 * WR), lds, 2 * KT, fa, fb, issue_a, issue_b, acc);
  } else {
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j) acc[hf][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int blocks32 = (rows + 32 * WR - 1 - wm * 32) / (32 * WR);   // row blocks of this wave that hold rows
    static_assert(MI <= 2, "loop variants for 0, 1 and 2 row blocks");
    if (blocks32 >= MI) {
      Core::template run<MI>(lds, 2 * KT, fa, fb, issue_a, issue_b, acc);
    } else if (MI > 1 && blocks32 == 1) {
      Core::template run<1>(lds, 2 * KT, fa, fb, issue_a, issue_b, acc);
    } else {
      Core::template run<0>(lds, 2 * KT, fa, fb, issue_a, issue_b, acc);   // its loads and barriers only
      return;
    }
  }

  // ---- epilogue.  The MFMAs computed (X W)^T per 16 x 16 block: a lane holds ONE row, lane % 16, and FOUR consecutive
  // columns, 4 (lane / 16) .. +3.  Stored straight from there a row would leave in 8- or
  // 16-byte pieces, and partial-line writes are slow in the L2.  Each wave passes 32 rows at a time through an LDS
  // region of its own and reads them back with the lanes laid along the rows, so that a store instruction writes
  // contiguous pieces of rows.  No barrier: the region is private and the LDS runs a wave's instructions in order.
  constexpr int COLS = 32 * NJ;
  constexpr int ESZ = (MODE != 1 || OUT_BF16) ? 2 : 4;
  constexpr int ROW_BYTES = COLS * ESZ;
  constexpr int CH = ROW_BYTES / 16;
  constexpr int RPI = 64 / CH;
  constexpr int SWZ_DIV = ROW_BYTES >= 256 ? 1 : 256 / ROW_BYTES;   // chunk q of row r sits at slot q ^ swz(r)
  constexpr int PIECE = 32 * ROW_BYTES;            // one staged block of 32 rows
  static_assert(3 * PIECE <= Core::LDS_BYTES / (2 * WR) || (!SAVE && PIECE <= Core::LDS_BYTES / (2 * WR)), "staging region");
  auto swz = [&](int r) { return (r / SWZ_DIV) & (CH - 1); };
  char* const ep = lds + wave * (Core::LDS_BYTES / (2 * WR));
  const int rd_row = lane / CH, rd_chunk = lane % CH;
  const int wrow = wm * 32;
  // where this lane's values of fragment (i, j) of the 32 rows go
  auto piece = [&](int i, int j) -> char* {
    const int r = i * 16 + lane % 16, boff = (j * 16 + lane / 16 * 4) * ESZ;
    return ep + r * ROW_BYTES + ((((boff >> 4) ^ swz(r))) << 4) + (boff & 15);
  };
  auto store_lines = [&](const char* from, int mi, char* dst_wave, size_t ld_bytes, bool streaming) {
#pragma unroll
    for (int j = 0; j < 32 / RPI; ++j) {
      const int r = j * RPI + rd_row;
      const u32x4 v = *(const u32x4*)(from + r * ROW_BYTES + ((rd_chunk ^ swz(r)) << 4));
      if (wrow + mi * 32 * WR + r < rows) {
        u32x4* dst = (u32x4*)(dst_wave + (size_t)(mi * 32 * WR + r) * ld_bytes + rd_chunk * 16);
        if (streaming) __builtin_nontemporal_store(v, dst); else *dst = v;
      }
    }
  };
  if constexpr (MODE == 2) {
    // p | q come in as whole lines, requested one pass ahead, go through the staging region to the lanes that hold the
    // matching dH values, and da | db leave the same way
    constexpr int LINES = 32 / RPI;
    u32x4 pl[2][LINES], ql[2][LINES];
    const size_t ld_bytes = (size_t)ld_aux * 2;
    char* const aux_wave = (char*)aux + (size_t)(row0 + wrow) * ld_bytes + (nt * Core::BN + wn * COLS) * 2;
    auto fetch = [&](int pass, int buf) {
      const int mi = pass / 2, hf = pass % 2;
#pragma unroll
      for (int j = 0; j < LINES; ++j) {
        const int r = mi * 32 * WR + j * RPI + rd_row;
        pl[buf][j] = ql[buf][j] = u32x4{0u, 0u, 0u, 0u};
        if (wrow + r < rows) {
          const char* src = aux_wave + (size_t)r * ld_bytes + hf * Core::HW * 2 + rd_chunk * 16;
          pl[buf][j] = *(const u32x4*)src;
          ql[buf][j] = *(const u32x4*)(src + ld_aux);   // q sits ld_aux / 2 columns to the right of p
        }
      }
    };
    fetch(0, 0);
#pragma unroll
    for (int pass = 0; pass < 2 * MI; ++pass) {
      const int mi = pass / 2, hf = pass % 2;
      if (wrow + mi * 32 * WR >= rows) break;
      if (pass + 1 < 2 * MI) fetch(pass + 1, (pass + 1) % 2);
#pragma unroll
      for (int j = 0; j < LINES; ++j) {
        const int r = j * RPI + rd_row;
        char* q = ep + r * ROW_BYTES + ((rd_chunk ^ swz(r)) << 4);
        *(u32x4*)q = pl[pass % 2][j];
        *(u32x4*)(q + PIECE) = ql[pass % 2][j];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j) {
          char* q = piece(i, j);
          const uint2 pv = *(const uint2*)q, qv = *(const uint2*)(q + PIECE);
          const float dp[4] = {bf16_lo(pv.x), bf16_hi(pv.x), bf16_lo(pv.y), bf16_hi(pv.y)};
          const float dq[4] = {bf16_lo(qv.x), bf16_hi(qv.x), bf16_lo(qv.y), bf16_hi(qv.y)};
          float da[4], db[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float dh = acc[hf][2 * mi + i][j][c];
            da[c] = dh * dp[c];
            db[c] = dh * dq[c];
          }
          *(uint2*)q = make_uint2(pack_bf16(da[0], da[1]), pack_bf16(da[2], da[3]));
          *(uint2*)(q + PIECE) = make_uint2(pack_bf16(db[0], db[1]), pack_bf16(db[2], db[3]));
        }
      store_lines(ep, mi, aux_wave + hf * Core::HW * 2, ld_bytes, false);
      store_lines(ep + PIECE, mi, aux_wave + hf * Core::HW * 2 + ld_aux, ld_bytes, false);
    }
    return;
  }
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    if (wrow + mi * 32 * WR >= rows) break;
#pragma unroll
    for (int hf = 0; hf < (MODE == 0 ? 1 : 2); ++hf) {
      const int col0 = (MODE == 0 ? nt * Core::HW : nt * Core::BN + hf * Core::HW) + wn * COLS;
      char* out_wave = (char*)out + ((size_t)(row0 + wrow) * ldo + col0) * ESZ;
      char* aux_wave = (char*)aux + ((size_t)(row0 + wrow) * ld_aux + col0) * 2;
      if constexpr (MODE == 0 && SAVE) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2 * NJ; ++j) {
            char* dst = piece(i, j);
            float hv[4], pv[4], qv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float a = acc[0][2 * mi + i][j][c], b = acc[1][2 * mi + i][j][c];
              const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-a));
              qv[c] = a * sg;
              hv[c] = qv[c] * b;
              pv[c] = b * sg * (1.0f + a - qv[c]);
            }
            *(uint2*)dst = make_uint2(pack_bf16(hv[0], hv[1]), pack_bf16(hv[2], hv[3]));
            *(uint2*)(dst + PIECE) = make_uint2(pack_bf16(pv[0], pv[1]), pack_bf16(pv[2], pv[3]));
            *(uint2*)(dst + 2 * PIECE) = make_uint2(pack_bf16(qv[0], qv[1]), pack_bf16(qv[2], qv[3]));
          }
        store_lines(ep, mi, out_wave, (size_t)ldo * ESZ, false);
        store_lines(ep + PIECE, mi, aux_wave, (size_t)ld_aux * 2, false);
        store_lines(ep + 2 * PIECE, mi, aux_wave + ld_aux, (size_t)ld_aux * 2, false);
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2 * NJ; ++j) {
            char* dst = piece(i, j);
            float v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
              v[c] = MODE == 0 ? silu(acc[0][2 * mi + i][j][c]) * acc[1][2 * mi + i][j][c] : acc[hf][2 * mi + i][j][c];
            if (ESZ == 2)
              *(uint2*)dst = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            else
              *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
          }
        store_lines(ep, mi, out_wave, (size_t)ldo * ESZ, MODE == 1 && !OUT_BF16);   // fp32 rows are read once, by the combine
      }
    }
  }
}

template <int MODE, bool OUT_BF16, bool SAVE, bool B_TR, int WR, int MI, int NJ, int DA, int DB, int OCC>
__global__ __launch_bounds__(128 * WR, OCC) void panel_gemm_kernel(
    const uint16_t* __restrict__ A, int lda, const int* __restrict__ row_src, int n_src_rows, int src_k,
    const int* __restrict__ offsets, int g_begin, int ng, int R_cap, int K, int n_tiles_n, int band,
    WeightTable wt, int ldw, int k_split, void* __restrict__ out, int ldo, void* aux, int ld_aux) {
  using Core = PanelGemm<WR, MI, NJ, DA, DB, false, B_TR>;
  constexpr int SH = Core::BM == 64 ? 6 : Core::BM == 128 ? 7 : 8;
  static_assert((1 << SH) == Core::BM, "tile height");
  constexpr bool QUARTERS = Core::BM == 256;
  __shared__ __attribute__((aligned(1024))) char lds[Core::LDS_BYTES];

  // ---- block -> tile: bands of `band` row tiles, walked column by column; a left-over tile has four blocks
  RowTiles<SH> tiles;
  tiles.init(offsets, g_begin, ng, R_cap);
  const int total = tiles.total * n_tiles_n;
  const int rest = QUARTERS ? total % 256 : 0, whole = rest > 0 && rest <= QUARTERS_MAX ? total - rest : total;
  int idx = tile_of_block<32 * Core::BLOCKS_PER_CU>(blockIdx.x, whole + 4 * (total - whole));
  if (idx < 0) return;
  const int quarter = idx < whole ? -1 : (idx - whole) % 4;
  if (quarter >= 0) idx = whole + (idx - whole) / 4;
  const int b0 = idx / (band * n_tiles_n) * band;
  const int in_band = idx - b0 * n_tiles_n;
  const int height = min(band, tiles.total - b0);
  const RowTile t = tiles.find(b0 + in_band % height, g_begin);
  const Tile tile{t.g, t.row0, t.rows, in_band / height};
  if constexpr (QUARTERS) {
    static_assert(PanelGemm<WR, MI / 2, NJ / 2, 4, 6, false, B_TR>::LDS_BYTES <= Core::LDS_BYTES, "a quarter's rings fit the tile's");
    if (quarter >= 0) {   // row half and column half
      const int below = quarter / 2 * (Core::BM / 2);
      const Tile q{tile.g, tile.row0 + below, min(tile.rows - below, Core::BM / 2), tile.nt * 2 + quarter % 2};
      if (q.rows > 0)
        panel_tile<MODE, OUT_BF16, SAVE, B_TR, WR, MI / 2, NJ / 2, 4, 6>(lds, q, A, lda, row_src, n_src_rows, src_k, K, wt, ldw, k_split, out, ldo, aux, ld_aux);
      return;
    }
  }
  panel_tile<MODE, OUT_BF16, SAVE, B_TR, WR, MI, NJ, DA, DB>(lds, tile, A, lda, row_src, n_src_rows, src_k, K, wt, ldw, k_split, out, ldo, aux, ld_aux);
}

// Estimated time of a round of large tiles of b row blocks of 64: whole[0] + whole[1] b, with half of the columns half[0] + half[1] b
struct Heights {
  int lo, hi;              // b may be lo .. hi
  float whole[2], half[2];
};

// The height of the large tiles by estimated time, from the groups' rows: whole rounds of tiles of the average height, and one of the
// tallest if tiles are left over.  count(b): row tiles of height up to b in all groups; rcp: 1 / x
template <class Count, class Rcp>
__host__ __device__ __forceinline__ int pick_height(const Heights& h, int n_tiles_n, Count&& count, Rcp&& rcp) {
  const float blocks = (float)count(1);
  int best = h.hi;
  float best_us = 0.f;
#pragma unroll
  for (int b = 5; b >= 2; --b) {
    if (b > h.hi || b < h.lo) continue;
    const int row_tiles = count(b), n = row_tiles * n_tiles_n, rest = n % 256;
    const float mean = blocks * rcp((float)row_tiles);
    const float tail = rest == 0 ? 0.f : rest <= QUARTERS_MAX ? h.half[0] + h.half[1] * (float)((b + 1) / 2)
                       : rest <= HALVES_MAX ? h.half[0] + h.half[1] * (float)b : h.whole[0] + h.whole[1] * (float)b;
    const float us = (float)(n / 256) * (h.whole[0] + h.whole[1] * mean) + tail;
    if (b == h.hi || us < best_us) {
      best = b;
      best_us = us;
    }
  }
  return best;
}

template <int MODE, bool OUT_BF16, bool SAVE, bool B_TR>
__global__ __launch_bounds__(256, 1) void tall_gemm_kernel(
    const uint16_t* __restrict__ A, int lda, const int* __restrict__ row_src, int n_src_rows, int src_k,
    const int* __restrict__ offsets, int g_begin, int ng, int R_cap, int K, int n_tiles_n, int band, Heights heights,
    WeightTable wt, int ldw, int k_split, void* __restrict__ out, int ldo, void* aux, int ld_aux) {
  using Core = TallGemm<5, 2, 2, 4, B_TR>;
  using Half = TallGemm<5, 1, 2, 4, B_TR>;
  static_assert(Half::LDS_BYTES <= Core::LDS_BYTES, "a half's rings fit the tile's");
  __shared__ __attribute__((aligned(1024))) char lds[Core::LDS_BYTES];

  // ---- block -> tile: bands of `band` row tiles, walked column by column; a left-over tile has several blocks
  TallTiles tiles;
  tiles.load(offsets, g_begin, ng, R_cap);
  tiles.split(__builtin_amdgcn_readfirstlane(pick_height(heights, n_tiles_n, [&](int b) { return tiles.count(b); },
                                                         [](float x) { return __builtin_amdgcn_rcpf(x); })));
  const int total = tiles.total * n_tiles_n;
  const int rest = total % 256, pieces = rest <= QUARTERS_MAX ? 4 : 2;
  const int whole = rest <= HALVES_MAX ? total - rest : total;
  int idx = tile_of_block<32>(blockIdx.x, whole + pieces * (total - whole));
  if (idx < 0) return;
  const int piece = idx < whole ? -1 : (idx - whole) % pieces;
  if (piece >= 0) idx = whole + (idx - whole) / pieces;
  const int b0 = idx / (band * n_tiles_n) * band;
  const int in_band = idx - b0 * n_tiles_n;
  const int height = min(band, tiles.total - b0);
  const RowTile t = tiles.find(b0 + in_band % height, g_begin);
  Tile tile{t.g, t.row0, t.rows, in_band / height};
  if (piece >= 0) {
    tile.nt = tile.nt * 2 + piece % 2;
    if (pieces == 4) {
      const int upper = (t.rows + 127) / 128 * 64;
      if (piece / 2) {
        tile.row0 += upper;
        tile.rows -= upper;
        if (tile.rows <= 0) return;
      } else {
        tile.rows = min(tile.rows, upper);
      }
    }
    panel_tile<MODE, OUT_BF16, SAVE, B_TR, 2, 5, 1, 2, 4, true>(lds, tile, A, lda, row_src, n_src_rows, src_k, K, wt, ldw, k_split, out, ldo, aux, ld_aux);
    return;
  }
  panel_tile<MODE, OUT_BF16, SAVE, B_TR, 2, 5, 2, 2, 4, true>(lds, tile, A, lda, row_src, n_src_rows, src_k, K, wt, ldw, k_split, out, ldo, aux, ld_aux);
}

// Tile shape by estimated time.  A launch of B tiles runs B / (256 per_cu) full rounds and a rest; a round with one
// (two) workgroups on a CU takes `start` plus k times the measured cost per k.  The costs are a fit to 60 shapes x 3
// GEMMs (1 to 128 groups of 8 to 8000 rows, d and f from 256 to 7168), timed with MFMAs 32x32x16 and with every rest of 256 x 256 tiles a round of
// its own; picking by it was 2 % slower on average than the best of the three each time.  With the present loop it is 3.4 % slower
// (gate/up) and 3.8 % (down) over 60 shapes drawn alike, at most 1.42x.  Part of that are rests that now run as quarters: one round and a
// few tiles, which the estimate sends to 128 x 256, would be faster in 256 x 256 (gate/up, d = 2048, f = 1024: 264 tiles 69.0 us against 65.6, 320 tiles
// 74.5 against 73.1; d = 6144: 184.6 against 172.5 and 204.6 against 187.9).  B is estimated from
// the row capacity, which was the number of rows in those 60: a group of rows ends half a tile early on average, empty ones
// included.  Where the capacity is a multiple of the rows the estimate is of another launch (64 experts, 16 groups, 2110 of
// 6018 rows, d = 2048, f = 1408: gate/up 46 us in 128 x 256 tiles, down 30 us in 256 x 256).  A shape whose rows do not fit the loads' 32-bit
// offsets (256 rows of more than 8.3 million elements) is not taken; the entry points see to it that 64 rows do.
struct Shape {
  int bm, bn, per_cu;
  double start, round[2];   // us; us per 1000 k
};
constexpr Shape SHAPES[3] = {{256, 256, 1, 3.5, {22.3, 0.}}, {128, 256, 2, 4.2, {14.1, 29.9}}, {64, 128, 2, 3.8, {4.8, 12.9}}};

int pick_shape(const feplb::GroupedGemm& a, int weight_cols) {
  int best = -1;
  double best_us = 0.;
  for (int i = 0; i < 3; ++i) {
    const Shape& s = SHAPES[i];
    const bool fits = (a.row_src || feplb::rows_fit_32_bits(s.bm, a.lda)) && (!a.w_nk || feplb::rows_fit_32_bits(s.bn / 2, a.ldw));
    if (!fits && i < 2) continue;
    const double m = (double)a.R_cap / s.bm + 0.5 * a.ng;
    const double tiles = (m > a.ng ? m : a.ng) * (weight_cols / s.bn);
    const double full = (double)(long)(tiles / (256 * s.per_cu)), rest = tiles - full * (256 * s.per_cu);
    const double tail = rest <= 0. ? 0. : s.round[rest > 256 ? 1 : 0];
    const double us = s.start + a.K * 1e-3 * (full * s.round[s.per_cu - 1] + tail);
    if (best < 0 || us < best_us) {
      best = i;
      best_us = us;
    }
  }
  return best;
}

template <int MODE, bool OUT_BF16, bool SAVE, bool B_TR, int WR, int MI, int NJ, int DA, int DB, int OCC>
hipError_t launch(const feplb::GroupedGemm& a, hipStream_t s) {
  using Core = PanelGemm<WR, MI, NJ, DA, DB, false, B_TR>;
  const int n_tiles_n = a.N / (MODE == 0 ? Core::HW : Core::BN);
  const long row_tiles = a.R_cap / Core::BM + a.ng;
  const int band = Core::BM == 256 ? 8 : 16;   // a run of tiles is about as many bytes of rows as of weights
  hipLaunchKernelGGL((panel_gemm_kernel<MODE, OUT_BF16, SAVE, B_TR, WR, MI, NJ, DA, DB, OCC>), dim3(blocks_for_tiles(row_tiles * n_tiles_n + (Core::BM == 256 ? 3 * QUARTERS_MAX : 0))),
                     dim3(128 * WR), 0, s, (const uint16_t*)a.A, a.lda, a.row_src, a.n_src_rows, a.src_k, a.offsets, a.g_begin, a.ng,
                     a.R_cap, a.K, n_tiles_n, band, *a.weights, a.ldw, a.k_split, a.out, a.ldo, a.aux, a.ld_aux);
  return hipGetLastError();
}

// tiles of up to b row blocks in a launch, at most
long most_tiles(const feplb::GroupedGemm& a, int b, int n_tiles_n) { return ((long)a.R_cap / (64 * b) + a.ng) * n_tiles_n; }

// The heights that a launch may take, and what they cost: a fit to 1975 launches drawn over the layer's sizes, each at the four heights, timed
// inside layer steps, where the weights come from memory (`tensors` of 64 rows x 128 columns in 16 bits leave per block and CU).  Off by 10 % in
// the root mean square; the height picked by it is 0.7 % slower than the best of the four.  (Constants from launches timed back to back, whose weights the
// memory-side cache then holds, took lower tiles: 2.5 % slower than the best, plain, and 5 % gate/up.)
Heights tall_heights(const feplb::GroupedGemm& a, bool gate_up, int tensors, int n_tiles_n) {
  Heights h{5, 5, {0.f, 0.f}, {0.f, 0.f}};
  if (!(a.row_src || feplb::rows_fit_32_bits(320, a.lda))) h.lo = h.hi = 4;   // 256 rows do, see use_tall
  while (h.lo > 2 && most_tiles(a, h.lo - 1, n_tiles_n) - most_tiles(a, h.hi, n_tiles_n) <= 512) --h.lo;   // at most two surplus workgroups per CU
  const float k = 1e-3f * a.K, t = (float)tensors;
  if (gate_up) {
    h.whole[0] = 3.1f + 8.f * k;
    h.whole[1] = 0.9f * t + 3.2f * k;
    h.half[0] = 6.8f * k;
    h.half[1] = 1.6f * t + 1.9f * k;
  } else {
    h.whole[0] = 4.4f + 5.8f * k;
    h.whole[1] = 0.5f * t + 3.7f * k;
    h.half[0] = 2.7f + 6.2f * k;
    h.half[1] = 0.1f * t + 2.2f * k;
  }
  return h;
}
int tall_tensors(bool gate_up, bool save, bool out_bf16) { return gate_up ? (save ? 3 : 1) : out_bf16 ? 2 : 4; }

template <int MODE, bool OUT_BF16, bool SAVE, bool B_TR>
hipError_t launch_tall(const feplb::GroupedGemm& a, hipStream_t s) {
  using Core = TallGemm<5, 2, 2, 4, B_TR>;
  const int n_tiles_n = a.N / (MODE == 0 ? Core::HW : Core::BN);
  const Heights h = tall_heights(a, MODE == 0, tall_tensors(MODE == 0, SAVE, OUT_BF16), n_tiles_n);
  const long blocks = most_tiles(a, h.lo, n_tiles_n) + (3 * QUARTERS_MAX > HALVES_MAX ? 3 * QUARTERS_MAX : HALVES_MAX);
  hipLaunchKernelGGL((tall_gemm_kernel<MODE, OUT_BF16, SAVE, B_TR>), dim3(blocks_for_tiles(blocks)), dim3(256), 0, s, (const uint16_t*)a.A, a.lda,
                     a.row_src, a.n_src_rows, a.src_k, a.offsets, a.g_begin, a.ng, a.R_cap, a.K, n_tiles_n, 8, h, *a.weights, a.ldw, a.k_split, a.out,
                     a.ldo, a.aux, a.ld_aux);
  return hipGetLastError();
}

// Does a launch that pick_shape gives to shape 0 or 1 run in tall tiles instead?  Measured inside layer steps, some 4500 launches drawn over the layer's
// sizes, each in that shape and in tall tiles at the height that pick_height takes: geometric mean of the gain, and its first and last tenth.  `tiles`
// are those of the shape, and like it estimated from the row capacity; a fourth of the launches had rows for a part of it only.
//   In the place of 256 x 256, plain, K >= 1280:
//     more than half a round of 256 and up to one, which lower tiles fill better: 1.043 (0.93, 1.21).  Rows for a quarter of a round, which run as
//     quarters of 256 x 256, lose (capacity for 178 tiles, rows for 60: 13 -> 18 us), rows for half of one gain more (for 163 and 60 % of them: 41 -> 29).
//     K = 768 to 1279 1.037 (0.86, 1.23), left out for its first tenth;
//     two rounds and a rest, more than quarters take, that tiles of 320 rows save, 577 to 656 tiles: 1.034 (0.95, 1.15), e.g. 16 groups of about 512 rows,
//     d = 4096, f = 1536, down 126 -> 111 us, dXp 214 -> 193.  Fewer 0.986 (0.92, 1.05);
//     more tiles: K < 2048 0.984 (0.93, 1.05), up to four columns of tiles 0.967 (0.92, 1.03; few tiles share a row of A, which then comes from memory);
//     other 1.001 (0.95, 1.05), taken, since copies beside such a launch find CUs free sooner (replicas' weights staged beside it, 6214 rows,
//     d = 6144, f = 2048: a layer step of 645 to 658 us instead of 673 to 677).
//   Gate/up, more than eight rounds: K < 2048 0.876, to 3071 0.951, to 4095 0.994, to 6143 1.009, from there on, rows for the whole capacity, 1.019 (80387
//     rows, d = 7168, f = 2048 3296 -> 3192 us), for a part of it 0.984; fewer rounds, K >= 6144 1.019 (0.92, 1.16).
//   In the place of 128 x 256 where those would be more than one to a CU, plain, K >= 2048: 1.099 (0.95, 1.30), smaller K 0.986, up to one to a CU 0.991;
//   gate/up, K >= 3072: 1.074 (0.93, 1.30); K = 2048 to 3071, a rest of up to a quarter after a round of 512 1.033 (0.89, 1.21), else 0.973; smaller K 0.905.
bool use_tall(const feplb::GroupedGemm& a, int mode, int weight_cols, int shape) {
  const double tiles = ((double)a.R_cap / SHAPES[shape].bm + 0.5 * a.ng) * (weight_cols / 256);
  if (mode == 2 || shape == 2 || !(a.row_src || feplb::rows_fit_32_bits(256, a.lda))) return false;
  if (shape == 1) return a.K >= (mode == 0 ? 3072 : 2048) ? tiles > 256. : mode == 0 && a.K >= 2048 && tiles > 512. && tiles <= 640.;
  if (mode == 0) return a.K >= 6144 && tiles > 8 * 256.;
  if (a.K < 1280) return false;
  return tiles <= 256. ? tiles > 128. : tiles > 2 * 256. + QUARTERS_MAX && (tiles <= 656. || (a.K >= 2048 && weight_cols > 1024));
}

template <int MODE, bool OUT_BF16, bool SAVE, bool B_TR>
hipError_t launch_shape(const feplb::GroupedGemm& a, hipStream_t s) {
  const int weight_cols = MODE == 0 ? 2 * a.N : a.N, shape = pick_shape(a, weight_cols);
  if constexpr (MODE != 2) {
    if (use_tall(a, MODE, weight_cols, shape)) return launch_tall<MODE, OUT_BF16, SAVE, B_TR>(a, s);
  }
  switch (shape) {
    case 0: return launch<MODE, OUT_BF16, SAVE, B_TR, 4, 2, 2, 3, 3, 2>(a, s);
    case 1: return launch<MODE, OUT_BF16, SAVE, B_TR, 2, 2, 2, 2, 3, 2>(a, s);
    default: return launch<MODE, OUT_BF16, SAVE, B_TR, 2, 1, 1, 3, 6, 2>(a, s);
  }
}

}  // namespace

namespace feplb {

// compiled in parts, for the sake of the build's time
#if !defined(FEPLB_GEMM_PART)
int gemm_tile_rows(const GroupedGemm& a, bool gate_up) { return SHAPES[pick_shape(a, gate_up ? 2 * a.N : a.N)].bm; }
int gemm_tall_rows(const GroupedGemm& a, bool gate_up, bool save, bool out_bf16, const int* offsets) {
  const int weight_cols = gate_up ? 2 * a.N : a.N, n_tiles_n = weight_cols / 256;
  if (!use_tall(a, gate_up ? 0 : 1, weight_cols, pick_shape(a, weight_cols))) return 0;
  auto count = [&](int b) {
    int n = 0;
    for (int g = 0; g < a.ng; ++g) {
      const int lo = offsets[g] < a.R_cap ? offsets[g] : a.R_cap, hi = offsets[g + 1] < a.R_cap ? offsets[g + 1] : a.R_cap;
      if (hi > lo) n += ((hi - lo + 63) / 64 + b - 1) / b;
    }
    return n;
  };
  return 64 * pick_height(tall_heights(a, gate_up, tall_tensors(gate_up, save, out_bf16), n_tiles_n), n_tiles_n, count, [](float x) { return 1.f / x; });
}
hipError_t launch_gate_up(const GroupedGemm& a, hipStream_t s) {
  return a.aux ? launch_gate_up_keeping(a, s) : launch_shape<0, true, false, true>(a, s);
}
#elif FEPLB_GEMM_PART == 1
hipError_t launch_gate_up_keeping(const GroupedGemm& a, hipStream_t s) { return launch_shape<0, true, true, true>(a, s); }
#elif FEPLB_GEMM_PART == 2
hipError_t launch_plain_gemm(const GroupedGemm& a, bool out_bf16, hipStream_t s) {
  if (a.w_nk) return launch_plain_gemm_nk(a, out_bf16, s);
  return out_bf16 ? launch_shape<1, true, false, true>(a, s) : launch_shape<1, false, false, true>(a, s);
}
#elif FEPLB_GEMM_PART == 3
hipError_t launch_plain_gemm_nk(const GroupedGemm& a, bool out_bf16, hipStream_t s) {
  return out_bf16 ? launch_shape<1, true, false, false>(a, s) : launch_shape<1, false, false, false>(a, s);
}
#elif FEPLB_GEMM_PART == 4
hipError_t launch_dswiglu(const GroupedGemm& a, hipStream_t s) {
  return a.w_nk ? launch_shape<2, true, false, false>(a, s) : launch_shape<2, true, false, true>(a, s);
}
#endif

}  // namespace feplb
