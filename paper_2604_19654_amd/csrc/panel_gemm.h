// Main loop shared by the grouped GEMMs, and the mapping from workgroups to ragged tiles.
//
// A workgroup of 2 WR wavefronts (WR wave rows x 2 wave columns) computes a tile of BM = 32 WR MI rows
// x BN = 128 NJ columns.  The contraction runs in tiles of 64.  The second operand of a tile is taken in
// two halves of HW = 64 NJ columns: sub-step u = 2 t + half multiplies the tile's BM x 64 first operand
// with a 64 x HW half of the second, 16 MI NJ MFMAs 16x16x32 per wave.  The first operand's fragments
// stay in registers over both halves.  LDS holds DA tiles of the first operand and a ring of DB half
// tiles of the second, filled by LDS-DMA loads in rows of 128 bytes or more, i.e. whole memory lines.
//
// MFMAs of 16 x 16 x 32, not 32 x 32 x 16: the same flops per cycle and the same LDS reads, but half of the accumulator
// words read and written per flop, and on a chip limited by power that is speed.  93580 x 6144 x 4096: 3308 -> 3099 us (1424 ->
// 1520 TFLOP/s); all grouped GEMMs of the large shapes 1.03x (weight gradients) to 1.08x, small ones unchanged.
//
// What bounds it.  On large shapes the chip is limited by power and by moving operands, not by the pipeline: the matrix
// pipes are busy 80 % of the time at a clock that has come down to 1.65 to 1.85 GHz (gate/up, 93580 and 37490 rows,
// d = 6144, f = 2048), and, measured with MFMAs 32 x 32 x 16, ring depths, band heights, s_setprio and the order of LDS reads between the MFMAs change
// nothing (+-0.5 %).  The loop with its loads taken out, which multiplies the same operands again and again, runs 1.3x as
// fast (93580 x 6144 x 4096: 3500 -> 2690 us).  What did move it is data movement:
// requesting the loads of a sub-step spread over its four slices instead of in one burst behind the
// barrier (93580 x 6144 x 4096: 4040 -> 3550 us), and neighbouring runs of tiles on all XCDs at once
// (tile_of_block below: 3550 -> 3340 us).
//
// Operand layouts.  "Rows": k-contiguous; a line of LDS is 64 k of one row (128 bytes), read with 16-byte
// reads; 16-byte slot p of row r holds k-chunk p ^ ((r >> 1) & 7), so that 16 consecutive rows hit 16
// different bank groups.  "Cols" (A_TR, B_TR): the k index runs over the rows as they lie in memory; a
// line of LDS is one k-row of the panel's columns, read with the transposing ds_read_b64_tr_b16; the
// 64-byte groups of a k-row are XOR-ed with the row, and the halves of a group with its bit 3, so that the eight
// k-rows that half a wave reads 32 bytes each of cover all banks.
//
// Pipeline.  A sub-step is four slices: 32 k of half of a wave's columns, of the other half, then the other 32 k of both.
// One barrier per sub-step, between the third and the fourth slice: there every wave holds the last fragments
// of half tile u, and half tile u+1 (and, if u was a first half, the first operand of the next tile) has landed.  Behind the barrier half tile u+DB is requested into the stage
// just freed, and behind the barrier of a first half tile t+DA of the first operand.  The LDS-DMA
// loads complete in issue order, so the barrier waits with a counted vmcnt for the loads it needs only.
// Requests past the end of the contraction re-read its last tile into stages nobody reads.
#pragma once
#include <numeric>
#include <type_traits>
#include "gemm_device.h"

namespace feplb {
namespace dev {

constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | ((vm >> 4) << 14); }

template <int WR, int MI, int NJ, int DA, int DB, bool A_TR, bool B_TR>
struct PanelGemm {
  static constexpr int BM = 32 * WR * MI;
  static constexpr int HW = 64 * NJ;
  static constexpr int BN = 2 * HW;
  static constexpr int A_BYTES = BM * 128;
  static constexpr int B_BYTES = HW * 128;
  static constexpr int LDS_BYTES = DA * A_BYTES + DB * B_BYTES;
  static constexpr int BLOCKS_PER_CU = 163840 / LDS_BYTES;
  static constexpr int LA = A_BYTES / 1024 / (2 * WR), LB = B_BYTES / 1024 / (2 * WR);   // wavefront loads of 1 KB per wave and stage
  static constexpr int PERIOD = std::lcm(DB, 2 * DA);   // sub-steps after which both rings are back at their start

  // Requests of interval u, between the barriers of sub-steps u and u+1, in this order: half tile u+DB (LB
  // loads), then A_EVEN (u even) or A_ODD (u odd) loads of first-operand tile u/2 + DA.  With DA > 2 the
  // tile is requested over both intervals.  An interval's loads are spread over four slots: slice 3 of
  // sub-step u and slices 0..2 of sub-step u+1.
  static constexpr int A_EVEN = DA > 2 ? (LA + 1) / 2 : LA, A_ODD = LA - A_EVEN;
  static constexpr int interval_loads(int j) { return LB + ((j & 1) == 0 ? A_EVEN : A_ODD); }
  static constexpr int slot_end(int j, int q) { return interval_loads(j) * (q + 1) / 4; }

  // younger loads that may still be in flight at the barrier of a sub-step of this parity
  static constexpr int in_flight(bool odd) {
    auto intervals = [](int j0, int u) {
      int n = 0;
      for (int j = j0; j < u; ++j) n += interval_loads(j);
      return n;
    };
    const int u = 64 + (odd ? 1 : 0);
    const int jb = u + 1 - DB;                                    // interval that requested half tile u+1
    int n = intervals(jb + 1, u) + interval_loads(jb) - LB;
    if (!odd) {
      const int ja = u + 2 - 2 * DA + (A_ODD > 0 ? 1 : 0);        // interval whose last loads complete tile u/2+1
      const int na = intervals(ja + 1, u);
      n = na < n ? na : n;
    }
    return n;
  }
  // the prologue makes the requests of all intervals before -1 and of slot 0 of interval -1; of those,
  // the ones behind the last load of tile 0 and half tile 0
  static constexpr int FIRST = -(2 * DA > DB ? 2 * DA : DB);
  static constexpr int in_flight_start() {
    int n = 0;
    for (int j = FIRST; j < 0; ++j) {
      const int end = j == -1 ? slot_end(j, 0) : interval_loads(j);
      for (int x = 0; x < end; ++x) {
        const bool b = x < LB;
        const int t = -((1 - j) / 2) + DA;
        if (b ? j < -DB : t < 0) continue;
        if (b ? j == -DB : t == 0) n = 0; else ++n;
      }
    }
    return n;
  }

  // An MFMA takes 16 rows of either operand and 32 k: lane l holds k 8 (l / 16) .. +7 of row (or column) l % 16.
  // A wave's rows and columns come in blocks of 32, i.e. two fragments: fragment i is half i % 2 of block i / 2.
  template <int STRIDE>   // rows between the wave's blocks
  struct FragRows {
    uint32_t base[2];
    __device__ __forceinline__ void init(int first_row, int lane) {
      const int r = first_row + lane % 16, h = lane / 16;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) base[ks] = r * 128 + (((4 * ks + h) ^ ((r >> 1) & 7)) << 4);
    }
    __device__ __forceinline__ bf16x8 read(const char* stage, int i, int ks) const {
      return *(const bf16x8*)(stage + base[ks] + (i / 2 * STRIDE + i % 2 * 16) * 128);
    }
  };
  template <int NB, int BLOCKS, int STRIDE>   // panel of 64 NB columns (a k-row is 128 NB bytes); the wave's blocks and the columns between them
  struct FragCols {
    static constexpr int ROW = 128 * NB;
    uint32_t base[2 * BLOCKS];
    __device__ __forceinline__ void init(int first_col, int lane) {
      const int r = (lane / 16) * 8 + (lane % 16) / 4;
#pragma unroll
      for (int i = 0; i < 2 * BLOCKS; ++i) {
        const int col = first_col + i / 2 * STRIDE + i % 2 * 16 + (lane % 4) * 4;
        base[i] = r * ROW + (cols_slot<NB>(r, col / 8) << 4) + (col % 8) * 2;
      }
    }
    // lane s of a 16-lane group addresses 4 columns of k-row s/4 and gets the 4 k-values of column s
    __device__ __forceinline__ bf16x8 read(const char* stage, int i, int ks) const {
      typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
      const char* p = stage + base[i] + ks * 32 * ROW;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 4 * ROW));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };
  // row block mi of wave row wm is block mi WR + wm of the tile: a tile that ends early leaves all SIMDs the same work
  using FragA = std::conditional_t<A_TR, FragCols<WR * MI / 2, MI, 32 * WR>, FragRows<32 * WR>>;
  using FragB = std::conditional_t<B_TR, FragCols<NJ, NJ, 32>, FragRows<32>>;

  // row (or k-row) and 16-byte piece that a lane of load `idx` of a stage reads from memory
  static __device__ __forceinline__ int rows_row(int idx, int lane) { return idx * 8 + lane / 8; }
  static __device__ __forceinline__ int rows_chunk(int idx, int lane) { return (lane % 8) ^ ((rows_row(idx, lane) >> 1) & 7); }
  template <int NB>
  static __device__ __forceinline__ int cols_row(int idx, int lane) { return idx * (8 / NB) + lane / (8 * NB); }
  // 16-byte slot of k-row r that holds piece p of its columns, and (the same map) the piece in slot p: the 64-byte groups
  // are XOR-ed with the k-row, and the halves of a group with its bit 3
  template <int NB>
  static __device__ __forceinline__ int cols_slot(int r, int p) {
    const int x = NB == 1 ? (r >> 1) & 1 : r & 3;
    return p ^ (x << 2) ^ (((r >> 3) & 1) << 1);
  }
  template <int NB>
  static __device__ __forceinline__ int cols_chunk(int idx, int lane) { return cols_slot<NB>(cols_row<NB>(idx, lane), lane % (8 * NB)); }

  // issue_a(stage, t, i), issue_b(stage, u, i): load i of this wave's share of tile t / half tile u to LDS
  // byte address `stage`; each operand's loads are asked for in order.  ME: this wave's row blocks that hold
  // rows (0 .. MI); the other accumulators are left alone.  U = 2 x the number of k tiles.
  template <int ME, class IA, class IB>
  static __device__ __forceinline__ void run(char* lds, int U, const FragA& fa, const FragB& fb, IA&& issue_a, IB&& issue_b,
                                             f32x4 (&acc)[2][2 * MI][2 * NJ]) {
    char* const lds_b = lds + DA * A_BYTES;
    const uint32_t a_off = lds_offset(lds), b_off = lds_offset(lds_b);
    bf16x8 af[2][ME > 0 ? 2 * ME : 1];
    bf16x8 bf[2][NJ];
    constexpr int B_READS = (B_TR ? 2 : 1) * NJ, A_READS = (A_TR ? 2 : 1) * ME;
    // quarter q of the first operand's tile: half of the fragments of 32 k
    auto read_a = [&](int stage, int q) {
      if constexpr (ME > 0) {
#pragma unroll
        for (int i = 0; i < ME; ++i) af[q / 2][q % 2 * ME + i] = fa.read(lds + stage * A_BYTES, q % 2 * ME + i, q / 2);
      }
    };
    // slice s of a half tile: 32 k (s / 2) of half of the wave's columns (s % 2)
    auto read_b = [&](int stage, int s) {
      if constexpr (ME > 0) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) bf[s & 1][j] = fb.read(lds_b + stage * B_BYTES, s % 2 * NJ + j, s / 2);
      }
    };
    auto mfma = [&](int half, int s) {
      if constexpr (ME > 0) {
#pragma unroll
        for (int i = 0; i < 2 * ME; ++i)
#pragma unroll
          for (int jj = 0; jj < NJ; ++jj) {
            const int j = i % 2 ? NJ - 1 - jj : jj;   // there and back: neighbouring MFMAs share an operand (0.4 % on large shapes)
            // second operand first: the product comes out transposed, a lane holds one row and four consecutive columns
            f32x4& c = acc[half][i][s % 2 * NJ + j];
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[s & 1][j], af[s / 2][i], c, 0, 0, 0);
          }
      }
    };
    // load x of interval u; j = u modulo PERIOD
    auto request = [&](auto jc, int u, auto xc) {
      constexpr int j = decltype(jc)::value + 4 * PERIOD, x = decltype(xc)::value;
      if constexpr (x < LB)
        issue_b(b_off + (j % DB) * B_BYTES, u + DB, x);
      else
        issue_a(a_off + (j / 2 % DA) * A_BYTES, (u >> 1) + DA, x - LB + ((j & 1) ? A_EVEN : 0));
    };
    auto slot = [&](auto jc, int u, auto qc) {
      constexpr int j = decltype(jc)::value + 4 * PERIOD, q = decltype(qc)::value;
      constexpr int lo = q == 0 ? 0 : slot_end(j, q - 1), hi = slot_end(j, q);
      range<lo, hi>([&](auto xc) { request(jc, u, xc); });
    };
    range<FIRST, 0>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      constexpr int end = j == -1 ? slot_end(j, 0) : interval_loads(j);
      range<0, end>([&](auto xc) {
        constexpr int x = decltype(xc)::value;
        constexpr bool wanted = x < LB ? j >= -DB : j >= -2 * DA;
        if constexpr (wanted) request(jc, j, xc);
      });
    });
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(in_flight_start(), 15));
    __syncthreads();
    read_a(0, 0);
    read_a(0, 1);
    read_b(0, 0);

    // the first operand's quarters are read a slice each: 0 and 1 of the next tile in the last two slices of a second
    // half, when the present tile's are done with, 2 and 3 in the first two of the first half that follows
    auto step = [&](auto sc, int u) {
      constexpr int s = decltype(sc)::value;         // u mod PERIOD
      constexpr int half = s & 1, sb = s % DB, sb_next = (s + 1) % DB, sa = s / 2 % DA, sa_next = (s / 2 + 1) % DA;
      constexpr std::integral_constant<int, s - 1> before{};
      auto slice = [&](auto kc) {
        constexpr int q = decltype(kc)::value;
        slot(before, u - 1, std::integral_constant<int, q + 1>{});
        read_b(sb, q + 1);
        if (half == 0 && q < 2) read_a(sa, q + 2);
        if (half == 1 && q == 2) read_a(sa_next, 0);
        mfma(half, q);
        interleave<B_READS + (((half == 0 && q < 2) || (half == 1 && q == 2)) ? A_READS : 0), 2 * ME * NJ>();
        __builtin_amdgcn_sched_barrier(0);
      };
      slice(std::integral_constant<int, 0>{});
      slice(std::integral_constant<int, 1>{});
      slice(std::integral_constant<int, 2>{});
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(in_flight(half == 1), 0));
      __syncthreads();
      slot(sc, u, std::integral_constant<int, 0>{});
      read_b(sb_next, 0);
      if (half == 1) read_a(sa_next, 1);
      mfma(half, 3);
      interleave<B_READS + (half == 1 ? A_READS : 0), 2 * ME * NJ>();
      __builtin_amdgcn_sched_barrier(0);
    };
    int u = 0;
    for (; u + PERIOD <= U; u += PERIOD) range<0, PERIOD>([&](auto sc) { step(sc, u + decltype(sc)::value); });
    tail<0>(step, u, U);
    __builtin_amdgcn_s_waitcnt(0);   // requests past the end must land before the stages are reused
    __syncthreads();
  }

 private:
  template <int LO, int HI, class F>
  static __device__ __forceinline__ void range(F&& f) {
    if constexpr (LO < HI) {
      f(std::integral_constant<int, LO>{});
      range<LO + 1, HI>(f);
    }
  }
  template <int S, class F>
  static __device__ __forceinline__ void tail(F& step, int u, int U) {
    if constexpr (S < PERIOD) {
      if (u + S < U) {
        step(std::integral_constant<int, S>{}, u + S);
        step(std::integral_constant<int, S + 1>{}, u + S + 1);
        tail<S + 2>(step, u, U);
      }
    }
  }
  // a slice's LDS reads spread over its MFMAs
  template <int R, int M>
  static __device__ __forceinline__ void interleave() {
    if constexpr (M > 0) {
      constexpr int per = (R + M - 1) / M;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x100, per, 0);   // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one MFMA
      }
    }
  }
};

// ---- ragged row tiles

struct RowTile {
  int g, row0, rows;   // group, first row, number of rows
};

// inclusive prefix sum over the 64 lanes of a wavefront (row shifts inside rows of 16 lanes, then row broadcasts)
__device__ __forceinline__ int wave_prefix_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// The row tiles of height 2^SH of groups [g_begin, g_begin + ng), ng <= 128, found by every wave for itself from
// the groups' row offsets (lane l holds groups l and 64 + l): no table, no launch to build one.
template <int SH>
struct RowTiles {
  int lo0, hi0, lo1, hi1, end0, end1, total;   // end: tiles up to and including the lane's group
  __device__ __forceinline__ void init(const int* __restrict__ offsets, int g_begin, int ng, int R_cap) {
    static_assert(FEPLB_MAX_GROUPS <= 128, "two groups per lane");
    const int lane = threadIdx.x % 64;
    auto tiles = [](int lo, int hi) { return hi > lo ? (hi - lo + (1 << SH) - 1) >> SH : 0; };
    lo0 = hi0 = lo1 = hi1 = 0;
    if (lane < ng) {
      lo0 = min(offsets[g_begin + lane], R_cap);
      hi0 = min(offsets[g_begin + lane + 1], R_cap);
    }
    end0 = wave_prefix_sum(tiles(lo0, hi0));
    total = __builtin_amdgcn_readlane(end0, 63);
    end1 = 0x7fffffff;
    if (ng > 64) {
      if (64 + lane < ng) {
        lo1 = min(offsets[g_begin + 64 + lane], R_cap);
        hi1 = min(offsets[g_begin + 64 + lane + 1], R_cap);
      }
      end1 = total + wave_prefix_sum(tiles(lo1, hi1));
      total = __builtin_amdgcn_readlane(end1, 63);
    }
  }
  __device__ __forceinline__ RowTile find(int m, int g_begin) const {   // m < total
    int a = __popcll(__ballot(end0 <= m)), lo, hi, first;
    if (a < 64) {
      lo = __builtin_amdgcn_readlane(lo0, a);
      hi = __builtin_amdgcn_readlane(hi0, a);
      first = a ? __builtin_amdgcn_readlane(end0, a - 1) : 0;
    } else {
      const int b = __popcll(__ballot(end1 <= m));
      lo = __builtin_amdgcn_readlane(lo1, b);
      hi = __builtin_amdgcn_readlane(hi1, b);
      first = b ? __builtin_amdgcn_readlane(end1, b - 1) : __builtin_amdgcn_readlane(end0, 63);
      a = 64 + b;
    }
    RowTile t;
    t.g = g_begin + a;
    t.row0 = lo + ((m - first) << SH);
    t.rows = min(1 << SH, hi - t.row0);
    return t;
  }
};

// Position in the launch's sequence of `total` tiles that block b computes, or -1.  Workgroups are dealt round-robin
// to the 8 XCDs, each with its own L2.  Runs of PATCH tiles (what an XCD has in work at a time) go to the XCDs in turn:
// tiles of a run share panels in the XCD's L2, and neighbouring runs, in work on all XCDs at once, share theirs in the
// memory-side cache.  What is left after whole deals is split evenly, so no XCD is idle for the last round.  (A contiguous
// eighth of the sequence per XCD: 6 % slower at 93580 rows, d = 6144, f = 2048.)
template <int PATCH>
__device__ __forceinline__ int tile_of_block(int b, int total) {
  const int xcd = b % XCDS, slot = b / XCDS;
  const int deals = total / (XCDS * PATCH);
  if (slot < deals * PATCH) return (slot / PATCH * XCDS + xcd) * PATCH + slot % PATCH;
  const int done = deals * (XCDS * PATCH), rest = slot - deals * PATCH;
  const int per = (total - done + XCDS - 1) / XCDS;
  const int idx = done + xcd * per + rest;
  return rest < per && idx < total ? idx : -1;
}
// workgroups that cover every tile of any sequence of at most `total` tiles
inline unsigned blocks_for_tiles(long total) { return (unsigned)((total + XCDS - 1) / XCDS * XCDS); }

}  // namespace dev
}  // namespace feplb
