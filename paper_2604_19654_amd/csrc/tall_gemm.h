// The grouped GEMMs' loop for tall tiles: up to 320 rows x 256 columns by four wavefronts, one per SIMD.
//
// A wave multiplies up to 160 x 128 (5 row blocks of 32), so that an operand read from LDS is used more often than by the eight
// wavefronts of panel_gemm.h.  Inside layer steps a round of 256 tiles takes 6 to 8 us per 1000 k and 3.2 to 3.7 more for every 64 rows of height
// (tall_heights in ffn_gemm.hip), so that heights can be chosen to fill whole rounds of the 256 CUs: 16 groups of about 512 rows, d = 4096,
// f = 1536 (two tiles of five or four blocks each in the place of two or three of 256 rows), profiled in a training step: down 126 -> 111 us,
// dXp 214 -> 193.  Over many rounds, back to back, against 256 x 256 by eight wavefronts: 93580 rows, d = 6144, f = 2048 gate/up 3135 -> 3112 us,
// down 1874 -> 1807, dXp 3318 -> 3222.  What bounds it is the power limit: 256 x 256
// by four wavefronts keeps the matrix pipes busy 82 % of the time at 1.82 GHz where eight do 83 % at 1.69 GHz (gate/up of the large shape, profiled), with a
// third fewer LDS reads; back to back, hot, that is 1 to 3 %.
//
// The rings of four wavefronts hold fewer k ahead (two tiles of A, four half tiles of the weights), so launches whose operands come from memory and that are
// short (small K), read a row of A for few columns, or have few tiles are faster in the other shapes (use_tall in ffn_gemm.hip has both sides).
//
// With one wave per SIMD nothing hides behind another wave's MFMAs: the order of MFMAs, LDS reads and loads is fixed in the source, a
// fragment read behind every other MFMA and a load behind every fourth (reads ahead of a slice's MFMAs, as the compiler places them: 7 % slower).
// The accumulators take up to 320 of 512 registers; the MFMAs are inline assembly with the accumulator as source and result, since the
// compiler's own choice moved accumulators between registers inside the loop (-19 %).  What the compiler then does not know about them stands at
// the two statements with wait states below.
//
// Pipeline, rings, LDS layout and fragments are those of panel_gemm.h.
#pragma once
#include "panel_gemm.h"

namespace feplb {
namespace dev {

template <int MI, int NJ, int DA, int DB, bool B_TR>
struct TallGemm : PanelGemm<2, MI, NJ, DA, DB, false, B_TR> {
  using Base = PanelGemm<2, MI, NJ, DA, DB, false, B_TR>;
  using typename Base::FragA;
  using typename Base::FragB;
  using Base::A_BYTES;
  using Base::B_BYTES;
  using Base::LA;
  using Base::LB;
  static constexpr int PERIOD = Base::PERIOD;
  static_assert(PERIOD == 4, "k are multiples of 128, 4 sub-steps");
  static constexpr int AGPR_FRAGS = 16 / NJ;   // accumulator fragments from here on are left to the vector registers

  // Requests of interval u, between the barriers of sub-steps u and u+1, in this order: half tile u+DB (LB
  // loads), then even(la) (u even) or la - even(la) (u odd) loads of first-operand tile u/2 + DA.  With DA > 2 the
  // tile is requested over both intervals.  An interval's loads are spread over four slots: slice 3 of
  // sub-step u and slices 0..2 of sub-step u+1.  la: loads of a first-operand tile by this wave, fewer than LA if it ends early.
  static constexpr int even(int la) { return DA > 2 ? (la + 1) / 2 : la; }
  static constexpr int interval_loads(int la, int j) { return LB + ((j & 1) == 0 ? even(la) : la - even(la)); }
  static constexpr int slot_end(int la, int j, int q) { return interval_loads(la, j) * (q + 1) / 4; }
  static constexpr int SLOT_MAX = (LB + LA + 3) / 4;

  // younger loads that may still be in flight at the barrier of a sub-step of this parity
  static constexpr int in_flight(int la, bool odd) {
    auto intervals = [la](int j0, int u) {
      int n = 0;
      for (int j = j0; j < u; ++j) n += interval_loads(la, j);
      return n;
    };
    const int u = 64 + (odd ? 1 : 0);
    const int jb = u + 1 - DB;                                          // interval that requested half tile u+1
    int n = intervals(jb + 1, u) + interval_loads(la, jb) - LB;
    if (!odd) {
      const int ja = u + 2 - 2 * DA + (la > even(la) ? 1 : 0);          // interval whose last loads complete tile u/2+1
      const int na = intervals(ja + 1, u);
      n = na < n ? na : n;
    }
    return n;
  }
  // the prologue makes the requests of all intervals before -1 and of slot 0 of interval -1; of those,
  // the ones behind the last load of tile 0 and half tile 0
  static constexpr int FIRST = -(2 * DA > DB ? 2 * DA : DB);
  static constexpr int in_flight_start(int la) {
    int n = 0;
    for (int j = FIRST; j < 0; ++j) {
      const int end = j == -1 ? slot_end(la, j, 0) : interval_loads(la, j);
      for (int x = 0; x < end; ++x) {
        const bool b = x < LB;
        const int t = -((1 - j) / 2) + DA;
        if (b ? j < -DB : t < 0) continue;
        if (b ? j == -DB : t == 0) n = 0; else ++n;
      }
    }
    return n;
  }

  // issue_a(stage, t, i), issue_b(stage, u, i): load i of this wave's share of tile t / half tile u to LDS
  // byte address `stage`; each operand's loads are asked for in order.  ME: row blocks of a wave that may hold
  // rows (1 .. MI): the others are neither loaded nor multiplied, and their accumulators are not set.  U = 2 x the number of k tiles,
  // a multiple of PERIOD.
  template <int ME, class IA, class IB>
  static __device__ __forceinline__ void run(char* lds, int U, const FragA& fa, const FragB& fb, IA&& issue_a, IB&& issue_b,
                                             f32x4 (&acc)[2][2 * MI][2 * NJ]) {
    constexpr int la = LA / MI * ME;
    char* const lds_b = lds + DA * A_BYTES;
    const uint32_t a_off = lds_offset(lds), b_off = lds_offset(lds_b);
    bf16x8 af[2][2 * ME];
    bf16x8 bf[2][NJ];
    // fragment i of quarter q of the first operand's tile (half of the fragments of 32 k)
    auto read_a = [&](int stage, int q, int i) { af[q / 2][q % 2 * ME + i] = fa.read(lds + stage * A_BYTES, q % 2 * ME + i, q / 2); };
    // fragment j of slice s of a half tile: 32 k (s / 2) of half of the wave's columns (s % 2)
    auto read_b = [&](int stage, int s, int j) { bf[s & 1][j] = fb.read(lds_b + stage * B_BYTES, s % 2 * NJ + j, s / 2); };
    // MFMA m of a slice; second operand first: the product comes out transposed, a lane holds one row and four consecutive columns
    auto mfma = [&](int half, int s, auto mc) {
      constexpr int m = decltype(mc)::value, i = m / NJ;
      constexpr int j = i % 2 ? NJ - 1 - m % NJ : m % NJ;   // there and back: neighbouring MFMAs share an operand (0.4 % on large shapes)
      const bf16x8 a = af[s / 2][i], b = bf[s & 1][j];
      f32x4& c = acc[half][i][s % 2 * NJ + j];
      if constexpr (i < AGPR_FRAGS)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(b), "v"(a));
      else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(b), "v"(a));
    };
    // load x of interval u; j = u modulo PERIOD
    auto request = [&](auto jc, int u, auto xc) {
      constexpr int j = decltype(jc)::value + 4 * PERIOD, x = decltype(xc)::value;
      if constexpr (x < LB)
        issue_b(b_off + (j % DB) * B_BYTES, u + DB, x);
      else
        issue_a(a_off + (j / 2 % DA) * A_BYTES, (u >> 1) + DA, x - LB + ((j & 1) ? even(la) : 0), la);
    };
    // loads lo .. hi - 1 of slot q of interval u
    auto slot = [&](auto jc, int u, auto qc, auto lo, auto hi) {
      constexpr int j = decltype(jc)::value + 4 * PERIOD, q = decltype(qc)::value;
      constexpr int begin = q == 0 ? 0 : slot_end(la, j, q - 1), end = slot_end(la, j, q);
      constexpr int l = begin + decltype(lo)::value, h = begin + decltype(hi)::value;
      range<l, (h < end ? h : end)>([&](auto xc) { request(jc, u, xc); });
    };
    range<FIRST, 0>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      constexpr int end = j == -1 ? slot_end(la, j, 0) : interval_loads(la, j);
      range<0, end>([&](auto xc) {
        constexpr int x = decltype(xc)::value;
        constexpr bool wanted = x < LB ? j >= -DB : j >= -2 * DA;
        if constexpr (wanted) request(jc, j, xc);
      });
    });
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int i = 0; i < 2 * ME; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j) acc[hf][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(in_flight_start(la), 15));
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < ME; ++i) read_a(0, q, i);
#pragma unroll
    for (int j = 0; j < NJ; ++j) read_b(0, 0, j);

    // the first operand's quarters are read a slice each: 0 and 1 of the next tile in the last two slices of a second
    // half, when the present tile's are done with, 2 and 3 in the first two of the first half that follows
    auto step = [&](auto sc, int u) {
      constexpr int s = decltype(sc)::value;         // u mod PERIOD
      constexpr int half = s & 1, sb = s % DB, sb_next = (s + 1) % DB, sa = s / 2 % DA, sa_next = (s / 2 + 1) % DA;
      auto slice = [&](auto kc) {
        constexpr int q = decltype(kc)::value;
        constexpr int M = 2 * ME * NJ;
        constexpr int R = NJ + ((half == 0) == (q < 2) ? ME : 0);   // fragments read for the next slices
        auto read = [&](int r) {
          if (r < NJ) read_b(q < 3 ? sb : sb_next, (q + 1) % 4, r);
          else read_a(half == 0 ? sa : sa_next, (q + 2) % 4, r - NJ);
        };
        auto load = [&](auto lo, auto hi) {
          if constexpr (q < 3) slot(std::integral_constant<int, s - 1>{}, u - 1, std::integral_constant<int, q + 1>{}, lo, hi);
          else slot(sc, u, std::integral_constant<int, 0>{}, lo, hi);
        };
        if constexpr (q == 3) {
          __builtin_amdgcn_s_waitcnt(waitcnt_imm(in_flight(la, half == 1), 0));
          __syncthreads();
        }
        constexpr int EVERY = R <= M / 2 ? 2 : 1, PER = M >= 4 * SLOT_MAX ? 4 : M >= SLOT_MAX ? M / SLOT_MAX : 1;
        range<0, M>([&](auto mc) {
          constexpr int m = decltype(mc)::value, x = m / PER;
          mfma(half, q, mc);
          if constexpr (m % EVERY == 0 && m / EVERY < R) read(m / EVERY);
          if constexpr (m == M - 1) load(std::integral_constant<int, x>{}, std::integral_constant<int, SLOT_MAX>{});
          else if constexpr (m % PER == PER - 1) load(std::integral_constant<int, x>{}, std::integral_constant<int, x + 1>{});
          __builtin_amdgcn_sched_barrier(0);
        });
      };
      range<0, 4>(slice);
    };
    int u = 0;
    for (; u + PERIOD <= U; u += PERIOD) {
      range<0, PERIOD>([&](auto sc) { step(sc, u + decltype(sc)::value); });
      // The compiler does not know that the MFMAs take 4 passes to write their results.  Where control branches it may copy accumulators to
      // other registers: the wait states ahead of such a copy (7, a test reads the built code for them) stand here.
      asm volatile("s_nop 7");
    }
    __builtin_amdgcn_s_waitcnt(0);   // requests past the end must land before the stages are reused
    __syncthreads();
    // The wait states between the last MFMAs and a read of their results, which the compiler does not see in inline assembly; nothing
    // that uses an accumulator can move ahead of its empty statement.
    asm volatile("s_nop 15\n\ts_nop 3");
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int i = 0; i < 2 * ME; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j)
          if (i < AGPR_FRAGS) asm volatile("" : "+a"(acc[hf][i][j]));
          else asm volatile("" : "+v"(acc[hf][i][j]));
  }

 private:
  template <int LO, int HI, class F>
  static __device__ __forceinline__ void range(F&& f) {
    if constexpr (LO < HI) {
      f(std::integral_constant<int, LO>{});
      range<LO + 1, HI>(f);
    }
  }
};

// ---- tiles of any height

// The row tiles of groups [g_begin, g_begin + ng), ng <= 128, found by every wave for itself from the groups' row
// offsets (lane l holds groups l and 64 + l): no table, no launch to build one.  Heights are multiples of 64 up to 64 b; a group
// of n rows has as few tiles as that allows and all of one height but the last (the tiles of a launch then take about as long as each other).
struct TallTiles {
  int lo0, hi0, lo1, hi1;   // rows
  int h0, h1, end0, end1;   // height in blocks of 64 rows; tiles up to and including the lane's group
  int total;
  bool two;
  __device__ __forceinline__ void load(const int* __restrict__ offsets, int g_begin, int ng, int R_cap) {
    static_assert(FEPLB_MAX_GROUPS <= 128, "two groups per lane");
    const int lane = threadIdx.x % 64;
    lo0 = hi0 = lo1 = hi1 = 0;
    two = ng > 64;
    if (lane < ng) {
      lo0 = min(offsets[g_begin + lane], R_cap);
      hi0 = max(min(offsets[g_begin + lane + 1], R_cap), lo0);
    }
    if (64 + lane < ng) {
      lo1 = min(offsets[g_begin + 64 + lane], R_cap);
      hi1 = max(min(offsets[g_begin + 64 + lane + 1], R_cap), lo1);
    }
  }
  static __device__ __forceinline__ int blocks(int lo, int hi) { return (hi - lo + 63) / 64; }
  // row tiles of height up to 64 b, all groups
  __device__ __forceinline__ int count(int b) const {
    int n = (blocks(lo0, hi0) + b - 1) / b;
    if (two) n += (blocks(lo1, hi1) + b - 1) / b;
    return __builtin_amdgcn_readlane(wave_prefix_sum(n), 63);
  }
  __device__ __forceinline__ void split(int b) {
    auto tiles = [b](int n, int& h) {
      const int t = (n + b - 1) / b;
      h = t > 1 ? (n + t - 1) / t : max(n, 1);
      return (n + h - 1) / h;
    };
    end0 = wave_prefix_sum(tiles(blocks(lo0, hi0), h0));
    total = __builtin_amdgcn_readlane(end0, 63);
    end1 = 0x7fffffff;
    h1 = 1;
    if (two) {
      end1 = total + wave_prefix_sum(tiles(blocks(lo1, hi1), h1));
      total = __builtin_amdgcn_readlane(end1, 63);
    }
  }
  __device__ __forceinline__ RowTile find(int m, int g_begin) const {   // m < total
    int a = __popcll(__ballot(end0 <= m)), lo, hi, first, h;
    if (a < 64) {
      lo = __builtin_amdgcn_readlane(lo0, a);
      hi = __builtin_amdgcn_readlane(hi0, a);
      h = __builtin_amdgcn_readlane(h0, a);
      first = a ? __builtin_amdgcn_readlane(end0, a - 1) : 0;
    } else {
      const int b = __popcll(__ballot(end1 <= m));
      lo = __builtin_amdgcn_readlane(lo1, b);
      hi = __builtin_amdgcn_readlane(hi1, b);
      h = __builtin_amdgcn_readlane(h1, b);
      first = b ? __builtin_amdgcn_readlane(end1, b - 1) : __builtin_amdgcn_readlane(end0, 63);
      a = 64 + b;
    }
    RowTile t;
    t.g = g_begin + a;
    t.row0 = lo + (m - first) * h * 64;
    t.rows = min(h * 64, hi - t.row0);
    return t;
  }
};

}  // namespace dev
}  // namespace feplb
