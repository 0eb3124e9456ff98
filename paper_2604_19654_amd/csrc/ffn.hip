// Ragged grouped SwiGLU expert FFN on bf16 MFMA (paper Section 3.1: expert
// compute is a Grouped GEMM; Sections 1 and 2.3: its speed depends on each
// expert's batch size and it must not fragment into per-expert launches).
//
// Forward: two grouped GEMMs, each ONE launch for a whole range of groups (ffn_gemm.hip):
//   gate_up : H[r,:]  = bf16( silu(x_r Wg[g]) * (x_r Wu[g]) ),  x_r = Xp[r,:] or, with row_src,
//             the token row X[row_src[r] / k, :] gathered while it is loaded
//   down    : Yp[r,:] = H[r,:] Wd[g]
// The training form of gate_up also keeps, for the backward pass, the two partial derivatives of
// its output with respect to the products a = x Wg and b = x Wu,
//   p = dH/da = b s (1 + a (1 - s)),   q = dH/db = a s,   s = sigmoid(a)        (bf16).
// The backward pass computes the input gradients (Section 3.2 times it as well) with the same kernel:
//   dswiglu : dH = dYp Wd^T, then [da | db] = [dH p | dH q], written over [p | q]
//   plain   : dXp = [da | db] [Wg | Wu]^T
// and the weight gradients with the ragged GEMM of ffn_backward.hip.  All launches find their tiles
// from offsets[] (device memory, ragged, possibly empty groups): the host never needs R.
#include "common.h"
#include "gemm_device.h"

namespace {
using namespace feplb::dev;

// The workspace, which no kernel uses any more and callers still size and pass: 16 bytes per 256-row tile, in the worst split
// over the groups, and one more; then one word per possible group.
size_t table_bytes(int R_cap, int ng) { return (size_t)(R_cap / 256 + ng + 2) * 16; }

}  // namespace

extern "C" size_t feplb_grouped_ffn_workspace_bytes(int32_t R_cap, int32_t G) {
  if (R_cap < 0 || G < 0) return 0;
  return table_bytes(R_cap, G) + FEPLB_MAX_GROUPS * sizeof(int);
}

namespace {
int32_t forward_impl(const void* Xp, const int32_t* row_src, int32_t T, int32_t k,
                     const int32_t* offsets, int32_t g_begin,
                     int32_t g_end, int32_t R_cap, int32_t d, int32_t f,
                     const void* const* w_gate, const void* const* w_up,
                     const void* const* w_down, void* H, void* AB, void* Yp,
                     int32_t yp_dtype, int32_t phases, bool needs_ws, void* ws, size_t ws_bytes,
                     void* stream) {
  FEPLB_REQUIRE(g_begin >= 0 && g_end >= g_begin && R_cap >= 0 && d >= 0 && f >= 0, FEPLB_EINVAL,
                "grouped_ffn: negative size or empty range reversed");
  FEPLB_REQUIRE(g_end <= FEPLB_MAX_GROUPS, FEPLB_ESHAPE, "grouped_ffn: g_end=%d above %d", g_end,
                FEPLB_MAX_GROUPS);
  FEPLB_REQUIRE((phases & ~FEPLB_FFN_ALL) == 0 && phases != 0, FEPLB_EINVAL,
                "grouped_ffn: phases=%d", phases);
  FEPLB_REQUIRE(yp_dtype == FEPLB_F32 || yp_dtype == FEPLB_BF16, FEPLB_EINVAL,
                "grouped_ffn: unknown yp_dtype %d", yp_dtype);
  // (both k extents, d and f, are then multiples of 128: the k loop runs two 64-wide steps per trip)
  FEPLB_REQUIRE(d % 256 == 0 && f % 128 == 0 && d > 0 && f > 0, FEPLB_ESHAPE,
                "grouped_ffn: need d %% 256 == 0 and f %% 128 == 0 (d=%d f=%d)", d, f);
  const int ng = g_end - g_begin;
  if (ng == 0 || R_cap == 0) return FEPLB_OK;
  FEPLB_REQUIRE(offsets, FEPLB_EINVAL, "grouped_ffn: null offsets");
  const bool do_up = phases & FEPLB_FFN_GATE_UP, do_down = phases & FEPLB_FFN_DOWN;
  const int rows = R_cap < 64 ? R_cap : 64;   // of the smallest tile; 64 rows of each weight matrix are a k tile
  FEPLB_REQUIRE((!do_up || ((row_src || feplb::rows_fit_32_bits(rows, d)) && feplb::rows_fit_32_bits(64, f))) &&
                    (!do_down || (feplb::rows_fit_32_bits(rows, f) && feplb::rows_fit_32_bits(64, d))),
                FEPLB_ESHAPE, "grouped_ffn: 64 rows do not fit 32-bit byte offsets (d=%d f=%d)", d, f);
  if (do_up) {
    FEPLB_REQUIRE(Xp && H && w_gate && w_up, FEPLB_EINVAL, "grouped_ffn: null Xp/H/w_gate/w_up");
    if (row_src) {
      // the kernel addresses a gathered row as a 32-bit byte offset from X
      FEPLB_REQUIRE(T > 0 && k > 0 && (uint64_t)T * (uint64_t)d * 2 <= 0xffffffffull, FEPLB_ESHAPE,
                    "grouped_ffn: gathering needs T > 0, k > 0 and T*d*2 < 4 GiB (T=%d k=%d d=%d)", T, k, d);
    }
    FEPLB_REQUIRE(feplb::aligned16(Xp) && feplb::aligned16(H) && feplb::aligned16(AB), FEPLB_EALIGN,
                  "grouped_ffn: Xp/H/AB not 16-byte aligned");
  }
  if (do_down) {
    FEPLB_REQUIRE(Yp && H && w_down, FEPLB_EINVAL, "grouped_ffn: null Yp/H/w_down");
    FEPLB_REQUIRE(feplb::aligned16(Yp) && feplb::aligned16(H), FEPLB_EALIGN,
                  "grouped_ffn: Yp/H not 16-byte aligned");
  }
  WeightTable up_tab{}, down_tab{};
  for (int g = g_begin; g < g_end; ++g) {
    if (do_up) {
      FEPLB_REQUIRE(w_gate[g] && w_up[g], FEPLB_EINVAL, "grouped_ffn: null weights of group %d", g);
      FEPLB_REQUIRE(feplb::aligned16(w_gate[g]) && feplb::aligned16(w_up[g]), FEPLB_EALIGN,
                    "grouped_ffn: weights of group %d not 16-byte aligned", g);
      up_tab.w0[g] = w_gate[g];
      up_tab.w1[g] = w_up[g];
    }
    if (do_down) {
      FEPLB_REQUIRE(w_down[g], FEPLB_EINVAL, "grouped_ffn: null w_down of group %d", g);
      FEPLB_REQUIRE(feplb::aligned16(w_down[g]), FEPLB_EALIGN,
                    "grouped_ffn: w_down of group %d not 16-byte aligned", g);
      down_tab.w0[g] = w_down[g];
      down_tab.w1[g] = nullptr;
    }
  }
  if (needs_ws) {
    const size_t need = table_bytes(R_cap, ng);
    FEPLB_REQUIRE(ws && ws_bytes >= need, FEPLB_EWORKSPACE, "grouped_ffn: workspace %zu < %zu", ws_bytes, need);
    FEPLB_REQUIRE(feplb::aligned16(ws), FEPLB_EALIGN, "grouped_ffn: workspace not 16-byte aligned");
  }
  hipStream_t s = (hipStream_t)stream;
  if (do_up) {
    const feplb::GroupedGemm a{Xp, d, row_src, T, k, offsets, g_begin, ng, R_cap, d, f, &up_tab, f, false, d, H, f, AB, 2 * f};
    FEPLB_HIP(feplb::launch_gate_up(a, s));
  }
  if (do_down) {
    const feplb::GroupedGemm a{H, f, nullptr, 0, 1, offsets, g_begin, ng, R_cap, f, d, &down_tab, d, false, f, Yp, d, nullptr, 0};
    FEPLB_HIP(feplb::launch_plain_gemm(a, yp_dtype == FEPLB_BF16, s));
  }
  return FEPLB_OK;
}
}  // namespace

extern "C" int32_t feplb_grouped_ffn(const void* Xp, const int32_t* row_src, int32_t T, int32_t k,
                                     const int32_t* offsets, int32_t g_begin,
                                     int32_t g_end, int32_t R_cap, int32_t d, int32_t f,
                                     const void* const* w_gate, const void* const* w_up,
                                     const void* const* w_down, void* H, void* Yp,
                                     int32_t yp_dtype, int32_t phases, void* ws, size_t ws_bytes,
                                     void* stream) {
  return forward_impl(Xp, row_src, T, k, offsets, g_begin, g_end, R_cap, d, f, w_gate, w_up, w_down, H,
                      nullptr, Yp, yp_dtype, phases, true, ws, ws_bytes, stream);
}

extern "C" int32_t feplb_grouped_ffn_static(const void* Xp, const int32_t* row_src, int32_t T, int32_t k,
                                            const int32_t* offsets, int32_t g_begin, int32_t g_end,
                                            int32_t R_cap, int32_t d, int32_t f, const void* const* w_gate,
                                            const void* const* w_up, const void* const* w_down, void* H,
                                            void* Yp, int32_t yp_dtype, int32_t phases, void* stream) {
  FEPLB_REQUIRE(g_begin >= 0 && g_end >= g_begin && R_cap >= 0, FEPLB_EINVAL,
                "grouped_ffn_static: negative size or empty range reversed");
  const size_t need = feplb_grouped_ffn_workspace_bytes(R_cap, g_end - g_begin);
  FEPLB_REQUIRE(need <= (size_t)FEPLB_STATIC_WS_BYTES, FEPLB_ESHAPE,
                "grouped_ffn_static: R_cap=%d rows in %d groups need %zu bytes of tile table, the built-in scratch "
                "holds %d; use feplb_grouped_ffn with a workspace", R_cap, g_end - g_begin, need, FEPLB_STATIC_WS_BYTES);
  return forward_impl(Xp, row_src, T, k, offsets, g_begin, g_end, R_cap, d, f, w_gate, w_up, w_down, H,
                      nullptr, Yp, yp_dtype, phases, false, nullptr, 0, stream);
}

extern "C" int32_t feplb_grouped_ffn_train(const void* Xp, const int32_t* row_src, int32_t T, int32_t k,
                                           const int32_t* offsets, int32_t g_begin,
                                           int32_t g_end, int32_t R_cap, int32_t d, int32_t f,
                                           const void* const* w_gate, const void* const* w_up,
                                           const void* const* w_down, void* H, void* AB, void* Yp,
                                           int32_t yp_dtype, int32_t phases, void* ws, size_t ws_bytes,
                                           void* stream) {
  FEPLB_REQUIRE(AB || !(phases & FEPLB_FFN_GATE_UP), FEPLB_EINVAL, "grouped_ffn_train: null AB");
  return forward_impl(Xp, row_src, T, k, offsets, g_begin, g_end, R_cap, d, f, w_gate, w_up, w_down, H,
                      AB, Yp, yp_dtype, phases, true, ws, ws_bytes, stream);
}

extern "C" size_t feplb_grouped_ffn_backward_wt_bytes(int32_t n_groups, int32_t d, int32_t f) {
  if (n_groups < 0 || d < 0 || f < 0) return 0;
  return (size_t)n_groups * 3 * (size_t)d * (size_t)f * 2;
}

extern "C" int32_t feplb_grouped_ffn_backward(const void* Xp, const int32_t* offsets, int32_t g_begin,
                                              int32_t g_end, int32_t R_cap, int32_t d, int32_t f,
                                              const void* const* w_gate, const void* const* w_up,
                                              const void* const* w_down, const void* H, void* AB,
                                              const void* dYp, void* dXp, int32_t dxp_dtype,
                                              void* const* dw_gate, void* const* dw_up,
                                              void* const* dw_down, void* WT, size_t wt_bytes,
                                              int32_t phases, void* ws, size_t ws_bytes, void* stream) {
  FEPLB_REQUIRE(g_begin >= 0 && g_end >= g_begin && R_cap >= 0 && d >= 0 && f >= 0, FEPLB_EINVAL,
                "grouped_ffn_backward: negative size or empty range reversed");
  FEPLB_REQUIRE(g_end <= FEPLB_MAX_GROUPS, FEPLB_ESHAPE, "grouped_ffn_backward: g_end=%d above %d", g_end,
                FEPLB_MAX_GROUPS);
  FEPLB_REQUIRE((phases & ~(FEPLB_BWD_ALL | FEPLB_BWD_ACCUMULATE | FEPLB_BWD_DIRECT)) == 0 && (phases & FEPLB_BWD_ALL) != 0,
                FEPLB_EINVAL, "grouped_ffn_backward: phases=%d", phases);
  FEPLB_REQUIRE(!(phases & FEPLB_BWD_DIRECT) || (phases & FEPLB_BWD_DGRAD), FEPLB_EINVAL,
                "grouped_ffn_backward: DIRECT without DGRAD (phases=%d)", phases);
  FEPLB_REQUIRE(dxp_dtype == FEPLB_F32 || dxp_dtype == FEPLB_BF16, FEPLB_EINVAL,
                "grouped_ffn_backward: unknown dxp_dtype %d", dxp_dtype);
  FEPLB_REQUIRE(d % 256 == 0 && f % 256 == 0 && d > 0 && f > 0, FEPLB_ESHAPE,
                "grouped_ffn_backward: need d %% 256 == 0 and f %% 256 == 0 (d=%d f=%d)", d, f);
  const int ng = g_end - g_begin;
  if (ng == 0) return FEPLB_OK;
  const bool do_t = phases & FEPLB_BWD_TRANSPOSE, do_d = phases & FEPLB_BWD_DGRAD, do_w = phases & FEPLB_BWD_WGRAD;
  const bool must_direct = phases & FEPLB_BWD_DIRECT;
  FEPLB_REQUIRE(!do_w || R_cap >= 32, FEPLB_ESHAPE, "grouped_ffn_backward: WGRAD needs R_cap >= 32 (R_cap=%d)", R_cap);
  FEPLB_REQUIRE(offsets, FEPLB_EINVAL, "grouped_ffn_backward: null offsets");
  // offsets inside the smallest tile travel as 32-bit byte offsets
  FEPLB_REQUIRE((uint64_t)(2 * (size_t)f + d) * 64 * 2 <= 0xffffffffull, FEPLB_ESHAPE, "grouped_ffn_backward: d, f too large");
  if (do_t || must_direct) {
    FEPLB_REQUIRE(w_gate && w_up && w_down, FEPLB_EINVAL, "grouped_ffn_backward: null weight tables");
    for (int g = g_begin; g < g_end; ++g) {
      FEPLB_REQUIRE(w_gate[g] && w_up[g] && w_down[g], FEPLB_EINVAL, "grouped_ffn_backward: null weights of group %d", g);
      FEPLB_REQUIRE(feplb::aligned16(w_gate[g]) && feplb::aligned16(w_up[g]) && feplb::aligned16(w_down[g]),
                    FEPLB_EALIGN, "grouped_ffn_backward: weights of group %d not 16-byte aligned", g);
    }
  }
  if (do_t || (do_d && !must_direct)) {
    const size_t need_wt = feplb_grouped_ffn_backward_wt_bytes(ng, d, f);
    FEPLB_REQUIRE(WT && wt_bytes >= need_wt, FEPLB_EWORKSPACE, "grouped_ffn_backward: WT %zu < %zu", wt_bytes, need_wt);
    FEPLB_REQUIRE(feplb::aligned16(WT), FEPLB_EALIGN, "grouped_ffn_backward: WT not 16-byte aligned");
  }
  // The input gradients read the weights themselves.  Only where they are not given (a call without TRANSPOSE may leave
  // them out, or misaligned) are the transposes read that an earlier call has left in WT: every call that asks for them
  // writes them, since it cannot know whether a later one will rely on them.
  bool direct = do_d && w_gate && w_up && w_down;
  for (int g = g_begin; direct && g < g_end; ++g)
    direct = w_gate[g] && w_up[g] && w_down[g] && feplb::aligned16(w_gate[g]) && feplb::aligned16(w_up[g]) &&
             feplb::aligned16(w_down[g]);
  if (do_d) {
    FEPLB_REQUIRE(AB && dYp && dXp, FEPLB_EINVAL, "grouped_ffn_backward: null AB/dYp/dXp");
    FEPLB_REQUIRE(feplb::aligned16(AB) && feplb::aligned16(dYp) && feplb::aligned16(dXp), FEPLB_EALIGN,
                  "grouped_ffn_backward: AB/dYp/dXp not 16-byte aligned");
  }
  if (do_w) {
    FEPLB_REQUIRE(Xp && H && AB && dYp && dw_gate && dw_up && dw_down, FEPLB_EINVAL,
                  "grouped_ffn_backward: null Xp/H/AB/dYp or gradient tables");
    FEPLB_REQUIRE(feplb::aligned16(Xp) && feplb::aligned16(H) && feplb::aligned16(AB) && feplb::aligned16(dYp),
                  FEPLB_EALIGN, "grouped_ffn_backward: Xp/H/AB/dYp not 16-byte aligned");
    for (int g = g_begin; g < g_end; ++g) {
      FEPLB_REQUIRE(dw_gate[g] && dw_up[g] && dw_down[g], FEPLB_EINVAL, "grouped_ffn_backward: null gradient of group %d", g);
      FEPLB_REQUIRE(feplb::aligned16(dw_gate[g]) && feplb::aligned16(dw_up[g]) && feplb::aligned16(dw_down[g]),
                    FEPLB_EALIGN, "grouped_ffn_backward: gradient of group %d not 16-byte aligned", g);
    }
  }
  {
    const size_t need = table_bytes(R_cap, ng) + FEPLB_MAX_GROUPS * sizeof(int);
    FEPLB_REQUIRE(ws && ws_bytes >= need, FEPLB_EWORKSPACE, "grouped_ffn_backward: workspace %zu < %zu", ws_bytes, need);
    FEPLB_REQUIRE(feplb::aligned16(ws), FEPLB_EALIGN, "grouped_ffn_backward: workspace not 16-byte aligned");
  }
  hipStream_t s = (hipStream_t)stream;
  const size_t df = (size_t)d * f;
  if (do_t) {
    // per group: Wd^T [d,f], then Wg^T [f,d] and Wu^T [f,d], the last two forming [2f,d]
    uint16_t* wt0 = (uint16_t*)WT;
    FEPLB_HIP(feplb::launch_transpose(w_down, g_begin, ng, f, d, wt0, 3 * df, s));
    FEPLB_HIP(feplb::launch_transpose(w_gate, g_begin, ng, d, f, wt0 + df, 3 * df, s));
    FEPLB_HIP(feplb::launch_transpose(w_up, g_begin, ng, d, f, wt0 + 2 * df, 3 * df, s));
  }
  WeightTable down_tab{}, gu_tab{};
  for (int g = g_begin; g < g_end; ++g) {
    const uint16_t* base = (const uint16_t*)WT + (size_t)(g - g_begin) * 3 * df;
    down_tab.w0[g] = direct ? w_down[g] : base;
    gu_tab.w0[g] = direct ? w_gate[g] : base + df;
    gu_tab.w1[g] = direct ? w_up[g] : nullptr;
  }
  if (do_w && R_cap > 0)   // dW_down = H^T dYp: before DGRAD, which does not touch H or dYp
    FEPLB_HIP(feplb::launch_wgrad(H, f, f, dYp, d, d, offsets, g_begin, ng, R_cap, dw_down, nullptr, d, d, phases & FEPLB_BWD_ACCUMULATE, s));
  if (do_d && R_cap > 0) {   // dH = dYp Wd^T, turned into [da | db] in place over the saved [p | q]
    const feplb::GroupedGemm a{dYp, d, nullptr, 0, 1, offsets, g_begin, ng, R_cap, d, f, &down_tab, direct ? d : f, direct, d,
                               nullptr, 0, AB, 2 * f};
    FEPLB_HIP(feplb::launch_dswiglu(a, s));
  }
  if (do_w && R_cap > 0)   // [dW_gate | dW_up] = Xp^T [da | db]
    FEPLB_HIP(feplb::launch_wgrad(Xp, d, d, AB, 2 * f, 2 * f, offsets, g_begin, ng, R_cap, dw_gate, dw_up, f, f, phases & FEPLB_BWD_ACCUMULATE, s));
  if (do_d && R_cap > 0) {   // dXp = [da | db] [Wg | Wu]^T
    const feplb::GroupedGemm a{AB, 2 * f, nullptr, 0, 1, offsets, g_begin, ng, R_cap, 2 * f, d, &gu_tab, direct ? f : d, direct,
                               direct ? f : 2 * f, dXp, d, nullptr, 0};
    FEPLB_HIP(feplb::launch_plain_gemm(a, dxp_dtype == FEPLB_BF16, s));
  }
  return FEPLB_OK;
}

namespace {
// the sizes of the call that launches this GEMM; false for one of the weight gradients'
bool sizes_of(int32_t gemm, int32_t R_cap, int32_t n_groups, int32_t d, int32_t f, feplb::GroupedGemm& a) {
  a.R_cap = R_cap;
  a.ng = n_groups;
  switch (gemm) {
    case FEPLB_GEMM_GATE_UP: a.K = a.lda = d; a.N = a.ldw = f; return true;
    case FEPLB_GEMM_DOWN: a.K = a.lda = f; a.N = a.ldw = d; return true;
    case FEPLB_GEMM_DH: a.K = a.lda = a.ldw = d; a.N = f; a.w_nk = true; return true;
    case FEPLB_GEMM_DXP: a.K = a.lda = 2 * f; a.N = d; a.ldw = f; a.w_nk = true; return true;
    default: return false;
  }
}
}  // namespace

extern "C" int32_t feplb_grouped_ffn_tile_rows(int32_t gemm, int32_t R_cap, int32_t n_groups, int32_t d, int32_t f) {
  if (R_cap < 0 || n_groups < 1 || n_groups > FEPLB_MAX_GROUPS || d < 256 || f < 128) return 0;
  feplb::GroupedGemm a{};
  if (sizes_of(gemm, R_cap, n_groups, d, f, a)) return feplb::gemm_tile_rows(a, gemm == FEPLB_GEMM_GATE_UP);
  switch (gemm) {
    case FEPLB_GEMM_DW_DOWN: return feplb::wgrad_tile_rows(R_cap, n_groups, f, d);
    case FEPLB_GEMM_DW_GATE_UP: return feplb::wgrad_tile_rows(R_cap, n_groups, d, 2 * f);
    default: return 0;
  }
}

extern "C" int32_t feplb_grouped_ffn_tall_rows(int32_t gemm, int32_t out, int32_t R_cap, int32_t n_groups, int32_t d, int32_t f,
                                               const int32_t* offsets) {
  if (R_cap < 0 || n_groups < 1 || n_groups > FEPLB_MAX_GROUPS || d < 256 || f < 128 || !offsets) return 0;
  feplb::GroupedGemm a{};
  if (gemm == FEPLB_GEMM_DH || !sizes_of(gemm, R_cap, n_groups, d, f, a)) return 0;
  return feplb::gemm_tall_rows(a, gemm == FEPLB_GEMM_GATE_UP, out != 0, out == FEPLB_BF16, offsets);
}
