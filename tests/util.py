"""Helpers shared by the tests: tensor -> float64 arrays, the float tolerance."""
import os
import re

import numpy as np
import torch


def f64(t: torch.Tensor) -> np.ndarray:
    """Exact widening of a (bf16 / fp32) tensor to a float64 NumPy array on the host."""
    return t.detach().to("cpu").to(torch.float64).numpy()


def i64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to("cpu").numpy()


# Float bar of the build: max-abs-err <= 2e-2 relative to output RMS for bf16 with
# fp32 accumulation, read per token row against the unrounded float64 oracle
# (a row's scale is set by its combine weights, so one global RMS would put the
# bound below the bf16 rounding step of the largest rows).
ROW_TOL = 2e-2


# Float bars for the backward pass, which the benchmark spec does not state.  The library stores
# the derivatives p = dH/da, q = dH/db of the SwiGLU product, the activations H and the gradients
# da = dH p, db = dH q in bf16 (da, db and H are MFMA operands), and the float64 oracle stores
# nothing rounded.  One bf16 rounding perturbs a value by a relative 2^-9 at most, about 1e-3 in
# the root mean square; every gradient term carries two of them (the stored derivative and the
# stored product, or H alone for dW_down), so the error of an output row, taken in the root mean
# square over the row, is about sqrt(2) * 1e-3 .. 3e-3 of the row's RMS whatever the number of
# rows summed (error and value grow alike).  A float64 computation that only rounds those five
# tensors measures 0.0027 .. 0.004 on every shape tried, from one-row groups to thousands of
# rows.  BWD_RMS_TOL is 1e-2.
# The largest single error of a row is heavy-tailed instead: da is a product of three random
# factors, and a one-row group has no sum to average over, so that same computation reaches
# 0.01 .. 0.035 of the row RMS.  BWD_MAX_TOL = 8e-2 (four times the forward bar) only guards
# against isolated wrong elements; the RMS bar is the one that carries the parity claim.
BWD_RMS_TOL = 1e-2
BWD_MAX_TOL = 8e-2


def row_rms_err(got: np.ndarray, want: np.ndarray) -> np.ndarray:
    """rms_i(got - want) / rms_i(want) per row; all-zero oracle rows must match exactly."""
    err = np.sqrt(((got - want) ** 2).mean(axis=1))
    rms = np.sqrt((want ** 2).mean(axis=1))
    out = np.zeros_like(err)
    nz = rms > 0
    out[nz] = err[nz] / rms[nz]
    out[~nz] = np.where(err[~nz] == 0, 0.0, np.inf)
    return out


def row_rel_err(got: np.ndarray, want: np.ndarray) -> np.ndarray:
    """max_i |got - want| / rms_i(want) per row; rows whose oracle value is all
    zero must match exactly (reported as 0 or inf)."""
    err = np.abs(got - want).max(axis=1)
    rms = np.sqrt((want ** 2).mean(axis=1))
    out = np.zeros_like(err)
    nz = rms > 0
    out[nz] = err[nz] / rms[nz]
    out[~nz] = np.where(err[~nz] == 0, 0.0, np.inf)
    return out


def bf16_rounding_excess(got: np.ndarray, want: np.ndarray) -> float:
    """For an INTERMEDIATE kept in bf16 (the SwiGLU activations H): every element
    must sit within one bf16 rounding step of the oracle value, plus a small
    allowance (1e-3 of the row RMS) for fp32 accumulation order and the fast
    exponential.  H rows are heavy-tailed (a product of two near-Gaussians), so
    their largest element's rounding step alone can exceed 2e-2 of the row RMS;
    the 2e-2 bar applies to the layer's outputs, not to this intermediate.
    Returns max over elements of |err| / allowed (<= 1 passes)."""
    rms = np.sqrt((want ** 2).mean(axis=1, keepdims=True))
    allowed = 2.0 ** -8 * np.abs(want) + 1e-3 * rms + 1e-30
    return float((np.abs(got - want) / allowed).max())


# ---------------------------------------------------------------------------------------------
# What the storage formats of the path cost, element by element.
#
# The path keeps two tensors in bf16 on purpose: the SwiGLU activations H (they are the down
# GEMM's MFMA operand) and the layer's output Y.  Everything else is fp32 (accumulators, expert
# outputs Yp, the combine's sum).  Against the unrounded float64 oracle an element of Y therefore
# carries
#   (1) the output rounding: at most half a bf16 step of the value that is rounded,
#       hu(v) = 2^(floor(log2 |v|) - 8);
#   (2) the H roundings, pushed through the down projection and the combine:
#       e_i = sum_j w_j sum_f dH[j,f] Wd_j[f,i] with |dH[j,f]| <= hu(H[j,f]).  The roundings of
#       different elements are independent and, to the accuracy needed here, uniform in their
#       interval (variance hu^2 / 3), so e_i is a sum of thousands of independent bounded terms
#       with standard deviation sigma_i = sqrt( sum_j w_j^2 sum_f hu(H[j,f])^2 / 3 * Wd_j[f,i]^2 );
#   (3) fp32 accumulation and the hardware exponential / reciprocal: relative 1e-5 at most,
#       carried as 1e-5 |Y_i| and as a 2 % widening of sigma (H is rounded from an fp32 value
#       that is itself off by that much).
# Bound per element: hu(|Y_i| + n sigma_i) + n sigma_i + 1e-5 |Y_i| with n = 7 (a Gaussian tail
# of 3e-12 per element; the largest check looks at 4e8 elements).
# ---------------------------------------------------------------------------------------------
FORMAT_NSIGMA = 7.0


def bf16_half_ulp(v: np.ndarray) -> np.ndarray:
    """Half the spacing of bf16 numbers around |v| (8 significand bits): 2^(floor(log2|v|) - 8)."""
    a = np.maximum(np.abs(v), 2.0 ** -126)
    return np.exp2(np.floor(np.log2(a)) - 8.0)


def h_rounding_variance(orc, x_rows: np.ndarray, weights) -> tuple:
    """For rows x of one expert: the oracle's (H, Yp) and, per element of Yp, the variance of the
    error that rounding H to bf16 causes: (hu(H)^2 / 3) @ (Wd^2)."""
    h, y = orc.ffn_rows(x_rows, *weights)
    wd = np.asarray(weights[2], dtype=np.float64)
    return h, y, (bf16_half_ulp(h) ** 2 / 3.0) @ (wd * wd)


def format_bound(value: np.ndarray, variance: np.ndarray, output_bf16: bool) -> np.ndarray:
    """Element-wise bound described above for a result `value` whose H-rounding variance is given."""
    ns = FORMAT_NSIGMA * 1.02 * np.sqrt(variance)
    b = ns + 1e-5 * np.abs(value) + 1e-30
    if output_bf16:
        b = b + bf16_half_ulp(np.abs(value) + ns)
    return b


def layer_tokens_with_format_bound(orc, x_rows, ids_rows, w_rows, keep_rows, weights_of):
    """The layer's result for a batch of tokens, expert by expert like orc.moe_tokens, together
    with the element-wise format bound of Y.  Returns (Y [m,d], bound [m,d])."""
    x = np.asarray(x_rows, dtype=np.float64)
    ids_rows = np.asarray(ids_rows)
    keep_rows = np.asarray(keep_rows, dtype=bool)
    w_rows = np.asarray(w_rows, dtype=np.float64)
    out = np.zeros_like(x)
    var = np.zeros_like(x)
    for e in sorted(set(int(v) for v in ids_rows[keep_rows])):
        tok, slot = np.nonzero((ids_rows == e) & keep_rows)      # a token names an expert at most once
        _, y, v = h_rounding_variance(orc, x[tok], weights_of(e))
        wj = w_rows[tok, slot][:, None]
        out[tok] += wj * y
        var[tok] += wj * wj * v
    return out, format_bound(out, var, output_bf16=True)


def _ffn_gemm_constant(name):
    with open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_19654_amd", "csrc",
                           "ffn_gemm.hip")) as fh:
        return int(re.search(rf"{name} = (\d+);", fh.read()).group(1))


def how_256_row_tiles_run(sizes, columns):
    """What a grouped GEMM in 256 x 256 tiles makes of groups of these sizes and a weight of `columns` columns: "whole" tiles,
    "quarters" of 128 x 128, or "both" (whole rounds of 256 tiles, and so few left over that they run as quarters)."""
    most = _ffn_gemm_constant("QUARTERS_MAX")
    tiles = sum(-(-n // 256) for n in sizes) * (columns // 256)
    rest = tiles % 256
    return "whole" if rest == 0 or rest > most else "quarters" if rest == tiles else "both"


def how_tall_tiles_run(sizes, height, columns):
    """What a grouped GEMM in tall tiles of up to `height` rows makes of groups of these sizes: whole rounds of 256 tiles, and how the tiles left over
    run: "whole", as "halves" of their columns, as "quarters", or "none"."""
    tiles = 0
    for n in sizes:
        blocks = -(-n // 64)
        if blocks:
            split = -(-blocks // (height // 64))
            tiles += -(-blocks // -(-blocks // split))   # all of one height but the last
    rounds, rest = divmod(tiles * (columns // 256), 256)
    return rounds, ("none" if rest == 0 else "quarters" if rest <= _ffn_gemm_constant("QUARTERS_MAX") else
                    "halves" if rest <= _ffn_gemm_constant("HALVES_MAX") else "whole")


def _spread(n, sizes):
    return [sizes[i * 7919 // 13 % len(sizes)] for i in range(n)]


# d, f, row capacity and group sizes, at the edges of the tall tiles' blocks of 64 rows, at which the grouped GEMMs run in tall tiles: together every
# product in every height, with left-over tiles of every kind, in less than a round and in more, and with more groups than a wavefront has lanes.  A
# host test holds the list to that.
TALL_CASES = [
    (2048, 1536, 5500, [2]),
    (2048, 2048, 24000, [84, 128, 70, 606, 3, 4, 240]),
    (3072, 1536, 3000, [84, 128, 70, 606, 3, 4, 240]),
    (2048, 2048, 4000, [195, 3, 213, 257, 15, 314, 65, 490, 449]),
    (3072, 1536, 3000, [257, 37, 111, 56, 65, 261, 321, 641, 623, 124]),
    (2048, 2048, 4000, [257, 37, 111, 56, 65, 261, 321, 641, 623, 124]),
    (3072, 1536, 4000, [393, 66, 257, 128, 63, 128, 334, 31, 138, 450, 65, 646]),
    (3072, 1024, 6000, [355, 24, 449, 383, 321, 321, 384, 319, 43, 210, 63, 129, 380, 255, 128, 384, 577, 13, 177, 13, 348, 192]),
    (2048, 2048, 5500, _spread(128, [0, 1, 2, 17, 33, 63, 64, 65])),
    (3072, 1024, 9500, _spread(128, [0, 1, 2, 17, 33, 63, 64, 65])),
    (2048, 2048, 16000, _spread(100, [1, 2, 3, 15, 16, 17, 31, 33, 63, 64, 65, 66, 127, 128, 129, 191, 192, 193, 255, 256, 257, 319, 320, 321])),
]
