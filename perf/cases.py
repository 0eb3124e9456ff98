"""Performance cases of the MoE layer: what one expert-parallel rank computes for a batch of tokens.

Three kinds of pass, all through the package's public entry points:

  forward     one layer step of a share without replicas (`runner.step`): router, permutation,
              grouped SwiGLU FFN, combine.  With `graph` the step recorded by
              `RankLayer.capture_forward` is replayed, as small calls are served.
  rebalanced  one layer step that plans on the host from the router's counts, stages the replicas'
              weights and runs static and dynamic experts (`runner.step`).
  train       a training step of the layer: router, permutation with its row copy, training forward,
              combine, then the whole backward down to dX, the router's gradient and the fp32 weight
              gradients; with `micro` = 2 over two micro-batches, the second accumulating.

A case is: tokens T, model width d, expert width f, experts E, choices per token k, expert-parallel
ranks P (this rank holds E / P experts), popularity of the experts, the storage type of the expert
outputs (forward: `yp`) or of the row gradients (train: `dxp`), and `cap`: whether the layer's
buffers hold exactly this batch's rows ("exact") or any batch's (T * k rows, "all").
"""
import math

import numpy as np
import torch

import workloads
from paper_2604_19654_amd import binding as B
from paper_2604_19654_amd import runner
from paper_2604_19654_amd.training import FfnTrainingStep

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, kind, T, d, f, E, k, P, pop, pop_seed, **options):
    c = dict(name=name, kind=kind, T=T, d=d, f=f, E=E, k=k, P=P, pop=pop, pop_seed=pop_seed)
    c.update(options)
    return c


def listed():
    forward = dict(yp="f32", cap="exact", graph=False)
    train = dict(dxp="f32", micro=1)
    return [
        # the repository's smallest workload (C1): a step as long as its launches
        _case("forward_tiny", "forward", 512, 256, 512, 8, 2, 1, "uniform", 1001, **forward),
        # a decode-sized batch at full model width, replayed as a graph with buffers for any batch:
        # a few rows per expert, so the weights' bytes are the work
        _case("forward_decode_graph", "forward", 96, 4096, 1536, 128, 8, 8, "uniform", 1002, yp="f32", cap="all", graph=True),
        # an odd-sized small micro-batch with bf16 expert outputs and buffers for any batch
        _case("forward_small_bf16", "forward", 1003, 2048, 1408, 64, 6, 4, "dirichlet", 21, yp="bf16", cap="all", graph=False),
        # balanced share of eight ranks (C2): every expert has about 512 rows
        _case("forward_balanced", "forward", 8192, 4096, 1536, 128, 8, 8, "uniform", 1002, **forward),
        # the straggler's skewed share (C3): two experts see almost every token, half see none
        _case("forward_skewed", "forward", 8192, 4096, 1536, 128, 8, 8, "zipf", 1003, **forward),
        # large share of four ranks (C5)
        _case("forward_large", "forward", 32768, 7168, 2048, 128, 8, 4, "dirichlet", 1005, **forward),
        # a short micro-batch of the rebalanced share, tokens not a round number
        _case("rebalanced_short", "rebalanced", 8 * 777, 6144, 2048, 128, 8, 8, "zipf", 1004, yp="f32", cap="exact"),
        # the rebalanced share at full size (C4), the default benchmark
        _case("rebalanced_full", "rebalanced", 8 * 16384, 6144, 2048, 128, 8, 8, "zipf", 1004, yp="f32", cap="exact"),
        # training step of the smallest workload
        _case("train_tiny", "train", 512, 256, 512, 8, 2, 1, "uniform", 1001, **train),
        # training step with gradient accumulation over two odd-sized micro-batches, bf16 row gradients
        _case("train_ragged_micro", "train", 2501, 2560, 768, 64, 4, 4, "zipf", 23, dxp="bf16", micro=2),
        # training step of the balanced share
        _case("train_balanced", "train", 8192, 4096, 1536, 128, 8, 8, "uniform", 1002, **train),
        # training step of the large share: the most work of all
        _case("train_large", "train", 32768, 7168, 2048, 128, 8, 4, "dirichlet", 1005, **train),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    most_flops = max(work(c)["flops"] for c in listed())
    most_bytes = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(["forward", "forward", "forward", "rebalanced", "train", "train", "train"])
        step_f = 256 if kind == "train" else 128
        d = 256 * max(1, round(_log_uniform(rng, 1, 28)))
        f = step_f * max(1, round(_log_uniform(rng, 256, 2048) / step_f))
        E, P = rng.choice([(8, 1), (16, 2), (32, 2), (64, 4), (64, 8), (96, 8), (128, 4), (128, 8), (128, 16), (256, 8)])
        k = rng.randint(1, min(8, E // P))
        c = dict(kind=kind, d=d, f=f, E=E, k=k, P=P, pop_seed=rng.randrange(1 << 20))
        if kind == "forward":
            T = int(_log_uniform(rng, 32, 65536))
            c.update(T=T, pop=rng.choice(["uniform", "zipf", "dirichlet"]), yp=rng.choice(["f32", "f32", "bf16"]),
                     cap=rng.choice(["exact", "all"]) if T * k * d * 4 < (4 << 30) else "exact",
                     graph=T <= 4096 and rng.random() < 0.5)
        elif kind == "rebalanced":
            if E // P < 8 or P < 2:
                continue
            c.update(T=P * int(_log_uniform(rng, 256, 16384)), pop="zipf", yp=rng.choice(["f32", "bf16"]), cap="exact")
        else:
            c.update(T=int(_log_uniform(rng, 256, 32768)), pop=rng.choice(["uniform", "zipf", "dirichlet"]),
                     dxp=rng.choice(["f32", "f32", "bf16"]), micro=rng.choice([1, 1, 2]))
        w = work(c)
        # the buffers of a state, three of which have to fit the card
        rows = min(c["T"] * k, int(1.3 * _share(c)[0]) + 1)
        state = (E // P + 4) * d * f * 3 * (12 if kind == "train" else 2) + c["T"] * d * 8 * c.get("micro", 1) + rows * (d * 14 + f * 8)
        if w["flops"] <= most_flops and w["bytes"] <= most_bytes and state < (40 << 30):
            return c


def _override(case, seed):
    c = dict(T=case["T"], d=case["d"], f=case["f"], E=case["E"], k=case["k"], P=case["P"], pop=case["pop"],
             pop_seed=case["pop_seed"], seed=seed, n_dyn=0, rank=0)
    if case["kind"] == "rebalanced":
        c.update(n_dyn=4, rank=-1)
    return c


def prepare(case, seed):
    if case["kind"] != "train":
        cap = case["T"] * case["k"] if case["cap"] == "all" else None
        p = runner.prepare("C1", device=DEV, yp_dtype=DTYPES[case["yp"]], r_cap=cap, **_override(case, seed))
        p.wl.drop_weights()
        replay = None
        if case.get("graph"):
            runner.step(p)
            replay = p.layer.capture_forward(p.wl.logits, p.wl.X, p.groups, p.weights)
        return dict(case=case, p=p, replay=replay)
    return _prepare_train(case, seed)


def _prepare_train(case, seed):
    T, d, E, k, P = case["T"], case["d"], case["E"], case["k"], case["P"]
    i32 = dict(dtype=torch.int32, device=DEV)
    bf16 = dict(dtype=torch.bfloat16, device=DEV)
    batches, weights, rows = [], None, 1
    for m in range(case["micro"]):
        wl = workloads.make("C1", device=DEV, **_override(case, seed + m))
        experts = [int(e) for e in wl.local_experts()]
        if weights is None:
            mats = [wl.expert_weights(e) for e in experts]
            weights = tuple([w[i] for w in mats] for i in range(3))
            groups = [(e, 0, B.ORD_MAX) for e in experts]
        wl.drop_weights()
        _, _, counts = B.feplb_route_topk(wl.logits, k)
        rows = max(rows, int(counts[experts].sum().item()))
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed + m + 77)
        dY = torch.empty((T, d), dtype=torch.float32, device=DEV).normal_(generator=gen).to(torch.bfloat16)
        batches.append((wl.logits, wl.X, dY))
    step = FfnTrainingStep(rows, len(groups), d, case["f"], device=DEV, dxp_dtype=DTYPES[case["dxp"]])
    R_cap = step.R_cap
    # the weight gradients of all experts lie in one tensor per matrix, as an optimiser keeps them
    grads = []
    for name in ("dW_gate", "dW_up", "dW_down"):
        shape = getattr(step, name)[0].shape
        setattr(step, name, None)
        whole = torch.empty((len(groups),) + tuple(shape), dtype=torch.float32, device=DEV)
        setattr(step, name, list(whole.unbind(0)))
        grads.append(whole)
    bufs = dict(
        ids=torch.empty((T, k), **i32), w=torch.empty((T, k), dtype=torch.float32, device=DEV), counts=torch.empty((E,), **i32),
        offsets=torch.zeros((len(groups) + 1,), **i32), row_src=torch.empty((R_cap,), **i32), inv=torch.empty((T * k,), **i32),
        ws=torch.empty((B.feplb_permute_workspace_bytes(T, k, E, len(groups)),), dtype=torch.uint8, device=DEV),
        Xp=torch.zeros((R_cap, d), **bf16), dYp=torch.zeros((R_cap, d), **bf16), Y=torch.empty((T, d), **bf16), dX=torch.empty((T, d), **bf16),
        dw=torch.empty((T, k), dtype=torch.float32, device=DEV), ones=torch.ones((T, k), dtype=torch.float32, device=DEV),
        dlogits=torch.empty((T, E), dtype=torch.float32, device=DEV))
    return dict(case=case, batches=batches, weights=weights, groups=groups, step=step, grads=grads, bufs=bufs)


def run(state):
    case = state["case"]
    if case["kind"] != "train":
        p, b = state["p"], state["p"].layer.buf
        if state["replay"] is not None:
            state["replay"].replay()
            Y = b.Y
        else:
            Y = runner.step(p)
        return dict(Y=Y, topk_ids=b.topk_ids, topk_w=b.topk_w, counts=b.counts)
    T, d, E, k = case["T"], case["d"], case["E"], case["k"]
    b, st = state["bufs"], state["step"]
    wg, wu, wd = state["weights"]
    for m, (logits, X, dY) in enumerate(state["batches"]):
        B.feplb_route_topk(logits, k, b["ids"], b["w"], b["counts"])
        B.feplb_permute(b["ids"], E, state["groups"], X, st.R_cap, b["Xp"], b["offsets"], b["row_src"], b["inv"], b["ws"])
        st.forward(b["Xp"], b["offsets"], wg, wu, wd)
        B.feplb_unpermute_combine(st.Yp, b["inv"], b["w"], T, k, d, b["Y"])
        B.feplb_combine_backward(dY, st.Yp, b["inv"], b["w"], T, k, d, b["dYp"], b["dw"])
        st.backward(b["Xp"], b["offsets"], wg, wu, wd, b["dYp"], phases=B.BWD_ALL | (B.BWD_ACCUMULATE if m else 0))
        B.feplb_unpermute_combine(st.dXp, b["inv"], b["ones"], T, k, d, b["dX"])
        B.feplb_route_topk_backward(b["ids"], b["w"], b["dw"], E, b["dlogits"])
    return dict(Y=b["Y"], dX=b["dX"], dlogits=b["dlogits"], counts=b["counts"],
                dW_gate=state["grads"][0], dW_up=state["grads"][1], dW_down=state["grads"][2])


def _share(case):
    """Expected rows of this rank's share and how many of its experts see any, from the case alone:
    the choices of a few thousand tokens drawn on the CPU."""
    n = 2048
    wl = workloads.make("C1", device="cpu", T=n, d=8, f=8, E=case["E"], k=case["k"], P=case["P"], pop=case["pop"],
                        pop_seed=case["pop_seed"], seed=1, n_dyn=0, rank=-1 if case["kind"] == "rebalanced" else 0)
    picks = torch.bincount(torch.topk(wl.logits, case["k"], dim=1).indices.reshape(-1), minlength=case["E"]).numpy()
    picks = picks.astype(np.float64) * (case["T"] / n)
    per = case["E"] // case["P"]
    loads = picks.reshape(case["P"], per)
    if case["kind"] == "rebalanced":
        mean = picks.sum() / case["P"]
        r = int(np.argmin(np.abs(2 * loads.sum(axis=1) - mean)))
        return max(mean, loads[r].sum()), int((loads[r] >= 0.5).sum()) + 4
    return loads[0].sum(), max(1, int((loads[0] >= 0.5).sum()))


def work(case):
    T, d, f, E, k = (case[x] for x in ("T", "d", "f", "E", "k"))
    rows, experts = _share(case)
    local = E // case["P"]
    weights = experts * 3 * d * f * 2
    tokens = min(T, rows)                     # rows of X that any local expert needs
    forward = T * E * 4 + T * k * 8 + tokens * d * 2 + weights + T * d * 2
    if case["kind"] != "train":
        staged = 2 * 4 * 3 * d * f * 2 if case["kind"] == "rebalanced" else 0
        return {"bytes": float(forward + staged), "flops": float(6.0 * d * f * rows)}
    # backward: dY and X in, dX and dlogits out, the weights once more, the fp32 gradients of every local
    # expert; the activations H and the two derivatives of each row are kept from the forward pass
    kept = rows * 3 * f * 2
    backward = 2 * T * d * 2 + T * E * 4 + weights + local * 3 * d * f * 4 + kept
    m = case["micro"]
    # another micro-batch reads and writes the gradients of the experts it reaches
    more = (m - 1) * experts * 3 * d * f * 4
    return {"bytes": float(m * (forward + kept + backward) + more), "flops": float(m * 18.0 * d * f * rows)}


def tolerance(case):
    # The path rounds H, the derivatives p and q, da and db, dYp and its outputs Y and dX to bf16 (2^-9
    # relative at most), everything else is fp32.  Sums in another order move a value across a rounding
    # boundary now and then: against the same path written with torch products in fp32 and in fp64, at the
    # same storage types, the outputs differ by 1e-5 .. 3.1e-4 in the 2-norm and by up to two bf16 steps
    # (1.6e-2) in single values; four times that is stated.  Ids and counts are whole numbers: equal.
    return {"rel": 1.2e-3, "max": 0.06}
