"""Performance cases of the MoE expert-layer path: what a training program asks of the library.

Each case is one kind of call sequence ("do") at one size:

  train     one training step of the layer over a batch: per micro-batch the permutation, the expert
            FFN forward, the combine, the backward of all of it; then the weight gradients.  The
            routing is replayed, so the batch's plan is known beforehand and its tables are resident.
            form "gated":      row gather and combine backward folded into the GEMMs, weight gradients
                               once per batch, forward on transposed weight copies (made in the step:
                               the parameters change with every optimizer step);
            form "plain":      the same with the combine's backward as a pass of its own;
            form "accumulate": gathered rows in memory, weight gradients added up in memory after
                               every micro-batch, replica gradients returned to their home experts.
  forward   forward pass only (log-probabilities, evaluation) of one micro-batch, weights as stored.
  plan      control plane of a batch: histograms, their way to the host, plan, tables to the device.
  hist      load histograms of the replayed routing of many layers in one call.
  dispatch  token movement alone: permutation with row gather, gated combine, combine backward.
  replica   the layer-shared replica buffer: parameter push and gradient pull with the default grid.

Routing is drawn as a Zipf-biased router's: normal logits plus log weights over a random order of
the experts, top-k, gates softmaxed over the selected ones.  Activations and upstream gradients are
N(0,1), weights N(0, 0.02), all rounded to bf16 once.
"""
import math

import numpy as np
import torch

import paper_2605_08639_amd as rl

DEV = "cuda"
TABLES = ("inst_ptr", "inst_rows", "inst_group", "group_offset", "group_expert", "group_dw_slot")


def _layer(name, do, E, k, h, hff, T, n_mb, EP, r, zipf, **more):
    return dict(name=name, do=do, E=E, k=k, h=h, hff=hff, T=T, n_mb=n_mb, EP=EP, r=r, zipf=zipf, **more)


def listed():
    return [
        # the smallest useful layer: every launch and every host call counts
        _layer("train_tiny", "train", 8, 2, 128, 256, 512, 1, 4, 1, 1.2, form="gated"),
        # sizes that divide nothing, several micro-batches, gradients accumulated in memory
        _layer("train_ragged", "train", 16, 4, 256, 192, 777, 3, 4, 2, 1.2, form="accumulate"),
        # a short sequence through a layer of many small experts: a handful of rows per expert
        _layer("forward_short", "forward", 128, 8, 2048, 768, 256, 1, 8, 2, 1.0),
        # many experts of moderate size (Qwen3-30B-A3B-shaped): groups from a few rows to a few thousand
        _layer("train_many_experts", "train", 128, 8, 2048, 768, 8192, 4, 8, 2, 1.0, form="gated"),
        # the same layer with gradients accumulated per micro-batch, half-size micro-batches
        _layer("train_accumulate", "train", 128, 8, 2048, 768, 4096, 2, 8, 2, 1.0, form="accumulate"),
        # long micro-batches with extreme hot spots (Qwen3-235B-A22B-shaped): the largest work
        _layer("train_large", "train", 128, 8, 4096, 1536, 16384, 4, 16, 2, 1.5, form="gated"),
        # few, wide experts (Mixtral-8x7B-shaped)
        _layer("train_wide_experts", "train", 8, 2, 4096, 14336, 4096, 2, 8, 1, 1.5, form="plain"),
        # weights far larger than the rows (DeepSeek-V3-shaped): streaming 22 GB of parameters
        _layer("forward_deepseek", "forward", 256, 8, 7168, 2048, 4096, 1, 32, 2, 1.2),
        # the control plane of the largest batch
        _layer("plan_batch", "plan", 128, 8, 4096, 1536, 16384, 32, 16, 2, 1.5),
        # replayed routing of 64 layers x 16 micro-batches
        _layer("hist_layers", "hist", 128, 8, 2048, 768, 8192, 1024, 8, 2, 1.0),
        # rows moved to the experts and back
        _layer("dispatch_combine", "dispatch", 128, 8, 4096, 1536, 8192, 1, 16, 2, 1.2),
        # eight live replicas of a Qwen3-30B-A3B-shaped layer
        _layer("replica_buffer", "replica", 128, 8, 2048, 768, 8192, 1, 8, 2, 1.0, live=8),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(rng, lo, hi, of):
    return max(lo, min(hi, int(round(_log_uniform(rng, lo, hi) / of)) * of))


def _fits(c):
    """No drawn case is larger than the largest listed one, in memory or in time."""
    E, h, hff, N, n_mb, do = c["E"], c["h"], c["hff"], c["T"] * c["k"], c["n_mb"], c["do"]
    w = 6.0 * E * h * hff                                     # bf16 weights
    if do == "train":
        held = 2 * w + 2 * w * (1 + c["EP"] * c["r"] / E) + n_mb * N * (6.0 * hff + 8.0 * h) + N * (4.0 * hff + 4.0 * h)
        ms = 18e3 * h * hff * N * n_mb / 6e14 + (n_mb * 3 + 6) * w / 3.5e9
        return held < 30e9 and ms < 60
    if do == "forward":
        return w + N * (6.0 * hff + 4.0 * h) < 26e9 and 6e3 * h * hff * N / 6e14 + w / 3.5e9 < 20
    if do == "dispatch":
        return 6.0 * N * h < 8e9
    if do == "replica":
        return 6.0 * w < 30e9
    return 4.0 * N * n_mb < 3e8 and c["n_mb"] * E <= 1 << 18


def draw(rng):
    while True:
        do = rng.choice(("train", "train", "train", "forward", "forward", "plan", "hist", "dispatch", "replica"))
        E = rng.choice((8, 16, 32, 64, 128, 256))
        EP = rng.choice([p for p in (1, 2, 4, 8, 16, 32) if p <= E])
        c = dict(do=do, E=E, k=rng.randint(1, min(8, E)), h=_multiple(rng, 128, 7168, 64), hff=_multiple(rng, 128, 14336 if E <= 16 else 2048, 64),
                 T=int(_log_uniform(rng, 32, 16384)), n_mb=1, EP=EP, r=rng.randint(0, 2), zipf=round(rng.uniform(0.8, 1.5), 2))
        if do == "train":
            c["n_mb"] = rng.randint(1, 4)
            # the combine's backward is a pass of its own where the experts are wide
            c["form"] = rng.choice(("plain" if c["hff"] >= 4096 else "gated", "accumulate"))
        elif do == "plan":
            c["n_mb"] = rng.randint(1, 32)
            c["r"] = max(c["r"], 1)
        elif do == "hist":
            c["n_mb"] = int(_log_uniform(rng, 1, 1024))
        elif do == "replica":
            c["r"] = max(c["r"], 1)
            c["live"] = rng.randint(1, c["EP"] * c["r"])
        if _fits(c):
            return c


# ---------------------------------------------------------------------------------------------
def _route(case, n_mb, gen):
    """ids [n_mb,T,k] int32 and gates [n_mb,T,k] fp32; the hot experts move from micro-batch to micro-batch."""
    E, k, T = case["E"], case["k"], case["T"]
    log_w = -case["zipf"] * torch.log(torch.arange(1, E + 1, device=DEV, dtype=torch.float32))
    ids = torch.empty((n_mb, T, k), dtype=torch.int32, device=DEV)
    gates = torch.empty((n_mb, T, k), dtype=torch.float32, device=DEV)
    for mb in range(n_mb):
        order = torch.randperm(E, generator=gen, device=DEV)
        bias = torch.empty(E, device=DEV)
        bias[order] = log_w
        top, at = torch.topk(torch.randn((T, E), generator=gen, device=DEV) + bias, k, dim=1)
        ids[mb] = at
        gates[mb] = torch.softmax(top, dim=1)
    return ids, gates


def _bf16(gen, shape, std=1.0):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=gen)


def _weights(case, gen, blocks):
    h, hff = case["h"], case["hff"]
    return [_bf16(gen, (blocks, hff, h), 0.02), _bf16(gen, (blocks, hff, h), 0.02), _bf16(gen, (blocks, h, hff), 0.02)]


def _ranks_per_node(case):
    return min(case["EP"], 8)


def _tables(plan):
    return {key: torch.from_numpy(plan[key]).to(DEV, non_blocking=True) for key in TABLES}


class State:
    """Everything a program keeps between steps: inputs, weights, plan tables, buffers, workspaces."""

    def __init__(self, case, seed):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed)
        self.case, do = case, case["do"]
        E, k, h, hff, T, n_mb, EP, r = (case[x] for x in ("E", "k", "h", "hff", "T", "n_mb", "EP", "r"))
        N, G = T * k, EP * (E // EP + r)
        self.N, self.G = N, G
        self.err = rl.new_err_flag(DEV)
        bf = lambda *s: torch.empty(s, dtype=torch.bfloat16, device=DEV)
        i32 = lambda *s: torch.empty(s, dtype=torch.int32, device=DEV)
        f32 = lambda *s: torch.empty(s, dtype=torch.float32, device=DEV)
        ws = lambda which: torch.empty(max(rl.workspace_bytes(which, T, k, E, G, h, hff), 1), dtype=torch.uint8, device=DEV)
        if do == "replica":
            slots = EP * r
            self.W = _weights(case, gen, E + slots)
            self.dW = [f32(*w.shape).normal_(generator=gen) for w in self.W]
            table = torch.full((slots,), -1, dtype=torch.int32, device=DEV)
            live = torch.randperm(slots, generator=gen, device=DEV)[:case["live"]]
            table[live] = torch.randint(0, E, (case["live"],), generator=gen, device=DEV, dtype=torch.int32)
            self.replica_expert = table
            return
        if do == "hist":                                     # the routing of a few micro-batches stands for all of them
            few = min(n_mb, 8)
            ids, _ = _route(case, few, gen)
            self.ids = ids.repeat((n_mb + few - 1) // few, 1, 1)[:n_mb].contiguous()
            self.counts = i32(n_mb, E)
            return
        self.ids, self.gates = _route(case, n_mb, gen)
        self.counts = i32(n_mb, E)
        if do == "plan":
            return
        rl.relibra_route_hist(self.ids, E, counts=self.counts, err_flag=self.err)
        self.tabs = _tables(rl.relibra_plan(self.counts.cpu().numpy(), k, EP, _ranks_per_node(case), r))
        self.X = [_bf16(gen, (T, h)) for _ in range(n_mb)]
        self.Out = bf(n_mb, T, h)
        self.row_of, self.src_of, self.ws_perm = i32(N), i32(N), ws(rl.WS_PERMUTE)
        if do == "dispatch":
            self.dOut = _bf16(gen, (T, h))
            self.Y = _bf16(gen, (N, h))
            self.Xrows, self.dY, self.dgate = bf(N, h), bf(N, h), f32(T, k)
            return
        self.W = _weights(case, gen, E)
        self.Gt, self.U, self.Yrows = bf(N, hff), bf(N, hff), bf(N, h)
        if do == "forward":
            self.A, self.row_tok, self.ws = bf(N, hff), i32(N), ws(rl.WS_FFN_FWD)
            return
        form = case["form"]
        keep = 1 if form == "accumulate" else n_mb           # batched weight gradients keep every micro-batch's rows
        self.dOut = [_bf16(gen, (T, h)) for _ in range(n_mb)]
        self.A = [bf(N, hff) for _ in range(keep)]
        self.ws = [ws(rl.WS_FFN_BWD) for _ in range(keep)]
        self.dXrows, self.dX, self.dgate = bf(N, h), bf(n_mb, T, h), f32(n_mb, T, k)
        slots = E + EP * r
        self.dW = [f32(slots, hff, h), f32(slots, hff, h), f32(slots, h, hff)]
        if form == "accumulate":
            self.Xrows, self.dY = bf(N, h), [bf(N, h)]
            return
        self.row_tok = [i32(N) for _ in range(n_mb)]
        self.ws_wgrad = ws(rl.WS_WGRAD_BATCHED)
        self.WT = [bf(E, h, hff), bf(E, h, hff), bf(E, hff, h)]
        if form == "gated":
            self.row_gate, self.ws_dgate = f32(N), ws(rl.WS_DGATE)
        else:
            self.dY = [bf(N, h) for _ in range(n_mb)]


def prepare(case, seed):
    return State(case, seed)


# ---------------------------------------------------------------------------------------------
def _permute(s, mb, X=None, Xrows=None):
    t = s.tabs
    rl.relibra_permute(s.ids[mb], t["inst_ptr"][mb], t["inst_rows"][mb], t["inst_group"][mb], t["group_offset"][mb], X, s.case["E"], s.G,
                       row_of=s.row_of, src_of=s.src_of, Xrows=Xrows, workspace=s.ws_perm, err_flag=s.err)


def _micro_batch_gated(s, mb):
    T, k, E = s.case["T"], s.case["k"], s.case["E"]
    go, ge, slot = s.tabs["group_offset"][mb], s.tabs["group_expert"][mb], s.tabs["group_dw_slot"][mb]
    _permute(s, mb)
    rl.relibra_row_tokens(s.src_of, k, T, row_tok=s.row_tok[mb], err_flag=s.err)
    rl.relibra_row_gates(s.src_of, s.gates[mb], row_gate=s.row_gate, err_flag=s.err)
    rl.relibra_moe_ffn_fwd_gated(s.X[mb], s.row_tok[mb], s.row_gate, go, ge, *s.WT, Gt=s.Gt, U=s.U, A=s.A[mb], Ag=s.A[mb], Yrows=s.Yrows,
                                 workspace=s.ws[mb], err_flag=s.err, flags=rl.FWD_TRANSPOSED_WEIGHTS)
    rl.relibra_unpermute_combine(rl.COMBINE_SUM, s.Yrows, s.row_of, T, k, out_tok=s.Out[mb], err_flag=s.err)
    rl.relibra_moe_ffn_bwd_gated(s.dOut[mb], s.row_tok[mb], s.row_gate, s.Gt, s.U, go, ge, slot, *s.W, src_of=s.src_of, E=E,
                                 dXrows=s.dXrows, dgate=s.dgate[mb], workspace=s.ws[mb], dgate_scratch=s.ws_dgate, err_flag=s.err)
    rl.relibra_unpermute_combine(rl.COMBINE_SUM, s.dXrows, s.row_of, T, k, out_tok=s.dX[mb], err_flag=s.err)


def _micro_batch_plain(s, mb):
    T, k, E = s.case["T"], s.case["k"], s.case["E"]
    go, ge, slot = s.tabs["group_offset"][mb], s.tabs["group_expert"][mb], s.tabs["group_dw_slot"][mb]
    accumulate = s.case["form"] == "accumulate"
    i = 0 if accumulate else mb
    if accumulate:
        _permute(s, mb, s.X[mb], s.Xrows)
        rl.relibra_moe_ffn_fwd(s.Xrows, go, ge, *s.W, Gt=s.Gt, U=s.U, A=s.A[i], Yrows=s.Yrows, workspace=s.ws[i], err_flag=s.err)
    else:
        _permute(s, mb)
        rl.relibra_row_tokens(s.src_of, k, T, row_tok=s.row_tok[mb], err_flag=s.err)
        rl.relibra_moe_ffn_fwd_gather(s.X[mb], s.row_tok[mb], go, ge, *s.WT, Gt=s.Gt, U=s.U, A=s.A[i], Yrows=s.Yrows,
                                      workspace=s.ws[i], err_flag=s.err, flags=rl.FWD_TRANSPOSED_WEIGHTS)
    rl.relibra_unpermute_combine(rl.COMBINE_FWD, s.Yrows, s.row_of, T, k, gates=s.gates[mb], out_tok=s.Out[mb], err_flag=s.err)
    rl.relibra_unpermute_combine(rl.COMBINE_BWD, s.Yrows, s.row_of, T, k, gates=s.gates[mb], tok=s.dOut[mb], out_rows=s.dY[i],
                                 dgate=s.dgate[mb], err_flag=s.err)
    flags = (0 if mb == 0 else rl.BWD_ACCUMULATE) if accumulate else rl.BWD_DEFER_WGRAD
    rl.relibra_moe_ffn_bwd(s.dY[i], s.Xrows if accumulate else None, s.Gt, s.U, s.A[i], go, ge, slot, *s.W, *s.dW, E=E, flags=flags,
                           dXrows=s.dXrows, workspace=s.ws[i], err_flag=s.err)
    rl.relibra_unpermute_combine(rl.COMBINE_SUM, s.dXrows, s.row_of, T, k, out_tok=s.dX[mb], err_flag=s.err)


def _train(s):
    c, t = s.case, s.tabs
    form, n_mb, E = c["form"], c["n_mb"], c["E"]
    if form != "accumulate":
        for w, wt in zip(s.W, s.WT):
            rl.relibra_transpose_experts(w, wt)
    for mb in range(n_mb):
        (_micro_batch_gated if form == "gated" else _micro_batch_plain)(s, mb)
    if form != "accumulate":
        mbs = [dict(X=s.X[mb], row_tok=s.row_tok[mb], A=s.A[mb], bwd_workspace=s.ws[mb], inst_ptr=t["inst_ptr"][mb],
                    inst_group=t["inst_group"][mb], group_offset=t["group_offset"][mb],
                    **(dict(dOut=s.dOut[mb]) if form == "gated" else dict(dYrows=s.dY[mb]))) for mb in range(n_mb)]
        rl.relibra_moe_ffn_wgrad_batched(mbs, E, *s.dW, workspace=s.ws_wgrad, err_flag=s.err)
    return dict(Out=s.Out, dX=s.dX, dgate=s.dgate, dWg=s.dW[0][:E], dWu=s.dW[1][:E], dWd=s.dW[2][:E], err=s.err)


def _forward(s):
    T, k = s.case["T"], s.case["k"]
    _permute(s, 0)
    rl.relibra_row_tokens(s.src_of, k, T, row_tok=s.row_tok, err_flag=s.err)
    rl.relibra_moe_ffn_fwd_gather(s.X[0], s.row_tok, s.tabs["group_offset"][0], s.tabs["group_expert"][0], *s.W, Gt=s.Gt, U=s.U, A=s.A,
                                  Yrows=s.Yrows, workspace=s.ws, err_flag=s.err)
    rl.relibra_unpermute_combine(rl.COMBINE_FWD, s.Yrows, s.row_of, T, k, gates=s.gates[0], out_tok=s.Out[0], err_flag=s.err)
    return dict(Out=s.Out, Gt=s.Gt, U=s.U, A=s.A, err=s.err)


def _plan(s):
    c = s.case
    rl.relibra_route_hist(s.ids, c["E"], counts=s.counts, err_flag=s.err)
    plan = rl.relibra_plan(s.counts.cpu().numpy(), c["k"], c["EP"], _ranks_per_node(c), c["r"])
    return dict(_tables(plan), counts=s.counts, before=plan["max_load_before"], after=plan["max_load_after"], err=s.err)


def _hist(s):
    rl.relibra_route_hist(s.ids, s.case["E"], counts=s.counts, err_flag=s.err)
    return dict(counts=s.counts, err=s.err)


def _dispatch(s):
    T, k = s.case["T"], s.case["k"]
    _permute(s, 0, s.X[0], s.Xrows)
    rl.relibra_unpermute_combine(rl.COMBINE_FWD, s.Y, s.row_of, T, k, gates=s.gates[0], out_tok=s.Out[0], err_flag=s.err)
    rl.relibra_unpermute_combine(rl.COMBINE_BWD, s.Y, s.row_of, T, k, gates=s.gates[0], tok=s.dOut, out_rows=s.dY, dgate=s.dgate,
                                 err_flag=s.err)
    return dict(row_of=s.row_of, src_of=s.src_of, Xrows=s.Xrows, Out=s.Out, dY=s.dY, dgate=s.dgate, err=s.err)


def _replica(s):
    c = s.case
    rl.relibra_replica_push(*s.W, s.replica_expert, c["E"], c["EP"], c["r"], err_flag=s.err)
    rl.relibra_replica_pull(*s.dW, s.replica_expert, c["E"], c["EP"], c["r"], err_flag=s.err)
    return dict(Wg=s.W[0], Wu=s.W[1], Wd=s.W[2], dWg=s.dW[0], dWu=s.dW[1], dWd=s.dW[2], err=s.err)


_RUN = dict(train=_train, forward=_forward, plan=_plan, hist=_hist, dispatch=_dispatch, replica=_replica)


def run(state):
    return _RUN[state.case["do"]](state)


# ---------------------------------------------------------------------------------------------
def _live_experts(case):
    """Experts with at least one row in a batch of this routing (drawn once more, on the host)."""
    rng, E = np.random.default_rng(0), case["E"]
    live = set()
    for _ in range(case["n_mb"]):
        bias = -case["zipf"] * np.log(np.arange(1, E + 1))
        rng.shuffle(bias)
        logits = rng.standard_normal((min(case["T"], 4096), E)) + bias
        live.update(np.argpartition(-logits, case["k"] - 1, axis=1)[:, :case["k"]].ravel().tolist())
    return len(live)


def work(case):
    E, k, h, hff, T, n_mb, do = (case[x] for x in ("E", "k", "h", "hff", "T", "n_mb", "do"))
    N, w = T * k, 1.0 * h * hff
    live_experts = _live_experts(case) if do in ("train", "forward") else 0
    if do == "train":        # tokens and gradients in and out, routing and gates, weights read, weight gradients written
        return dict(bytes=n_mb * (8.0 * T * h + 12.0 * N) + 3 * w * (2 * live_experts + 4 * E), flops=18.0 * w * N * n_mb)
    if do == "forward":      # ... and the activations kept for a backward pass
        return dict(bytes=4.0 * T * h + 8.0 * N + 6.0 * N * hff + 6.0 * w * live_experts, flops=6.0 * w * N)
    if do in ("plan", "hist"):
        return dict(bytes=4.0 * N * n_mb + 4.0 * E * n_mb, flops=0)
    if do == "dispatch":     # X -> rows; rows -> combined; dOut and rows -> gradient rows and dgate
        return dict(bytes=(2.0 * T * h + 2.0 * N * h + 12.0 * N) + (2.0 * N * h + 2.0 * T * h + 4.0 * N) + (2.0 * T * h + 4.0 * N * h + 4.0 * N), flops=0)
    # push: a live slot's parameters read and written; pull: slot and home gradients read, home written
    return dict(bytes=case["live"] * 3 * w * (2 * 2 + 4 * 3), flops=0)


def tolerance(case):
    do = case["do"]
    if do in ("plan", "hist", "replica"):
        return "exact"       # whole numbers; copies and single fp32 additions in a fixed order
    if do == "dispatch":
        return {"rel": 4e-3}  # one bf16 rounding of an fp32 sum (1.1e-3); copies and indices are exact
    # bf16 operands and intermediates, fp32 accumulation: 2.4e-3 to 3.8e-3 against the same path in
    # 64 bits, so up to 5e-3 between two implementations
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------------------------
# What `run` returns, in 64 bits.  Inputs are the state's (drawn once more from the seed); the
# rows' order is spelled out from the plan's tables, which the program has in hand.
def _rows_by_definition(s, mb):
    """Expert of every assignment and its row: an expert's assignments in ascending order fill its instances one after the other."""
    ids = s.ids[mb].reshape(-1).long()
    t = {key: s.tabs[key][mb].cpu().tolist() for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset")}
    row_of = torch.empty_like(ids)
    for e in range(s.case["E"]):
        at, taken = torch.nonzero(ids == e).reshape(-1), 0
        for i in range(t["inst_ptr"][e], t["inst_ptr"][e + 1]):
            n, first = t["inst_rows"][i], t["group_offset"][t["inst_group"][i]]
            row_of[at[taken:taken + n]] = first + torch.arange(n, device=DEV)
            taken += n
    return ids, row_of


def _exact_layer(s, backward):
    c = s.case
    E, k, h, hff, T, n_mb, N = c["E"], c["k"], c["h"], c["hff"], c["T"], c["n_mb"], s.N
    f64 = lambda *shape: torch.zeros(shape, dtype=torch.float64, device=DEV)
    Out, dX, dgate = f64(n_mb, T, h), f64(n_mb, T, h), f64(n_mb, N)
    saved = None if backward else [f64(N, hff) for _ in range(3)]
    dW = [f64(E, hff, h), f64(E, hff, h), f64(E, h, hff)] if backward else None
    routes = [s.ids[mb].reshape(-1).long() if backward else _rows_by_definition(s, mb) for mb in range(n_mb)]
    for e in range(E):
        Wg, Wu, Wd = (w[e].double() for w in s.W)
        for mb in range(n_mb):
            at = torch.nonzero((routes[mb] if backward else routes[mb][0]) == e).reshape(-1)
            if at.numel() == 0:
                continue
            tok, gate = at // k, s.gates[mb].reshape(-1)[at].double()[:, None]
            x = s.X[mb][tok].double()
            G, U = x @ Wg.T, x @ Wu.T
            sig = torch.sigmoid(G)
            A = G * sig * U
            Y = A @ Wd.T
            Out[mb].index_add_(0, tok, gate * Y)
            if not backward:
                for whole, part in zip(saved, (G, U, A)):
                    whole[routes[mb][1][at]] = part
                continue
            dO = s.dOut[mb][tok].double()
            dgate[mb][at] = (dO * Y).sum(1)
            dY = gate * dO
            dA = dY @ Wd
            dG, dU = dA * U * sig * (1 + G * (1 - sig)), dA * G * sig
            dX[mb].index_add_(0, tok, dG @ Wg + dU @ Wu)
            for whole, part in zip(dW, (dG.T @ x, dU.T @ x, dY.T @ A)):
                whole[e] += part
    if not backward:
        return dict(Out=Out, Gt=saved[0], U=saved[1], A=saved[2], err=None)
    return dict(Out=Out, dX=dX, dgate=dgate.view(n_mb, T, k), dWg=dW[0], dWu=dW[1], dWd=dW[2], err=None)


def exact(case, seed):
    do, E, k, T, n_mb = (case[x] for x in ("do", "E", "k", "T", "n_mb"))
    s = prepare(case, seed)
    if do in ("train", "forward"):
        return _exact_layer(s, do == "train")
    if do in ("plan", "hist"):
        counts = torch.stack([torch.bincount(s.ids[mb].reshape(-1), minlength=E) for mb in range(n_mb)]).int()
        return dict(counts=counts, err=None)
    if do == "dispatch":
        _, row_of = _rows_by_definition(s, 0)
        tok = torch.arange(s.N, device=DEV) // k
        src_of = torch.empty_like(row_of)
        src_of[row_of] = torch.arange(s.N, device=DEV)
        gate, y, dO = s.gates[0].reshape(-1).double()[:, None], s.Y[row_of].double(), s.dOut[tok].double()
        dY = torch.empty((s.N, case["h"]), dtype=torch.float64, device=DEV)
        dY[row_of] = gate * dO
        return dict(row_of=row_of.int(), src_of=src_of.int(), Xrows=s.X[0][tok[src_of]].double(),
                    Out=(gate * y).view(T, k, -1).sum(1)[None], dY=dY, dgate=(dO * y).sum(1).view(T, k), err=None)
    table = s.replica_expert.cpu().tolist()
    W, dW = [w.clone() for w in s.W], [g.double() for g in s.dW]
    for slot, e in enumerate(table):
        if e >= 0:
            for w, g in zip(W, dW):
                w[E + slot] = w[e]
                g[e] += g[E + slot]
    W = [w.double() for w in W]
    return dict(Wg=W[0], Wu=W[1], Wd=W[2], dWg=dW[0], dWu=dW[1], dWd=dW[2], err=None)
