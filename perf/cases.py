"""The work a user of this library has it do, as cases that can be timed and compared between two builds.

Every case goes through the public entry points of ``paper_2112_13509_amd.binding``: scoring of candidate grids
(flat statistics, the two encoders, one entry of V per worker), the online update and its transfer-learning form
with replay mixing, and the trigger / selection on stored scores.  Inputs follow the distributions of
``paper_2112_13509_amd.workloads``; models, grids and minibatches come from that module, the large statistics arrays
are drawn on the GPU.

About the compared outputs: with fp32 arithmetic the chosen index is one of them.  With bf16 arithmetic it is not,
because the best two candidates of many scenarios lie closer together than bf16 rounding (an exact evaluation chooses
another one in about three scenarios of ten); there the scores and the score of the chosen candidate are compared, and,
where V of the chosen candidate is asked for, V, which is computed anew from the chosen index.
"""
import math

import torch

from paper_2112_13509_amd import binding as ab
from paper_2112_13509_amd import workloads as wl

DEV = "cuda:0"


# --------------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------------
def listed():
    return [
        # The paper's own operating point: one job, 64 candidates, a small network; a latency-bound call.
        dict(name="one_job_small_net", kind="score", dtype="f32", S=1, L=16, hidden="64,64", P=8, Q=8, scores=True,
             per_scenario=False, static=False),
        # One job that asks the large bf16 network, from a serving loop that hands over no workspace.
        dict(name="one_job_large_net", kind="score", dtype="bf16", S=1, L=128, hidden="1024,1024,1024,1024", P=16, Q=16,
             scores=True, per_scenario=False, static=True),
        # fp32 batch scoring over a fine grid, only the choice wanted.
        dict(name="batch_fine_grid_f32", kind="score", dtype="f32", S=1024, L=128, hidden="256,256", P=64, Q=64,
             scores=False, per_scenario=False, static=False),
        # A few hundred jobs on the large network; layer count, job count and grid on no tile boundary.
        dict(name="ragged_large_net", kind="score", dtype="bf16", S=777, L=101, hidden="1024,1024,1024,1024", P=15, Q=17,
             scores=True, per_scenario=False, static=False),
        # The benchmark's main workload: a whole cluster's history re-scored on the large network.
        dict(name="batch_large_net", kind="score", dtype="bf16", S=65536, L=128, hidden="1024,1024,1024,1024", P=16, Q=16,
             scores=True, per_scenario=False, static=False),
        # Transformer-like jobs of mixed layer counts through the per-tensor encoder.
        dict(name="tensor_encoder_batch", kind="encoder", te="mlp", S=8192, L=400, hidden="512,512", P=32, Q=32, mixed=True),
        # The same jobs through the temporal (LSTM) encoder, every job with all its layers.
        dict(name="lstm_encoder_batch", kind="encoder", te="lstm", S=8192, L=400, hidden="512,512", P=32, Q=32, mixed=False),
        # Per-worker speeds: every job brings its own grid and wants V of the pair that was chosen.
        dict(name="per_worker_speeds", kind="workers", S=300, L=64, n=8, hidden="512,512,512", P=16, Q=16, per_scenario=True),
        # Online adaptation at the configured minibatch: forward, backward and Adam, bf16 products.
        dict(name="update_minibatch", kind="update", dtype="bf16", B=4096, L=128, hidden="512,512,512", n=0, loss="mse",
             first=0, mix=False),
        # A handful of fresh observations adapt a small fp32 network.
        dict(name="update_small_f32", kind="update", dtype="f32", B=200, L=16, hidden="64,64", n=0, loss="mse", first=0,
             mix=False),
        # Transfer learning as the paper has it: fresh rows mixed with the offline pool, lower layers frozen.
        dict(name="adapt_tail_replay", kind="update", dtype="bf16", B=1000, L=128, hidden="512,512,512", n=8, loss="l2norm",
             first=2, mix=True),
        # The Optimization Trigger over stored scores of a whole batch.
        dict(name="trigger_batch", kind="decide", op="trigger", S=65536, C=256, pad=0),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


F32_NETS = ["64,64", "128,128", "256,256", "256,128,64", "256,256,256"]
BF16_NETS = ["512,512", "512,512,512", "1024,512,256", "1024,1024,1024,1024"]
# No drawn case costs more than the listed ones of its arithmetic (operations of one pass; sizes off the tile
# boundaries take longer for the same count).
MOST_F32, MOST_BF16 = 5.4e11, 6.0e13


def _fit(case):
    """The case with its scenario count cut down until its operations fit."""
    most = MOST_F32 if case.get("dtype") == "f32" else MOST_BF16
    f = work(case)["flops"]
    if f > most:
        case["S"] = max(1, int(case["S"] * most / f))
    return case


def draw(rng):
    kind = rng.choice(["score_f32", "score_bf16", "score_bf16", "mlp", "lstm", "workers", "update", "update", "adapt", "decide"])
    if kind == "score_f32":
        return _fit(dict(kind="score", dtype="f32", S=_logint(rng, 1, 4096), L=_logint(rng, 8, 128), hidden=rng.choice(F32_NETS),
                         P=rng.randint(5, 64), Q=rng.randint(5, 64), scores=rng.random() < 0.5, per_scenario=rng.random() < 0.3,
                         static=False))
    if kind == "score_bf16":
        case = _fit(dict(kind="score", dtype="bf16", S=_logint(rng, 1, 65536), L=_logint(rng, 16, 128),
                         hidden=rng.choice(BF16_NETS), P=rng.randint(8, 32), Q=rng.randint(8, 32), scores=rng.random() < 0.7,
                         per_scenario=rng.random() < 0.3, static=False))
        case["static"] = case["S"] * case["P"] * case["Q"] <= 4096 and rng.random() < 0.5
        return case
    if kind in ("mlp", "lstm"):
        return _fit(dict(kind="encoder", te=kind, S=_logint(rng, 16, 8192), L=_logint(rng, 50, 400), hidden=rng.choice(BF16_NETS[:3]),
                         P=rng.randint(8, 32), Q=rng.randint(8, 32), mixed=rng.random() < 0.6))
    if kind == "workers":
        return _fit(dict(kind="workers", S=_logint(rng, 1, 4096), L=_logint(rng, 16, 128), n=rng.choice([2, 4, 8, 16]),
                         hidden=rng.choice(BF16_NETS), P=rng.randint(8, 24), Q=rng.randint(8, 24),
                         per_scenario=rng.random() < 0.5))
    if kind in ("update", "adapt"):
        small = rng.random() < 0.3
        hidden = rng.choice(F32_NETS[:4] if small else BF16_NETS[:3])
        n = rng.choice([0, 0, 4, 8])
        return dict(kind="update", dtype="f32" if small else "bf16", B=_logint(rng, 64, 8192), L=_logint(rng, 16, 128),
                    hidden=hidden, n=n, loss="l2norm" if n and rng.random() < 0.5 else "mse",
                    first=rng.randint(1, len(_widths(hidden))) if kind == "adapt" else 0, mix=kind == "adapt")
    return dict(kind="decide", op=rng.choice(["trigger", "select"]), S=_logint(rng, 64, 65536), C=_logint(rng, 32, 1024),
                pad=rng.choice([0, 0, 1, 32]))


def _widths(text):
    return [int(x) for x in text.split(",")]


# --------------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _stats(g, S, L, bytes_lo, bytes_hi, position=False):
    """Raw per-layer statistics [S, L, 3 or 4]: forward and backward ms, tensor bytes(, position)."""
    n = lambda: torch.randn(S, L, generator=g, device=DEV)
    t = [torch.exp(wl.TIME_MU + wl.TIME_SIGMA * n()), torch.exp(wl.TIME_MU + wl.TIME_SIGMA * n()),
         torch.exp(math.log(bytes_lo) + math.log(bytes_hi / bytes_lo) * torch.rand(S, L, generator=g, device=DEV))]
    if position:
        t.append((torch.arange(L, device=DEV) / max(L - 1, 1)).expand(S, L))
    return torch.stack(t, dim=2).contiguous()


def _scalars(g, S, onehots):
    """Raw scalars [S, 2 + 2 onehots]: workers, bandwidth, two-way one-hots."""
    cols = [2.0 ** torch.randint(1, 5, (S,), generator=g, device=DEV).float(),
            wl.BW_LO + (wl.BW_HI - wl.BW_LO) * torch.rand(S, generator=g, device=DEV)]
    for _ in range(onehots):
        b = torch.randint(0, 2, (S,), generator=g, device=DEV)
        cols += [(b == 0).float(), (b == 1).float()]
    return torch.stack(cols, dim=1).contiguous()


def _grids(g, w, S, per_scenario):
    part, cred = torch.from_numpy(w.part).to(DEV), torch.from_numpy(w.cred).to(DEV)
    if not per_scenario:
        return part, cred
    # a job's grid: the common one, its partition sizes scaled by up to a factor of two, its credits by up to 25 %
    a = torch.exp2(2.0 * torch.rand(S, 1, generator=g, device=DEV) - 1.0)
    b = 1.0 + 0.25 * torch.rand(S, 1, generator=g, device=DEV)
    return (part * a).contiguous(), (cred * b).contiguous()


class _Scoring:
    """Model, inputs, outputs and workspace of one scoring problem."""

    def __init__(self, w, dyn, scal, part, cred, scores=True, layers_of=None, static=False, n_v=0):
        S, C = dyn.shape[0], part.shape[-1] * cred.shape[-1]
        self.desc, self.params = ab.desc_from_workload(w), ab.Params.from_workload(w, DEV)
        self.dyn, self.scal, self.part, self.cred, self.layers_of = dyn, scal, part, cred, layers_of
        self.scores = torch.empty(S, C, device=DEV) if scores else None
        self.best_idx = torch.empty(S, dtype=torch.int32, device=DEV)
        self.best_score = torch.empty(S, device=DEV)
        self.v = torch.empty(S, n_v, device=DEV) if n_v else None
        self.static = static
        self.ws = None if static else ab.alloc_workspace(self.desc, S, C, device=DEV)

    def run(self):
        if self.static:
            ab.ab_score_candidates_static(self.desc, self.params, self.dyn, self.scal, self.part, self.cred, self.scores,
                                          self.best_idx, self.best_score, layers_of=self.layers_of)
        else:
            ab.ab_score_candidates(self.desc, self.params, self.dyn, self.scal, self.part, self.cred, self.scores,
                                   self.best_idx, self.best_score, self.ws, layers_of=self.layers_of, v_best=self.v)
        out = [self.best_score]
        if self.scores is not None:
            out.append(self.scores)
        if self.v is not None:
            out.append(self.v)
        if self.desc.compute_dtype == ab.AB_F32:
            out.append(self.best_idx)
        return out


class _Update:
    """Model with its optimiser state, a minibatch (or two pools to mix it from) and a workspace."""

    def __init__(self, case, seed):
        B, hidden, self.mix = case["B"], _widths(case["hidden"]), case["mix"]
        n_old, n_new = 4 * B, max(1, B // 2)
        u = wl.make_update(N=n_old + n_new if self.mix else B, batch=B, L=case["L"], hidden=hidden, dtype=case["dtype"],
                           seed=seed, n_workers=case["n"], loss_kind=case["loss"])
        self.desc = ab.desc_from_workload(u)
        self.params = ab.Params(u.W, u.b, case["dtype"], DEV, trainable=True)
        self.first, self.loss = case["first"], torch.zeros(1, device=DEV)
        x, y = torch.from_numpy(u.x_raw).to(DEV), torch.from_numpy(u.target).to(DEV)
        self.x, self.y = x, y
        if self.mix:
            # a quarter of the minibatch from the fresh rows, the rest from the offline pool
            self.pools = (x[:n_new].contiguous(), y[:n_new].contiguous(), x[n_new:].contiguous(), y[n_new:].contiguous())
            g = _gen(seed)
            fresh = torch.rand(B, generator=g, device=DEV) < 0.25
            new = torch.randint(0, n_new, (B,), generator=g, device=DEV)
            old = -1 - torch.randint(0, n_old, (B,), generator=g, device=DEV)
            self.pick = torch.where(fresh, new, old).to(torch.int32)
            self.x, self.y = torch.empty_like(x[:B]), torch.empty_like(y[:B])
        self.ws = ab.alloc_workspace(self.desc, B=B, device=DEV)

    def run(self):
        p = self.params
        if self.mix:
            ab.ab_replay_mix(*self.pools, self.pick, self.x, self.y)
        if self.first:
            ab.ab_online_update_tail(self.desc, p, self.x, self.y, self.first, loss_out=self.loss, workspace=self.ws)
        else:
            ab.ab_online_update(self.desc, p, self.x, self.y, loss_out=self.loss, workspace=self.ws)
        k = self.first
        out = [self.loss, p.step, p.W[k:], p.b[k:], p.W_master[k:], p.mW[k:], p.vW[k:], p.mb[k:], p.vb[k:]]
        return out + [self.x, self.y] if self.mix else out


class _Decide:
    """A stored score matrix (rows padded by some columns) and what the decision on it reads and writes."""

    def __init__(self, case, seed):
        g, S, C = _gen(seed), case["S"], case["C"]
        self.op, self.C = case["op"], C
        # a job's predicted speeds: smooth over the candidates, around 1, with some candidates equally good
        self.scores = 1.0 + 0.2 * torch.randn(S, 1, generator=g, device=DEV) \
            + torch.round(50.0 * torch.randn(S, C + case["pad"], generator=g, device=DEV)) / 1000.0
        self.current = torch.randint(0, C, (S,), generator=g, device=DEV).to(torch.int32)
        at = self.scores.gather(1, self.current.long()[:, None])[:, 0]
        self.observed = (at * (1.0 + 0.1 * torch.randn(S, generator=g, device=DEV))).contiguous()
        self.best_idx = torch.empty(S, dtype=torch.int32, device=DEV)
        self.best_score, self.gain = torch.empty(S, device=DEV), torch.empty(S, device=DEV)
        self.reconfigure = torch.empty(S, dtype=torch.uint8, device=DEV)
        self.adapt = torch.empty(S, dtype=torch.uint8, device=DEV)

    def run(self):
        if self.op == "select":
            ab.ab_select_best(self.scores, self.best_idx, self.best_score, C_=self.C)
            return [self.best_idx, self.best_score]
        ab.ab_trigger(self.scores, self.current, self.best_idx, self.reconfigure, self.observed, self.gain, self.adapt,
                      C_=self.C)
        return [self.best_idx, self.gain, self.reconfigure, self.adapt]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "update":
        return _Update(case, seed)
    if kind == "decide":
        return _Decide(case, seed)
    g, S, L, hidden, P, Q = _gen(seed), case["S"], case["L"], _widths(case["hidden"]), case["P"], case["Q"]
    if kind == "score":
        w = wl.make_scoring("flat", 1, L, hidden, P, Q, 16 * wl.KIB, 64 * wl.MIB, 1.0, 64.0, False, case["dtype"], seed)
        part, cred = _grids(g, w, S, case["per_scenario"])
        return _Scoring(w, _stats(g, S, L, 4 * wl.KIB, 400 * wl.MIB), _scalars(g, S, 1), part, cred, case["scores"],
                        static=case["static"])
    if kind == "encoder":
        make, sizes = (wl.make_lstm_encoder, {}) if case["te"] == "lstm" else (wl.make_tensor_encoder, {"te_hidden": [128, 128]})
        w = make(case["te"], 1, hidden, P=P, Q=Q, dtype="bf16", seed=seed, n_blocks=0, per_block=1, extra=L, **sizes)
        layers_of = torch.randint((L + 1) // 2, L + 1, (S,), generator=g, device=DEV).to(torch.int32) if case["mixed"] else None
        part, cred = _grids(g, w, S, False)
        return _Scoring(w, _stats(g, S, L, wl.KIB, 256 * wl.MIB, position=True), _scalars(g, S, 2), part, cred, False,
                        layers_of=layers_of)
    w = wl.make_per_worker("workers", S, L, case["n"], hidden, P, Q, "bf16", seed)
    part, cred = _grids(g, w, S, case["per_scenario"])
    return _Scoring(w, torch.from_numpy(w.dyn).to(DEV), torch.from_numpy(w.scal).to(DEV), part, cred, True, n_v=case["n"])


def run(state):
    return state.run()


# --------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct implementations may be apart
# --------------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "decide":
        per = 8 if case["op"] == "select" else 18
        return {"bytes": case["S"] * (4 * case["C"] + per), "flops": case["S"] * case["C"]}
    hidden = _widths(case["hidden"])
    if kind == "update":
        es = 2 if case["dtype"] == "bf16" else 4
        F, n, B, first = 3 * case["L"] + 6, max(1, case["n"]), case["B"], case["first"]
        widths = [F] + hidden + [n]
        par = [a * b + b for a, b in zip(widths, widths[1:])]
        fwd = 2 * B * sum(par)
        dw = 2 * B * sum(par[first:])
        dx = 2 * B * sum(par[first + 1:])
        rows = 4 * B * (F + n) * (3 if case["mix"] else 1)
        return {"bytes": rows + es * sum(par) + (24 + es) * sum(par[first:]), "flops": fwd + dw + dx}
    S, C = case["S"], case["P"] * case["Q"]
    if kind == "encoder":
        layers = case["L"] * (0.75 if case["mixed"] else 1.0)
        per_layer, enc, block = (2 * (4 * 128 + 128 * 128), 4 * 128 + 128 * 128, 128) if case["te"] == "mlp" else \
            (2 * (4 * 32 + 256 * 96 + 256 * 128), 4 * 32 + 256 * 96 + 256 * 128, 64)
        enc_flops, Fs, raw, n_out, n_v = S * layers * per_layer, block + 6, S * (layers * 4 + 6) * 4, 1, 0
        es, scores, per_scenario = 2, False, False
    else:
        K, Ns = (case["n"], 6 + 2 * case["n"]) if kind == "workers" else (3, 4)
        enc, enc_flops, Fs, raw = 0, 0, K * case["L"] + Ns, S * (K * case["L"] + Ns) * 4
        n_out, n_v = (case["n"], case["n"]) if kind == "workers" else (1, 0)
        es = 4 if case.get("dtype") == "f32" else 2
        scores, per_scenario = kind == "workers" or case["scores"], case["per_scenario"]
    chain = 2 * sum(a * b for a, b in zip(hidden, hidden[1:]))
    flops = enc_flops + 2 * S * Fs * hidden[0] + S * C * (3 * hidden[0] + chain + 2 * hidden[-1])
    if n_v:
        flops += S * (chain + 2 * hidden[-1] * n_v)
    widths = [Fs + 2] + hidden + [n_out]
    par = enc + sum(a * b for a, b in zip(widths, widths[1:]))
    grid = 4 * (case["P"] + case["Q"]) * (S if per_scenario else 1)
    out = 8 * S + (4 * S * C if scores else 0) + 4 * S * n_v
    return {"bytes": raw + es * par + grid + out, "flops": flops}


def tolerance(case):
    if case["kind"] == "decide":
        return "exact"
    if case.get("dtype") == "f32":
        # Sums of at most a few hundred fp32 terms.  The update divides every gradient by its own magnitude in its first
        # steps, so an entry that is all rounding moves by a whole learning rate: 2e-3 against parameters of about 0.1.
        # The chosen index may differ where two candidates are equal to fp32 rounding.
        return {"rel": 1e-4, "max": 5e-2} if case["kind"] == "update" else {"rel": 1e-5, "differ": 0.01}
    # bf16 operands, fp32 accumulation: activations round to 8 bits, on one side or the other of a boundary.
    return {"rel": 1e-2}
