"""Performance cases: the work that a user of this library has it do, through its public calls.

Every case is a plain dict; the graphs are synthetic stand-ins with the node count, edge count, degree shape and share of
edges inside subgraphs of the repository's workloads (and of generic graphs between them), made on the GPU from a seed.

  kind      train     gco_train for `epochs` epochs, then what a caller takes home: the loss of every epoch, the probabilities and
                      the trained networks; with `embed` from fresh parameters every time, as random restarts do, and back come
                      the trained embeddings too: the whole checkpoint of a small model
            finetune  the same for the first `listed` subgraphs, with the conflict penalty on some of their nodes
            infer     forward pass, probabilities, loss of every subgraph
            readout   rounding with both repairs, cross edges, cross nodes and conflict edges of a trained model
            job       upload of graph and parameters, training, probabilities, rounding: a graph seen for the first time
  n, m      nodes, undirected edges aimed at (duplicates that come up are dropped)
  hub       expected degree of the largest node (power law with exponent gamma), 0 = every node alike
  local     share of the edges drawn inside a subgraph
  parts, skew   subgraphs and the relative spread of their sizes
  layers, dim, storage, problem, norm, shared, embed_trained, gumbel   the model, as in gco_config
"""
import ctypes
import math

import numpy as np
import torch

from paper_2511_09261_amd import binding

_MODEL = dict(problem="mis", norm="sym", layers=2, dim=16, storage="fp32", shared=False, embed_trained=True, gumbel=False,
              lr=5e-3)


def _case(name, kind, n, m, parts, **more):
    c = dict(_MODEL, name=name, kind=kind, n=n, m=m, parts=parts, hub=0, gamma=2.2, local=0.5, skew=0.0, epochs=0, embed=False,
             listed=0)
    c.update(more)
    return c


def listed():
    return [
        # The default model (two layers, width 16, fp32) on a graph of a few hundred nodes, as in the G(200, 0.05) workload: the
        # smallest call, nothing but launches and latency.
        _case("tiny", "train", 200, 962, 1, local=1.0, lr=1e-2, epochs=200, embed=True),
        # Max-Cut on a sparse graph of ten thousand nodes of about equal degree, width 32, fp32, 8 subgraphs.
        _case("small-maxcut", "train", 10_000, 15_000, 8, local=0.7, problem="maxcut", dim=32, epochs=30, embed=True),
        # Facebook-shaped graph, 16 subgraphs, width 64, bf16.
        _case("facebook-shaped", "train", 4_039, 88_234, 16, hub=1_000, gamma=2.5, local=0.11, dim=64, storage="bf16",
              epochs=100, embed=True),
        # Youtube-shaped graph, 64 subgraphs, three layers of width 64, bf16: the benchmark's workload.
        _case("youtube-shaped", "train", 1_134_890, 2_987_624, 64, hub=28_000, local=0.26, layers=3, dim=64, storage="bf16",
              epochs=20),
        # A quarter of the 50-regular two-million-node workload: width 128, bf16, most edges cut.
        _case("regular-wide", "train", 499_999, 12_500_000, 64, local=0.044, layers=3, dim=128,
              storage="bf16", lr=2e-3, epochs=8),
        # The default model on a large power-law graph: fp32 storage where bandwidth counts.
        _case("large-default", "train", 700_001, 1_850_000, 48, hub=9_000, local=0.4, skew=0.3, epochs=20),
        # fp32 storage at width 64, three layers, row-mean normalisation, one weight set for all subgraphs; a partition that
        # keeps most edges (communities), ragged subgraphs.
        _case("communities-fp32", "train", 150_001, 900_000, 24, hub=2_000, gamma=2.5, local=0.9, skew=0.5, norm="mean",
              layers=3, dim=64, shared=True, epochs=20),
        # The one-layer model with Gumbel-softmax inputs of which only the weights are trained, on a collaboration-shaped graph.
        _case("one-layer", "train", 18_772, 198_050, 4, hub=500, gamma=2.5, local=0.6, norm="mean", layers=1, dim=64,
              embed_trained=False, gumbel=True, epochs=100),
        # Fine-tuning round of the coordination stage: 6 of 64 subgraphs with the penalty on some nodes.
        _case("fine-tune", "finetune", 600_000, 1_600_000, 64, hub=12_000, local=0.3, layers=3, dim=64, storage="bf16",
              epochs=20, listed=6),
        # Forward pass, probabilities and loss at full size.
        _case("infer", "infer", 1_134_890, 2_987_624, 64, hub=28_000, local=0.26, layers=3, dim=64, storage="bf16"),
        # What follows training: rounding, repair inside subgraphs and over all edges, cross edges, conflicts.
        _case("read-out", "readout", 1_134_890, 2_987_624, 64, hub=28_000, local=0.26, epochs=10),
        # A graph that the library has not seen: upload and preprocessing count as much as the training.
        _case("whole-job", "job", 300_007, 1_200_000, 32, hub=5_000, local=0.5, skew=0.2, layers=3, dim=64, storage="bf16",
              epochs=30),
    ]


def draw(rng):
    n = int(round(150 * (1_000_000 / 150) ** rng.random()))
    kind = rng.choice(["train"] * 6 + ["finetune", "infer", "readout", "job"])
    storage = rng.choice(["fp32", "fp32", "bf16", "bf16"])
    dim = rng.choice([64, 64, 128] if storage == "bf16" else [8, 16, 16, 32, 64, 128])
    while n * dim > 1_134_890 * 64:
        n = n * 2 // 3
    degree = 1.3 * 20 ** rng.random()
    m = int(n * min(degree, n / 16, 4_000_000 / n))
    parts = max(1, min(256, n // 50, int(n ** (0.55 * rng.random()))))
    layers = rng.choice([1, 2, 2, 3, 3])
    one = layers == 1
    c = _case("", kind, n, m, parts, hub=rng.choice([0, int(n ** 0.7) // 2]), gamma=rng.choice([2.2, 2.5]),
              local=round(0.05 + 0.9 * rng.random(), 2), skew=rng.choice([0.0, 0.3, 0.6]), layers=layers, dim=dim,
              storage=storage, problem=rng.choice(["mis", "maxcut"]) if storage == "fp32" else "mis", norm=rng.choice(["sym", "sym", "mean"]),
              shared=rng.random() < 0.2, embed_trained=not (one and rng.random() < 0.5), gumbel=one and rng.random() < 0.5)
    del c["name"]
    if kind in ("train", "finetune", "job"):
        c["epochs"] = max(4, min(25, int(15 * 1_134_890 * 64 / max(1, n * dim * layers))))
        c["embed"] = kind == "train" and n * dim <= 400_000
    if dim == 128:
        c["lr"] = 2e-3
    if kind == "readout":
        c["epochs"] = 5
        c["storage"] = "fp32"  # probabilities that do not hang on bf16 rounding
        c["problem"] = "mis"
    if kind == "finetune":
        c["listed"] = max(1, parts // 8)
        c["problem"] = "mis"
    return c


# --- inputs ------------------------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _graph(case, gen):
    """rowptr int64[n+1], col int32[nnz], part int32[n] on the GPU, in an order of the nodes that says nothing about them."""
    n, P, dev = case["n"], case["parts"], "cuda"
    # sizes of the subgraphs; node v of the inner order belongs to part_of[v]
    share = 1.0 + case["skew"] * (2.0 * torch.rand(P, generator=gen, device=dev, dtype=torch.float64) - 1.0)
    ends = torch.round(torch.cumsum(share, 0) / share.sum() * (n - P)).to(torch.int64) + torch.arange(1, P + 1, device=dev)
    part_of = torch.searchsorted(ends, torch.arange(n, device=dev), right=True)
    starts = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), ends[:-1]])
    # weights: all alike, or a power law whose largest expected degree is `hub`, spread over the subgraphs at random
    rank = torch.randperm(n, generator=gen, device=dev).to(torch.float64)
    if case["hub"]:
        a = 1.0 / (case["gamma"] - 1.0)
        lo, hi = 0.0, float(n)
        for _ in range(40):
            i0 = 0.5 * (lo + hi)
            w = (rank + 1.0 + i0) ** -a
            if 2.0 * case["m"] * (1.0 + i0) ** -a / float(w.sum()) > case["hub"]:
                lo = i0
            else:
                hi = i0
    else:
        w = torch.ones(n, dtype=torch.float64, device=dev)
    cum = torch.cumsum(w, 0)
    before = torch.cat([torch.zeros(1, dtype=torch.float64, device=dev), cum])

    def pick(lo, hi):
        x = lo + (hi - lo) * torch.rand(lo.shape[0], generator=gen, device=dev, dtype=torch.float64)
        return torch.searchsorted(cum, x).clamp_(max=n - 1)

    m = case["m"]
    zero, total = torch.zeros(m, dtype=torch.float64, device=dev), cum[-1].expand(m)
    u = pick(zero, total)
    inside = torch.rand(m, generator=gen, device=dev) < case["local"]
    k = part_of[u]
    v = pick(torch.where(inside, before[starts[k]], zero), torch.where(inside, before[ends[k]], total))
    name = torch.randperm(n, generator=gen, device=dev)  # inner order -> the caller's order
    u, v = name[u], name[v]
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.minimum(u, v) * n + torch.maximum(u, v))
    u, v = key // n, key % n
    both = torch.sort(torch.cat([u * n + v, v * n + u])).values
    row, col = both // n, (both % n).to(torch.int32)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    part = torch.empty(n, dtype=torch.int32, device=dev)
    part[name] = part_of.to(torch.int32)
    return rowptr, col, part


def _inputs(case, seed):
    gen = _generator(seed)
    # the number of cross edges is an output of the read-out: its graph is the same for every seed, the model is not
    rowptr, col, part = _graph(case, _generator(case["m"]) if case["kind"] == "readout" else gen)
    n, d, L = case["n"], case["dim"], case["layers"]
    sets = 1 if case["shared"] else case["parts"]
    x = {"rowptr": rowptr, "col": col, "part": part}
    x["E"] = 0.1 * torch.randn(n, d, generator=gen, device="cuda")
    if case["gumbel"]:
        x["U"] = (torch.rand(n, d, generator=gen, device="cuda") * (1 - 2.0 ** -20) + 2.0 ** -22)
    x["W"] = []
    for layer in range(1, L + 1):
        out = d if layer < L else 1
        a = math.sqrt(6.0 / (d + out))
        x["W"].append(a * (2.0 * torch.rand(sets, d, out, generator=gen, device="cuda") - 1.0))
    if case["kind"] == "finetune":  # the penalty sits on one node in 50 of the listed subgraphs
        hit = (part < case["listed"]) & (torch.rand(n, generator=gen, device="cuda") < 0.02)
        x["penalty"] = torch.where(hit, 3.0, 0.0).to(torch.float32)
    return x


def _context(case):
    return binding.Context(problem=case["problem"], num_layers=case["layers"], dim=case["dim"], norm=case["norm"],
                           storage=case["storage"], weight_sharing=case["shared"], train_embed=case["embed_trained"],
                           lr=case["lr"])


def _set_params(case, ctx, x):
    if case["gumbel"]:
        ctx.set_params_gumbel(x["E"], x["U"], 1.0, x["W"])
    else:
        ctx.set_params(x["E"], x["W"])


def prepare(case, seed):
    x = {k: [w.cpu().numpy() for w in v] if isinstance(v, list) else v.cpu().numpy() for k, v in _inputs(case, seed).items()}
    ctx = _context(case)
    state = {"case": case, "ctx": ctx, "x": x}
    if case["kind"] == "job":
        return state
    ctx.upload_graph(case["n"], x["rowptr"], x["col"], x["part"], case["parts"])
    _set_params(case, ctx, x)
    if case["kind"] == "finetune":
        ctx.set_linear_penalty(x["penalty"])
        ctx.forward()  # the probabilities of the subgraphs that sit out
        state["parts"] = np.arange(case["listed"], dtype=np.int32)
    if case["kind"] == "readout":
        ctx.train(case["epochs"], return_loss=False)
        ctx.forward()
        ctx.sync()
    return state


# --- one pass ----------------------------------------------------------------------------------------------------------------

def _networks(ctx):
    """The weights alone (gco_get_params without the embeddings, which stay on the GPU)."""
    sets, d, L = ctx.num_weight_sets, ctx.dim, ctx.num_layers
    Ws = [np.empty((sets, d, d if layer < L else 1), dtype=np.float32) for layer in range(1, L + 1)]
    status = ctx.lib.gco_get_params(ctx.h, None, (ctypes.c_void_p * L)(*(W.ctypes.data for W in Ws)))
    if status != binding.OK:
        raise binding.GcoError(status, ctx.last_error())
    return Ws


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "infer":
        ctx.forward()
        p = ctx.get_probs()
        total, per_part = ctx.loss()
        return {"p": p, "loss": total, "loss per subgraph": per_part}
    if kind == "readout":
        x_local, obj_local, before, after_local = ctx.round_repair(0.5, "local")
        u, v = ctx.cut_edges()
        in_conflict = np.zeros(ctx.n, dtype=np.uint8)
        for ends in ctx.conflict_edges(x_local):
            in_conflict[ends] = 1
        cross = ctx.cross_mask()
        x, obj, _, after = ctx.round_repair(0.5, "all")
        return {"x local": x_local, "x": x, "u": u, "v": v, "in conflict": in_conflict, "cross": cross,
                "counts": np.array([obj_local, before, after_local, obj, after], dtype=np.int64)}
    x = state["x"]
    if kind == "job":
        ctx.upload_graph(case["n"], x["rowptr"], x["col"], x["part"], case["parts"])
    if kind == "job" or case["embed"]:
        _set_params(case, ctx, x)
    if kind == "finetune":
        loss = ctx.train_subset(case["epochs"], state["parts"])
    else:
        loss = ctx.train(case["epochs"])
    out = {"loss": loss, "p": ctx.get_probs()}
    if case["embed"]:
        out["E"], Ws = ctx.get_params()
    else:
        Ws = _networks(ctx)
    for i, W in enumerate(Ws):
        out["W%d" % (i + 1)] = W
    if kind == "job":
        out["x"], out["size"], _, _ = ctx.round_repair(0.5, "local")
    return out


# --- what a pass cannot do without -------------------------------------------------------------------------------------------

def work(case):
    n, d, L = float(case["n"]), float(case["dim"]), case["layers"]
    nnz_all = 2.0 * case["m"]
    s = 2.0 if case["storage"] == "bf16" else 4.0
    sets = 1 if case["shared"] else case["parts"]
    part = 1.0
    if case["kind"] == "finetune":
        part = case["listed"] / case["parts"]
    nl, nnz = n * part, nnz_all * part * (case["local"] + (1 - case["local"]) / case["parts"])
    idx = 4 * nnz + 4 * nl  # the local CSR
    weights = sets * part * ((L - 1) * d * d + d) * 4
    fwd = max(1, L - 1) * (idx + nl * d * s) + (L - 1) * nl * d * s + idx + 12 * nl + weights
    loss = idx + 12 * nl
    # gradient rows in and out of every hidden layer, the activations they meet, the optimizer's state
    bwd = idx + 8 * nl + (L - 1) * (idx + 3 * nl * d * s) + 7 * weights
    bwd += (24 * nl * d + (2 * nl * d if s == 2 else 0)) if case["embed_trained"] else nl * d * s
    dense = 2 * nl * d * (d if L > 1 else 1) * max(1, L - 1)
    flops = dense + 2 * d * (nnz + nl) * max(1, L - 1)
    p_out = 4 * n
    if case["kind"] == "infer":
        return {"bytes": 2 * fwd + loss + p_out, "flops": 2 * flops}
    if case["kind"] == "readout":
        cut = nnz_all / 2 * (1 - case["local"])
        return {"bytes": 2 * (4 * nnz_all + 8 * n + 5 * n) + 4 * nnz + 4 * nnz_all + 8 * n + 8 * cut + 2 * n, "flops": nnz_all}
    w = {"bytes": case["epochs"] * (fwd + loss + bwd) + p_out + weights, "flops": case["epochs"] * 3 * flops}
    if case["embed"]:
        w["bytes"] += 4 * n * d
    if case["kind"] == "job":
        w["bytes"] += 4 * nnz_all + 12 * n + 4 * n * d + 8 * nnz + 4 * nnz_all + 8 * n
    return w


def tolerance(case):
    # About four times what the three launch forms of the scalar layer, whose sums run in different orders, differ by over two
    # passes.  Training enlarges a rounding: Adam's first steps follow the sign of a gradient however small it is.
    if case["kind"] == "readout":  # whole numbers; the probabilities they come from may differ in the last bits
        return {"rel": 0.0, "differ": 1e-3}
    if case["kind"] == "infer":
        return {"rel": 1e-3, "max": 0.05} if case["storage"] == "bf16" else {"rel": 1e-6, "max": 1e-4}
    return {"rel": 0.02, "max": 0.99, "differ": 5e-3} if case["storage"] == "bf16" else {"rel": 0.005, "max": 0.99, "differ": 1e-3}


# --- the same in 64 bits -----------------------------------------------------------------------------------------------------

def _f(x):
    """A hyper-parameter as the C ABI takes it: a 32-bit float."""
    return float(np.float32(x))


class _Exact:
    """The model of gco.h in float64 on plain torch operations."""

    def __init__(self, case, seed):
        self.case = case
        x = _inputs(case, seed)
        n, dev = case["n"], "cuda"
        order = torch.argsort(x["part"].to(torch.int64), stable=True)  # subgraph by subgraph
        place = torch.empty(n, dtype=torch.int64, device=dev)
        place[order] = torch.arange(n, device=dev)
        row = torch.repeat_interleave(torch.arange(n, device=dev), x["rowptr"][1:] - x["rowptr"][:-1])
        col = x["col"].to(torch.int64)
        inside = x["part"][row] == x["part"][col]
        self.row, self.col = place[row[inside]], place[col[inside]]
        self.order, self.place = order, place
        part = x["part"].to(torch.int64)[order]
        self.bounds = [0] + torch.cumsum(torch.bincount(part, minlength=case["parts"]), 0).tolist()
        deg = torch.bincount(self.row, minlength=n).to(torch.float64)
        if case["norm"] == "sym":
            self.sa = self.sb = (deg + 1).rsqrt()
        else:
            self.sa, self.sb = 1.0 / (deg + 1), torch.ones_like(deg)
        maxcut = case["problem"] == "maxcut"
        self.q = 2.0  # Max-Cut's coefficient, and alpha
        self.c = -deg if maxcut else -torch.ones_like(deg)
        if "penalty" in x:
            self.c = self.c + x["penalty"].to(torch.float64)[order]
        self.E = x["E"].to(torch.float64)[order]
        if case["gumbel"]:
            self.E = torch.softmax(self.E - torch.log(-torch.log(x["U"].to(torch.float64)[order])), dim=1)
        self.W = [w.to(torch.float64) for w in x["W"]]
        self.parts = list(range(case["parts"]))
        if case["kind"] == "finetune":
            self.parts = list(range(case["listed"]))
        self.state = [[torch.zeros_like(t) for t in [self.E] + self.W] for _ in range(2)]

    def neighbours(self, X):
        out = torch.zeros_like(X)
        step = max(1, (1 << 27) // (X.shape[1] if X.dim() > 1 else 1))
        for i in range(0, self.row.shape[0], step):
            out.index_add_(0, self.row[i:i + step], X[self.col[i:i + step]])
        return out

    def apply(self, X, a, b):  # diag(a) (A + I) diag(b) X
        if X.dim() > 1:
            a, b = a[:, None], b[:, None]
        Y = b * X
        return a * (Y + self.neighbours(Y))

    def per_part(self, fn, *rows):
        """fn(k, rows of subgraph k ...) of every subgraph, one after another."""
        if self.case["shared"]:
            return [fn(0, *rows)]
        return [fn(k, *(r[self.bounds[k]:self.bounds[k + 1]] for r in rows)) for k in range(self.case["parts"])]

    def forward(self):
        self.H, self.A = [self.E], []
        for W in self.W[:-1]:
            self.A.append(self.apply(self.H[-1], self.sa, self.sb))
            self.H.append(torch.relu(torch.cat(self.per_part(lambda k, a: a @ W[k], self.A[-1]))))
        self.t = torch.cat(self.per_part(lambda k, h: (h @ self.W[-1][k])[:, 0], self.H[-1]))
        self.p = torch.sigmoid(self.apply(self.t, self.sa, self.sb))
        self.s = self.neighbours(self.p)
        term = self.p * (self.c + 0.5 * self.q * self.s)
        self.loss_of = torch.stack([term[self.bounds[k]:self.bounds[k + 1]].sum() for k in range(self.case["parts"])])
        return float(self.loss_of[self.parts].sum())

    def gradients(self):
        gz = (self.c + self.q * self.s) * self.p * (1 - self.p)
        mine = torch.zeros_like(gz)
        for k in self.parts:
            mine[self.bounds[k]:self.bounds[k + 1]] = 1.0
        gt = self.apply(gz * mine, self.sb, self.sa)
        gW = [torch.stack(self.per_part(lambda k, h, g: h.T @ g[:, None], self.H[-1], gt))]
        G = torch.cat(self.per_part(lambda k, g: g[:, None] * self.W[-1][k][:, 0], gt))
        for layer in range(len(self.W) - 2, -1, -1):
            G = G * (self.H[layer + 1] > 0)
            gW.insert(0, torch.stack(self.per_part(lambda k, a, g: a.T @ g, self.A[layer], G)))
            W = self.W[layer]
            G = self.apply(torch.cat(self.per_part(lambda k, g: g @ W[k].T, G)), self.sb, self.sa)
        return [G] + gW

    def step(self, count):
        grads = self.gradients()
        lr, b1, b2, eps = _f(self.case["lr"]), _f(0.9), _f(0.999), _f(1e-8)
        live = torch.zeros(self.case["n"], 1, dtype=torch.float64, device="cuda")
        on = torch.zeros(self.W[0].shape[0], 1, 1, dtype=torch.float64, device="cuda")
        for k in self.parts:
            live[self.bounds[k]:self.bounds[k + 1]] = 1.0
            on[0 if self.case["shared"] else k] = 1.0
        for i, g in enumerate(grads):
            if i == 0 and not self.case["embed_trained"]:
                continue
            t = self.E if i == 0 else self.W[i - 1]
            m, v = self.state[0][i], self.state[1][i]
            m.mul_(b1).add_(g, alpha=1 - b1)
            v.mul_(b2).addcmul_(g, g, value=1 - b2)
            t -= (live if i == 0 else on) * lr * (m / (1 - b1 ** count)) / (torch.sqrt(v / (1 - b2 ** count)) + eps)


def exact(case, seed):
    if case["kind"] == "readout":
        return None
    with torch.no_grad():
        e = _Exact(case, seed)
        if case["kind"] == "infer":
            total = e.forward()
            return {"p": e.p[e.place], "loss": total, "loss per subgraph": e.loss_of}
        loss = []
        for i in range(case["epochs"]):
            loss.append(e.forward())
            e.step(i + 1)
        p = e.p[e.place]
        out = {"loss": torch.tensor(loss, dtype=torch.float64), "p": p}
        if case["embed"]:
            out["E"] = e.E[e.place]
        for i, W in enumerate(e.W):
            out["W%d" % (i + 1)] = W
        if case["kind"] == "job":
            out["x"], out["size"] = None, None
        return out
