"""Timed cases: the work a CPRA program has this library do, over the range of
its sizes, through the public Python entry points (``CPRASolver``, ``api`` and
``WarmStartNet``).

A case is a dict of plain values.  ``kind`` says which call it is:

* ``train``    -- replayed CPRA training steps of a solver (forward, loss,
                  backward, Adam), returning the logits, dR/dZ, the gradient
                  and the per-graph loss terms.  A network with hidden ReLU layers is
                  kept small or has its encoder frozen: between two correctly
                  rounded runs a hidden unit on the edge of its ReLU may fall
                  either way, and at 1e7 units one does.  The large steps
                  therefore train the embedding and the output layer.
* ``layer``    -- forward and backward of one message-passing layer (a
                  one-layer model), alone or with one weight set per graph.
* ``forward``  -- the logits of a whole network.
* ``decode``   -- rounding and exact evaluation of all heads.
* ``diversity``-- pairwise Hamming matrix, histogram and distinct count.
* ``warm``     -- warm-start inference: structural features and the BF16 network.

Graphs are random near-regular graphs or block-diagonal unions of Erdos-Renyi
graphs, drawn on the GPU from the seed.  GEMM plans are the library's own
choice, as in ``solve``.
"""

import math

import numpy as np
import torch

from paper_2402_02190_amd import api
from paper_2402_02190_amd.solver import CPRAConfig, CPRASolver, gamma_schedule
from paper_2402_02190_amd.warmstart import WarmStartNet

GAMMA = (-2.0, 0.1)


def listed():
    return [
        # The smallest problem of the presets (3-regular, N = 100, GCN 2x32, S = 10): ten
        # replayed steps, bound by launches and latency.
        dict(name="train_100", kind="train", n=100, degree=3, graphs=1, problem="mis",
             layer="gcn", layers=2, hidden=32, S=10, nu=0.0, weights="", frozen=0, steps=10),
        # 27 MaxCut instances of one 3-regular structure, one per head (the multi-instance
        # comparison's joint run): S = 27 leaves every head row unaligned.
        dict(name="train_instances", kind="train", n=2000, degree=3, graphs=1, problem="maxcut",
             layer="gcn", layers=2, hidden=64, S=27, nu=0.0, weights="edge", frozen=0, steps=1),
        # Fine-tuning 500 fresh heads on a frozen encoder (the second stage of the two-stage
        # scheme, weighted MIS on a 20-regular graph of 8,000 nodes, GraphSAGE 2x256).
        dict(name="finetune_heads", kind="train", n=8000, degree=20, graphs=1, problem="mis",
             layer="sage", layers=2, hidden=256, S=500, nu=0.0, weights="node", frozen=1, steps=1),
        # The batched workload: 256 Erdos-Renyi graphs of 500..5000 nodes, MaxCut with the
        # diversity term, the embedding and the output layer (64 -> 32) trained.
        dict(name="train_batch", kind="train", n=2750, degree=7, graphs=256, problem="maxcut",
             layer="gcn", layers=1, hidden=64, S=32, nu=0.1, weights="", frozen=0, steps=1),
        # The embedding and output layer (128 -> 64) of the 20-regular N = 100,000 workload.
        dict(name="train_100k", kind="train", n=100_000, degree=20, graphs=1, problem="mis",
             layer="gcn", layers=1, hidden=128, S=64, nu=0.0, weights="", frozen=0, steps=1),
        # A hidden GraphSAGE layer of the 5-regular N = 10,000 workload, both directions.
        dict(name="layer_10k", kind="layer", n=10_000, degree=5, graphs=1, layer="sage",
             d_in=256, d_out=256, per_graph=0),
        # A hidden GCN layer of the 20-regular N = 100,000 workload, both directions.
        dict(name="layer_100k", kind="layer", n=100_000, degree=20, graphs=1, layer="gcn",
             d_in=128, d_out=128, per_graph=0),
        # A hidden layer of 32 Erdos-Renyi graphs, every graph with its own weights.
        dict(name="layer_per_graph", kind="layer", n=2750, degree=7, graphs=32, layer="gcn",
             d_in=64, d_out=64, per_graph=1),
        # The logits of the whole N = 100,000 network (3-layer GCN 128, S = 64).
        dict(name="forward_100k", kind="forward", n=100_000, degree=20, graphs=1, layer="gcn",
             layers=3, hidden=128, S=64),
        # Rounding and scoring its 64 heads (done whenever a run reports its solutions).
        dict(name="decode_100k", kind="decode", n=100_000, degree=20, graphs=1, problem="mis", S=64),
        # Diversity of the 100 solutions of the N = 10,000 workload.
        dict(name="diversity_10k", kind="diversity", n=10_000, S=100),
        # A warm start for an unseen 5-regular graph of 50,000 nodes (BF16 network 3x64, S = 32).
        dict(name="warm_50k", kind="warm", n=50_000, degree=5, graphs=1, layers=3, hidden=64, S=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "shallow", "batch", "finetune", "layer", "layer", "layer",
                       "per_graph", "forward", "decode", "diversity", "warm"])
    degree = rng.choice([3, 4, 5, 7, 10, 15, 20])
    widths = [32, 48, 64, 96, 100, 128, 33, 57, 250, 256]
    heads = [8, 10, 27, 32, 50, 64, 100, 128, 200]
    if kind == "train":
        hidden = rng.choice([16, 32, 33, 48, 64])
        n = _log_int(rng, 60, 120_000 // hidden)
        weights = rng.choice(["", "", "edge", "node"])
        return dict(kind="train", n=n, degree=min(degree, 10), graphs=1,
                    problem="mis" if weights == "node" else rng.choice(["mis", "maxcut"]),
                    layer=rng.choice(["gcn", "sage"]), layers=2, hidden=hidden, S=rng.choice(heads),
                    nu=rng.choice([0.0, 0.1]), weights=weights, frozen=0, steps=rng.choice([1, 5]))
    if kind == "shallow":
        return dict(kind="train", n=_log_int(rng, 3000, 100_000), degree=degree, graphs=1,
                    problem=rng.choice(["mis", "maxcut"]), layer=rng.choice(["gcn", "sage"]),
                    layers=1, hidden=rng.choice([32, 64, 100, 128]), S=rng.choice([10, 32, 50, 64]),
                    nu=rng.choice([0.0, 0.1]), weights="", frozen=0, steps=1)
    if kind == "batch":
        return dict(kind="train", n=_log_int(rng, 300, 2750), degree=rng.choice([4, 5, 6, 7, 8]),
                    graphs=_log_int(rng, 2, 200), problem="maxcut", layer=rng.choice(["gcn", "sage"]),
                    layers=1, hidden=rng.choice([32, 64]), S=rng.choice([16, 27, 32]), nu=0.1,
                    weights="", frozen=0, steps=1)
    if kind == "finetune":
        return dict(kind="train", n=_log_int(rng, 500, 8000), degree=degree, graphs=1, problem="mis",
                    layer="sage", layers=2, hidden=rng.choice([64, 128, 256]),
                    S=rng.choice([100, 201, 330, 500]), nu=0.0, weights="node", frozen=1, steps=1)
    if kind == "layer":
        return dict(kind="layer", n=_log_int(rng, 300, 100_000), degree=degree, graphs=1,
                    layer=rng.choice(["gcn", "sage"]), d_in=rng.choice(widths[:7]),
                    d_out=rng.choice(widths[:7]), per_graph=0) if rng.random() < 0.6 else \
            dict(kind="layer", n=_log_int(rng, 300, 20_000), degree=degree, graphs=1,
                 layer=rng.choice(["gcn", "sage"]), d_in=rng.choice(widths),
                 d_out=rng.choice(widths), per_graph=0)
    if kind == "per_graph":
        return dict(kind="layer", n=_log_int(rng, 300, 2750), degree=rng.choice([4, 5, 6, 7, 8]),
                    graphs=_log_int(rng, 2, 48), layer=rng.choice(["gcn", "sage"]),
                    d_in=rng.choice([32, 57, 64]), d_out=rng.choice([27, 32, 64]), per_graph=1)
    if kind == "forward":
        return dict(kind="forward", n=_log_int(rng, 1000, 100_000), degree=degree, graphs=1,
                    layer=rng.choice(["gcn", "sage"]), layers=rng.choice([2, 3]),
                    hidden=rng.choice([32, 64, 100, 128]), S=rng.choice([10, 27, 32, 50, 64]))
    if kind == "decode":
        graphs = rng.choice([1, 1, 1, 8])
        return dict(kind="decode", n=_log_int(rng, 500, 100_000) // graphs, degree=degree,
                    graphs=graphs, problem=rng.choice(["mis", "maxcut"]),
                    S=rng.choice([10, 27, 32, 50, 64])) \
            if rng.random() < 0.7 else \
            dict(kind="decode", n=_log_int(rng, 500, 20_000), degree=degree, graphs=1,
                 problem=rng.choice(["mis", "maxcut"]), S=rng.choice([100, 128, 200, 333]))
    if kind == "diversity":
        return dict(kind="diversity", n=_log_int(rng, 100, 10_000), S=rng.choice([7, 10, 32, 64, 100]))
    return dict(kind="warm", n=_log_int(rng, 1000, 50_000), degree=min(degree, 10), graphs=1,
                layers=rng.choice([2, 3]), hidden=rng.choice([32, 64]), S=rng.choice([32, 64]))


# ---- inputs -----------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _graph(c, gen):
    """(row_ptr, col_idx, graph_ptr, rows) on the GPU: a near-regular graph (union of
    random permutations and, for an odd degree, a matching), or a union of
    Erdos-Renyi graphs of about n/5 .. 9n/5 nodes and mean degree 4/7 .. 10/7 of
    `degree`; loops and repeated edges dropped, rows sorted, symmetric."""
    dev, G, d = "cuda", c["graphs"], c["degree"]
    if G == 1:
        n = c["n"]
        ptr = torch.tensor([0, n], device=dev)
        us, vs = [], []
        ids = torch.arange(n, device=dev)
        for _ in range(d // 2):
            us.append(ids)
            vs.append(torch.randperm(n, generator=gen, device=dev))
        if d % 2:
            p = torch.randperm(n, generator=gen, device=dev)[: n - n % 2].view(-1, 2)
            us.append(p[:, 0])
            vs.append(p[:, 1])
        u, v = torch.cat(us), torch.cat(vs)
    else:
        x = np.random.default_rng(c["n"]).random(G)  # the sizes belong to the case
        sizes = torch.from_numpy((c["n"] * (0.2 + 1.6 * x)).astype(np.int64)).to(dev)
        deg = d * (4 / 7 + 6 / 7 * torch.rand(G, generator=gen, device=dev))
        ptr = torch.zeros(G + 1, dtype=torch.long, device=dev)
        ptr[1:] = sizes.cumsum(0)
        n = int(ptr[-1])
        m = (sizes * deg / 2).long()
        who = torch.repeat_interleave(torch.arange(G, device=dev), m)
        u, v = (ptr[who] + (torch.rand(who.numel(), generator=gen, device=dev, dtype=torch.float64)
                            * sizes[who]).long() for _ in range(2))
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.minimum(u, v) * n + torch.maximum(u, v))
    lo, hi = key // n, key % n
    both = torch.sort(torch.cat([lo * n + hi, hi * n + lo])).values
    rows, cols = both // n, both % n
    row_ptr = torch.zeros(n + 1, dtype=torch.long, device=dev)
    row_ptr[1:] = torch.bincount(rows, minlength=n).cumsum(0)
    return row_ptr, cols, ptr, rows


def _device_graph(row_ptr, cols, ptr):
    i32 = [t.to(torch.int32).cpu().numpy() for t in (row_ptr, cols, ptr)]
    return api.DeviceGraph(i32[0], i32[1], None, i32[2] if len(i32[2]) > 2 else None)


def _dims(layers, d_in, hidden, d_out):
    w = [d_in] + [hidden] * (layers - 1) + [d_out]
    return list(zip(w[:-1], w[1:]))


def _params(kind, n, dims, groups, gen):
    """Flat float32 parameters: the embedding, then per layer Ws, Wn and (SAGE) b."""
    parts = [torch.randn(n * dims[0][0], generator=gen, device="cuda")]
    for i, o in dims:
        b = 1 / math.sqrt(i)
        for _ in range(2):
            parts.append((2 * torch.rand(groups * o * i, generator=gen, device="cuda") - 1) * b)
        if kind == "sage":
            parts.append((2 * torch.rand(groups * o, generator=gen, device="cuda") - 1) * b)
    return torch.cat(parts)


def _edge_weights(rows, cols, n, S, gen):
    """Symmetric integer weights U{1..4}, one column per head."""
    lo, hi = torch.minimum(rows, cols), torch.maximum(rows, cols)
    _, eid = torch.unique(lo * n + hi, return_inverse=True)
    w = torch.randint(1, 5, (int(eid.max()) + 1 if eid.numel() else 1, S), generator=gen, device="cuda")
    return w[eid].float()


def _solutions(rows, cols, n, S, gen):
    """Logits of trained heads: independent sets (a node is in where its random priority
    beats its neighbours'), a quarter of the heads at random (their penalty is too small)."""
    pr = torch.rand(n, S, generator=gen, device="cuda")
    best = torch.zeros(n, S, device="cuda").scatter_reduce_(
        0, rows[:, None].expand(-1, S), pr[cols], "amax", include_self=True)
    x = pr > best
    loose = S // 4
    x[:, :loose] = torch.rand(n, loose, generator=gen, device="cuda") > 0.5
    size = 2 + 10 * torch.rand(n, S, generator=gen, device="cuda")
    return torch.where(x, size, -size)


def _inputs(c, seed):
    """Everything drawn for a case, shared by prepare and exact."""
    gen = _gen(seed)
    k = c["kind"]
    d = {}
    if k == "diversity":
        n, S = c["n"], c["S"]
        base = torch.rand(n, max(1, S // 2), generator=gen, device="cuda") < 0.4
        pick = torch.randint(0, base.shape[1], (S,), generator=gen, device="cuda")
        flip = torch.rand(n, S, generator=gen, device="cuda") < 0.02
        flip[:, torch.rand(S, generator=gen, device="cuda") < 0.3] = False
        d["X"] = (base[:, pick] ^ flip).to(torch.uint8)
        return d
    row_ptr, cols, ptr, rows = _graph(c, gen)
    n = int(row_ptr.numel() - 1)
    d.update(row_ptr=row_ptr, cols=cols, ptr=ptr, rows=rows, n=n)
    if k == "train":
        d["dims"] = _dims(c["layers"], c["hidden"], c["hidden"], c["S"])
        d["params"] = _params(c["layer"], n, d["dims"], 1, gen)
        if c["weights"] == "edge":
            d["edge_weight"] = _edge_weights(rows, cols, n, c["S"], gen)
        if c["weights"] == "node":
            d["node_weight"] = torch.rand(n, c["S"], generator=gen, device="cuda")
        d["lam"] = np.logspace(-1.0, 1.0, c["S"]).astype(np.float32) if c["problem"] == "mis" else None
    elif k == "layer":
        d["dims"] = [(c["d_in"], c["d_out"])]
        d["params"] = _params(c["layer"], n, d["dims"], c["graphs"] if c["per_graph"] else 1, gen)
        d["dZ"] = torch.randn(n, c["d_out"], generator=gen, device="cuda")
    elif k == "forward":
        d["dims"] = _dims(c["layers"], c["hidden"], c["hidden"], c["S"])
        d["params"] = _params(c["layer"], n, d["dims"], 1, gen)
    elif k == "decode":
        d["Z"] = _solutions(rows, cols, n, c["S"], gen)
    else:
        d["dims"] = _dims(c["layers"], 16, c["hidden"], c["S"])
        d["rand"] = 2 * torch.rand(n, 14, generator=gen, device="cuda") - 1
        d["weights"] = [tuple((2 * torch.rand(*s, generator=gen, device="cuda") - 1) / math.sqrt(i)
                              for s in ((o, i), (o, i), (o,))) for i, o in d["dims"]]
    return d


def _layer_kind(c):
    return api.SAGE if c["layer"] == "sage" else api.GCN


def prepare(case, seed):
    c, d = case, _inputs(case, seed)
    k = c["kind"]
    s = {"case": c}
    if k == "diversity":
        n, S = c["n"], c["S"]
        s.update(X=d["X"], D=torch.empty(S, S, dtype=torch.int32, device="cuda"),
                 hist=torch.empty(n + 1, dtype=torch.int64, device="cuda"),
                 unique=torch.empty(1, dtype=torch.int32, device="cuda"))
        return s
    dg = _device_graph(d["row_ptr"], d["cols"], d["ptr"])
    n = d["n"]
    s["graph"] = dg
    if k == "train":
        cfg = CPRAConfig(problem=c["problem"], layer_kind=c["layer"], n_layers=c["layers"],
                         hidden=c["hidden"], S=c["S"], nu=c["nu"], gamma_start=GAMMA[0],
                         gamma_end=GAMMA[1], T=2000, train_from_layer=c["frozen"])
        host = {w: d[w].cpu().numpy() for w in ("node_weight", "edge_weight") if w in d}
        sol = CPRASolver(dg, cfg, d["lam"], **host)
        sol.params.copy_(d["params"])
        if c["frozen"]:
            sol.forward()  # saves the frozen prefix, which the steps start from
            sol.set_reuse_frozen_prefix(True)
        sol.capture(steps_per_graph=c["steps"])
        s["sol"] = sol
    elif k in ("layer", "forward"):
        hidden = d["dims"][-1][0]
        s["cfg"] = api.make_model_cfg(_layer_kind(c), len(d["dims"]), d["dims"][0][0], hidden,
                                      d["dims"][-1][1],
                                      weight_groups=c["graphs"] if c.get("per_graph") else 0)
        s["params"] = d["params"]
        s["Z"] = torch.empty(n, d["dims"][-1][1], device="cuda")
        s["ws"] = torch.empty(max(256, api.model_workspace_bytes(dg, s["cfg"])), dtype=torch.uint8,
                              device="cuda")
        if k == "layer":
            s["dZ"] = d["dZ"]
            s["grads"] = torch.empty_like(d["params"])
    elif k == "decode":
        G, S = c["graphs"], c["S"]
        i64 = dict(dtype=torch.int64, device="cuda")
        s.update(Z=d["Z"], X=torch.empty(n, S, dtype=torch.uint8, device="cuda"),
                 value=torch.empty(G * S, **i64), viol=torch.empty(G * S, **i64),
                 ham=torch.empty(G, **i64),
                 ws=torch.empty(api.round_eval_workspace_bytes(dg, S), dtype=torch.uint8, device="cuda"))
    else:
        net = WarmStartNet(c["layers"], 16, c["hidden"], c["S"], 14)
        net.params.copy_(torch.cat([t.reshape(-1) for w in d["weights"] for t in w]))
        s.update(net=net, rand=d["rand"], ws=net.workspace(dg),
                 feat=torch.empty(n, 16, dtype=torch.int16, device="cuda"),
                 tri=torch.empty(n, dtype=torch.int64, device="cuda"))
    return s


def run(state):
    s = state
    k = s["case"]["kind"]
    if k == "train":
        sol = s["sol"]
        sol.run(s["case"]["steps"])
        g0 = sol.offsets[1 + 3 * sol.cfg.train_from_layer] if sol.cfg.train_from_layer else 0
        return {"Z": sol.Z, "dZ": sol.dZ, "grads": sol.grads[g0:], "terms": sol.terms}
    if k == "layer":
        api.model_forward(s["graph"], s["cfg"], s["params"], s["Z"], s["ws"])
        api.model_backward(s["graph"], s["cfg"], s["params"], s["dZ"], s["grads"], s["ws"])
        return {"Z": s["Z"], "grads": s["grads"]}
    if k == "forward":
        return {"Z": api.model_forward(s["graph"], s["cfg"], s["params"], s["Z"], s["ws"])}
    if k == "decode":
        problem = api.MIS if s["case"]["problem"] == "mis" else api.MAXCUT
        api.round_eval(s["graph"], problem, s["Z"], s["X"], s["value"], s["viol"], None, s["ham"],
                       ws=s["ws"])
        return {"X": s["X"], "value": s["value"], "violations": s["viol"], "pair_hamming": s["ham"]}
    if k == "diversity":
        api.pairwise_hamming(s["X"], s["D"], s["hist"], s["unique"])
        return {"D": s["D"], "hist": s["hist"], "unique": s["unique"]}
    net = s["net"]
    api.node_features(s["graph"], net.in_dim, s["rand"], s["feat"], s["tri"])
    return {"feat": s["feat"], "triangles": s["tri"], "Zw": net.forward(s["graph"], s["feat"], s["ws"])}


# ---- work -------------------------------------------------------------------
def _sizes(c):
    n = c["n"] * c["graphs"]
    return n, n * c["degree"]


def work(case):
    c = case
    k = c["kind"]
    if k == "diversity":
        S = c["S"]
        return {"bytes": c["n"] * S + 4 * S * S + 8 * (c["n"] + 1), "flops": 0}
    n, nnz = _sizes(c)
    csr = 4 * (n + nnz)
    if k == "train":
        dims = _dims(c["layers"], c["hidden"], c["hidden"], c["S"])
        S = c["S"]
        if c["frozen"]:  # the saved input of the last layer and its aggregate
            i, o = dims[-1]
            per = 28 * (2 * i * o + o) + 4 * n * i * (1 if o < i else 2) + 8 * n * S
            fl = 8 * n * i * o
        else:
            w = sum(2 * i * o + (o if c["layer"] == "sage" else 0) for i, o in dims)
            per = 28 * (n * c["hidden"] + w) + 8 * n * S
            fl = sum(12 * n * i * o for i, o in dims)
        fl += 2 * nnz * S
        per += csr + (4 * nnz * S if c["weights"] == "edge" else 0) + (4 * n * S if c["weights"] == "node" else 0)
        return {"bytes": c["steps"] * per, "flops": c["steps"] * fl}
    if k == "layer":
        i, o = c["d_in"], c["d_out"]
        w = 2 * i * o * (c["graphs"] if c["per_graph"] else 1)
        return {"bytes": csr + 4 * n * (2 * i + 2 * o) + 8 * w,
                "flops": 12 * n * i * o + 2 * nnz * (min(i, o) * 2)}
    if k == "forward":
        dims = _dims(c["layers"], c["hidden"], c["hidden"], c["S"])
        return {"bytes": csr + 4 * n * (dims[0][0] + c["S"]) + sum(8 * i * o for i, o in dims),
                "flops": sum(4 * n * i * o + nnz * min(i, o) for i, o in dims)}
    if k == "decode":
        return {"bytes": csr + 5 * n * c["S"] + 16 * c["graphs"] * c["S"], "flops": 0}
    dims = _dims(c["layers"], 16, c["hidden"], c["S"])
    return {"bytes": csr + n * (14 * 4 + 16 * 2 + 8 + 4 * c["S"]) + sum(8 * i * o for i, o in dims),
            "flops": sum(4 * n * i * o + nnz * i for i, o in dims)}


# ---- the same in 64 bits -------------------------------------------------------
def _mean(d, X):
    """M X over the CSR, rows with no neighbour 0."""
    Y = torch.zeros_like(X).index_add_(0, d["rows"], X[d["cols"]])
    return Y * d["inv_deg"][:, None]


def _mean_rows(d, X):
    return _Mean.apply(X, d)


class _Mean(torch.autograd.Function):
    @staticmethod
    def forward(ctx, X, d):
        ctx.d = d
        return _mean(d, X)

    @staticmethod
    def backward(ctx, dY):
        d = ctx.d  # M^T = A D^-1 on a symmetric pattern
        dY = dY * d["inv_deg"][:, None]
        return torch.zeros_like(dY).index_add_(0, d["rows"], dY[d["cols"]]), None


def _network(d, flat, n, dims, kind, groups=1):
    at = n * dims[0][0]
    H = flat[:at].view(n, -1)
    for k, (i, o) in enumerate(dims):
        ws = flat[at: at + groups * o * i].view(groups, o, i)
        wn = flat[at + groups * o * i: at + 2 * groups * o * i].view(groups, o, i)
        at += 2 * groups * o * i
        b = None
        if kind == "sage":
            b = flat[at: at + groups * o].view(groups, o)
            at += groups * o
        A = _mean_rows(d, H)
        if groups == 1:
            Y = H @ ws[0].T + A @ wn[0].T + (0 if b is None else b[0])
        else:
            p = d["ptr"].tolist()
            Y = torch.cat([H[x:y] @ ws[g].T + A[x:y] @ wn[g].T + (0 if b is None else b[g])
                           for g, (x, y) in enumerate(zip(p[:-1], p[1:]))])
        H = Y if k == len(dims) - 1 else torch.relu(Y)
    return H


def _terms(c, d, P):
    """Per-graph loss terms [G, S + 2] of the relaxed solutions P."""
    n, S = P.shape
    w = d["edge_weight"].double() if "edge_weight" in d else None
    nb = P[d["cols"]] if w is None else w * P[d["cols"]]
    AP = torch.zeros_like(P).index_add(0, d["rows"], nb)
    if c["problem"] == "mis":
        lam = torch.from_numpy(d["lam"]).to(P.device).double()
        nw = d["node_weight"].double() if "node_weight" in d else 1.0
        per = P * (0.5 * lam * AP - nw)
    else:
        if w is None:
            deg = (d["row_ptr"][1:] - d["row_ptr"][:-1]).double()[:, None]
        else:
            deg = torch.zeros_like(P).index_add(0, d["rows"], w)
        per = P * (AP - deg)
    phi = (1 - (2 * P - 1) ** 2).sum(1, keepdim=True)
    psi = -S * P.std(dim=1, unbiased=False, keepdim=True)
    graph = torch.repeat_interleave(torch.arange(d["ptr"].numel() - 1, device=P.device),
                                    d["ptr"][1:] - d["ptr"][:-1])
    cols = torch.cat([per, phi, psi], 1)
    return torch.zeros(d["ptr"].numel() - 1, S + 2, dtype=P.dtype, device=P.device).index_add(0, graph, cols)


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    k = c["kind"]
    if k in ("decode", "diversity"):
        return None  # whole numbers
    deg = (d["row_ptr"][1:] - d["row_ptr"][:-1]).double()
    d["inv_deg"] = torch.where(deg > 0, 1 / deg.clamp_min(1), torch.zeros_like(deg))
    n = d["n"]
    if k == "warm":
        # in full precision (the network itself keeps its activations in bfloat16)
        tri = torch.zeros(n, dtype=torch.float64, device="cuda")  # near-regular: a handful in all
        H = torch.cat([deg[:, None] / 16, tri[:, None], d["rand"].double()], 1)
        for i, (ws, wn, b) in enumerate(d["weights"]):
            H = H @ ws.double().T + _mean(d, H) @ wn.double().T + b.double()
            H = H if i == len(d["weights"]) - 1 else torch.relu(H)
        return {"feat": None, "triangles": None, "Zw": H}
    flat = d["params"].double()
    if k == "forward":
        return {"Z": _network(d, flat, n, d["dims"], c["layer"])}
    flat.requires_grad_(True)
    if k == "layer":
        Z = _network(d, flat, n, d["dims"], c["layer"], c["graphs"] if c["per_graph"] else 1)
        Z.backward(d["dZ"].double())
        return {"Z": Z.detach(), "grads": flat.grad}
    m, v = torch.zeros_like(flat), torch.zeros_like(flat)
    g0 = 0
    if c["frozen"]:
        g0 = n * d["dims"][0][0]
        for i, o in d["dims"][: c["frozen"]]:
            g0 += 2 * i * o + (o if c["layer"] == "sage" else 0)
    for t in range(c["steps"]):
        flat = flat.detach().requires_grad_(True)
        gamma = gamma_schedule(t, 2000, *GAMMA)
        Z = _network(d, flat, n, d["dims"], c["layer"])
        Z.retain_grad()
        T = _terms(c, d, torch.sigmoid(Z))
        S = c["S"]
        R = (T[:, :S].sum() + gamma * T[:, S].sum()) + (c["nu"] * T[:, S + 1].sum() if c["nu"] else 0.0)
        R.backward()
        g = flat.grad.clone()
        g[:g0] = 0
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        step = 1e-3 * (m / (1 - 0.9 ** (t + 1))) / ((v / (1 - 0.999 ** (t + 1))).sqrt() + 1e-8)
        flat = flat.detach() - torch.where(g == 0, torch.zeros_like(step), step) if c["frozen"] \
            else flat.detach() - step
    return {"Z": Z.detach(), "dZ": Z.grad, "grads": g[g0:], "terms": T.detach()}
