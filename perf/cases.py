"""Workloads whose time matters to a program built on this library.

Each case is one relational-GNN layer (or a two-layer model) on a synthetic heterogeneous graph: a serving call
(forward only) or a training pass (forward and backward), called through the C ABI binding or the autograd front
end as a program would.  Graph shapes follow the library's own workloads: relation frequencies are Zipf distributed,
in-degrees follow a capped power law, sources are uniform, and in HGT graphs every relation ties a source node type
to a destination node type.  The graph handle, the parameters and the buffers are made once (`prepare`); a pass
(`run`) is the layer calls alone.
"""
import math

import numpy as np
import torch

from paper_2412_04747_amd import autograd as A
from paper_2412_04747_amd import binding as B

SLOPE = 0.2


def _case(name, layer, mode, nodes, rels, edges, d_in, d_out, dtype="f32", api="autograd", heads=1, types=1, tied=True,
          zipf=1.1, hub=0.05, self_loop=False, relu=False, mu=False):
    c = dict(layer=layer, mode=mode, nodes=nodes, rels=rels, edges=edges, d_in=d_in, d_out=d_out, dtype=dtype, api=api,
             heads=heads, types=types, tied=tied, zipf=zipf, hub=hub, self_loop=self_loop, relu=relu, mu=mu)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: scoring a small graph online with one RGCN layer; a few launches, all latency
        _case("rgcn_infer_tiny", "rgcn", "infer", 1000, 8, 10000, 32, 32, api="abi", zipf=0.0, hub=0.0),
        # training one RGAT layer on a small graph (tens of thousands of nodes): many short kernels in a row
        _case("rgat_train_small", "rgat", "train", 20000, 50, 200000, 64, 64),
        # full-graph training step of a two-layer RGAT model, loss and all, on a graph of the same kind
        _case("rgat_model_step", "model", "train", 50021, 47, 500119, 64, 64),
        # the flagship: RGAT forward and backward on a graph of a million nodes and ten million edges
        _case("rgat_train_large", "rgat", "train", 1000000, 200, 10000000, 64, 64, api="abi", zipf=1.2),
        # serving a mid-size graph: RGAT forward with nothing kept for a backward pass, sizes of no round number
        _case("rgat_infer_mid", "rgat", "infer", 300007, 37, 3000017, 64, 64, api="abi"),
        # multi-head attention, training, mid-size
        _case("rgat_heads_train", "rgat", "train", 250013, 101, 2500003, 64, 64, heads=4),
        # the widest fp32 layer: 128 features, training
        _case("rgat_wide_train", "rgat", "train", 200003, 60, 2000003, 128, 128),
        # RGCN as it is usually trained: self-loop weight, 1/c normalisation, ReLU, input narrower than the output
        _case("rgcn_train_mid", "rgcn", "train", 120011, 45, 1200007, 32, 64, self_loop=True, relu=True),
        # knowledge-graph RGCN in bf16: many relations, most of them small, most (source, relation) pairs with one edge
        _case("rgcn_train_kg_bf16", "rgcn", "train", 2500000, 500, 16000000, 128, 128, dtype="bf16", api="abi", zipf=1.0, hub=0.02),
        # HGT training in bf16 on a large typed graph: four heads, every relation tied to its node types
        _case("hgt_train_large_bf16", "hgt", "train", 2000000, 30, 20000000, 128, 128, dtype="bf16", api="abi", heads=4, types=8, zipf=1.0),
        # the same layer on a graph of a tenth of that size
        _case("hgt_train_mid_bf16", "hgt", "train", 200017, 17, 2000029, 128, 128, dtype="bf16", api="abi", heads=4, types=5, zipf=1.0),
        # HGT training in fp32 on a small typed graph, with the prior on (relation, head)
        _case("hgt_train_small", "hgt", "train", 30011, 12, 300007, 64, 64, heads=4, types=4, zipf=1.0, mu=True),
    ]


def draw(rng):
    kind = rng.choice(["rgcn_infer", "rgcn_train", "rgcn_bf16", "rgat_infer", "rgat_train", "hgt_train", "hgt_bf16", "model"])
    top = {"rgcn_bf16": 8e6, "rgat_train": 4e6, "hgt_train": 1.5e6, "hgt_bf16": 8e6, "model": 1.5e6}.get(kind, 6e6)
    low = 1e4
    edges = int(math.exp(rng.uniform(math.log(low), math.log(top))))
    nodes = max(64, int(edges / rng.uniform(5.0, 15.0)))
    rels = int(math.exp(rng.uniform(math.log(4), math.log(500 if "hgt" not in kind else 60))))
    zipf, hub = rng.choice([1.0, 1.1, 1.2]), rng.choice([0.02, 0.05])
    layer = kind.split("_")[0]
    mode = "infer" if kind.endswith("infer") else "train"
    if layer == "hgt":
        bf16 = kind == "hgt_bf16"
        d, heads = (128, rng.choice([4, 8])) if bf16 else rng.choice([(32, 2), (64, 4), (64, 2), (128, 4)])
        return _case(None, layer, mode, nodes, rels, edges, d, d, dtype="bf16" if bf16 else "f32", api="abi" if bf16 else "autograd",
                     heads=heads, types=rng.randint(2, 8), tied=rng.random() < 0.85, zipf=zipf, hub=hub, mu=rng.random() < 0.5)
    if kind == "rgcn_bf16":
        d = rng.choice([128, 128, 128, 64])
        return _case(None, layer, mode, nodes, rels, edges, d, d, dtype="bf16", api="abi", zipf=zipf, hub=hub,
                     self_loop=rng.random() < 0.3, relu=rng.random() < 0.3)
    d_in, d_out = rng.choice([(32, 32), (64, 64), (64, 64), (128, 128), (32, 64), (64, 32)])
    if layer == "rgcn":
        loop = rng.random() < 0.6
        return _case(None, layer, mode, nodes, rels, edges, d_in, d_out, api="abi" if mode == "infer" else "autograd", zipf=zipf,
                     hub=hub, self_loop=loop, relu=loop)
    if layer == "model":
        return _case(None, layer, mode, nodes, rels, edges, 64, 64, zipf=zipf, hub=hub)
    heads = rng.choice([1, 1, 2, 4]) if d_out >= 64 else 1
    return _case(None, layer, mode, nodes, rels, edges, d_in, d_out, api="abi" if mode == "infer" else rng.choice(["autograd", "abi"]),
                 heads=heads, zipf=zipf, hub=hub)


# ---------------------------------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 31) + 17)
    return g


def _pick(gen, weights, n):
    """n indices drawn with probability proportional to weights (float64)."""
    cdf = torch.cumsum(weights, 0)
    u = torch.rand(n, device="cuda", dtype=torch.float64, generator=gen) * cdf[-1]
    return torch.searchsorted(cdf, u, right=True).clamp_(max=len(weights) - 1)


def _ints(gen, lo, hi, n):
    return torch.randint(lo, hi, (n,), device="cuda", generator=gen)


def _rel_probs(rels, zipf):
    p = 1.0 / np.arange(1, rels + 1, dtype=np.float64) ** zipf
    return p / p.sum()


def _popular(gen, nodes, n, hub):
    """Destinations with power-law popularity (exponent 2.1); the most popular expects hub * nodes edges or fewer."""
    if hub <= 0:
        return _ints(gen, 0, nodes, n)
    u = torch.rand(nodes, device="cuda", dtype=torch.float64, generator=gen)
    raw = (1.0 - u) ** (-1.0 / 1.1)
    cap = max(hub * nodes, 8.0)
    lo, hi = 1.0, float(raw.max())
    if n * hi / float(raw.sum()) > cap:
        for _ in range(30):
            mid = 0.5 * (lo + hi)
            if n * mid / float(raw.clamp(max=mid).sum()) > cap:
                hi = mid
            else:
                lo = mid
        raw = raw.clamp(max=0.5 * (lo + hi))
    return _pick(gen, raw, n)


def _edges(case, gen):
    """(src, dst, rel, node types, rel -> source type, rel -> destination type); the last three None with one type."""
    N, R, E, T = case["nodes"], case["rels"], case["edges"], case["types"]
    rel = _pick(gen, torch.as_tensor(_rel_probs(R, case["zipf"]), device="cuda"), E)
    if T == 1:
        return _ints(gen, 0, N, E), _popular(gen, N, E, case["hub"]), rel, None, None, None
    sizes = np.maximum(1, np.floor(_rel_probs(T, 1.0) * N)).astype(np.int64)
    sizes[0] += N - sizes.sum()
    start = np.concatenate([[0], np.cumsum(sizes)])
    ntype = torch.repeat_interleave(torch.arange(T, device="cuda"), torch.as_tensor(sizes, device="cuda"))
    if not case["tied"]:
        return _ints(gen, 0, N, E), _popular(gen, N, E, case["hub"]), rel, ntype, None, None
    # more frequent relations lie between the larger node types, as they do in practice: round robin over the types
    rst, rdt = np.arange(R) % T, (np.arange(R) // T + np.arange(R)) % T
    cnt = torch.bincount(rel, minlength=R).cpu().numpy()
    src, dst = [], []
    for r in range(R):
        a, b, n = int(rst[r]), int(rdt[r]), int(cnt[r])
        src.append(_ints(gen, int(start[a]), int(start[a + 1]), n))
        dst.append(_popular(gen, int(sizes[b]), n, case["hub"]) + int(start[b]))
    rel = torch.repeat_interleave(torch.arange(R, device="cuda"), torch.as_tensor(cnt, device="cuda"))
    mix = torch.randperm(E, device="cuda", generator=gen)          # edge lists arrive in no particular order
    return torch.cat(src)[mix], torch.cat(dst)[mix], rel[mix], ntype, rst, rdt


def _normal(gen, var, *shape):
    return torch.randn(*shape, device="cuda", generator=gen) * math.sqrt(var)


def _tensors(case, gen):
    """The layer's tensors: features N(0, 1), weights N(0, 1 / fan in), output gradient N(0, 1)."""
    N, R, T, k, d, H = (case[x] for x in ("nodes", "rels", "types", "d_in", "d_out", "heads"))
    t = {"X": _normal(gen, 1.0, N, k)}
    if case["layer"] == "rgcn":
        t["W"] = _normal(gen, 1.0 / k, R, k, d)
        if case["self_loop"]:
            t["W0"] = _normal(gen, 1.0 / k, k, d)
    elif case["layer"] == "hgt":
        dh = d // H
        for name in ("Wk", "Wq", "Wv", "Wo"):
            t[name] = _normal(gen, 1.0 / d, T, d, d)
        t["Watt"], t["Wmsg"] = _normal(gen, 1.0 / dh, R, H, dh, dh), _normal(gen, 1.0 / dh, R, H, dh, dh)
        if case["mu"]:
            t["mu"] = 1.0 + 0.25 * _normal(gen, 1.0, R, H)
    else:
        for s in ("", "2") if case["layer"] == "model" else ("",):
            t["W" + s] = _normal(gen, 1.0 / k, R, k, d)
            t["w_s" + s], t["w_t" + s] = _normal(gen, 1.0 / d, R, d), _normal(gen, 1.0 / d, R, d)
    if case["layer"] == "model":
        t["rows"] = torch.randperm(N, device="cuda", generator=gen)[: max(N // 10, 1)]
        t["labels"] = _ints(gen, 0, d, len(t["rows"]))
    elif case["mode"] == "train":
        t["dOut"] = _normal(gen, 1.0, N, d)
    if case["dtype"] == "bf16":
        t = {n: v.to(torch.bfloat16) for n, v in t.items()}
    return t


PARAMS = {"rgcn": ("W", "W0"), "rgat": ("W", "w_s", "w_t"), "hgt": ("Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg", "mu"),
          "model": ("W", "w_s", "w_t", "W2", "w_s2", "w_t2")}


def prepare(case, seed):
    gen = _gen(seed)
    src, dst, rel, ntype, rst, rdt = _edges(case, gen)
    i32 = lambda x: None if x is None else (x.cpu().numpy() if torch.is_tensor(x) else x).astype(np.int32)
    g = A.Graph(case["nodes"], case["rels"], i32(src), i32(dst), i32(rel), i32(ntype), case["types"], i32(rst), i32(rdt))
    t = _tensors(case, gen)
    st = {"case": case, "graph": g, "t": t}
    if case["api"] == "autograd":
        for n in ("X",) + PARAMS[case["layer"]]:
            if n in t and not (case["layer"] == "model" and n == "X"):
                t[n].requires_grad_()
        return st
    layer = {"rgcn": B.RGNN_LAYER_RGCN, "rgat": B.RGNN_LAYER_RGAT, "hgt": B.RGNN_LAYER_HGT}[case["layer"]]
    desc = B.make_desc(B.RGNN_BF16 if case["dtype"] == "bf16" else B.RGNN_F32, case["d_in"], case["d_out"], case["heads"], SLOPE,
                       B.RGNN_NORM_IN_DEGREE_PER_REL, B.RGNN_ACT_RELU if case["relu"] else B.RGNN_ACT_NONE)
    fwd, bwd, saved = B.rgnn_workspace_bytes(g.handle, layer, desc)
    buf = lambda n: torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    st["desc"] = desc
    st["out"] = torch.empty(case["nodes"], case["d_out"], device="cuda")
    if case["mode"] == "infer":          # nothing is kept for a backward call: its tensors become scratch
        st["saved"], st["ws"] = None, buf(fwd + 256 + saved)
    else:
        st["saved"], st["ws"] = buf(saved), buf(max(fwd, bwd))
        st["grads"] = {"d" + n: torch.empty(t[n].shape, device="cuda") for n in ("X",) + PARAMS[case["layer"]] if n in t}
    return st


# ---------------------------------------------------------------------------------------------- one pass

def _run_autograd(st):
    case, g, t = st["case"], st["graph"], st["t"]
    if case["layer"] == "model":
        h = A.rgat(g, t["X"], t["W"], t["w_s"], t["w_t"], SLOPE)
        logits = A.rgat(g, torch.relu(h), t["W2"], t["w_s2"], t["w_t2"], SLOPE)
        loss = torch.nn.functional.nll_loss(torch.log_softmax(logits[t["rows"]], dim=1), t["labels"])
        names = PARAMS["model"]
        grads = torch.autograd.grad(loss, [t[n] for n in names])
        return {"logits": logits.detach(), **{"d" + n: x for n, x in zip(names, grads)}}
    if case["layer"] == "rgat":
        out = A.rgat(g, t["X"], t["W"], t["w_s"], t["w_t"], SLOPE, case["heads"])
    elif case["layer"] == "rgcn":
        out = A.rgcn(g, t["X"], t["W"], t.get("W0"), "in_degree_per_rel", "relu" if case["relu"] else "none")
    else:
        out = A.hgt(g, *[t[n] for n in ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg")], t.get("mu"))
    names = [n for n in ("X",) + PARAMS[case["layer"]] if n in t]
    grads = torch.autograd.grad(out, [t[n] for n in names], t["dOut"])
    return {"out": out.detach(), **{"d" + n: x for n, x in zip(names, grads)}}


def run(state):
    case = state["case"]
    if case["api"] == "autograd":
        return _run_autograd(state)
    g, d, t, out, saved, ws = state["graph"].handle, state["desc"], state["t"], state["out"], state["saved"], state["ws"]
    stream = torch.cuda.current_stream().cuda_stream
    train = case["mode"] == "train"
    gr = state.get("grads", {})
    if case["layer"] == "rgcn":
        B.rgnn_rgcn_fwd(g, d, t["X"], t["W"], t.get("W0"), out, saved, ws, stream)
        if train:
            B.rgnn_rgcn_bwd(g, d, t["X"], t["W"], t.get("W0"), out, saved, t["dOut"], gr["dX"], gr["dW"], gr.get("dW0"), ws, stream)
    elif case["layer"] == "rgat":
        B.rgnn_rgat_fwd(g, d, t["X"], t["W"], t["w_s"], t["w_t"], out, saved, ws, stream)
        if train:
            B.rgnn_rgat_bwd(g, d, t["X"], t["W"], t["w_s"], t["w_t"], out, saved, t["dOut"], gr["dX"], gr["dW"], gr["dw_s"],
                            gr["dw_t"], ws, stream)
    else:
        w = [t[n] for n in ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg")] + [t.get("mu")]
        B.rgnn_hgt_fwd(g, d, *w, out, saved, ws, stream)
        if train:
            B.rgnn_hgt_bwd(g, d, *w, out, saved, t["dOut"], *[gr["d" + n] for n in ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg")],
                           gr.get("dmu"), ws, stream)
    return {"out": out, **gr}


# ---------------------------------------------------------------------------------------------- cost and accuracy

def _pairs(case):
    """Expected number of distinct (source, relation) pairs: what a typed linear has to be applied to."""
    N, R, E, T = case["nodes"], case["rels"], case["edges"], case["types"]
    e = E * _rel_probs(R, case["zipf"])
    n = np.full(R, float(N))
    if T > 1 and case["tied"]:
        n = np.maximum(1.0, np.floor(_rel_probs(T, 1.0) * N))[np.arange(R) % T]
    return float((n * -np.expm1(e * np.log1p(-1.0 / np.maximum(n, 2.0)))).sum())


def work(case):
    """Inputs and outputs once (features, edge list, weights, gradients); products of the typed linears on distinct
    (source, relation) pairs and of the node linears, and the multiply-adds of the edges' weighted sums and dots."""
    N, R, T, E, k, d, H = (case[x] for x in ("nodes", "rels", "types", "edges", "d_in", "d_out", "heads"))
    b = 2 if case["dtype"] == "bf16" else 4
    train = case["mode"] == "train"
    P = _pairs(case)
    if case["layer"] == "hgt":
        par = 4 * T * d * d + 2 * R * d * d // H
        mm = 2 * P * d * d + 2 * N * d * d            # key and message per pair (weights folded), query and output per node
        edge = 2 * E * d
    elif case["layer"] == "rgcn":
        par = R * k * d + (k * d if case["self_loop"] else 0)
        mm = P * k * d + (N * k * d if case["self_loop"] else 0)
        edge = E * d
    else:
        par, mm, edge = R * k * d + 2 * R * d, P * k * d, 2 * E * d
    io = N * k * b + 12 * E + par * b + N * d * 4
    if train:
        io += N * d * b + N * k * 4 + par * 4
    mult = 3 if train else 1
    if case["layer"] == "model":          # two layers; the input's gradient is not needed
        io, mult = N * k * 4 + 12 * E + 2 * par * 4 * 2 + N * d * 4, 6
    return {"bytes": float(io), "flops": float(2 * mult * (mm + edge))}


def tolerance(case):
    """About four times the largest error seen against 64 bits: 5e-3 for HGT with bf16 rows, 2e-3 for RGCN with bf16 rows,
    2e-6 in fp32.  RGAT and the two-layer model are allowed more: an edge whose logit (or a unit whose activation)
    lies within rounding of zero takes the other side of the kink in another implementation, which moves the gradient rows
    of its two endpoints by a finite amount (a few such edges in millions: up to 1.3e-4 seen)."""
    if case["dtype"] == "bf16" and case["d_out"] == 128:
        return {"rel": 2e-2 if case["layer"] == "hgt" else 8e-3}
    kink = case["layer"] == "model" or (case["layer"] == "rgat" and case["mode"] == "train")
    return {"rel": 5e-4 if kink else 1e-5}


# ---------------------------------------------------------------------------------------------- 64-bit evaluation

CHUNK = 1 << 20      # edges at a time


def _by_relation(src, dst, rel, R):
    """Edges in relation order as (relation, slice) pieces of at most CHUNK edges."""
    order = torch.argsort(rel, stable=True)
    src, dst = src[order], dst[order]
    cnt = torch.bincount(rel, minlength=R).cpu().tolist()
    pieces, at = [], 0
    for r, n in enumerate(cnt):
        pieces += [(r, slice(i, min(i + CHUNK, at + n))) for i in range(at, at + n, CHUNK)]
        at += n
    return src, dst, rel[order], pieces


def _heads(x, H):
    return x.view(len(x), H, -1)


def _rgat64(N, e, X, W, w_s, w_t, H, dOut_fn):
    """RGAT forward, then backward for the output gradient dOut_fn(out) (None: forward only)."""
    src, dst, rel, pieces = e
    E, d = len(src), W.shape[2]
    zero = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.float64)
    z, S, out = zero(E, H), zero(N, H), zero(N, d)
    for r, q in pieces:
        z[q] = (_heads(X[src[q]] @ W[r] * w_s[r], H) + _heads(X[dst[q]] @ W[r] * w_t[r], H)).sum(-1)
    att = torch.exp(torch.where(z > 0, z, SLOPE * z))
    S.index_add_(0, dst, att)
    att /= S[dst]
    for r, q in pieces:
        out.index_add_(0, dst[q], (att[q].unsqueeze(-1) * _heads(X[src[q]] @ W[r], H)).flatten(1))
    if dOut_fn is None:
        return out, None
    dO = dOut_fn(out)
    gbar = _heads(dO * out, H).sum(-1)
    dX, dW, dws, dwt = zero(*X.shape), zero(*W.shape), zero(*w_s.shape), zero(*w_t.shape)
    for r, q in pieces:
        xs, xt, go = X[src[q]], X[dst[q]], _heads(dO[dst[q]], H)
        hs, ht = xs @ W[r], xt @ W[r]
        dz = att[q] * ((go * _heads(hs, H)).sum(-1) - gbar[dst[q]]) * torch.where(z[q] > 0, 1.0, SLOPE)
        full = dz.repeat_interleave(d // H, 1)
        dhs = (att[q].unsqueeze(-1) * go).flatten(1) + full * w_s[r]
        dht = full * w_t[r]
        dX.index_add_(0, src[q], dhs @ W[r].t())
        dX.index_add_(0, dst[q], dht @ W[r].t())
        dW[r] += xs.t() @ dhs + xt.t() @ dht
        dws[r] += (full * hs).sum(0)
        dwt[r] += (full * ht).sum(0)
    return out, {"dX": dX, "dW": dW, "dw_s": dws, "dw_t": dwt}


def _rgcn64(N, e, t, case):
    src, dst, rel, pieces = e
    X, W, W0 = t["X"], t["W"], t.get("W0")
    _, inv, cnt = torch.unique(rel * N + dst, return_inverse=True, return_counts=True)
    c = (1.0 / cnt.double())[inv].unsqueeze(1)
    out = X @ W0 if W0 is not None else torch.zeros(N, W.shape[2], device="cuda", dtype=torch.float64)
    for r, q in pieces:
        out.index_add_(0, dst[q], c[q] * (X[src[q]] @ W[r]))
    if case["relu"]:
        out = torch.relu(out)
    if case["mode"] == "infer":
        return {"out": out}
    dO = t["dOut"] * (out > 0) if case["relu"] else t["dOut"]
    dX, dW = (dO @ W0.t() if W0 is not None else torch.zeros_like(X)), torch.zeros_like(W)
    for r, q in pieces:
        g = c[q] * dO[dst[q]]
        dX.index_add_(0, src[q], g @ W[r].t())
        dW[r] += X[src[q]].t() @ g
    res = {"out": out, "dX": dX, "dW": dW}
    if W0 is not None:
        res["dW0"] = X.t() @ dO
    return res


def _hgt64(N, e, ntype, t, case):
    src, dst, rel, pieces = e
    T, R, H, d = case["types"], case["rels"], case["heads"], case["d_out"]
    dh = d // H
    rows = [torch.nonzero(ntype == k).flatten() for k in range(T)]
    zero = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.float64)

    def linear(x, w):
        y = zero(N, d)
        for k in range(T):
            y[rows[k]] = x[rows[k]] @ w[k]
        return y

    def linear_bwd(x, w, dy):
        dx, dw = zero(N, d), zero(T, d, d)
        for k in range(T):
            dx[rows[k]] = dy[rows[k]] @ w[k].t()
            dw[k] = x[rows[k]].t() @ dy[rows[k]]
        return dx, dw

    diag = lambda w: torch.block_diag(*w)
    scale = (t["mu"] if "mu" in t else torch.ones(R, H, device="cuda", dtype=torch.float64)) / math.sqrt(dh)
    X = t["X"]
    K, Q, V = linear(X, t["Wk"]), linear(X, t["Wq"]), linear(X, t["Wv"])
    raw, S, Z = zero(len(src), H), zero(N, H), zero(N, d)
    for r, q in pieces:
        raw[q] = _heads((K[src[q]] @ diag(t["Watt"][r])) * Q[dst[q]], H).sum(-1)
    att = torch.exp(raw * scale[rel])
    S.index_add_(0, dst, att)
    att /= S[dst]
    for r, q in pieces:
        Z.index_add_(0, dst[q], (att[q].unsqueeze(-1) * _heads(V[src[q]] @ diag(t["Wmsg"][r]), H)).flatten(1))
    res = {"out": linear(Z, t["Wo"])}
    dZ, res["dWo"] = linear_bwd(Z, t["Wo"], t["dOut"])
    gbar = _heads(dZ * Z, H).sum(-1)
    dK, dQ, dV = zero(N, d), zero(N, d), zero(N, d)
    dA, dM, dmu = zero(R, H, dh, dh), zero(R, H, dh, dh), zero(R, H)
    for r, q in pieces:
        Ba, Bm = diag(t["Watt"][r]), diag(t["Wmsg"][r])
        k, v, go = K[src[q]], V[src[q]], dZ[dst[q]]
        dl = att[q] * (_heads(go * (v @ Bm), H).sum(-1) - gbar[dst[q]])
        dm = (att[q].unsqueeze(-1) * _heads(go, H)).flatten(1)
        w = (dl * scale[r]).repeat_interleave(dh, 1)
        dka = w * Q[dst[q]]
        dQ.index_add_(0, dst[q], w * (k @ Ba))
        dK.index_add_(0, src[q], dka @ Ba.t())
        dV.index_add_(0, src[q], dm @ Bm.t())
        gA, gM = k.t() @ dka, v.t() @ dm
        for h in range(H):
            s = slice(h * dh, (h + 1) * dh)
            dA[r, h] += gA[s, s]
            dM[r, h] += gM[s, s]
        dmu[r] += (dl * raw[q]).sum(0) / math.sqrt(dh)
    dX = zero(N, d)
    for n, g in (("k", dK), ("q", dQ), ("v", dV)):
        dx, res["dW" + n] = linear_bwd(X, t["W" + n], g)
        dX += dx
    res.update(dX=dX, dWatt=dA, dWmsg=dM)
    if "mu" in t:
        res["dmu"] = dmu
    return {n: res[n] for n in ("out", "dX", "dWk", "dWq", "dWv", "dWo", "dWatt", "dWmsg", "dmu") if n in res}


def exact(case, seed):
    gen = _gen(seed)
    src, dst, rel, ntype, _, _ = _edges(case, gen)
    t = {n: v.double() if v.is_floating_point() else v for n, v in _tensors(case, gen).items()}
    N, e = case["nodes"], _by_relation(src, dst, rel, case["rels"])
    if case["layer"] == "rgcn":
        return _rgcn64(N, e, t, case)
    if case["layer"] == "hgt":
        return _hgt64(N, e, ntype, t, case)
    if case["layer"] == "rgat":
        fn = (lambda out: t["dOut"]) if case["mode"] == "train" else None
        out, gr = _rgat64(N, e, t["X"], t["W"], t["w_s"], t["w_t"], case["heads"], fn)
        return {"out": out, **(gr or {})}

    def loss_grad(h):
        h = h.clone().requires_grad_()
        loss = torch.nn.functional.nll_loss(torch.log_softmax(h[t["rows"]], dim=1), t["labels"])
        return torch.autograd.grad(loss, h)[0]

    h1, _ = _rgat64(N, e, t["X"], t["W"], t["w_s"], t["w_t"], 1, None)
    logits, g2 = _rgat64(N, e, torch.relu(h1), t["W2"], t["w_s2"], t["w_t2"], 1, loss_grad)
    _, g1 = _rgat64(N, e, t["X"], t["W"], t["w_s"], t["w_t"], 1, lambda out: g2["dX"] * (out > 0))
    return {"logits": logits, **{n: g1[n] for n in ("dW", "dw_s", "dw_t")}, **{n + "2": g2[n] for n in ("dW", "dw_s", "dw_t")}}
