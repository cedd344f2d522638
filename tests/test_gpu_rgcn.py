"""RGCN layer on the GPU vs the CPU oracle, element by element."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2412_04747_amd import synth
from parity import check, TOL_F32, TOL_BF16

pytestmark = pytest.mark.gpu


def _launches(call):
    """Names of the kernels a call launches."""
    import torch
    from paper_2412_04747_amd import binding as B
    torch.cuda.synchronize()
    B.rgnn_profile_start()
    call()
    return set(B.rgnn_profile_stop())


def _run(N, R, src, dst, rel, p, d, norm, act, self_loop, bwd=True, tag="", dtype="f32", d_in=None, one_launch=None):
    """one_launch: whether the forward is the one of a small graph (None: either)."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    print(f"rgcn case {tag}: N={N} R={R} E={len(src)} d={d} norm={norm} act={act} W0={self_loop}", flush=True)
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, norm, act, self_loop, dtype=dtype, d_in=d_in)
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    W0 = p["W0"] if self_loop else None
    L.load(p["X"], p["W"], W0, p["dOut"])
    names = _launches(L.fwd)
    assert one_launch is None or ("rgcn_small_fwd" in names) == one_launch, names
    want = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], W0, norm, act)
    check(L.out, want, tol, "out")
    if bwd:
        if act != "none":
            # the activation's mask is a decision taken from `out`: both sides take it from the same
            # values (the backward call receives `out` as an argument), so that an output within
            # rounding distance of zero cannot flip a whole gradient entry
            L.out.copy_(torch.from_numpy(np.ascontiguousarray(want, dtype=np.float32)))
        L.bwd()
        torch.cuda.synchronize()
        wg = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], W0, p["dOut"], norm, act, out=want)
        for k, v in L.grads().items():
            check(v, wg[k], tol, k)
    g.close()


def test_config1_forward():
    c = synth.config(1)
    _run(c["N"], c["R"], c["src"], c["dst"], c["rel"], c, 32, "in_degree_per_rel", "none", False, bwd=False, tag="C1")


# 700 edges of one relation at one destination: more than the forward of a small graph in one launch takes, so the general plan runs
@pytest.mark.parametrize("hub", [0, 700])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward_backward_all_options(d, hub):
    rng, src, dst, rel, _ = synth.tiny(40 + d, N=700, R=5, E=6000)
    dst[:hub], rel[:hub] = 6, 2
    p = synth.rgcn_params(rng, 700, 5, d, d, self_loop=True)
    one = d < 128 and hub == 0
    _run(700, 5, src, dst, rel, p, d, "in_degree_per_rel", "none", True, tag=f"d{d}", one_launch=one)
    _run(700, 5, src, dst, rel, p, d, "none", "relu", True, tag=f"d{d}-relu", one_launch=one)
    _run(700, 5, src, dst, rel, p, d, "none", "none", False, tag=f"d{d}-plain", one_launch=one)


@pytest.mark.parametrize("d_in,d", [(32, 64), (64, 32)])
def test_input_width_differs_from_output_width(d_in, d):
    rng, src, dst, rel, _ = synth.tiny(45 + d, N=700, R=5, E=6000)
    dst[:800], rel[:800] = 9, 2         # a hub cut into pieces
    p = synth.rgcn_params(rng, 700, 5, d_in, d, self_loop=True)
    _run(700, 5, src, dst, rel, p, d, "in_degree_per_rel", "none", True, tag=f"widths-{d_in}-{d}", d_in=d_in, one_launch=False)
    _run(700, 5, src, dst, rel, p, d, "none", "relu", True, tag=f"widths-{d_in}-{d}-loop-relu", d_in=d_in, one_launch=False)
    _run(700, 5, src, dst, rel, p, d, "none", "relu", False, tag=f"widths-{d_in}-{d}-relu", d_in=d_in, one_launch=False)


@pytest.mark.parametrize("norm,act,loop", [("in_degree_per_rel", "none", False), ("none", "relu", True), ("in_degree_per_rel", "none", True)])
@pytest.mark.parametrize("d_in,d", [(32, 32), (32, 64), (64, 32), (64, 64)])
def test_small_graph_in_one_launch(d_in, d, norm, act, loop):
    """Destinations with runs of 1, 8, 9, 31, 32, 33 and 256 edges, with 7, 8, 9, 16 and 17 runs (eight half wavefronts take a
    destination's runs in turn), and without any."""
    rng = np.random.default_rng(d_in + 2 * d)
    runs = [(v, 0, n) for v, n in enumerate((1, 8, 9, 31, 32, 33, 256))]
    for v, n in enumerate((7, 8, 9, 16, 17), start=20):
        runs += [(v, r, 1 + r % 3) for r in range(n)]
    N, R = 60, 20
    dst = np.concatenate([np.full(n, v) for v, _, n in runs]).astype(np.int32)
    rel = np.concatenate([np.full(n, r) for _, r, n in runs]).astype(np.int32)
    src = rng.integers(0, N, len(dst)).astype(np.int32)
    p = synth.rgcn_params(rng, N, R, d_in, d, self_loop=True)
    _run(N, R, src, dst, rel, p, d, norm, act, loop, tag=f"one-launch-{d_in}-{d}", d_in=d_in, one_launch=True)


@pytest.mark.parametrize("d_in,d", [(32, 32), (32, 64), (64, 32), (64, 64)])
def test_small_graph_with_rows_at_the_ends_of_the_range(d_in, d):
    """The one-launch forward of a small graph: rows of subnormal numbers, whose sums and products are whole multiples of 2^-29 that
    24 bits hold (256 rows of at most 63 units, 64 products with weights of at most 7), so the result is exact; and rows of 1.5 * 2^127,
    whose mean fp32 holds where their sum overflows."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng = np.random.default_rng(d_in + d)
    lengths = [1, 2, 7, 8, 9, 31, 32, 33, 64, 255, 256]
    N, R = 40, 12                                          # nodes 20.. are the sources; destination 0 has all lengths, then one each
    runs = [(0, r, n) for r, n in enumerate(lengths) if n < 64] + [(1 + r, r, n) for r, n in enumerate(lengths)]
    dst = np.concatenate([np.full(n, v) for v, _, n in runs]).astype(np.int32)
    rel = np.concatenate([np.full(n, r) for _, r, n in runs]).astype(np.int32)
    src = rng.integers(20, 38, len(dst)).astype(np.int32)
    big = np.array([(15, 11, 38)] * 128, np.int32)         # one destination of 128 rows near the largest number
    dst, rel, src = np.concatenate([dst, big[:, 0]]), np.concatenate([rel, big[:, 1]]), np.concatenate([src, big[:, 2]])
    X = rng.integers(-63, 64, (N, d_in)) * 2.0 ** -149
    W = rng.integers(-7, 8, (R, d_in, d)) * 2.0 ** 120
    X[38], W[11] = 0, 0
    X[38, 5], W[11, 5, 3] = 1.5 * 2.0 ** 127, 1
    g = Graph(N, R, src, dst, rel)
    for norm in ("none", "in_degree_per_rel"):
        L = RgcnLayer(g, d, norm, d_in=d_in)
        L.load(X.astype(np.float32), W.astype(np.float32))
        assert "rgcn_small_fwd" in _launches(L.fwd)
        got = L.out.cpu().numpy().astype(np.float64)
        if norm == "none":
            want = np.zeros((N, d))
            np.add.at(want, dst[:-128], np.einsum("ek,ekd->ed", X[src[:-128]], W[rel[:-128]]))
            assert np.array_equal(np.delete(got, 15, 0), np.delete(want, 15, 0))
            assert np.isinf(got[15, 3])
        else:
            assert got[15, 3] == 1.5 * 2.0 ** 127 and (np.delete(got[15], 3) == 0).all()
            cnt = 2.0 ** 5                                  # a run of 32 rows: an exact mean
            e = (dst == 1 + lengths.index(32)) & (rel == lengths.index(32))
            assert np.array_equal(got[1 + lengths.index(32)], np.einsum("ek,kd->d", X[src[e]], W[lengths.index(32)]) / cnt)
    g.close()


@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("d", [32, 64])
def test_small_graph_whose_output_takes_the_place_of_its_input(d, shift):
    """Without a self-loop the forward may write `out` over X, wholly or from some row on: X has been read by then, whatever the
    size of the graph."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng, src, dst, rel, _ = synth.tiny(90 + d, N=600, R=5, E=5000)
    p = synth.rgcn_params(rng, 600, 5, d, d)
    g = Graph(600, 5, src, dst, rel)
    L = RgcnLayer(g, d)
    L.load(p["X"], p["W"])
    buf = torch.empty((600 + shift) * d, device="cuda")
    buf[:600 * d] = L.X.flatten()
    L.X, L.out = buf[:600 * d].view(600, d), buf[shift * d:].view(600, d)
    L.fwd()
    torch.cuda.synchronize()
    check(L.out, O.rgcn_fwd(600, src, dst, rel, p["X"], p["W"], None, "in_degree_per_rel", "none"), TOL_F32, "out")
    g.close()


@pytest.mark.parametrize("k,loop,N,E,hub,rels,one", [
    (32, False, 4000, 19397, 0, 0, True), (32, False, 4000, 19398, 0, 0, False),             # nodes and runs
    (32, False, 13698, 1, 0, 0, True), (32, False, 13699, 1, 0, 0, False),
    (64, True, 4000, 11625, 0, 0, True), (64, True, 4000, 11626, 0, 0, False),
    (64, True, 8650, 0, 0, 0, True), (64, True, 8651, 0, 0, 0, False),
    (32, False, 4000, 27576, 40, 40, True), (32, False, 4000, 27577, 40, 40, False),         # ... with a destination that is cut
    (32, False, 500, 300, 428, 1, True), (32, False, 500, 300, 429, 1, False),               # edges of one destination
    (64, True, 500, 300, 339, 1, True), (64, True, 500, 300, 340, 1, False),
    (32, False, 500, 300, 400, 10, True),                                                    # ... in short runs
    (32, False, 500, 300, 104, 104, True), (32, False, 500, 300, 105, 105, False),           # relations of one destination
    (64, False, 500, 300, 64, 64, True), (64, False, 500, 300, 65, 65, False), (64, False, 500, 300, 256, 256, False)])
def test_either_side_of_the_small_graph_rule(k, loop, N, E, hub, rels, one):
    """The largest graphs of the one-launch forward and the smallest beyond it: which plan runs, and its results."""
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng = np.random.default_rng(N + E + hub)
    R = max(40, rels)
    pick = rng.permutation((N - 1) * 40)[:E]               # a run per edge, none at node N - 1
    dst, rel = np.concatenate([pick // 40, np.full(hub, N - 1)]), np.concatenate([pick % 40, np.arange(hub) % max(rels, 1)])
    src, dst, rel = rng.integers(0, N, E + hub).astype(np.int32), dst.astype(np.int32), rel.astype(np.int32)
    p = synth.rgcn_params(rng, N, R, k, k, self_loop=True)
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, k, "in_degree_per_rel", "none", loop)
    W0 = p["W0"] if loop else None
    L.load(p["X"], p["W"], W0)
    names = _launches(L.fwd)
    assert ("rgcn_small_fwd" in names) == one and ("aggregate_fwd" in names) == (not one), names
    check(L.out, O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], W0, "in_degree_per_rel", "none"), TOL_F32, "out")
    g.close()


@pytest.mark.parametrize("d_in,d", [(32, 32), (32, 64), (64, 32), (64, 64)])
@pytest.mark.parametrize("N,R,E", [(1, 1, 0), (40000, 3, 70), (300, 40, 30000), (3000, 2, 40000)])
def test_self_loop_and_pairs_share_the_compute_units(N, R, E, d_in, d):
    """The self-loop's and the pairs' backward split the compute units by their rows: none, few and nearly all of them pairs."""
    rng = np.random.default_rng(N + E + d)
    src, dst = rng.integers(0, N, E).astype(np.int32), rng.integers(0, N, E).astype(np.int32)
    rel = rng.integers(0, R, E).astype(np.int32)
    p = synth.rgcn_params(rng, N, R, d_in, d, self_loop=True)
    _run(N, R, src, dst, rel, p, d, "in_degree_per_rel", "none", True, tag="shared-units", d_in=d_in)


def test_hub_and_isolated_nodes():
    rng, src, dst, rel, _ = synth.tiny(50, N=400, R=3, E=3000)
    dst[:1500] = 3          # hub far above the item length, many nodes left without in-edges
    src[:900] = 5           # one (src, rel) pair feeding many edges
    rel[:900] = 1
    p = synth.rgcn_params(rng, 400, 3, 64, 64, self_loop=True)
    _run(400, 3, src, dst, rel, p, 64, "in_degree_per_rel", "none", True, tag="hub", one_launch=False)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_relu_backward_from_the_gpus_own_output(dtype, d):
    """The ReLU mask of the backward call is taken from the `out` the GPU's own forward wrote (the other cases
    hand both sides the oracle's `out`).  So that no mask bit hangs on rounding, the inputs are built with
    every pre-activation at least 1e-3 away from 0: sources and destinations are disjoint node sets and the
    self-loop weight is the identity, hence a destination's own feature row shifts its own pre-activation only (a source's row
    also moves its destinations, so the nudging is repeated until nothing is left inside the margin)."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    N, R, E = 800, 4, 6000
    rng = np.random.default_rng(611)
    src = rng.integers(0, N // 2, E).astype(np.int32)
    dst = rng.integers(N // 2, N, E).astype(np.int32)
    dst[:900] = N // 2 + 3                                       # a hub
    rel = rng.integers(0, R, E).astype(np.int32)
    p = synth.rgcn_params(rng, N, R, d, d, self_loop=True)
    p["W0"] = np.eye(d, dtype=np.float32)
    if dtype == "bf16":
        p = {k: synth.round_to_bf16(v) for k, v in p.items()}
    margin = 4e-3 if dtype == "f32" else 3e-2                    # bf16: a step of X's grid is up to 2^-8 of |x|
    for _ in range(4):
        pre = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], p["W0"], "in_degree_per_rel", "none")
        near = np.abs(pre) < margin
        if not near.any():
            break
        X = p["X"].astype(np.float64)
        X[near] += np.where(pre[near] >= 0, 2 * margin, -2 * margin)
        p["X"] = synth.round_to_bf16(X.astype(np.float32)) if dtype == "bf16" else X.astype(np.float32)
    pre = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], p["W0"], "in_degree_per_rel", "none")
    assert np.abs(pre).min() >= 1e-3
    print(f"rgcn case relu-own-out {dtype} d={d}: min |pre-activation| {np.abs(pre).min():.2e}", flush=True)
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, "in_degree_per_rel", "relu", True, dtype=dtype)
    L.load(p["X"], p["W"], p["W0"], p["dOut"])
    L.fwd(); L.bwd()                                             # `out` stays the GPU's
    torch.cuda.synchronize()
    want = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], p["W0"], "in_degree_per_rel", "relu")
    check(L.out, want, tol, "out")
    assert np.array_equal(L.out.cpu().numpy() > 0, want > 0)
    wg = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], p["W0"], p["dOut"], "in_degree_per_rel", "relu", out=want)
    for k, v in L.grads().items():
        check(v, wg[k], tol, k)
    g.close()


def test_empty_graph():
    rng = np.random.default_rng(0)
    p = synth.rgcn_params(rng, 10, 2, 32, 32, self_loop=True)
    e = np.zeros(0, np.int32)
    _run(10, 2, e, e, e, p, 32, "in_degree_per_rel", "none", True, tag="empty")


@pytest.mark.parametrize("d", [32, 64, 128])
def test_small_bf16_all_options(d):
    rng, src, dst, rel, _ = synth.tiny(140 + d, N=700, R=5, E=6000)
    dst[:800] = 3
    p = synth.rgcn_params(rng, 700, 5, d, d, self_loop=True)
    p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(700, 5, src, dst, rel, p, d, "in_degree_per_rel", "none", True, tag=f"bf16-d{d}", dtype="bf16")
    _run(700, 5, src, dst, rel, p, d, "none", "relu", False, tag=f"bf16-d{d}-relu", dtype="bf16")


@pytest.mark.parametrize("dtype,d", [("f32", 32), ("bf16", 128)])
def test_many_single_entry_segments(dtype, d):
    """Thousands of destinations with one incoming edge, thousands with two to four, and as many
    (source, relation) pairs with one or two edges: the batched single-entry and short-segment
    aggregation paths, forward (destination-major) and backward (pair-major)."""
    rng = np.random.default_rng(77)
    N, R = 12000, 4
    dst = rng.permutation(N).astype(np.int32)              # every node: in-degree at least 1; 7000 of them exactly 1
    more = np.repeat(np.arange(5000, dtype=np.int32), rng.integers(1, 4, 5000))   # 5000 nodes with 2..4 incoming edges
    hub = rng.integers(0, 50, 600).astype(np.int32)        # a few busier ones on top
    dst = np.concatenate([dst, more, hub])
    src = rng.integers(0, N, len(dst)).astype(np.int32)
    rel = rng.integers(0, R, len(dst)).astype(np.int32)
    src[N:N + 6000] = src[:6000]; rel[N:N + 6000] = rel[:6000]   # 6000 (source, relation) pairs with two edges
    p = synth.rgcn_params(rng, N, R, d, d, self_loop=False)
    if dtype == "bf16":
        p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(N, R, src, dst, rel, p, d, "in_degree_per_rel", "none", False, tag=f"singles-{dtype}", dtype=dtype, one_launch=False)


def test_scaled_config5_bf16():
    c = synth.config(5, scale=0.01)          # knowledge-graph shaped: 500 relations, many with a handful of edges
    _run(c["N"], c["R"], c["src"], c["dst"], c["rel"], c, 128, "in_degree_per_rel", "none", False, tag="C5/100",
         dtype="bf16")


@pytest.mark.timeout(1100)
def test_config5_full_size_bf16():
    """2.5M nodes, 500 relations (100 of them with fewer than 100 edges), 16M edges, d=128, bf16 inputs."""
    c = synth.config(5)
    _run(c["N"], c["R"], c["src"], c["dst"], c["rel"], c, 128, "in_degree_per_rel", "none", False, tag="C5",
         dtype="bf16")


@pytest.mark.parametrize("norm", ["none", "in_degree_per_rel"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 128), ("f32", 64), ("f32", 32)])
def test_relation_sizes_around_the_row_tiles(dtype, d, norm):
    """Relations whose pairs fill the 64-row tiles of the typed linears exactly, less one and plus one, one of a single
    pair, an empty one and one of several tiles; a third of the pairs have two edges."""
    rng = np.random.default_rng(600 + d)
    sizes = [64, 1, 63, 0, 65, 128, 31, 33, 127, 129, 300, 16, 15]
    N, R = 310, len(sizes)
    src = np.concatenate([rng.permutation(N)[:n] for n in sizes])
    rel = np.repeat(np.arange(R), sizes)
    dst = rng.integers(0, N, len(src))
    two = rng.random(len(src)) < 0.33
    src, rel, dst = (np.concatenate([a, b]).astype(np.int32) for a, b in
                     ((src, src[two]), (rel, rel[two]), (dst, rng.integers(0, N, int(two.sum())))))
    p = synth.rgcn_params(rng, N, R, d, d, self_loop=True)
    if dtype == "bf16":
        p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(N, R, src, dst, rel, p, d, norm, "none", True, tag=f"tiles-{dtype}-d{d}", dtype=dtype)


@pytest.mark.parametrize("value", [3.39e38, float("inf")])
@pytest.mark.parametrize("where", ["X", "W", "dOut"])
def test_operands_beyond_the_range_of_bfloat16(where, value):
    """Width 128, fp32: an operand whose bfloat16 rounding is not finite (the largest fp32 values, infinity) takes the tile
    through the fp32 matrix instructions in the backward (RGCN's forward is on them throughout; HGT's forward has a test of
    its own).  One edge per destination, so every result row is one product; the other operand is scaled by 2^-126 for the
    finite value, which keeps the products near 1.  Errors are fp32 roundings of 128-term sums: at most 128 * 2^-24 of the
    sum of magnitudes, or 128 roundings of subnormal sums."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng = np.random.default_rng(41)
    N, R, d = 200, 3, 128
    src, dst = rng.permutation(N).astype(np.int32), np.arange(N, dtype=np.int32)
    rel = np.repeat(np.arange(R, dtype=np.int32), [70, 66, 64])
    p = synth.rgcn_params(rng, N, R, d, d)
    tiny = np.float32(2.0 ** -126) if np.isfinite(value) else np.float32(1.0)
    at = {"X": (src[5], 7), "W": (0, 7, 9), "dOut": (5, 11)}[where]
    p[where][at] = value
    for k in ("X", "W", "dOut"):
        if k != where and (where == "W") == (k != "W"):       # the operands that meet it in a product
            p[k] = p[k] * tiny
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, "none")
    L.load(p["X"], p["W"], None, p["dOut"])
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    X, W, dO = (p[k].astype(np.float64) for k in ("X", "W", "dOut"))
    with np.errstate(invalid="ignore"):
        out, dX, dW = np.zeros((N, d)), np.zeros((N, d)), np.zeros((R, d, d))
        mag = {"out": np.zeros((N, d)), "dX": np.zeros((N, d)), "dW": np.zeros((R, d, d))}
        for r in range(R):
            e = rel == r
            out[dst[e]], dX[src[e]], dW[r] = X[src[e]] @ W[r], dO[dst[e]] @ W[r].T, X[src[e]].T @ dO[dst[e]]
            mag["out"][dst[e]], mag["dX"][src[e]] = abs(X[src[e]]) @ abs(W[r]), abs(dO[dst[e]]) @ abs(W[r]).T
            mag["dW"][r] = abs(X[src[e]]).T @ abs(dO[dst[e]])
    top = float(np.finfo(np.float32).max)
    for name, got, want in (("out", L.out, out), ("dX", L.dX, dX), ("dW", L.dW, dW)):
        got = got.cpu().numpy().astype(np.float64)
        over = ~(mag[name] < top / 2)                # where fp32 partial sums may overflow only non-finite values are compared
        assert (np.isfinite(got) | over).all(), name
        bad = ~np.isfinite(want)
        assert (~np.isfinite(got[bad])).all(), name
        ok = ~over & np.isfinite(want)
        assert (np.abs(got - want)[ok] <= 128 * 2.0 ** -24 * mag[name][ok] + 128 * 2.0 ** -149).all(), name
    g.close()


@pytest.mark.parametrize("hub", [0, 700])
@pytest.mark.parametrize("N", [700, 701])
@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 32), ("bf16", 128)])
def test_relu_mask_of_an_output_off_the_16_byte_grid(dtype, d, N, hub):
    """The backward reads `out` four elements at a time where its address allows it: the same bits, masked one by one, when
    it does not; and the forward's activation (in the self-loop's epilogue, or that of the one launch of a small graph) is max(0, .)
    of the run without one."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng, src, dst, rel, _ = synth.tiny(70 + d, N=N, R=5, E=6000)
    dst[:hub], rel[:hub] = 6, 2
    p = synth.rgcn_params(rng, N, 5, d, d, self_loop=True)
    g = Graph(N, 5, src, dst, rel)
    outs = {}
    for act in ("none", "relu"):
        L = RgcnLayer(g, d, "in_degree_per_rel", act, True, dtype=dtype)
        L.load(p["X"], p["W"], p["W0"], p["dOut"])
        assert ("rgcn_small_fwd" in _launches(L.fwd)) == (dtype == "f32" and d < 128 and hub == 0)
        outs[act] = L.out.clone()
    assert torch.equal(outs["relu"], outs["none"].clamp(min=0))
    L.bwd()
    torch.cuda.synchronize()
    want = {k: v.clone() for k, v in L.grads().items()}
    buf = torch.empty(L.out.numel() + 1, device="cuda")
    L.out = buf[1:].view_as(outs["relu"]).copy_(outs["relu"])
    assert L.out.data_ptr() % 16 == 4
    L.bwd()
    torch.cuda.synchronize()
    for k, v in L.grads().items():
        assert torch.equal(v, want[k]), k
    g.close()


@pytest.mark.parametrize("exponent", [-126, -118, -112, -109, -104])
@pytest.mark.parametrize("where", ["dOut", "X and W"])
def test_backward_operands_of_small_magnitude(where, exponent):
    """Width 128, fp32: operands scaled by 2^exponent, where the low planes of a split into bfloat16 numbers would be subnormal
    or lost, against operands scaled up by as much (2^120 at most).  One edge per destination and per pair, so a row of dX is one
    product and dW a sum over a relation's rows: errors are fp32 roundings of sums of at most 128 terms, 128 * 2^-24 of the
    sum of magnitudes."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng = np.random.default_rng(43)
    N, R, d = 200, 3, 128
    src, dst = rng.permutation(N).astype(np.int32), np.arange(N, dtype=np.int32)
    rel = np.repeat(np.arange(R, dtype=np.int32), [70, 66, 64])
    p = synth.rgcn_params(rng, N, R, d, d)
    small, large = np.float32(2.0 ** exponent), np.float32(2.0 ** min(-exponent, 120))
    for k in ("X", "W", "dOut"):
        p[k] = p[k] * (small if (k == "dOut") == (where == "dOut") else large)
    p["dOut"][3, 40:80] = 0                              # zeros are no small numbers
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, "none")
    L.load(p["X"], p["W"], None, p["dOut"])
    L.bwd()
    torch.cuda.synchronize()
    X, W, dO = (p[k].astype(np.float64) for k in ("X", "W", "dOut"))
    for r in range(R):
        e = rel == r
        x, y = X[src[e]], dO[dst[e]]
        for name, got, want, mag in (("dX", L.dX[torch.as_tensor(src[e]).long()], y @ W[r].T, abs(y) @ abs(W[r]).T),
                                     ("dW", L.dW[r], x.T @ y, abs(x).T @ abs(y))):
            err = np.abs(got.cpu().numpy().astype(np.float64) - want)
            assert (err <= 128 * 2.0 ** -24 * mag).all(), (name, r, (err / mag).max())
    g.close()


def test_weight_gradient_of_long_chunks_bf16():
    """A relation of 16 row tiles per workgroup (two workgroups per compute unit).  Every product is 1 but the first of dW[0][0],
    2^28, where a unit in the last place is 32: that workgroup's share is off by at most half a unit per tile and per step of 16
    rows within the first tile.  The other shares are multiples of 32 and add up without error."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    d, tiles = 128, 16
    N = 2 * torch.cuda.get_device_properties(0).multi_processor_count * tiles * 64
    src = dst = np.arange(N, dtype=np.int32)
    g = Graph(N, 1, src, dst, np.zeros(N, np.int32))
    L = RgcnLayer(g, d, "none", dtype="bf16")
    ones = lambda *s: torch.ones(*s, device="cuda", dtype=torch.bfloat16)
    L.X, L.W, L.W0, L.dOut = ones(N, d), ones(1, d, d), None, ones(N, d)
    L.X[0, 0] = 2.0 ** 14
    L.dOut[0, 0] = 2.0 ** 14
    L.bwd()
    torch.cuda.synchronize()
    want = torch.full((d, d), float(N), device="cuda", dtype=torch.float64)
    want[0, :] += 2.0 ** 14 - 1
    want[:, 0] += 2.0 ** 14 - 1
    want[0, 0] = 2.0 ** 28 + N - 1
    err = (L.dW[0].double() - want).abs()
    assert err[0, 0].item() <= 16 * (tiles + 4), err[0, 0].item()
    err[0, 0] = 0
    assert err.max().item() == 0
    g.close()


def test_weight_gradient_of_many_shares():
    """fp32 self-loop weight whose gradient comes in a share per compute unit (one unit goes to the only pair), each the sum of one row
    tile or two: all products are 1 but the first of dW0[0][0], 2^33, where half a unit in the last place is 512, as much as eight
    shares of a tile.  An addition to the large number loses half a unit at most, and no more than what is added.  Halves of units:
      1  the other rows of its own share (at most 127)
      1  16 groups of lanes take the shares in turn, in two chains: the other seven shares of its own (512 with a second tile's)
      1  the group's second chain
      3  four chains of four groups
      2  and those by halves.
    One after the other 255 shares of 64 would lose 31.  (Up to 256 compute units; each further 256 add 1.)"""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    d = 64
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N = 64 * cus
    g = Graph(N, 1, np.zeros(1, np.int32), np.ones(1, np.int32), np.zeros(1, np.int32))
    L = RgcnLayer(g, d, "none", self_loop=True)
    ones = lambda *s: torch.ones(*s, device="cuda")
    L.X, L.W, L.W0, L.dOut = ones(N, d), ones(1, d, d), ones(d, d), ones(N, d)
    L.X[0, 0], L.dOut[0, 0] = 2.0 ** 17, 2.0 ** 16
    L.bwd()
    torch.cuda.synchronize()
    err = abs(float(L.dW0[0, 0].double()) - (2.0 ** 33 + N - 1))
    assert err <= 512 * (7 + -(-cus // 256)), err
    g.close()
