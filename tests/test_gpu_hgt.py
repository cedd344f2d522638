"""HGT layer (forward + backward) on the GPU vs the CPU oracle."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2412_04747_amd import synth
from parity import check, TOL_F32, TOL_BF16

pytestmark = pytest.mark.gpu

NAMES = ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg", "mu")


def _run(N, T, R, src, dst, rel, ntype, p, d, H, tag, dtype="f32", repeat=True):
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    print(f"hgt case {tag}: N={N} T={T} R={R} E={len(src)} d={d} H={H} mu={'yes' if p['mu'] is not None else 'no'}",
          flush=True)
    g = Graph(N, R, src, dst, rel, ntype if T > 1 else None, T)
    L = HgtLayer(g, d, H, with_mu=p["mu"] is not None, dtype=dtype)
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    L.load(*[p[k] for k in NAMES], dOut=p["dOut"])
    L.fwd()
    torch.cuda.synchronize()
    nt = ntype if T > 1 else None
    want = O.hgt_fwd(N, src, dst, rel, nt, *[p[k] for k in NAMES])
    check(L.out, want, tol, "out")
    L.bwd()
    torch.cuda.synchronize()
    wg = O.hgt_bwd(N, src, dst, rel, nt, *[p[k] for k in NAMES], p["dOut"])
    errs = {k: check(v, wg[k], tol, k) for k, v in L.grads().items()}
    print("   max rel errors:", {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    if not repeat:
        g.close()
        return
    out1 = L.out.clone()
    first = {k: v.clone() for k, v in L.grads().items()}
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    assert torch.equal(out1, L.out)
    for k, v in L.grads().items():
        assert torch.equal(first[k], v), k
    g.close()


@pytest.mark.parametrize("d,H,mu", [(64, 2, True), (64, 4, False), (128, 4, True), (32, 1, True)])
def test_small_typed(d, H, mu):
    rng, src, dst, rel, ntype = synth.tiny(90 + d + H, N=600, R=5, E=5000, T=3)
    p = synth.hgt_params(rng, 600, 3, 5, d, H, with_mu=mu)
    _run(600, 3, 5, src, dst, rel, ntype, p, d, H, f"small-d{d}-H{H}")


@pytest.mark.parametrize("d,H", [(64, 2), (32, 2), (128, 4), (128, 8)])     # (128, 8): softmax as a pass of its own
def test_small_typed_bf16(d, H):
    rng, src, dst, rel, ntype = synth.tiny(190 + d, N=700, R=6, E=6000, T=3)
    dst[:900] = 5                                   # a hub cut into pieces
    p = synth.hgt_params(rng, 700, 3, 6, d, H, with_mu=True)
    p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(700, 3, 6, src, dst, rel, ntype, p, d, H, f"bf16-d{d}-H{H}", dtype="bf16")


def test_hub_isolated_and_single_type():
    rng, src, dst, rel, ntype = synth.tiny(95, N=300, R=4, E=4000, T=1)
    dst[:2500] = 9
    src[:700] = 4
    rel[:700] = 2
    p = synth.hgt_params(rng, 300, 1, 4, 64, 2, with_mu=True)
    _run(300, 1, 4, src, dst, rel, ntype, p, 64, 2, "hub")


@pytest.mark.parametrize("dtype,d,H", [("f32", 64, 2), ("bf16", 128, 4)])
def test_many_single_entry_segments(dtype, d, H):
    """Thousands of destinations with one incoming edge and of pairs with one edge: the batched
    single-entry aggregation path with one coefficient per head."""
    rng = np.random.default_rng(78)
    N, T, R = 12000, 2, 3
    ntype = (np.arange(N) >= 7000).astype(np.int32)
    more = np.repeat(np.arange(5000), rng.integers(1, 4, 5000))         # 5000 nodes with 2..4 incoming edges
    dst = np.concatenate([rng.permutation(N), more, rng.integers(0, 40, 500)]).astype(np.int32)
    src = rng.integers(0, N, len(dst)).astype(np.int32)
    rel = rng.integers(0, R, len(dst)).astype(np.int32)
    src[N:N + 6000] = src[:6000]; rel[N:N + 6000] = rel[:6000]          # 6000 pairs with two edges
    p = synth.hgt_params(rng, N, T, R, d, H, with_mu=True)
    if dtype == "bf16":
        p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(N, T, R, src, dst, rel, ntype, p, d, H, f"singles-{dtype}", dtype=dtype)


@pytest.mark.parametrize("dtype,d,H", [("f32", 64, 2), ("f32", 32, 2), ("f32", 128, 4), ("bf16", 64, 4), ("bf16", 128, 4)])
def test_relations_tied_to_one_source_type(dtype, d, H):
    """Every relation draws its sources from one node type, so the library folds the key and message
    linears of the nodes into the per-relation weights.  Relation 4 has no edge, type 3 is never a
    source, types 0 and 1 serve several relations, and a hub and a pair with many edges are cut."""
    rng = np.random.default_rng(311 + d)
    N, T, R, E = 900, 4, 6, 8000
    ntype = rng.integers(0, T, N).astype(np.int32)
    rel_type = np.array([0, 1, 2, 0, 1, 0], np.int32)
    rel = rng.choice([0, 1, 2, 3, 5], E).astype(np.int32)
    by_type = [np.nonzero(ntype == t)[0] for t in range(T)]
    src = np.array([rng.choice(by_type[rel_type[r]]) for r in rel], np.int32)
    dst = rng.integers(0, N, E).astype(np.int32)
    dst[:1500] = 13
    src[:600] = by_type[1][0]; rel[:600] = 1
    p = synth.hgt_params(rng, N, T, R, d, H, with_mu=True)
    if dtype == "bf16":
        p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(N, T, R, src, dst, rel, ntype, p, d, H, f"tied-{dtype}-d{d}", dtype=dtype)


@pytest.mark.parametrize("dtype,d,H", [("f32", 32, 1), ("f32", 32, 2), ("f32", 64, 1), ("f32", 64, 4), ("f32", 128, 2),
                                       ("f32", 128, 8), ("bf16", 128, 2), ("bf16", 128, 4), ("bf16", 128, 8)])
def test_walk_lengths(dtype, d, H):
    """Destinations and pairs at the lengths where the edge walks change: none, one batch of four and its remainders, the
    shortest item that a whole wavefront takes (29 entries), the longest uncut item (32) and cut ones with a remainder."""
    rng = np.random.default_rng(400 + d + H)
    lengths = [0, 1, 2, 3, 4, 5, 7, 8, 9, 27, 28, 29, 30, 31, 32, 33, 61, 64, 65, 97, 130] * 3
    dst = np.repeat(np.arange(len(lengths)), lengths)
    E, N, T, R = len(dst), 150, 2, 3
    src = np.concatenate([np.repeat(np.arange(len(lengths)), rng.permutation(lengths)), rng.integers(0, N, 40)])[:E]
    src = np.concatenate([src, rng.integers(0, N, E - len(src))])
    rel = rng.integers(0, R, E)
    rel[:E // 2] = 1                                  # pairs of many edges too
    perm = rng.permutation(E)
    ntype = rng.integers(0, T, N).astype(np.int32)
    p = synth.hgt_params(rng, N, T, R, d, H, with_mu=True)
    if dtype == "bf16":
        p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(N, T, R, src.astype(np.int32)[perm], dst.astype(np.int32), rel.astype(np.int32), ntype, p, d, H, f"lengths-{dtype}-d{d}-H{H}",
         dtype=dtype)


@pytest.mark.parametrize("tied", [True, False])
@pytest.mark.parametrize("dtype,d,H", [("bf16", 128, 4), ("f32", 128, 4), ("f32", 64, 4)])
def test_relation_sizes_around_the_row_tiles(dtype, d, H, tied):
    """Relations whose pairs fill the 64-row tiles of the typed linears exactly, less one and plus one, a single pair, none,
    and several tiles, with sources of one node type per relation (folded weights, key and message half in one kernel)
    and of mixed types (node linears of their own)."""
    rng = np.random.default_rng(700 + d)
    sizes = [64, 1, 63, 0, 65, 128, 31, 129, 300]
    T, R, per = 3, len(sizes), 310
    N = T * per + 1
    ntype = np.minimum(np.arange(N) // per, T - 1).astype(np.int32)
    src, rel = [], np.repeat(np.arange(R), sizes)
    for r, n in enumerate(sizes):
        src.append(rng.permutation(per)[:n] + (per * (r % T) if tied else 0))
        if not tied and n > 1:
            src[-1][: n // 2] += per
    src = np.concatenate(src)
    dst = rng.integers(0, N, len(src))
    p = synth.hgt_params(rng, N, T, R, d, H, with_mu=True)
    if dtype == "bf16":
        p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
    _run(N, T, R, src.astype(np.int32), dst.astype(np.int32), rel.astype(np.int32), ntype, p, d, H, f"tiles-{dtype}-{tied}", dtype=dtype)


@pytest.mark.parametrize("d,H", [(32, 1), (64, 4)])
@pytest.mark.parametrize("N,R,E", [(1, 1, 1), (40000, 3, 0), (40000, 3, 70), (300, 40, 30000), (3000, 2, 40000)])
def test_nodes_and_pairs_share_the_compute_units(N, R, E, d, H):
    """The node and pair products of one launch split the compute units by their rows: none, few and nearly all of them pairs."""
    rng = np.random.default_rng(N + E + d)
    src, dst = rng.integers(0, N, E).astype(np.int32), rng.integers(0, N, E).astype(np.int32)
    rel = rng.integers(0, R, E).astype(np.int32)
    p = synth.hgt_params(rng, N, 1, R, d, H, with_mu=True)
    _run(N, 1, R, src, dst, rel, np.zeros(N, np.int32), p, d, H, "shared-units")


def _wide_case(seed, tied):
    """Width 128, four heads: 230 nodes of two types, five relations, 700 edges; with `tied` the sources of a relation are
    of one type."""
    rng = np.random.default_rng(seed)
    N, T, R, E = 230, 2, 5, 700
    ntype = (np.arange(N) >= 120).astype(np.int32)
    rel = rng.integers(0, R, E).astype(np.int32)
    src = rng.integers(0, N, E)
    if tied:
        src = np.where(rel % 2 == 0, src % 120, 120 + src % 110)
    dst = rng.integers(0, N, E).astype(np.int32)
    return N, T, R, src.astype(np.int32), dst, rel, ntype, synth.hgt_params(rng, N, T, R, 128, 4, with_mu=True)


@pytest.mark.parametrize("tied", [True, False])
@pytest.mark.parametrize("exponent", [-120, -116, -112, -109, -104])
def test_operands_of_small_magnitude(exponent, tied):
    """fp32: X scaled by 2^exponent and the node weights that it meets by 2^-exponent, so that every product is as without
    the scales and the errors relative to the largest entry stay below those of fp32 sums of 128 terms, 128 * 2^-24."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    N, T, R, src, dst, rel, ntype, p = _wide_case(800, tied)
    p["X"] = p["X"] * np.float32(2.0 ** exponent)
    for k in ("Wk", "Wq", "Wv"):
        p[k] = p[k] * np.float32(2.0 ** -exponent)
    g = Graph(N, R, src, dst, rel, ntype, T)
    L = HgtLayer(g, 128, 4)
    L.load(*[p[k] for k in NAMES], dOut=p["dOut"])
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    wg = O.hgt_bwd(N, src, dst, rel, ntype, *[p[k] for k in NAMES], p["dOut"])
    pairs = {"out": (L.out, O.hgt_fwd(N, src, dst, rel, ntype, *[p[k] for k in NAMES])), **{k: (v, wg[k]) for k, v in L.grads().items()}}
    for k, (got, want) in pairs.items():
        unit = np.abs(want).max()                       # `check` does not divide by less than 1e-30
        check(got.cpu().numpy().astype(np.float64) / unit, want / unit, 128 * 2.0 ** -24, k)
    g.close()


@pytest.mark.parametrize("tied", [True, False])
@pytest.mark.parametrize("value", [3.39e38, float("inf")])
@pytest.mark.parametrize("where", ["X", "Wv"])
def test_operands_beyond_the_range_of_bfloat16(where, value, tied):
    """fp32 forward with one operand whose bfloat16 rounding is not finite (the largest fp32 values, infinity): its unit of rows,
    or its weight's band, takes the fp32 matrix instructions.  For the finite value the operands that it meets are scaled by
    2^-126, which keeps the products near 1.  Rows that it does not reach keep the accuracy of fp32 sums of 128 terms; those
    that an infinity reaches are not finite."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    N, T, R, src, dst, rel, ntype, p = _wide_case(801, tied)
    u, c, finite = 130, 7, np.isfinite(value)
    if where == "X":
        if finite:
            for k in ("Wk", "Wq", "Wv"):
                p[k][:, c] *= np.float32(2.0 ** -126)
        p["X"][u, c] = value
        reached = (dst[:, None] == np.arange(N))[src == u].any(0) | (np.arange(N) == u)      # as a source or on its own as a destination
        reached &= np.isin(np.arange(N), dst)
    else:
        if finite:
            p["X"][:, c] *= np.float32(2.0 ** -126)
        p["Wv"][0, c, 9] = value
        reached = (dst[:, None] == np.arange(N))[ntype[src] == 0].any(0)
    g = Graph(N, R, src, dst, rel, ntype, T)
    L = HgtLayer(g, 128, 4)
    L.load(*[p[k] for k in NAMES], dOut=p["dOut"])
    L.fwd()
    torch.cuda.synchronize()
    got = L.out.cpu().numpy().astype(np.float64)
    if not finite:
        p[where][(u, c) if where == "X" else (0, c, 9)] = 0
    want = O.hgt_fwd(N, src, dst, rel, ntype, *[p[k] for k in NAMES])
    ok = np.full(N, True) if finite else ~reached
    assert ok.sum() > 0 and reached.sum() > 0
    check(got[ok], want[ok], 128 * 2.0 ** -24, "out")
    if not finite:
        assert (~np.isfinite(got[reached])).any(1).all()
    g.close()


@pytest.mark.parametrize("far", [-60.3, -20.7])
def test_small_attention_weights(far):
    """fp32: an edge far below the maximum, whose weight shows in a column that only its message has.  Identity weights make
    the logit the product of the first columns (mu undoes the scale), so the oracle's value is a few exponentials; the
    result is off by the exponential's last place, and one rounding per product, quotient and sum on the way: 16 * 2^-24.
    Destinations of one batch, of a wavefront's batches, and cut ones whose far edges share a piece with the near ones or not."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    d, H = 64, 4
    lists = ["ab", "aaaab", "a" * 29 + "bb", "a" * 64 + "b" * 6, "ab" * 20 + "a" * 60]
    N, big = 2 + len(lists), np.float32(2.0 ** 80)
    src = np.array([0 if c == "a" else 1 for w in lists for c in w], np.int32)
    dst = np.repeat(np.arange(2, N, dtype=np.int32), [len(w) for w in lists])
    X = np.zeros((N, d), np.float32)
    X[1, 0], X[1, 1], X[2:, 0] = far, big, 1
    I = np.eye(d, dtype=np.float32)[None]
    i = np.tile(np.eye(d // H, dtype=np.float32), (1, H, 1, 1))
    dOut = np.zeros((N, d), np.float32)
    dOut[2:, 1] = 1
    g = Graph(N, 1, src, dst, np.zeros(len(src), np.int32))
    L = HgtLayer(g, d, H)
    L.load(X, I, I, I, I, i, i, np.full((1, H), np.sqrt(d // H), np.float32), dOut)
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    w = np.exp(np.float64(np.float32(far)))
    att = np.array([w * k.count("b") / (k.count("a") + w * k.count("b")) for k in lists])
    out = L.out.cpu().numpy().astype(np.float64)[2:, 1]
    assert (np.abs(out - att * big) <= 16 * 2.0 ** -24 * att * big).all(), out / (att * big) - 1
    got = float(L.dX[1, 1])                                # the sum of the far edges' weights
    assert abs(got - att.sum()) <= 16 * 2.0 ** -24 * att.sum(), got / att.sum() - 1
    g.close()


@pytest.mark.parametrize("d,H", [(32, 1), (64, 4), (128, 2)])
def test_sums_of_the_unfolding(d, H):
    """fp32: dWmsg and dWv from the gradient of the folded weight, here all ones (one edge, X and dOut of ones), in sums of a
    2^24, where a unit in the last place is 2, and ones: four chains, or steps of four, lose at most one per addition."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    dh = d // H
    g = Graph(2, 1, np.zeros(1, np.int32), np.ones(1, np.int32), np.zeros(1, np.int32))
    L = HgtLayer(g, d, H)
    I = np.eye(d, dtype=np.float32)[None]
    Wv, Wmsg = np.ones((1, d, d), np.float32), np.ones((1, H, dh, dh), np.float32)
    Wv[0, 0] = 2.0 ** 24
    Wmsg[0, :, :, 0] = 2.0 ** 24
    L.load(np.ones((2, d), np.float32), np.zeros_like(I), I, Wv, I, np.ones_like(Wmsg), Wmsg, None, np.ones((2, d), np.float32))
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    assert (L.dWmsg.double() - (2.0 ** 24 + d - 1)).abs().max().item() <= d // 4 + 2
    assert (L.dWv.double() - (2.0 ** 24 + dh - 1)).abs().max().item() <= dh // 4 + 2
    g.close()


@pytest.mark.parametrize("d,H", [(32, 1), (64, 4), (128, 2)])
def test_sums_of_rows_in_batches(d, H):
    """fp32: a destination of 24 edges (equal logits) and a pair of 24 edges (one to each of 24 destinations) sum a 2^24, where a
    unit in the last place is 2, and 23 ones, in batches of four: the first batch loses at most one, the others none.  The
    destination's sum is then divided by 24: two more roundings."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    n = 24
    N = 2 * n + 2                                         # sources 0..n-1, their destination n, pair's source n + 1, its destinations
    src = np.concatenate([np.arange(n), np.full(n, n + 1)]).astype(np.int32)
    dst = np.concatenate([np.full(n, n), np.arange(n + 2, N)]).astype(np.int32)
    X, dOut = np.zeros((N, d), np.float32), np.zeros((N, d), np.float32)
    X[:n, 0], dOut[n + 2:, 0] = 1, 1
    X[0, 0] = dOut[n + 2, 0] = 2.0 ** 24
    I = np.eye(d, dtype=np.float32)[None]
    i = np.tile(np.eye(d // H, dtype=np.float32), (1, H, 1, 1))
    g = Graph(N, 1, src, dst, np.zeros(2 * n, np.int32))
    L = HgtLayer(g, d, H)
    L.load(X, np.zeros_like(I), I, I, I, i, i, None, dOut)
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    want = (2.0 ** 24 + n - 1) / n
    assert abs(float(L.out[n, 0]) - want) <= 1.0 / n + 2 * 2.0 ** -24 * want, float(L.out[n, 0]) - want
    assert abs(float(L.dX[n + 1, 0].double()) - (2.0 ** 24 + n - 1)) <= 1, float(L.dX[n + 1, 0])
    g.close()


@pytest.mark.parametrize("dtype,d,H", [("f32", 32, 1), ("f32", 64, 4), ("f32", 128, 2), ("bf16", 128, 4), ("bf16", 128, 8)])
def test_messages_near_the_top_of_the_range(dtype, d, H):
    """Destinations of 1 to 700 edges (one batch, a wavefront's batches, two pieces, many pieces) whose messages are all 2^126 in
    one column: so is their mean, although four of them exceed fp32.  It may be off by roundings, 8 * 2^-24 in fp32 and one
    of bf16.  With one edge a message near the bottom, 3 * 2^-127, passes unchanged."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    lengths = [1, 2, 3, 4, 5, 7, 24, 29, 32, 33, 40, 300, 700]
    N = len(lengths) + 3
    dst = np.append(np.repeat(np.arange(len(lengths)), lengths), N - 3).astype(np.int32)
    src = np.full(len(dst), N - 2, np.int32)
    src[-1] = N - 1
    X = np.zeros((N, d), np.float32)
    X[N - 2, 0], X[N - 1, 0] = 2.0 ** 126, 3 * 2.0 ** -127
    I = np.eye(d, dtype=np.float32)[None]
    i = np.tile(np.eye(d // H, dtype=np.float32), (1, H, 1, 1))
    g = Graph(N, 1, src, dst, np.zeros(len(src), np.int32))
    L = HgtLayer(g, d, H, dtype=dtype)
    L.load(X, np.zeros_like(I), np.zeros_like(I), I, I, i, i, None)
    L.fwd()
    torch.cuda.synchronize()
    got = L.out.cpu().numpy().astype(np.float64)[:, 0]
    tol = 2.0 ** -8 if dtype == "bf16" else 8 * 2.0 ** -24
    assert (np.abs(got[:len(lengths)] * 2.0 ** -126 - 1) <= tol).all(), got
    assert got[N - 3] == 3 * 2.0 ** -127
    g.close()


@pytest.mark.parametrize("dtype,d,H", [("bf16", 128, 8), ("bf16", 128, 2), ("f32", 64, 4)])
def test_logits_of_minus_infinity(dtype, d, H):
    """Edges whose logit overflows to minus infinity weigh nothing, also where they fill a destination's first batch, a lane
    group's share of a long item, or a whole piece of a cut destination: the result is the other edges' message, 5."""
    import torch
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    lists = ["aaaab", "a" * 8 + "bbb", "a" * 26 + "bbbb", "a" * 40 + "bbbb", "a" * 70 + "b", "a" * 64 + "b" * 90, "ab"]
    N = 2 + len(lists)
    src = np.array([0 if c == "a" else 1 for w in lists for c in w], np.int32)
    dst = np.repeat(np.arange(2, N, dtype=np.int32), [len(w) for w in lists])
    X = np.zeros((N, d), np.float32)
    X[0, 0], X[2:, 0], X[0, 1], X[1, 1] = -2.0 ** 70, 2.0 ** 64, 3, 5
    I = np.eye(d, dtype=np.float32)[None]
    i = np.tile(np.eye(d // H, dtype=np.float32), (1, H, 1, 1))
    dOut = np.zeros((N, d), np.float32)
    dOut[2:, 1] = 1
    g = Graph(N, 1, src, dst, np.zeros(len(src), np.int32))
    L = HgtLayer(g, d, H, dtype=dtype)
    L.load(X, I, I, I, I, i, i, None, dOut)
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    out = L.out.cpu().numpy()
    assert (np.abs(out[2:, 1] - 5) <= 5 * 8 * 2.0 ** -24).all(), out[2:, 1]
    dX = L.dX.cpu().numpy()
    assert dX[0, 1] == 0 and abs(dX[1, 1] - len(lists)) <= 2.0 ** -7 * len(lists), dX[:2, 1]
    g.close()


def test_scaled_config4_bf16():
    c = synth.config(4, scale=0.01)          # 20k nodes, 200k edges, 8 node types, 30 relations, d=128, H=4
    c["mu"] = None
    _run(c["N"], c["T"], c["R"], c["src"], c["dst"], c["rel"], c["ntype"], c, 128, 4, "C4/100", dtype="bf16")


@pytest.mark.timeout(1100)
def test_config4_full_size_bf16():
    """2M nodes of 8 types, 30 relations, 20M edges, hidden 128 in 4 heads, bf16 inputs."""
    c = synth.config(4)
    c["mu"] = None
    _run(c["N"], c["T"], c["R"], c["src"], c["dst"], c["rel"], c["ntype"], c, 128, 4, "C4", dtype="bf16", repeat=False)
