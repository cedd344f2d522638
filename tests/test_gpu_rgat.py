"""RGAT layer (forward + backward) on the GPU vs the CPU oracle."""
import numpy as np
import pytest

from oracle import layers as O
from oracle import graph_index
from paper_2412_04747_amd import synth
from parity import check, TOL_F32

pytestmark = pytest.mark.gpu


def _run(N, R, src, dst, rel, p, d, tag, slope=0.2, check_saved=True, dtype="f32", d_in=None):
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    from parity import TOL_BF16
    print(f"rgat case {tag}: N={N} R={R} E={len(src)} d={d} {dtype}", flush=True)
    TOL_F32 = TOL_BF16 if dtype == "bf16" else 1e-4        # the tolerance of this case, under the name used below
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d, slope, dtype=dtype, d_in=d_in)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    L.fwd()
    torch.cuda.synchronize()
    want, alpha, z = O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], slope, want_alpha=True)
    check(L.out, want, TOL_F32, "out")
    if check_saved and len(src):
        ix = graph_index.build(N, R, src, dst, rel)
        hs, s_dst, ms = (t.cpu().numpy() for t in L.saved_views())
        s_dst, ms = s_dst[:, 0], ms[:, 0]
        # what the forward keeps: the destination half of the logit per run, and per destination the
        # maximum m of the leaky-ReLU logits and s = sum exp(l - m); the backward rebuilds att from them
        X64, W64 = p["X"].astype(np.float64), p["W"].astype(np.float64)
        ht = np.einsum("qi,qij->qj", X64[ix["run_dst"]], W64[ix["run_rel"]])
        check(s_dst, (ht * p["w_t"].astype(np.float64)[ix["run_rel"]]).sum(1), TOL_F32, "s_dst")
        zz = z[ix["in_eid"]]                                   # logits in CSR order
        l = np.where(zz > 0, zz, slope * zz)
        deg = np.diff(ix["in_ptr"])
        has = deg > 0
        m_want = np.maximum.reduceat(l, ix["in_ptr"][:-1][has])
        s_want = np.add.reduceat(np.exp(l - np.repeat(m_want, deg[has])), ix["in_ptr"][:-1][has])
        assert np.abs(ms[has, 0] - m_want).max() <= TOL_F32 * max(np.abs(l).max(), 1.0)
        check(ms[has, 1], s_want, TOL_F32, "softmax sum")
        v_of = np.repeat(np.arange(N), deg)
        check(np.exp(l - ms[v_of, 0].astype(np.float64)) / ms[v_of, 1], alpha[ix["in_eid"]], TOL_F32, "att from (m, s)")
        pair_hs = np.einsum("pi,pij->pj", p["X"].astype(np.float64)[ix["pair_src"]], p["W"].astype(np.float64)[ix["pair_rel"]])
        check(hs, pair_hs, TOL_F32, "Hs")
    L.bwd()
    torch.cuda.synchronize()
    wg = O.rgat_bwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"], slope)
    errs = {k: check(v, wg[k], TOL_F32, k) for k, v in L.grads().items()}
    print("   max rel errors:", {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    # determinism: a second run gives bit-identical results (no atomics anywhere)
    first = {k: v.clone() for k, v in L.grads().items()}
    out1 = L.out.clone()
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    assert torch.equal(out1, L.out)
    for k, v in L.grads().items():
        assert torch.equal(first[k], v), k
    g.close()


@pytest.mark.parametrize("d", [32, 64, 128])
def test_small_random(d):
    rng, src, dst, rel, _ = synth.tiny(60 + d, N=500, R=6, E=4000)
    p = synth.rgat_params(rng, 500, 6, d, d)
    _run(500, 6, src, dst, rel, p, d, f"small-d{d}")


@pytest.mark.parametrize("d_in,d", [(32, 64), (64, 32)])
def test_input_width_differs_from_output_width(d_in, d):
    rng, src, dst, rel, _ = synth.tiny(75 + d, N=700, R=6, E=6000)
    dst[:900] = 11                                   # a hub cut into pieces
    src[900:1300] = 3; rel[900:1300] = 2             # one pair with many edges
    p = synth.rgat_params(rng, 700, 6, d_in, d)
    _run(700, 6, src, dst, rel, p, d, f"widths-{d_in}-{d}", d_in=d_in)


@pytest.mark.parametrize("d", [64, 128])
def test_single_head_bf16_inputs(d):
    """bf16 X, W, w_s, w_t, dOut (rounded once on the host; the oracle consumes the rounded values in fp64),
    fp32 sums and fp32 results: single-head RGAT against the oracle at the bf16 tolerance."""
    rng, src, dst, rel, _ = synth.tiny(90 + d, N=600, R=5, E=5000)
    dst[:900] = 7                                    # a hub cut into pieces
    p = {k: synth.round_to_bf16(v) for k, v in synth.rgat_params(rng, 600, 5, d, d).items()}
    _run(600, 5, src, dst, rel, p, d, f"bf16-d{d}", dtype="bf16")


def test_more_relations_than_a_grid_dimension_holds():
    """70,000 relations, nearly all without an edge: per-relation launches must not put the relation index on a grid
    dimension limited to 65,535, and w_s (9 MB) no longer fits in LDS, so the fused walks read it through the caches."""
    N, R, E, d = 300, 70000, 3000, 32
    rng = np.random.default_rng(97)
    src, dst = rng.integers(0, N, E).astype(np.int32), rng.integers(0, N, E).astype(np.int32)
    rel = rng.choice(np.array([0, 1, 65534, 65535, 65536, 69999]), E).astype(np.int32)
    dst[:700] = 5
    p = synth.rgat_params(rng, N, R, d, d)
    _run(N, R, src, dst, rel, p, d, "R=70000", check_saved=False)


def test_many_single_edge_destinations():
    """Thousands of destinations with exactly one incoming edge (softmax weight 1) next to a few
    busier ones: the batched single-entry aggregation path."""
    rng = np.random.default_rng(79)
    N, R, d = 12000, 5, 64
    more = np.repeat(np.arange(5000), rng.integers(1, 4, 5000))         # 5000 nodes with 2..4 incoming edges
    dst = np.concatenate([rng.permutation(N), more, rng.integers(0, 60, 800)]).astype(np.int32)
    src = rng.integers(0, N, len(dst)).astype(np.int32)
    rel = rng.integers(0, R, len(dst)).astype(np.int32)
    src[N:N + 6000] = src[:6000]; rel[N:N + 6000] = rel[:6000]          # 6000 pairs with two edges (backward short path)
    p = synth.rgat_params(rng, N, R, d, d)
    _run(N, R, src, dst, rel, p, d, "singles")


def _run_heads(N, R, src, dst, rel, p, d, H, tag, dtype="f32", slope=0.2, flags=0, d_in=None):
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    from parity import TOL_BF16
    print(f"rgat case {tag}: N={N} R={R} E={len(src)} d={d} heads={H} {dtype}", flush=True)
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d, slope, dtype=dtype, heads=H, flags=flags, d_in=d_in)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    L.fwd()
    torch.cuda.synchronize()
    want, alpha, z = O.rgat_heads_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], H, slope, want_alpha=True)
    check(L.out, want, tol, "out")
    ix = graph_index.build(N, R, src, dst, rel)
    # the backward rebuilds the attention weights from what the forward keeps: (max, sum) per (destination, head)
    _, _, ms = (t.cpu().numpy().astype(np.float64) for t in L.saved_views())
    zz = z[ix["in_eid"]]                                   # [E, H] logits in CSR order
    l = np.where(zz > 0, zz, slope * zz)
    v_of = np.repeat(np.arange(N), np.diff(ix["in_ptr"]))
    check(np.exp(l - ms[v_of, :, 0]) / ms[v_of, :, 1], alpha[ix["in_eid"]], tol, "att from (m, s)")
    L.bwd()
    torch.cuda.synchronize()
    wg = O.rgat_heads_bwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"], H, slope)
    errs = {k: check(v, wg[k], tol, k) for k, v in L.grads().items()}
    print("   max rel errors:", {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    first = {k: v.clone() for k, v in L.grads().items()}
    out1 = L.out.clone()
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    assert torch.equal(out1, L.out)
    for k, v in L.grads().items():
        assert torch.equal(first[k], v), k
    g.close()


@pytest.mark.parametrize("d,H", [(64, 2), (64, 4), (128, 8), (32, 2), (128, 2)])
def test_multi_head(d, H):
    rng, src, dst, rel, _ = synth.tiny(160 + d + H, N=800, R=6, E=7000)
    dst[:1200] = 4                                   # a hub cut into pieces
    src[:300] = 9; rel[:300] = 2                     # one pair with many edges
    p = synth.rgat_params(rng, 800, 6, d, d)
    _run_heads(800, 6, src, dst, rel, p, d, H, f"heads-d{d}-H{H}")


@pytest.mark.parametrize("d,H", [(64, 4), (32, 2)])
def test_multi_head_rows_written_per_pair(d, H):
    # the schedule without the row selector: every pair's gradient row is stored, also for the pairs with one edge
    rng, src, dst, rel, _ = synth.tiny(190 + d + H, N=800, R=6, E=7000)
    dst[:1200] = 4
    src[:300] = 9; rel[:300] = 2
    p = synth.rgat_params(rng, 800, 6, d, d)
    _run_heads(800, 6, src, dst, rel, p, d, H, f"heads-d{d}-H{H}-noselect", flags=4)       # RGNN_FLAG_NO_ROW_SELECT


@pytest.mark.parametrize("d_in,d,H,flags", [(32, 64, 4, 0), (64, 32, 2, 0), (32, 64, 2, 4)])
def test_multi_head_input_width_differs(d_in, d, H, flags):
    rng, src, dst, rel, _ = synth.tiny(195 + d + H, N=800, R=6, E=7000)
    dst[:1200] = 4
    src[:300] = 9; rel[:300] = 2
    p = synth.rgat_params(rng, 800, 6, d_in, d)
    _run_heads(800, 6, src, dst, rel, p, d, H, f"heads-{d_in}-{d}-H{H}-flags{flags}", flags=flags, d_in=d_in)


@pytest.mark.parametrize("d,H", [(32, 1), (32, 2), (64, 1), (64, 2), (64, 4), (128, 1), (128, 8)])
def test_node_with_runs_of_many_relations(d, H):
    """Destinations with runs of 1, 9, 17, 33 and 90 relations among neighbours with few: the shared walk of the run term (more
    than eight batches of 1, 2 or 4 runs) and the lone one, in a last wavefront that is not full."""
    N, R = 203, 90
    rng = np.random.default_rng(197 + d + H)
    parts = [(v, np.arange(n)) for v, n in ((5, 90), (6, 33), (7, 17), (8, 9), (9, 1), (120, 90), (202, 70), (201, 34))]
    dst = np.concatenate([np.full(len(r), v) for v, r in parts] + [rng.integers(0, N, 600)]).astype(np.int32)
    rel = np.concatenate([r for _, r in parts] + [rng.integers(0, R, 600)]).astype(np.int32)
    src = rng.integers(0, N, len(dst)).astype(np.int32)
    p = synth.rgat_params(rng, N, R, d, d)
    _run_heads(N, R, src, dst, rel, p, d, H, f"many-runs-d{d}-H{H}")


def test_multi_head_bf16_inputs_and_empty_relation():
    rng, src, dst, rel, _ = synth.tiny(171, N=600, R=5, E=5000)
    rel[rel == 3] = 1                                # relation 3 has no edge
    p = {k: synth.round_to_bf16(v) for k, v in synth.rgat_params(rng, 600, 5, 64, 64).items()}
    _run_heads(600, 5, src, dst, rel, p, 64, 4, "heads-bf16", dtype="bf16")


def test_multi_head_scaled_config3():
    c = synth.config(3, scale=0.02)                  # 20k nodes, 200k edges, 200 relations, power-law in-degree
    _run_heads(c["N"], c["R"], c["src"], c["dst"], c["rel"], c, 64, 4, "heads-C3/50")


def test_config2():
    c = synth.config(2)
    _run(c["N"], c["R"], c["src"], c["dst"], c["rel"], c, 64, "C2")


@pytest.mark.timeout(900)
def test_config3_full_size():
    """The benchmark's workload (10M edges, 200 relations, hubs of in-degree 50k), every output
    element against the oracle."""
    c = synth.config(3)
    _run(c["N"], c["R"], c["src"], c["dst"], c["rel"], c, 64, "C3", check_saved=False)


@pytest.mark.timeout(900)
def test_pair_tensors_of_more_than_2_to_32_elements():
    """72M edges over 4M nodes and 200 relations, nearly all (source, relation) pairs distinct: the
    per-pair tensors hold 68.8M rows of 64, more than 2^32 elements, so any 32-bit element index
    would wrap.  The leaky ReLU has a kink at z = 0: an edge whose logit is within fp32 rounding of
    0 may take the other branch on the GPU, which changes its gradient by a finite amount.  Such
    edges (|z| < 1e-5 by the oracle, a few hundred of 72M) are left out of the graph, so the rest is
    compared at the usual tolerance."""
    N, R, E, d = 4_000_000, 200, 72_000_000, 64
    rng = np.random.default_rng(4242)
    src, dst, rel = (rng.integers(0, n, E, dtype=np.int32) for n in (N, N, R))
    p = synth.rgat_params(rng, N, R, d, d)
    print("large case: generated", flush=True)
    _, _, z = O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], 0.2, want_alpha=True)
    keep = np.abs(z) >= 1e-5
    print(f"large case: {int((~keep).sum())} edges at the kink left out", flush=True)
    assert (~keep).sum() < 2000
    src, dst, rel = src[keep], dst[keep], rel[keep]
    assert len(np.unique(src.astype(np.int64) * R + rel)) * d > 2 ** 32
    _run(N, R, src, dst, rel, p, d, "beyond-2^32", check_saved=False)


@pytest.mark.parametrize("d", [32, 64, 128])
def test_edge_parallel_aggregation_flag(d):
    """The comparison schedule of the forward aggregation (atomic adds per edge): same result within the
    fp32 tolerance (the order of the additions is not fixed), backward unchanged."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    N, R, E = 600, 5, 6000
    rng, src, dst, rel, _ = synth.tiny(71 + d, N=N, R=R, E=E)
    dst[:2000] = 17                                    # a hub: thousands of atomic adds on one row
    p = synth.rgat_params(rng, N, R, d, d)
    print(f"rgat case edge-parallel d={d}", flush=True)
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d, flags=B.RGNN_FLAG_EDGE_PARALLEL_AGGREGATION)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    check(L.out, O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"]), TOL_F32, "out")
    wg = O.rgat_bwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    for k, v in L.grads().items():
        check(v, wg[k], TOL_F32, k)
    with pytest.raises(B.RgnnError):                   # not with several heads
        RgatLayer(g, d, heads=2, flags=B.RGNN_FLAG_EDGE_PARALLEL_AGGREGATION)
    g.close()


@pytest.mark.parametrize("n_hub", [33, 1025, 1700])
@pytest.mark.parametrize("d,H", [(32, 1), (64, 1), (128, 1), (64, 4), (64, 2), (128, 8)])
def test_one_segment_of_many_pieces(d, H, n_hub):
    """One destination and one (source, relation) pair hold most edges and are cut into 2 to 54 pieces, so that the pieces'
    sums are formed by small workgroups or, beyond 32 pieces per cut segment, by large ones on column ranges."""
    rng = np.random.default_rng(900 + n_hub)
    N, R, E = 60, 3, 2 * n_hub + 100
    src, dst, rel = (rng.integers(0, n, E).astype(np.int32) for n in (N, N, R))
    dst[:n_hub] = 7
    src[n_hub:2 * n_hub] = 11; rel[n_hub:2 * n_hub] = 2
    p = synth.rgat_params(rng, N, R, d, d)
    if H == 1:
        _run(N, R, src, dst, rel, p, d, f"pieces-d{d}-{n_hub}")
    else:
        _run_heads(N, R, src, dst, rel, p, d, H, f"pieces-d{d}-H{H}-{n_hub}")


@pytest.mark.parametrize("d,H", [(32, 2), (64, 1), (64, 4), (128, 1)])
def test_relations_of_many_run_pieces(d, H):
    """Relations whose run lists are cut at 32 runs: whole ones, and 2, 127, 128, 129 and 1025 pieces (64 lane groups sum a
    relation's pieces, four at a time)."""
    runs = [1, 32, 33, 127 * 32, 128 * 32, 128 * 32 + 1, 1024 * 32 + 7]
    N, R = max(runs), len(runs) + 1                                   # the last relation has no edge
    rng = np.random.default_rng(d + H)
    dst = np.concatenate([rng.permutation(N)[:n] for n in runs]).astype(np.int32)
    rel = np.repeat(np.arange(len(runs), dtype=np.int32), runs)
    src = rng.integers(0, N, len(dst)).astype(np.int32)
    p = synth.rgat_params(rng, N, R, d, d)
    if H == 1:
        _run(N, R, src, dst, rel, p, d, "run-pieces", check_saved=False)
    else:
        _run_heads(N, R, src, dst, rel, p, d, H, "run-pieces")


@pytest.mark.parametrize("H", [1, 4])
def test_overflowing_piece_of_a_cut_destination(H):
    """A destination of five pieces whose last one sums messages of 3e38 to infinity: infinity it stays (not NaN), in that
    column alone.  With w_s = w_t = 0 the other columns are the mean of their messages."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    d, n = 64, 150
    src, dst = np.zeros(n, np.int32), np.full(n, 3, np.int32)
    src[-8:] = 1
    X, W = np.zeros((4, d), np.float32), np.eye(d, dtype=np.float32)[None]
    X[0, 1] = X[1, 1] = 1
    X[1, 0] = 3e38
    w = np.zeros((1, d), np.float32)
    g = Graph(4, 1, src, dst, np.zeros(n, np.int32))
    L = RgatLayer(g, d, heads=H)
    L.load(X, W, w, w)
    L.fwd()
    torch.cuda.synchronize()
    got = L.out.cpu().numpy()[3]
    assert got[0] == np.inf and abs(got[1] - 1) <= 8 * 2.0 ** -24 and (got[2:] == 0).all(), got[:4]
    g.close()


def test_hub_empty_relation_isolated_nodes():
    rng, src, dst, rel, _ = synth.tiny(70, N=300, R=5, E=4000)
    rel[rel == 4] = 0       # relation 4 has no edge
    dst[:2500] = 11         # hub cut into many items; most nodes isolated
    src[:700] = 2           # a (src, rel) pair with hundreds of outgoing edges (cut pair-major segment)
    rel[:700] = 1
    p = synth.rgat_params(rng, 300, 5, 64, 64)
    _run(300, 5, src, dst, rel, p, 64, "hub")


def test_single_edge_and_empty():
    rng = np.random.default_rng(3)
    p = synth.rgat_params(rng, 5, 2, 64, 64)
    _run(5, 2, np.array([1], np.int32), np.array([3], np.int32), np.array([1], np.int32), p, 64, "one-edge")
    e = np.zeros(0, np.int32)
    _run(5, 2, e, e, e, p, 64, "empty", check_saved=False)


def test_edge_order_invariance_is_bitwise():
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    rng, src, dst, rel, _ = synth.tiny(80, N=200, R=4, E=2000)
    p = synth.rgat_params(rng, 200, 4, 64, 64)
    perm = rng.permutation(len(src))
    res = []
    for s, d_, r in ((src, dst, rel), (src[perm], dst[perm], rel[perm])):
        g = Graph(200, 4, s, d_, r)
        L = RgatLayer(g, 64)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
        L.fwd(); L.bwd()
        torch.cuda.synchronize()
        res.append([L.out.clone()] + [v.clone() for v in L.grads().values()])
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.timeout(300)
def test_more_parameters_than_one_row_of_workgroups():
    """4.2M relations, 32 -> 64 columns, and 8.38M, 32 -> 32: the launches that sum the weight gradient's shares and finish the parameter
    gradients have more workgroups of 256 threads than 2^32 lanes hold.  Fifty relations have edges; the gradients of the others are
    zero."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph
    rng = np.random.default_rng(88)
    N, E, used = 40000, 4000, 50
    for R, k, d in ((4_200_000, 32, 64), (8_388_000, 32, 32)):
        print(f"rgat case many parameters: R={R} {k}->{d}", flush=True)
        ids = np.sort(np.concatenate([[0, R - 1], rng.choice(np.arange(1, R - 1), used - 2, replace=False)]))
        src, dst = rng.integers(0, N, E).astype(np.int32), rng.integers(0, N, E).astype(np.int32)
        few = rng.integers(0, used, E).astype(np.int32)
        p = synth.rgat_params(rng, N, used, k, d)
        g = Graph(N, R, src, dst, ids[few].astype(np.int32))
        desc = B.make_desc(B.RGNN_F32, k, d, 1, 0.2)
        f, b, s = B.rgnn_workspace_bytes(g.handle, B.RGNN_LAYER_RGAT, desc)
        at = torch.as_tensor(ids, device="cuda")
        dev = lambda a: torch.from_numpy(a).cuda()
        def spread(a):
            t = torch.zeros((R,) + a.shape[1:], device="cuda")
            t[at] = dev(a)
            return t
        X, dO, W, ws, wt = dev(p["X"]), dev(p["dOut"]), spread(p["W"]), spread(p["w_s"]), spread(p["w_t"])
        e = lambda *shape: torch.full(shape, 7.0, device="cuda")
        out, dX, dW, dws, dwt = e(N, d), e(N, k), e(R, k, d), e(R, d), e(R, d)
        work, saved = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (max(f, b), s))
        B.rgnn_rgat_fwd(g.handle, desc, X, W, ws, wt, out, saved, work)
        B.rgnn_rgat_bwd(g.handle, desc, X, W, ws, wt, out, saved, dO, dX, dW, dws, dwt, work)
        torch.cuda.synchronize()
        a = (N, src, dst, few, p["X"], p["W"], p["w_s"], p["w_t"])
        check(out, O.rgat_fwd(*a), TOL_F32, "out")
        want = O.rgat_bwd(*a, p["dOut"])
        check(dX, want["dX"], TOL_F32, "dX")
        for name, got in (("dW", dW), ("dw_s", dws), ("dw_t", dwt)):
            check(got[at], want[name], TOL_F32, name)
            got[at] = 0
            for part in got.view(R, -1).split(1 << 20):
                assert not part.any(), name
        g.close()
        del X, dO, W, ws, wt, out, dX, dW, dws, dwt, work, saved, got, part
        torch.cuda.empty_cache()


@pytest.mark.timeout(300)
def test_more_folded_weights_than_a_launch_of_512_threads_holds():
    """2.1M relations of width 128, 137 GB of weights: the workgroups that fold them are more than 2^32 lanes hold at the 512 threads of the
    forward product, with which they share a launch where they are fewer.  Forty relations have edges."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph
    rng = np.random.default_rng(89)
    N, E, used, R, d = 3000, 4000, 40, 2_097_200, 128
    ids = np.sort(np.concatenate([[0, R - 1], rng.choice(np.arange(1, R - 1), used - 2, replace=False)]))
    src, dst = rng.integers(0, N, E).astype(np.int32), rng.integers(0, N, E).astype(np.int32)
    few = rng.integers(0, used, E).astype(np.int32)
    p = synth.rgat_params(rng, N, used, d, d)
    print(f"rgat case many folds: R={R} d={d}", flush=True)
    g = Graph(N, R, src, dst, ids[few].astype(np.int32))
    desc = B.make_desc(B.RGNN_F32, d, d, 1, 0.2)
    f, _, s = B.rgnn_workspace_bytes(g.handle, B.RGNN_LAYER_RGAT, desc)
    at = torch.as_tensor(ids, device="cuda")
    def spread(a):
        t = torch.zeros((R,) + a.shape[1:], device="cuda")
        t[at] = torch.from_numpy(a).cuda()
        return t
    X, W, ws, wt = torch.from_numpy(p["X"]).cuda(), spread(p["W"]), spread(p["w_s"]), spread(p["w_t"])
    out = torch.full((N, d), 7.0, device="cuda")
    work, saved = (torch.zeros(n, dtype=torch.uint8, device="cuda") for n in (f, s))
    B.rgnn_rgat_fwd(g.handle, desc, X, W, ws, wt, out, saved, work)
    torch.cuda.synchronize()
    check(out, O.rgat_fwd(N, src, dst, few, p["X"], p["W"], p["w_s"], p["w_t"]), TOL_F32, "out")
    g.close()
    del X, W, ws, wt, out, work, saved
    torch.cuda.empty_cache()


@pytest.mark.parametrize("R,tiles,apart", [(200, 1, False), (400, 1, True), (400, 1000, False)])
def test_folds_of_width_128_apart_from_the_product(R, tiles, apart):
    """The weight folds of the forward share the product's launch, unless there are many and its chunks hold about as many relations
    each (`tiles`: row tiles of relation 0, the others have one)."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    rng = np.random.default_rng(R + tiles)
    N, d = 64 * max(tiles, 8), 128
    rel = np.concatenate([np.repeat(np.arange(R), 3), np.zeros(64 * tiles - 3)]).astype(np.int32)
    src = np.concatenate([rng.integers(0, N, 3 * R), np.arange(64 * tiles - 3)]).astype(np.int32)
    dst = rng.integers(0, N, len(rel)).astype(np.int32)
    p = synth.rgat_params(rng, N, R, d, d)
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    B.rgnn_profile_start()
    L.fwd()
    assert ("fold_weight" in B.rgnn_profile_stop()) == apart
    check(L.out, O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"]), TOL_F32, "out")
    g.close()
