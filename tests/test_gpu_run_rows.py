"""Layers whose rows are kept per (destination, relation) run (large graphs with fewer runs than pairs) against the oracle."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2412_04747_amd import synth
from parity import check, TOL_F32
from test_gpu_hipgraph import _capture_and_replay
from test_gpu_workspace_bounds import _guarded, _intact

pytestmark = pytest.mark.gpu


def _graph(seed, E):
    """Destinations of 1 to thousands of edges, runs of one edge and of hundreds (cut into pieces), a hub source, and relations without
    an edge (11), with single-edge runs only (12), with runs of several edges only (13), with one run (14)."""
    rng = np.random.default_rng(seed)
    N, R = 9001 if E < 400000 else 40009, 15
    src = rng.integers(0, N, E)
    dst = (N * rng.random(E) ** 3).astype(np.int64)
    rel = rng.integers(0, 11, E)
    dst[:E // 16] = 5                                        # hub destination: runs and run lists
    src[E // 16:E // 8] = 7                                  # hub source
    rel[-400:-200] = 12; dst[-400:-200] = np.arange(200)
    rel[-200:-4] = 13; dst[-200:-4] = np.arange(196) // 2
    rel[-4:] = 14; dst[-4:] = 4000
    mix = rng.permutation(E)
    return N, R, *(a[mix].astype(np.int32) for a in (src, dst, rel)), rng


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("k,d,dtype,norm,act,loop,flags", [
    (32, 64, "f32", "in_degree_per_rel", "relu", True, 0), (64, 32, "f32", "none", "none", False, 32),
    (64, 64, "f32", "in_degree_per_rel", "none", True, 32), (32, 32, "f32", "none", "none", True, 0),
    (64, 64, "bf16", "in_degree_per_rel", "none", False, 0),
    (128, 128, "f32", "in_degree_per_rel", "none", False, 0), (128, 128, "f32", "none", "relu", True, 32)])
def test_rgcn(k, d, dtype, norm, act, loop, flags, saved):
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    E = 260011 if d in (32, 128) else 140003
    N, R, src, dst, rel, rng = _graph(31 + k + d, E)
    print(f"run rows rgcn {k}->{d} {dtype} {norm} {act} loop={loop} flags={flags} saved={saved}", flush=True)
    p = synth.rgcn_params(rng, N, R, k, d, self_loop=loop)
    tol = TOL_F32
    if dtype == "bf16":
        p = {n: v if v is None else synth.round_to_bf16(v) for n, v in p.items()}
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, norm, act, loop, dtype=dtype, flags=flags, d_in=k)
    L.load(p["X"], p["W"], p["W0"], p["dOut"])
    f, b, s = B.rgnn_workspace_bytes(g.handle, B.RGNN_LAYER_RGCN, L.desc)
    assert s > 0
    guards = []
    def area(n):
        big, mid = _guarded(n)
        guards.append(big)
        return mid
    L.saved = area(s) if saved else None
    L.ws = area(f)
    B.rgnn_profile_start()
    L.fwd()
    torch.cuda.synchronize()
    # a forward that keeps nothing takes the rows per pair below 30M elements, and the backward then sums the runs' inputs itself
    assert ("run_inputs" in B.rgnn_profile_stop()) == (saved or E * d >= 30000000)
    want = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], p["W0"], norm, act)
    check(L.out, want, tol, "out")
    if act != "none":                                        # (the mask from the same values on both sides)
        L.out.copy_(torch.from_numpy(np.ascontiguousarray(want, dtype=np.float32)))
    L.ws = area(b)
    for v in L.grads().values():
        v.fill_(1.0)
    B.rgnn_profile_start()
    L.bwd()
    torch.cuda.synchronize()
    assert ("run_inputs" in B.rgnn_profile_stop()) == (not saved)
    wg = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], p["W0"], p["dOut"], norm, act, out=want)
    for n, v in L.grads().items():
        check(v - (1.0 if flags else 0.0), wg[n], tol, n)
    for r in range(R):                                       # by relation: a small one would hide among the others
        check(L.dW[r] - (1.0 if flags else 0.0), wg["dW"][r], 4 * tol, f"dW[{r}]")
    for big in guards:
        _intact(big, "a buffer")
    first = {n: v.clone() for n, v in L.grads().items()}
    for v in L.grads().values():
        v.fill_(1.0)
    L.bwd()
    torch.cuda.synchronize()
    for n, v in L.grads().items():
        assert torch.equal(v, first[n]), n
    g.close()


@pytest.mark.parametrize("N,R,E,dsts,k,d,loop", [
    (3000, 4, 200000, 2500, 64, 64, False), (2000, 8, 140000, 1000, 32, 64, True), (3000, 4, 260000, 1500, 32, 32, False),
    (3000, 4, 260000, 1500, 64, 32, True), (6080, 8, 140000, 80, 64, 64, True)])
def test_rgcn_of_few_destinations(N, R, E, dsts, k, d, loop):
    """Graphs with fewer runs than pairs whose forward is the one launch of a small graph: its backward needs nothing of `saved`."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    rng = np.random.default_rng(N + E + k)
    print(f"run rows rgcn of few destinations N={N} R={R} E={E} {dsts} {k}->{d} loop={loop}", flush=True)
    src, dst, rel = (rng.integers(0, n, E).astype(np.int32) for n in (N, dsts, R))
    p = synth.rgcn_params(rng, N, R, k, d, self_loop=loop)
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, self_loop=loop, d_in=k)
    L.load(p["X"], p["W"], p["W0"], p["dOut"])
    L.saved.fill_(0xFF)
    B.rgnn_profile_start()
    L.fwd()
    L.bwd()
    torch.cuda.synchronize()
    rep = B.rgnn_profile_stop()
    a = (N, src, dst, rel, p["X"], p["W"], p["W0"])
    check(L.out, O.rgcn_fwd(*a), TOL_F32, "out")
    want = O.rgcn_bwd(*a, p["dOut"])
    for n, v in L.grads().items():
        check(v, want[n], TOL_F32, n)
    assert "rgcn_small_fwd" in rep and "run_inputs" not in rep and "aggregate_bwd_pair" in rep
    g.close()


def _popular(d, dtype, positive):
    """500 destinations with a run of 70 edges in each of four relations, every (source, relation) pair with one edge."""
    rng = np.random.default_rng(8)
    N, R = 40000, 4
    rel, dst = (a.ravel().astype(np.int32) for a in np.indices((R, 500, 70))[:2])
    src = np.concatenate([rng.permutation(N)[:35000] for _ in range(R)]).astype(np.int32)
    p = synth.rgcn_params(rng, N, R, d, d, self_loop=False)
    if positive:
        p["X"] = np.abs(p["X"])
    if dtype == "bf16":
        p = {n: v if v is None else synth.round_to_bf16(v) for n, v in p.items()}
    return N, R, src, dst, rel, p


def test_rgcn_rows_in_bf16_stay_per_pair():
    """Rows stored in bf16, of non-negative features: sums are fp32.  A message is rounded to bf16 by up to 2^-9 of it (1.1e-3 rms); 280 of them
    add up to a row of out of about 0.4 times the sum of their magnitudes, so the roundings average to 2e-4 of it (a row of a run in bf16:
    four roundings, 1e-3).  Without 1/c, the gradient row of a pair with one edge is dOut as given, and the products in dW are exact: fp32
    sums of 35000 terms."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    N, R, src, dst, rel, p = _popular(128, "bf16", True)
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, 128, "none", dtype="bf16")
    L.load(p["X"], p["W"], None, p["dOut"])
    L.fwd()
    L.bwd()
    torch.cuda.synchronize()
    a = (N, src, dst, rel, p["X"], p["W"], None)
    want = O.rgcn_bwd(*a, p["dOut"], "none")
    for n, got, ref, tol in (("out", L.out, O.rgcn_fwd(*a, "none"), 5e-4), ("dW", L.dW, want["dW"], 1e-5)):
        err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"rgcn bf16 rows per pair: {n} {err:.2e}", flush=True)
        assert err <= tol, (n, err)
    g.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 32), ("f32", 64), ("f32", 128)])
def test_rgcn_of_an_infinite_feature(dtype, d):
    """An infinite feature makes the rows of its destinations infinite, none of them NaN, and no other row; also of the source that is the
    last of its runs of 70 edges, whose row the batches of four read again past the end."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    N, R, src, dst, rel, p = _popular(d, dtype, False)
    if d == 32:
        src, dst, rel = np.concatenate([src] * 2), np.concatenate([dst, dst + 500]), np.concatenate([rel] * 2)
    u = [int(src[17]), int(src.max())]
    p["X"][u, 3] = np.inf
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, dtype=dtype)
    L.load(p["X"], p["W"])
    L.fwd()
    torch.cuda.synchronize()
    hit, times = np.unique(dst[np.isin(src, u)], return_counts=True)
    assert times.max() == 1                                  # (two infinities may cancel)
    row = torch.zeros(N, dtype=torch.bool, device="cuda")
    row[torch.as_tensor(hit, device="cuda").long()] = True
    assert torch.isinf(L.out[row]).all() and torch.isfinite(L.out[~row]).all()
    g.close()


def _area(guards, n):
    big, mid = _guarded(n)
    guards.append(big)
    return mid


@pytest.mark.parametrize("k,d,dtype,flags,spread", [
    (64, 64, "f32", 0, 1), (32, 64, "f32", 32, 1), (64, 32, "f32", 0, 1), (32, 32, "f32", 32, 1), (128, 128, "f32", 0, 1),
    (128, 128, "f32", 32, 9), (64, 64, "bf16", 0, 1)])       # (135 relations of width 128: their folded vectors do not fit in LDS)
def test_rgat(k, d, dtype, flags, spread):
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    E = {32: 810007, 64: 290011, 128: 300007}[d]
    N, R, src, dst, rel, rng = _graph(57 + k + d, E)
    R, rel = R * spread, rel * spread
    print(f"run rows rgat {k}->{d} {dtype} flags={flags} R={R}", flush=True)
    p = synth.rgat_params(rng, N, R, k, d)
    if dtype == "bf16":
        p = {n: synth.round_to_bf16(v) for n, v in p.items()}
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d, dtype=dtype, flags=flags, d_in=k)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    f, b, s = B.rgnn_workspace_bytes(g.handle, B.RGNN_LAYER_RGAT, L.desc)
    guards = []
    L.saved, L.ws = _area(guards, s), _area(guards, f)
    B.rgnn_profile_start()
    L.fwd()
    torch.cuda.synchronize()
    assert "run_inputs" in B.rgnn_profile_stop()
    a = (N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"])
    check(L.out, O.rgat_fwd(*a), TOL_F32, "out")
    out = L.out.clone()
    L.ws = _area(guards, b)
    base = 1.0 if flags else 0.0
    for v in L.grads().values():
        v.fill_(1.0)
    L.bwd()
    torch.cuda.synchronize()
    wg = O.rgat_bwd(*a, p["dOut"])
    for n, v in L.grads().items():
        check(v - base, wg[n], TOL_F32, n)
    for r in range(R):                                       # by relation: a small one would hide among the others
        for n in ("dW", "dw_s", "dw_t"):
            check(L.grads()[n][r] - base, wg[n][r], 4 * TOL_F32, f"{n}[{r}]")
    for big in guards:
        _intact(big, "a buffer")
    first = {n: v.clone() for n, v in L.grads().items()}
    # a forward that keeps nothing, in exactly the workspace reported for it (rows per pair at these sizes); the same bits again, and from the
    # static scratch
    guards2 = []
    L.out.fill_(7.0)
    B.rgnn_rgat_fwd(g.handle, L.desc, L.X, L.W, L.w_s, L.w_t, L.out, None, _area(guards2, (f + 255) // 256 * 256 + s))
    torch.cuda.synchronize()
    check(L.out, O.rgat_fwd(*a), TOL_F32, "out of a forward that keeps nothing")
    L.saved.fill_(0xFF)
    L.out.fill_(7.0)
    B.rgnn_rgat_fwd_static(g.handle, L.desc, L.X, L.W, L.w_s, L.w_t, L.out, L.saved)
    for v in L.grads().values():
        v.fill_(1.0)
    L.bwd()
    torch.cuda.synchronize()
    assert torch.equal(L.out, out)
    for n, v in L.grads().items():
        assert torch.equal(v, first[n]), n
    for big in guards2:
        _intact(big, "the workspace of an inference call")
    g.close()


@pytest.mark.parametrize("d", [32, 64, 128])
def test_rgat_of_logits_of_minus_infinity(d):
    """A relation whose destination halves overflow to minus infinity, in runs of every length: its edges weigh nothing, and nothing is NaN
    (in 64 bits the halves are -1e39, and the weights 0)."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    N, R, src, dst, rel, rng = _graph(3 + d, {32: 810007, 64: 290011, 128: 300007}[d])
    masked = 10
    other = np.bincount(dst[rel != masked], minlength=N) > 0
    rel[(rel == masked) & ~other[dst]] = 0                   # (every destination has another edge)
    p = synth.rgat_params(rng, N, R, d, d)
    p["X"][:, 0] = 10
    p["W"][masked][:, 0] = np.eye(d)[0]
    p["w_t"][masked] = 0
    p["w_t"][masked][0] = -1e38
    print(f"run rows rgat minus infinity d={d}: runs of {np.unique(np.unique(dst[rel == masked], return_counts=True)[1])[[0, 1, -1]]} edges", flush=True)
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    B.rgnn_profile_start()
    L.fwd()
    L.bwd()
    torch.cuda.synchronize()
    assert "run_inputs" in B.rgnn_profile_stop()
    a = (N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"])
    check(L.out, O.rgat_fwd(*a), TOL_F32, "out")
    want = O.rgat_bwd(*a, p["dOut"])
    for n, v in L.grads().items():
        check(v, want[n], TOL_F32, n)
    g.close()


@pytest.mark.parametrize("d,flags", [(32, 0), (64, 0), (128, 0), (128, 4)])
def test_rgat_edges_alone_in_their_destination(d, flags):
    """Their attention weight is 1 whatever the logit, so its gradient is 0, exactly: as much as a relation of such edges only has in dw_s and
    dw_t, and its destinations, which are nobody's sources, in dX.  (flags: rows per pair)"""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    N, R, src, dst, rel, rng = _graph(13 + d, {32: 850007, 64: 290011, 128: 300007}[d])
    src = np.concatenate([src, rng.integers(0, N, 500)]).astype(np.int32)
    dst, rel = (np.concatenate(x).astype(np.int32) for x in ((dst, N + np.arange(500)), (rel, np.full(500, R))))
    p = synth.rgat_params(rng, N + 500, R + 1, d, d)
    print(f"run rows rgat edges alone in their destination d={d} flags={flags}", flush=True)
    g = Graph(N + 500, R + 1, src, dst, rel)
    L = RgatLayer(g, d, flags=flags)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    L.fwd()
    B.rgnn_profile_start()
    L.bwd()
    torch.cuda.synchronize()
    assert ("source_walk" in B.rgnn_profile_stop()) == (flags == 0)
    assert not L.dw_s[R].any() and not L.dw_t[R].any() and not L.dX[N:].any()
    assert L.dw_s[:11].abs().max(1).values.min() > 0 and L.dX[:N].any()
    g.close()


@pytest.mark.parametrize("layer", ["rgat", "rgcn"])
@pytest.mark.parametrize("k,d,N,runs", [(64, 32, 30000, False), (32, 64, 30000, True), (64, 32, 80000, True)])
def test_widths_that_differ(layer, k, d, N, runs):
    """Narrower outputs on a graph of 20 edges per node, where rows per run save a seventh of a row per edge, and of 7.5, where they save
    two thirds; wider ones."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer, RgcnLayer
    R, E = 4, 600000
    rng = np.random.default_rng(k + N)
    src, rel = rng.integers(0, N, E).astype(np.int32), rng.integers(0, R, E).astype(np.int32)
    dst = (N * rng.random(E) ** 3).astype(np.int32)
    print(f"run rows {layer} {k}->{d} N={N}", flush=True)
    g = Graph(N, R, src, dst, rel)
    single = [int((np.diff(g.export(n)) == 1).sum()) for n in ("out_ptr", "run_ptr")]
    saved = (7 * (g.P - g.Q) - 2 * (single[0] - single[1])) / E
    assert saved < 0.2 if N == 30000 else saved > 0.6
    if layer == "rgat":
        p = synth.rgat_params(rng, N, R, k, d)
        L = RgatLayer(g, d, d_in=k)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"])
        want = O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"])
    else:
        p = synth.rgcn_params(rng, N, R, k, d)
        L = RgcnLayer(g, d, d_in=k)
        L.load(p["X"], p["W"])
        want = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"])
    B.rgnn_profile_start()
    L.fwd()
    torch.cuda.synchronize()
    assert ("run_inputs" in B.rgnn_profile_stop()) == runs
    check(L.out, want, TOL_F32, "out")
    g.close()


@pytest.mark.parametrize("layer,d,flags", [("rgat", 64, 0), ("rgat", 64, 32), ("rgat", 128, 0), ("rgcn", 64, 0)])
def test_input_gradient_over_the_input(layer, d, flags):
    """dX written over X: the same bits as in a buffer of its own (with flags: added to what that holds)."""
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer, RgcnLayer
    N, R, src, dst, rel, rng = _graph(71 + d, 300007)
    print(f"run rows {layer} dX over X d={d} flags={flags}", flush=True)
    g = Graph(N, R, src, dst, rel)
    if layer == "rgat":
        p = synth.rgat_params(rng, N, R, d, d)
        L = RgatLayer(g, d, flags=flags)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    else:
        p = synth.rgcn_params(rng, N, R, d, d, self_loop=True)
        L = RgcnLayer(g, d, self_loop=True, flags=flags)
        L.load(p["X"], p["W"], p["W0"], p["dOut"])
    L.fwd()
    for v in L.grads().values():
        v.zero_()
    L.dX.copy_(L.X)
    L.bwd()
    torch.cuda.synchronize()
    want = {n: v.clone() for n, v in L.grads().items()}
    L.dX = L.X
    for n, v in L.grads().items():
        if n != "dX":
            v.zero_()
    L.bwd()
    torch.cuda.synchronize()
    for n, v in L.grads().items():
        assert torch.equal(v, want[n]), n
    g.close()


@pytest.mark.parametrize("others", [0, 5000])
def test_rgat_of_nothing_but_minus_infinity(others):
    """Destinations all of whose logits are minus infinity, in one run of several edges: NaN, as a softmax gives, whether they are batched with
    thousands of others of one run or not.  The rest of the graph knows nothing of it."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    d = 64
    N, R, src, dst, rel, rng = _graph(23, 290011)
    at = N + np.arange(50 + others)                          # destinations of one run of three edges, the first 50 of the relation R
    src = np.concatenate([src, rng.integers(0, N, 3 * len(at))]).astype(np.int32)
    dst, rel = np.concatenate([dst, np.repeat(at, 3)]).astype(np.int32), np.concatenate([rel, np.where(np.repeat(at, 3) < N + 50, R, 0)]).astype(np.int32)
    p = synth.rgat_params(rng, N + len(at), R + 1, d, d)
    p["X"][:, 0] = 10
    p["W"][R][:, 0] = np.eye(d)[0]
    p["w_t"][R] = 0
    p["w_t"][R][0] = -1e38
    print(f"run rows rgat nothing but minus infinity, {others} others", flush=True)
    g = Graph(N + len(at), R + 1, src, dst, rel)
    L = RgatLayer(g, d)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"])
    B.rgnn_profile_start()
    L.fwd()
    torch.cuda.synchronize()
    assert "run_inputs" in B.rgnn_profile_stop()
    assert L.out[N:N + 50].isnan().all()
    want = O.rgat_fwd(N + len(at), src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"])
    rest = np.r_[0:N, N + 50:N + len(at)]
    check(L.out[torch.as_tensor(rest, device="cuda")], want[rest], TOL_F32, "out")
    g.close()


@pytest.mark.parametrize("n,fits", [(121, True), (160, False)])
def test_rgat_forward_that_keeps_nothing(n, fits):
    """Runs of nine edges.  Rows per run, from a workspace and from the static scratch; where that holds the rows per pair only, those from both."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    rng = np.random.default_rng(5)
    N, R, runs, d = 54000, 8, 1000 * n, 64
    q = np.repeat(np.arange(runs), 9)
    rel, dst, src = (q % R).astype(np.int32), (q // 3).astype(np.int32), np.empty(9 * runs, np.int32)
    for r in range(R):
        m = np.flatnonzero(rel == r)
        src[m] = rng.permutation(len(m)) % 25000
    g = Graph(N, R, src, dst, rel)
    p = synth.rgat_params(rng, N, R, d, d)
    L = RgatLayer(g, d)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"])
    f, _, s = B.rgnn_workspace_bytes(g.handle, B.RGNN_LAYER_RGAT, L.desc)
    guards, names, outs = [], [], []
    ws = _area(guards, (f + 255) // 256 * 256 + s)
    a = (L.X, L.W, L.w_s, L.w_t, L.out)
    for call in (L.fwd, lambda: B.rgnn_rgat_fwd(g.handle, L.desc, *a, None, ws), lambda: B.rgnn_rgat_fwd_static(g.handle, L.desc, *a, None)):
        L.out.fill_(7.0)
        B.rgnn_profile_start()
        call()
        torch.cuda.synchronize()
        names.append("run_inputs" in B.rgnn_profile_stop())
        outs.append(L.out.clone())
    check(outs[0], O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"]), TOL_F32, "out")
    check(outs[1], O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"]), TOL_F32, "out")
    assert names == [True, fits, fits] and torch.equal(outs[1], outs[2])
    _intact(guards[0], "the workspace")
    g.close()


FLAGS = [
    ("rgat", 64, 64, 16, 0), ("rgat", 64, 64, 1, 0), ("rgat", 64, 64, 4, 0), ("rgat", 32, 64, 2, 32), ("rgat", 128, 128, 16, 32), ("rgat", 64, 64, 0, 4),
    ("rgat", 128, 128, 0, 4), ("rgat", 64, 32, 0, 2), ("rgat", 64, 64, 16, 4), ("rgat", 64, 64, 4, 4 | 32), ("rgcn", 64, 64, 2, 0), ("rgcn", 32, 64, 4, 0),
    ("rgcn", 64, 64, 0, 4)]


@pytest.mark.parametrize("layer,k,d,forward,backward,in_place", [(*c, False) for c in FLAGS] + [(*c, True) for c in FLAGS if c[1] == c[2]])
def test_flags_of_one_call(layer, k, d, forward, backward, in_place):
    """A backward need not carry the flags of its forward, in one `saved` that is as large for both, also where the forward writes out over X."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer, RgcnLayer
    N, R, src, dst, rel, rng = _graph(5 + k + d, {32: 810007, 64: 290011, 128: 300007}[min(k, d)])
    print(f"run rows {layer} {k}->{d} flags {forward} then {backward} in_place={in_place}", flush=True)
    g = Graph(N, R, src, dst, rel)
    if layer == "rgat":
        p = synth.rgat_params(rng, N, R, k, d)
        a = (N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"])
        want, wg = O.rgat_fwd(*a), O.rgat_bwd(*a, p["dOut"])
        which, make, names = B.RGNN_LAYER_RGAT, RgatLayer, ("X", "W", "w_s", "w_t", "dOut")
    else:
        p = synth.rgcn_params(rng, N, R, k, d, self_loop=False)
        a = (N, src, dst, rel, p["X"], p["W"], None)
        want, wg = O.rgcn_fwd(*a), O.rgcn_bwd(*a, p["dOut"])
        which, make, names = B.RGNN_LAYER_RGCN, RgcnLayer, ("X", "W", "W0", "dOut")
    F, G = make(g, d, flags=forward, d_in=k), make(g, d, flags=backward, d_in=k)
    (f, _, s), (_, b, s2) = (B.rgnn_workspace_bytes(g.handle, which, L.desc) for L in (F, G))
    assert s == s2 > 0
    guards = []
    F.saved, F.ws, G.ws = _area(guards, s), _area(guards, f), _area(guards, b)
    F.saved.fill_(0xFF)
    for L in (F, G):
        L.load(*[p[n] for n in names])
    if in_place:
        F.out = F.X
    B.rgnn_profile_start()
    F.fwd()
    torch.cuda.synchronize()
    rep = B.rgnn_profile_stop()
    assert "run_inputs" in rep and ("single_logits" in rep) == (layer == "rgat" and forward & ~32 > 0 and not in_place)
    check(F.out, want, TOL_F32, "out")
    G.out, G.saved = F.out, F.saved
    base = 1.0 if backward & 32 else 0.0
    for v in G.grads().values():
        v.fill_(1.0)
    G.bwd()
    torch.cuda.synchronize()
    for n, v in G.grads().items():
        check(v - base, wg[n], TOL_F32, n)
    for big in guards:
        _intact(big, "a buffer")
    g.close()


@pytest.mark.parametrize("layer,dtype", [("rgat", "f32"), ("rgcn", "f32")])
def test_replays(layer, dtype):
    """Forward + backward recorded into a HIP graph: every replay leaves the bits of the eager calls."""
    from paper_2412_04747_amd.harness import Graph, RgatLayer, RgcnLayer
    d = 64
    N, R, src, dst, rel, rng = _graph(91, 290011)
    print(f"run rows replays {layer} {dtype}", flush=True)
    g = Graph(N, R, src, dst, rel)
    if layer == "rgat":
        p = synth.rgat_params(rng, N, R, d, d)
        L = RgatLayer(g, d)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    else:
        p = synth.rgcn_params(rng, N, R, d, d, self_loop=True)
        L = RgcnLayer(g, d, "in_degree_per_rel", "relu", True, dtype=dtype)
        L.load(p["X"], p["W"], p["W0"], p["dOut"])
    _capture_and_replay(L, lambda: [L.out, *L.grads().values()])
    g.close()


@pytest.mark.parametrize("layer,d", [("rgat", 64), ("rgat", 128), ("rgcn", 64), ("rgcn", 128)])
def test_memory_of_a_forward_without_gradients(layer, d):
    """Beside the graph's workspace: out, and what RGAT would have saved with its forward scratch; for RGCN nothing else."""
    import torch
    from paper_2412_04747_amd import autograd as A
    from paper_2412_04747_amd import binding as B
    N, R, src, dst, rel, _ = _graph(17, 300007)
    g = A.Graph(N, R, src, dst, rel)
    conv = A.RgatConv(R, d) if layer == "rgat" else A.RgcnConv(R, d)
    X = torch.randn(N, d, device="cuda")
    f, _, s = B.rgnn_workspace_bytes(g.handle, *((B.RGNN_LAYER_RGAT, B.make_desc(d_in=d, d_out=d)) if layer == "rgat" else
                                                 (B.RGNN_LAYER_RGCN, B.make_desc(d_in=d, d_out=d, norm=B.RGNN_NORM_IN_DEGREE_PER_REL))))
    with torch.no_grad():
        conv(g, X)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        conv(g, X)
        more = torch.cuda.max_memory_allocated() - before
    print(f"run rows memory {layer} {d}: {more} bytes, out {4 * N * d}, forward {f}, saved {s}", flush=True)
    assert s > 0 and more <= 4 * N * d + (f + s if layer == "rgat" else 0) + (1 << 20)
    g.close()


@pytest.mark.parametrize("layer,d", [("rgat", 64), ("rgat", 128), ("rgcn", 64)])
def test_autograd_without_gradients(layer, d):
    """A forward of the autograd front end that no backward follows keeps nothing and gives the same result up to rounding."""
    import torch
    from paper_2412_04747_amd import autograd as A
    N, R, src, dst, rel, rng = _graph(17, 290011)
    print(f"run rows without gradients {layer} {d}", flush=True)
    g = A.Graph(N, R, src, dst, rel)
    torch.manual_seed(3)
    conv = A.RgatConv(R, d) if layer == "rgat" else A.RgcnConv(R, d)
    X = torch.randn(N, d, device="cuda", requires_grad=True)
    out = conv(g, X)
    with torch.no_grad():
        again = conv(g, X)
    assert out.requires_grad and not again.requires_grad
    check(again, out.detach().cpu().numpy(), TOL_F32, "out")
    out.sum().backward()                                     # (the forward that keeps nothing has left what this one needs alone)
    first = X.grad.clone()
    X.grad = None
    conv(g, X).sum().backward()
    assert torch.equal(X.grad, first)
    g.close()
