"""The schedule / layout choice of the library: rgnn_schedule on real graphs agrees with the host-side pick made from
the edge list alone, and every forced alternative (desc.flags) gives the oracle's results too."""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest

from oracle import layers as O
from paper_2412_04747_amd import synth
from parity import check, TOL_F32, TOL_BF16
import test_work_lists as WL

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def wl():
    out = os.path.join(tempfile.mkdtemp(prefix="rgnn_wl_"), "libwl.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "host", "work_lists_shim.cpp")])
    return C.CDLL(out)


@pytest.mark.parametrize("cid,scale", [(1, 1.0), (2, 1.0), (3, 0.05), (4, 0.02), (5, 0.05)])
def test_library_pick_equals_host_pick(wl, cid, scale):
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph
    c = synth.config(cid, scale, graph_only=True)
    print(f"schedule case config {cid} x {scale}: N={c['N']} E={c['E']}", flush=True)
    g = Graph(c["N"], c["R"], c["src"], c["dst"], c["rel"], c.get("ntype") if c["T"] > 1 else None, c["T"])
    k = WL.graph_counts(c)
    layer = WL.LAYER[c["layer"]]
    import torch
    pair_ptr, cus, scalars = g.export("pair_ptr"), torch.cuda.get_device_properties(0).multi_processor_count, np.zeros(3, np.int32)
    def chunks(most):                 # of the pair tiles, `most` at most
        wl.wl_plan_tiles(pair_ptr.ctypes.data_as(C.c_void_p), c["R"], wl.wl_constant(WL.K["tile_rows"]), most)
        wl.wl_tiles_scalars(scalars.ctypes.data_as(C.c_void_p))
        return int(scalars[0])
    for flags in (0, 2, 4, 8, 2 | 4 | 8) + ((16, 1) if c["layer"] == "rgat" else ()):
        for heads in ((1, 4) if c["layer"] == "rgat" and not flags & 17 else (c["H"],)):
            desc = B.make_desc(B.RGNN_BF16 if c["dtype"] == "bf16" else B.RGNN_F32, c["d_out"], c["d_out"], heads, flags=flags)
            got = B.rgnn_schedule(g.handle, layer, desc)
            want = WL.pick(wl, c, k, heads=heads, flags=flags)
            want["tile_chunks"] = chunks(wl.wl_constant(WL.K["max_chunks"]))
            want["wide_chunks"] = chunks(cus * (2 if c["layer"] == "rgcn" and want["rows_bf16"] else 1))
            assert got == want, (flags, heads, {f: (got[f], want[f]) for f in got if got[f] != want[f]})
    g.close()


def _hub_graph(seed, N, R, E, T=1):
    rng, src, dst, rel, ntype = synth.tiny(seed, N=N, R=R, E=E, T=T)
    dst[:E // 5] = 3
    src[E // 5:E // 3] = 5; rel[E // 5:E // 3] = 1
    return rng, src, dst, rel, ntype


@pytest.mark.parametrize("flags", [2, 4, 16, 2 | 4 | 16, 1 | 2 | 4])
@pytest.mark.parametrize("d", [32, 64])
def test_rgat_forced_alternatives(flags, d):
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    N, R, E = 9000, 6, 40000
    rng, src, dst, rel, _ = _hub_graph(700 + d, N, R, E)
    print(f"schedule case rgat flags={flags} d={d}", flush=True)
    p = synth.rgat_params(rng, N, R, d, d)
    g = Graph(N, R, src, dst, rel)
    L = RgatLayer(g, d, flags=flags)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    check(L.out, O.rgat_fwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"]), TOL_F32, "out")
    wg = O.rgat_bwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    for k, v in L.grads().items():
        check(v, wg[k], TOL_F32, k)
    g.close()


@pytest.mark.parametrize("flags", [2, 4, 2 | 4])
def test_rgcn_bf16_forced_alternatives(flags):
    import torch
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    N, R, E, d = 9000, 6, 40000, 128
    rng, src, dst, rel, _ = _hub_graph(721, N, R, E)
    print(f"schedule case rgcn bf16 flags={flags}", flush=True)
    p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in synth.rgcn_params(rng, N, R, d, d).items()}
    g = Graph(N, R, src, dst, rel)
    L = RgcnLayer(g, d, "in_degree_per_rel", "none", False, dtype="bf16", flags=flags)
    L.load(p["X"], p["W"], None, p["dOut"])
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    want = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], None, "in_degree_per_rel", "none")
    check(L.out, want, TOL_BF16, "out")
    wg = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], None, p["dOut"], "in_degree_per_rel", "none", out=want)
    for k, v in L.grads().items():
        check(v, wg[k], TOL_BF16, k)
    g.close()


@pytest.mark.parametrize("loop", [True, False])
@pytest.mark.parametrize("k,d,norm,dtype", [(k, d, n, "f32") for k, d in ((32, 32), (64, 64), (32, 64), (64, 32))
                                            for n in ("in_degree_per_rel", "none")] +
                         [(d, d, "in_degree_per_rel", "bf16") for d in (32, 64)] +
                         [(128, 128, n, m) for n in ("in_degree_per_rel", "none") for m in ("f32", "f32 small")])
def test_rgcn_row_select(k, d, norm, dtype, loop):
    """fp32 rows: the rows of the single-edge pairs are read from the destinations' gradient rows.  Products and sums
    are those of the plain walk in the same order, so the gradients are the same bits; and they are the oracle's.  (small:
    some rows hold values below 2^-110, which take the fp32 matrix instructions at width 128.)"""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    N, R, E = 9001, 7, 40037
    rng, src, dst, rel, _ = _hub_graph(741 + k + d, N, R, E)
    rel[-1000:] = np.where(rel[-1000:] == 4, 3, rel[-1000:])
    print(f"schedule case rgcn row select {k}->{d} {norm} {dtype}", flush=True)
    p = synth.rgcn_params(rng, N, R, k, d, self_loop=loop)
    if dtype == "bf16":
        p = {n: v if v is None else synth.round_to_bf16(v) for n, v in p.items()}
    if dtype == "f32 small":
        dtype = "f32"
        p["dOut"][::101] *= np.float32(2.0 ** -114)
    g = Graph(N, R, src, dst, rel)
    want = O.rgcn_fwd(N, src, dst, rel, p["X"], p["W"], p["W0"], norm, "none")
    wg = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], p["W0"], p["dOut"], norm, "none", out=want)
    got = []
    for flags in (0, B.RGNN_FLAG_NO_ROW_SELECT):
        L = RgcnLayer(g, d, norm, "none", loop, dtype=dtype, flags=flags, d_in=k)
        assert B.rgnn_schedule(g.handle, B.RGNN_LAYER_RGCN, L.desc)["row_select"] == (flags == 0)
        L.load(p["X"], p["W"], p["W0"], p["dOut"])
        L.fwd(); L.bwd()
        torch.cuda.synchronize()
        check(L.out, want, TOL_F32, "out")
        got.append({n: v.clone() for n, v in L.grads().items()})
        for n, v in L.grads().items():
            check(v, wg[n], TOL_F32, n)
    for n in got[0]:
        assert torch.equal(got[0][n], got[1][n]), n
    g.close()


@pytest.mark.parametrize("small", [False, True])
def test_rgat_row_select_of_width_128(small):
    """As above for RGAT with one head, whose rows also carry a rank-1 term."""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    N, R, E, d = 3001, 5, 15013, 128
    rng, src, dst, rel, _ = _hub_graph(761, N, R, E)
    print(f"schedule case rgat row select d={d} small={small}", flush=True)
    p = synth.rgat_params(rng, N, R, d, d)
    if small:
        p["dOut"][::101] *= np.float32(2.0 ** -114)
    g = Graph(N, R, src, dst, rel)
    wg = O.rgat_bwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    got = []
    for flags in (0, B.RGNN_FLAG_NO_ROW_SELECT):
        L = RgatLayer(g, d, flags=flags)
        assert B.rgnn_schedule(g.handle, B.RGNN_LAYER_RGAT, L.desc)["row_select"] == (flags == 0)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
        L.fwd(); L.bwd()
        torch.cuda.synchronize()
        got.append({n: v.clone() for n, v in L.grads().items()})
        for n, v in L.grads().items():
            check(v, wg[n], TOL_F32, n)
    for n in got[0]:
        assert torch.equal(got[0][n], got[1][n]), n
    g.close()


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_hgt_unfolded_on_a_graph_that_could_fold(dtype, d):
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, HgtLayer
    c = synth.config(4, scale=0.002, graph_only=True)
    N, T, R, H = c["N"], c["T"], c["R"], 4
    print(f"schedule case hgt unfolded {dtype} d={d}: N={N} E={c['E']}", flush=True)
    rng = np.random.default_rng(733)
    p = synth.hgt_params(rng, N, T, R, d, H, with_mu=True)
    if dtype == "bf16":
        p = {k: synth.round_to_bf16(v) for k, v in p.items()}
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    g = Graph(N, R, c["src"], c["dst"], c["rel"], c["ntype"], T)
    names = ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg", "mu")
    want = O.hgt_fwd(N, c["src"], c["dst"], c["rel"], c["ntype"], *[p[k] for k in names])
    wg = O.hgt_bwd(N, c["src"], c["dst"], c["rel"], c["ntype"], *[p[k] for k in names], p["dOut"])
    sizes = {}
    for flags in (0, B.RGNN_FLAG_NO_WEIGHT_FOLDING | B.RGNN_FLAG_NO_BATCHED_WALKS):
        L = HgtLayer(g, d, H, with_mu=True, dtype=dtype, flags=flags)
        assert B.rgnn_schedule(g.handle, B.RGNN_LAYER_HGT, L.desc)["hgt_folded"] == (flags == 0)
        sizes[flags] = B.rgnn_workspace_bytes(g.handle, B.RGNN_LAYER_HGT, L.desc)[2]
        L.load(*[p[k] for k in names], p["dOut"])
        L.fwd(); L.bwd()
        torch.cuda.synchronize()
        check(L.out, want, tol, f"out flags={flags}")
        for k, v in L.grads().items():
            check(v, wg[k], tol, f"{k} flags={flags}")
    assert sizes[0] < max(sizes.values())            # the folded path saves the K and V rows
    g.close()


@pytest.mark.parametrize("layer,d,H", [("rgat", 64, 1), ("rgat", 64, 2), ("rgat", 32, 2), ("rgcn", 64, 1), ("hgt", 64, 4), ("hgt unfolded", 64, 4), ("hgt uneven", 64, 4)])
def test_chunks_of_many_relations(wl, layer, d, H):
    """1,500 relations of one row tile each: the fp32 backward takes the shorter chunks (twice as many here), HGT with folded weights the
    share of each list of the pairs in one chunk per compute unit, within the workspace that is reported for them and with the
    oracle's results.  (uneven: three of them have 400 tiles, and HGT takes the shorter chunks as well.)"""
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd import harness as Hn
    from test_gpu_workspace_bounds import _guarded, _intact
    N, R = 25600 if layer == "hgt uneven" else 400, 1500
    rng = np.random.default_rng(1500 + d)
    rel = np.repeat(np.arange(R, dtype=np.int32), 4)
    src, dst = rng.integers(0, N, len(rel)).astype(np.int32), rng.integers(0, N, len(rel)).astype(np.int32)
    if layer == "hgt uneven":
        rel = np.concatenate([rel, np.repeat(np.arange(3, dtype=np.int32), N)])
        src, dst = np.concatenate([src] + [np.arange(N)] * 3).astype(np.int32), np.concatenate([dst, rng.integers(0, N, 3 * N)]).astype(np.int32)
    g = Hn.Graph(N, R, src, dst, rel)
    if layer == "rgat":
        p = synth.rgat_params(rng, N, R, d, d)
        L = Hn.RgatLayer(g, d, heads=H)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
        a = (N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"])
        want = O.rgat_heads_bwd(*a, p["dOut"], H) if H > 1 else O.rgat_bwd(*a, p["dOut"])
    elif layer == "rgcn":
        p = synth.rgcn_params(rng, N, R, d, d)
        L = Hn.RgcnLayer(g, d, "none")
        L.load(p["X"], p["W"], None, p["dOut"])
        want = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], None, p["dOut"], "none", "none", out=np.zeros((N, d)))
    else:
        p = synth.hgt_params(rng, N, 1, R, d, H, with_mu=True)
        names = ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg", "mu")
        L = Hn.HgtLayer(g, d, H, flags=B.RGNN_FLAG_NO_WEIGHT_FOLDING if layer == "hgt unfolded" else 0)
        L.load(*[p[k] for k in names], dOut=p["dOut"])
        want = O.hgt_bwd(N, src, dst, rel, None, *[p[k] for k in names], p["dOut"])
    ptr, cus = g.export("pair_ptr"), torch.cuda.get_device_properties(0).multi_processor_count
    n = np.zeros((3, 3), np.int32)
    wl.wl_pair_share.argtypes = [C.c_longlong, C.c_longlong, C.c_int, C.c_int]
    for row, most in zip(n, (cus, wl.wl_constant(WL.K["wide_chunks"]) * cus, wl.wl_pair_share(g.P, N, cus, 2))):
        wl.wl_plan_tiles(ptr.ctypes.data_as(C.c_void_p), R, wl.wl_constant(WL.K["tile_rows"]), most)
        wl.wl_tiles_scalars(row.ctypes.data_as(C.c_void_p))
    code = WL.LAYER[layer.split()[0]]
    assert n[0, 0] < n[1, 0] and n[2, 0] < n[0, 0]
    assert B.rgnn_schedule(g.handle, code, L.desc)["wide_chunks"] == n[2 if layer == "hgt" else 1, 0]
    L.fwd()
    ws, L.ws = _guarded(B.rgnn_workspace_bytes(g.handle, code, L.desc)[1])
    L.bwd()
    torch.cuda.synchronize()
    _intact(ws, "backward workspace")
    for k, v in L.grads().items():
        check(v, want[k], TOL_F32, k)
    g.close()


@pytest.mark.parametrize("uneven", [False, True])
@pytest.mark.parametrize("layer,d,dtype", [("rgcn", 32, "f32"), ("rgcn", 64, "f32"), ("rgcn", 128, "f32"), ("rgcn", 128, "bf16"), ("rgat", 64, "f32")])
def test_weight_gradients_of_a_few_shares(layer, d, dtype, uneven):
    """Relations whose weight gradient is the sum of a few shares (one per compute unit that has tiles of the relation), an empty one
    among them: 1 to 10 shares of 1 to 40 row tiles, and 850 relations of one; 1 to 17, one of 150 and 60 of one, where four groups
    of lanes share the shares."""
    import torch
    from paper_2412_04747_amd import harness as Hn
    rng = np.random.default_rng(170 + d)
    tiles = [0] + list(range(1, 18)) + [150] + [1] * 60 if uneven else [0, 1, 2, 3, 5, 8, 12, 16, 20, 24, 28, 32, 36, 40] + [1] * 850
    N, R = 64 * max(tiles), len(tiles)
    src = np.concatenate([rng.permutation(N)[:64 * t] for t in tiles]).astype(np.int32)
    rel = np.repeat(np.arange(R, dtype=np.int32), [64 * t for t in tiles])
    dst = rng.integers(0, N, len(src)).astype(np.int32)
    print(f"schedule case few shares {layer} {dtype} d={d}: E={len(src)}", flush=True)
    g = Hn.Graph(N, R, src, dst, rel)
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    if layer == "rgat":
        p = synth.rgat_params(rng, N, R, d, d)
        L = Hn.RgatLayer(g, d)
        L.load(p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
        want = O.rgat_bwd(N, src, dst, rel, p["X"], p["W"], p["w_s"], p["w_t"], p["dOut"])
    else:
        p = synth.rgcn_params(rng, N, R, d, d)
        if dtype == "bf16":
            p = {k: (None if v is None else synth.round_to_bf16(v)) for k, v in p.items()}
        L = Hn.RgcnLayer(g, d, "none", dtype=dtype)
        L.load(p["X"], p["W"], None, p["dOut"])
        want = O.rgcn_bwd(N, src, dst, rel, p["X"], p["W"], None, p["dOut"], "none", "none", out=np.zeros((N, d)))
    L.fwd(); L.bwd()
    torch.cuda.synchronize()
    for k, v in L.grads().items():
        check(v, want[k], tol, k)
    for r in range(R):                                   # by relation: a lost share would hide among the others
        check(L.dW[r], want["dW"][r], tol, f"dW[{r}]")
    g.close()
