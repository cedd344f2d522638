"""Layers whose rows are kept per (destination, relation) run (large graphs with fewer runs than pairs) against the oracle."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2412_04747_amd import synth
from parity import check, TOL_F32, TOL_BF16
from test_gpu_workspace_bounds import _guarded, _intact

pytestmark = pytest.mark.gpu


def _graph(seed, E):
    """Destinations of 1 to thousands of edges, runs of one edge and of hundreds (cut into pieces), a hub source, and relations without
    an edge (11), with single-edge runs only (12), with runs of several edges only (13), with one run (14)."""
    rng = np.random.default_rng(seed)
    N, R = 9001, 15
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
    (128, 128, "f32", "in_degree_per_rel", "none", False, 0), (128, 128, "f32", "none", "relu", True, 32),
    (128, 128, "bf16", "in_degree_per_rel", "none", False, 0), (128, 128, "bf16", "none", "relu", True, 32)])
def test_rgcn(k, d, dtype, norm, act, loop, flags, saved):
    import torch
    from paper_2412_04747_amd import binding as B
    from paper_2412_04747_amd.harness import Graph, RgcnLayer
    E = 260011 if d == 32 or (d == 128 and dtype == "f32") else 140003
    N, R, src, dst, rel, rng = _graph(31 + k + d, E)
    print(f"run rows rgcn {k}->{d} {dtype} {norm} {act} loop={loop} flags={flags} saved={saved}", flush=True)
    p = synth.rgcn_params(rng, N, R, k, d, self_loop=loop)
    tol = TOL_F32
    if dtype == "bf16":
        p = {n: v if v is None else synth.round_to_bf16(v) for n, v in p.items()}
        tol = TOL_BF16 if d == 128 else TOL_F32
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
    assert ("run_inputs" in B.rgnn_profile_stop()) == (saved or (dtype == "f32" and E * d >= 30000000))
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
