"""RGAT, rows per pair: the destination halves of the logits against 64 bits, on both sides of the line between their two kernels."""
import numpy as np
import pytest

from paper_2412_04747_amd import synth
from parity import check, TOL_F32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,R,Q", [
    (64, 1, 3, 3071), (64, 1, 3, 3073), (32, 1, 1, 1025), (128, 1, 2, 2051), (64, 2, 3, 3074), (64, 4, 3, 3071), (64, 4, 3, 3075),
    (128, 8, 3, 3073), (128, 8, 38, 38 * 1024 + 3)])          # (the last: 152 KB of vectors, not in LDS)
def test_destination_halves(d, heads, R, Q):
    import torch
    from paper_2412_04747_amd.harness import Graph, RgatLayer
    print(f"halves d={d} heads={heads} R={R} Q={Q}", flush=True)
    rng = np.random.default_rng(d + heads + Q)
    q = np.arange(Q)
    N = Q // R + 1
    dst, rel, src = (q // R).astype(np.int32), (q % R).astype(np.int32), rng.integers(0, N, Q).astype(np.int32)
    mix = rng.permutation(Q)
    g = Graph(N, R, src[mix], dst[mix], rel[mix])
    assert g.Q == Q
    p = synth.rgat_params(rng, N, R, d, d)
    L = RgatLayer(g, d, heads=heads)
    L.load(p["X"], p["W"], p["w_s"], p["w_t"])
    L.fwd()
    torch.cuda.synchronize()
    W, w_t = p["W"].astype(np.float64), p["w_t"].astype(np.float64)
    dh = d // heads
    wtp = np.stack([np.einsum("rkc,rc->rk", W[:, :, h * dh:(h + 1) * dh], w_t[:, h * dh:(h + 1) * dh]) for h in range(heads)], 1)
    want = np.einsum("qk,qhk->qh", p["X"].astype(np.float64)[dst], wtp[rel])
    check(L.saved_views()[1], want, TOL_F32, "s_dst")
    g.close()
