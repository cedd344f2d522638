#!/usr/bin/env python3
"""Benchmark: RGAT layer forward+backward on one MI355X, edges/s.

One step = one pass of the whole hot path (rgnn_rgat_fwd + rgnn_rgat_bwd) over the
synthetic 1M-node / 200-relation / 10M-edge graph, inputs resident in HBM, graph index
built beforehand (the thesis also times the layer only, with preprocessing done before).
Prints ONE JSON line with the throughput, the roofline of the dominant kernel (timed live
with HIP events on the launch stream, through the library's profiling hooks) and the CPU
oracle timed on the host cores on the same inputs.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
FP32_MFMA_PEAK_TFLOPS = 157.3
BF16_MFMA_PEAK_TFLOPS = 2500.0
TRAFFIC_TSV = os.path.join(ROOT, "profiles", "rgat_c3_hbm_traffic_per_label.txt")


def library_sha16():
    """Hash of the HIP sources the library is built from: ties a committed counter summary to the kernels it measured."""
    import glob
    import hashlib
    h = hashlib.sha256()
    for f in sorted(glob.glob(os.path.join(ROOT, "paper_2412_04747_amd", "csrc", "*.h*"))):
        h.update(os.path.basename(f).encode())
        h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def counter_traffic(label, sha):
    """(bytes per step, source note) for a kernel label from the committed rocprofv3 --pmc summary of this command
    (FETCH_SIZE + WRITE_SIZE, calibrated), or (None, why) when the summary was taken from other kernel sources."""
    if not os.path.exists(TRAFFIC_TSV):
        return None, "no counter summary committed"
    rel = os.path.relpath(TRAFFIC_TSV, ROOT)
    rows, file_sha = {}, None
    for ln in open(TRAFFIC_TSV):
        if ln.startswith("# lib_sha16:"):
            file_sha = ln.split(":", 1)[1].strip()
        elif not ln.startswith("#"):
            f = ln.rstrip("\n").split("\t")
            rows[f[0]] = float(f[1]) + float(f[2])
    if file_sha != sha:
        return None, f"{rel} was measured on other kernel sources ({file_sha}, now {sha}): stale, not used"
    if label not in rows:
        return None, f"{rel} has no row for {label}"
    return rows[label], f"{rel} (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this command at lib_sha16 {sha}; not measured by this run)"


def run_row_work(name, E, N, P, Q, Q1, R, d, layer="rgat", n_dst=None):
    """algorithmic_work for the kernels of the plan that keeps rows per (destination, relation) run (RGCN, RGAT with one head; fp32
    rows); Q1 of the Q runs have one edge and read their source's row where it is."""
    M, Em = Q - Q1, E - Q1            # runs with several edges, and their edges
    row = d * 4
    mm = "hbm" if d == 128 else "mfma"
    w2 = d * d * 4
    rgat = layer == "rgat"
    table = {
        # per edge: source's row, source, relation and run (RGCN: coefficient); per run: the sum, s_dst and (max, sum)
        "run_inputs": ("hbm", Em * (row + (12 if rgat else 8)) + M * (row + (12 if rgat else 8)), 4.0 * Em * d),
        # input row(s), result row, gather index and place of the result
        "typed_linear_fwd": ("mfma", Q * (2 * row + 8) + R * w2, 2.0 * Q * d * d),
        # per run: its row; RGAT: tag, relation, s_dst, (max, sum) read or written; per node the result row and its item; RGAT: (max, sum)
        "aggregate_fwd": ("hbm", Q * (row + (20 if rgat else 0)) + N * (row + (16 if rgat else 8)), 4.0 * Q * d),
        # input row, gradient row, result row, both indices; RGAT: number, weight and product of the run
        "typed_linear_bwd": (mm, Q * (3 * row + (20 if rgat else 8)) + R * 2 * w2, 4.0 * Q * d * d),
        "typed_linear_loop_bwd": ("mfma", Q * (3 * row + 8) + R * 2 * w2 + N * 3 * row + 2 * w2, 4.0 * (Q + N) * d * d),
        "run_weights": ("hbm", Q * 16 + N * 8, 4.0 * Q),
        "run_stat": ("hbm", Q * 40 + Q1 * 4 + N * 12, 8.0 * Q),
        # per edge: the run's gradient row, its 16 bytes, three indices, dz; per node its row in and out
        "source_walk": ("hbm", E * (row + 32) + N * (2 * row + 16), 8.0 * E * d),
        # the nodes' rows, once for the pairs and once for the runs (structural: a block of nodes is read once for all relations);
        # per pair node and list ends, per edge dz, per run destination, index and ds_dst
        "block_sums": ("hbm", 2 * N * row + P * 12 + E * 4 + Q * 12, 2.0 * (P + Q) * d),
        "run_term": ("hbm", N * 2 * row + Q * 8, 2.0 * Q * d),
        "run_logit": ("hbm", Q * 12 + (N if n_dst is None else n_dst) * row, 2.0 * Q * d),
        # RGCN: per edge the run's gradient row, its index and coefficient
        "node_grad_sum": ("hbm", E * (row + 8) + N * (row + 16), 2.0 * E * d),
    }
    return table.get(name)


def run_row_steps(kern_ms, E, N, P, Q, Q1, d):
    """step_rooflines for the rows per run: the traversals of the forward, of the backward by source, and the sums of its parameter
    gradients and destination halves."""
    work = lambda *names: sum(run_row_work(n, E, N, P, Q, Q1, 0, d)[1] for n in names)
    return _steps(kern_ms, {
        "S3_traversal_fwd": (work("run_inputs", "aggregate_fwd"), ("run_inputs", "run_inputs.combine", "aggregate_fwd", "aggregate_fwd.combine")),
        "S4_traversal_bwd_src": (work("source_walk", "run_stat") + E * 8 + Q * 8, ("run_stat", "source_walk", "source_walk.combine", "ds_dst_sum")),
        "S5_sums_bwd": (work("block_sums", "run_term"), ("block_sums", "run_term")),
    })


def step_rooflines(kern_ms, E, N, P, P1, Q, d):
    """Single-head RGAT: the traversal steps as wholes against the HBM peak: all kernels that implement a step, over
    the bytes the step itself needs per edge / node / pair (listed with each step below), whatever else the kernels move."""
    row = 4 * d
    steps = {
        # S3 forward traversal: per edge the message row, pair id, a logit scalar and a 4-byte weight or its
        # equivalent (272 B at d = 64); per node the output row and 8 bytes of offsets / statistics
        "S3_traversal_fwd": (E * (row + 16) + N * (row + 8),
                             ("aggregate_fwd", "aggregate_fwd.combine", "edge_softmax", "edge_softmax.finish", "aggregate_fwd_edge_parallel")),
        # S4 backward, destination-major: per edge the message row, index, weight, dz store; per node the gradient row
        "S4_traversal_bwd_dst": (E * (row + 12) + N * row, ("edge_dot_bwd", "ds_dst_sum")),
        # S5 backward, pair-major, over the pairs with several edges (the others are served by the row selector):
        # per edge the gradient row, position, weight, dz, destination; per pair the stored row and its offset.  The launch
        # also walks the runs of the destination-side weight gradient: per run the destination's row, its id, run and ds_dst
        "S5_traversal_bwd_pair": ((E - P1) * (row + 16) + (P - P1) * (row + 4) + Q * (row + 12),
                                  ("pair_run_walks", "aggregate_bwd_pair.combine", "ds_src_sum")),
    }
    return _steps(kern_ms, steps)


def _steps(kern_ms, steps):
    out = {}
    for k, (nbytes, names) in steps.items():
        ms = sum(kern_ms.get(n, 0.0) for n in names)
        if ms > 0:
            gbs = nbytes / ms / 1e6
            out[k] = {"bound": "hbm", "bytes": nbytes, "ms": ms, "achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                      "frac": gbs / HBM_PEAK_GBS, "kernels": [n for n in names if n in kern_ms]}
    return out


def algorithmic_work(name, E, N, P, Q, R, T, d, H, P1=0, bf16=False, layer="rgat", sched=None, n_dst=None):
    """(bound, bytes, flops) one launch of kernel `name` must move / compute, or None where no model is kept
    (the small reduce / combine / finish kernels).  Gathered rows are counted once per reference (no cache
    reuse assumed) except where the reuse is structural: the runs of one destination are adjacent, so the
    per-run logit kernel reads a destination's row once (n_dst = destinations with an incoming edge).
    Index and scalar traffic as listed in the comments below.  Row tensors are 4-byte elements, except in
    the bfloat16 workloads at width 128, where inputs and intermediate rows are 2-byte elements (results
    handed back to the caller stay fp32).  `sched` is the library's pick for the call (rgnn_schedule)."""
    if name.endswith((".reduce", ".combine", ".finish")):
        return None
    sched = sched or {}
    n_dst = N if n_dst is None else n_dst
    half = bf16 and d == 128
    r32 = d * 4                       # an fp32 row
    row = d * 2 if half else r32      # an input / intermediate row
    wb = 2 if half else 4             # element size of a given weight
    if half:
        rows = {"typed_linear": P, "pair_linear": P, "node_linear": N}       # (the self-loop runs on fp32 copies: below)
        key = name.split(".")[0]
        n = next((v for k, v in rows.items() if key.startswith(k)), None)
        if n is not None:
            bound = "hbm"
            # one row in, one row out, + the gather index; backward: two rows in (both products in one kernel)
            segs = T if key.startswith("node_linear") else R
            w2 = d * d * (4 if key.startswith("pair_linear") else wb)       # block-diagonal weights are fp32
            if name == "pair_linear":          # key and message halves together: X row in, two rows out
                return (bound, n * (3 * row + 4) + 2 * segs * d * d * wb, 4.0 * n * d * d)
            if name == "pair_linear_bwd":      # key and message halves together: X row, two gradient rows in, one row out
                return (bound, n * (4 * row + 4) + 2 * segs * d * d * (wb + 4), 8.0 * n * d * d)
            out_row = r32 if key in ("node_linear_out", "node_linear_k_bwd", "node_linear_q_bwd", "node_linear_v_bwd") else row
            # unfolded, bf16 rows: the second and third node linear accumulate into dX (read + write of the fp32 row)
            extra = r32 if not sched.get("hgt_folded") and key in ("node_linear_q_bwd", "node_linear_v_bwd") else 0
            if key.endswith("_bwd"):
                return (bound, n * (2 * row + out_row + extra + 4) + segs * (w2 + d * d * 4), 4.0 * n * d * d)
            return (bound, n * (row + out_row + extra + 4) + segs * w2, 2.0 * n * d * d)
    w2 = d * d * 4
    # RGAT up to width 64: the gradient row of a single-edge pair is not stored per pair; the
    # backward typed linear reads att_e * dOut[dst_e] through a row selector (one index per pair; ds_src[p] and
    # the scale come as one pair of floats per pair and head)
    sel = bool(sched.get("row_select", layer == "rgat" and H == 1 and d <= 64)) and layer == "rgat"
    fused = bool(sched.get("fused_softmax", layer == "rgat" and H == 1))       # single-head RGAT: softmax inside the walks
    P1s = P1 if sel or H == 1 else 0      # single-edge pairs that the edge walk / the row selector serve
    # width 128: fp32 products by three bf16 planes on the bf16 matrix cores, bound by the rows, except the forward of RGAT and
    # RGCN, which stays on the fp32 instructions
    mm = "hbm" if d == 128 else "mfma"
    pair_fwd = (mm, P * (2 * row + 4) + R * w2, 2.0 * P * d * d)        # gathered row + stored row + pair_src
    pair_bwd = (mm, P * (3 * row + 4) + R * w2, 4.0 * P * d * d)        # dY row + gathered row + stored row
    node_fwd = (mm, N * (2 * row + 4) + T * w2, 2.0 * N * d * d)
    node_bwd = (mm, N * (3 * row + 4) + T * w2, 4.0 * N * d * d)
    out_dst = row if layer == "hgt" else r32                                  # HGT's Z / dQ are intermediates
    agg_dst = ("hbm", E * (row + 4 + 4 * H) + N * (out_dst + 8), 2.0 * E * d)  # row + in_pair + coefficient(s); out row + item
    table = {
        # RGAT: + s_src per pair and head; backward also reads ds_src
        "typed_linear_fwd": ("mfma", pair_fwd[1] + (P * 4 * H if layer == "rgat" and not fused else 0), pair_fwd[2]),
        # RGCN: the selector and the scale with the row selector, nothing without
        "typed_linear_bwd": (mm, pair_bwd[1] + ((P * (4 + 8 * H) if sel else P * 4 if H == 1 else 0) if layer == "rgat" else P * 8 if sched.get("row_select") else 0), pair_bwd[2]),
        "typed_linear_loop_bwd": ("mfma", pair_bwd[1] + (P * 8 if sched.get("row_select") else 0) + N * 3 * r32 + w2, pair_bwd[2] + 4.0 * N * d * d),
        "self_loop_fwd": ("mfma", N * 3 * r32 + w2, 2.0 * N * d * d),         # X row + out row read and written
        "self_loop_bwd": (mm, N * 3 * r32 + w2, 4.0 * N * d * d),
        # fused RGAT walk: row + in_pair + in_rel + in_run per edge, s_dst per run and head, out row + item + (m, s) per head per node
        "aggregate_fwd": ("hbm", E * (row + 12) + Q * 4 * H + N * (r32 + 8 + 8 * H), 4.0 * E * d) if fused else agg_dst,
        # the whole RGCN forward of a small graph: rows in and out, the edges' sources, every weight once
        "rgcn_small_fwd": ("hbm", 2 * N * r32 + E * 4 + Q * 8 + R * w2, 2.0 * Q * d * d),
        # the same sum edge by edge with atomic adds: + in_run and run_dst per edge, and the zero fill
        "aggregate_fwd_edge_parallel": ("hbm", agg_dst[1] + E * 8 + N * r32, 2.0 * E * d),
        # per edge: Hs row + in_pair + att + (att, dz) store; per node: dOut row + out row + item;
        # per single-edge pair (P1 of them): ds_src and its G row, or with the row selector att_e only
        # (fused: att is recomputed, so in_rel, in_run and s_dst are read instead of att, and (m, s) per node)
        # (several heads: (att, dz), s_dst, (m, s) and the single-edge pairs' entries once per head)
        "edge_dot_bwd": ("hbm", E * (row + 12 + 8 * H) + Q * 4 * H + N * (2 * row + 8 + 8 * H) + P1s * ((4 * H if sel else row) + 4 * H), 4.0 * E * d) if fused
                        else ("hbm", E * (row + 16) + N * (2 * row + 8) + P1 * ((4 if sel else row) + 4), 2.0 * E * d),
        # RGAT: only the E - P1 edges of the P - P1 pairs with several edges; coefficient = the (att, dz) pair;
        # with one head the walk also writes ds_src per pair.
        # RGCN: every edge; row + out_dst + coefficient
        # RGCN with the row selector: likewise only pairs with several edges (the typed-linear backward reads the
        # others' rows straight from the destinations' gradient rows)
        "aggregate_bwd_pair": ("hbm", (E - P1s) * (row + 8 + 8 * H) + (P - P1s) * (row + 8 + 4 * H), 2.0 * (E - P1s) * d) if layer == "rgat"
                              else ("hbm", (E - P1) * (row + 8) + (P - P1) * (row + 8), 2.0 * (E - P1) * d) if sched.get("row_select", half)
                              else ("hbm", E * (row + 8) + P * (row + 8), 2.0 * E * d),
        # RGAT: the two walks in one launch; per run X row + relrun_idx + run_dst + ds_dst per head
        "pair_run_walks": ("hbm", (E - P1s) * (row + 8 + 8 * H) + (P - P1s) * (row + 8 + 4 * H) + Q * (row + 8 + 4 * H), 2.0 * (E - P1s + Q * H) * d),
        "dst_side_wgrad": ("hbm", Q * (row + 12), 2.0 * Q * d),
        # per pair: dXp row + srcpair_idx; per run (RGAT): ds_dst + run_rel; per node: result row + 2 ptrs
        # (HGT on the folded path: two per-pair tensors are summed and the query part, an fp32 row per node, is added;
        #  the result is the layer's fp32 dX.  Several heads: one ds_dst per run and head.)
        "node_grad_sum": ("hbm", P * (2 * row + 4) + N * (2 * r32 + 8), 2.0 * P * d) if layer == "hgt" and sched.get("hgt_folded")
                         else ("hbm", P * (row + 4) + (Q * (4 + 4 * H) if layer == "rgat" else 0) + N * (out_dst + 8), 1.0 * P * d),
        # per edge: in_pair, in_run, s_src, s_dst, att write (reads of its own writes not counted)
        "edge_softmax": ("hbm", E * 20 + N * 8, 10.0 * E),
        # per run: run_dst, run_rel, s_dst; per destination with edges: its X row (its runs are adjacent)
        "run_logit": ("hbm", Q * 12 + n_dst * row, 2.0 * Q * d),
        # HGT
        "node_linear_k": node_fwd, "node_linear_q": node_fwd, "node_linear_v": node_fwd, "node_linear_out": node_fwd,
        "node_linear_k_bwd": node_bwd, "node_linear_q_bwd": node_bwd, "node_linear_v_bwd": node_bwd,
        "node_linear_out_bwd": node_bwd,
        "pair_linear_att": pair_fwd, "pair_linear_msg": pair_fwd,
        # several products in one launch: query and both pair linears (folded), or the node and the pair linears (unfolded)
        "node_pair_linears": (mm, node_fwd[1] + 2 * pair_fwd[1], node_fwd[2] + 2 * pair_fwd[2]),
        "node_linears": (mm, 3 * node_fwd[1], 3 * node_fwd[2]), "pair_linears": (mm, 2 * pair_fwd[1], 2 * pair_fwd[2]),
        "node_pair_linears_bwd": (mm, node_bwd[1] + 2 * pair_bwd[1], node_bwd[2] + 2 * pair_bwd[2]),
        "pair_linear_att_bwd": pair_bwd, "pair_linear_msg_bwd": pair_bwd,
        # the walks gather the key and the message row of a pair together (2 rows per edge).  Forward: + pair id; per node the
        # query row, the result row, (max, sum) per head and the item.  Backward: + pair id and the (att, dl) pair per head;
        # per node the query, gradient and result rows in, dQ out.  Pair-major: the query and gradient rows of the edge's
        # destination, position, destination and the (att, dl) pair per head; per pair the two gradient rows
        "hgt_attend_fwd": ("hbm", E * (2 * row + 4) + N * (2 * row + 8 + 8 * H), 4.0 * E * d + 10.0 * E * H),
        "hgt_attend_bwd": ("hbm", E * (2 * row + 4 + 8 * H) + N * (4 * row + 8 + 8 * H), 6.0 * E * d),
        "hgt_pair_bwd": ("hbm", E * (2 * row + 8 + 8 * H) + P * (2 * row + 8), 4.0 * E * d),
    }
    return table.get(name)


def make_layer(c, g, heads=0, flags=0):
    """-> (layer object, forward-only?) for workload dict c on graph g."""
    from paper_2412_04747_amd.harness import RgatLayer, RgcnLayer, HgtLayer
    d, dt = c["d_out"], c["dtype"]
    if c["layer"] == "rgat":
        L = RgatLayer(g, d, c["slope"], dtype=dt, heads=max(heads, 1), flags=flags)
        L.load(c["X"], c["W"], c["w_s"], c["w_t"], c["dOut"])
    elif c["layer"] == "rgcn":
        L = RgcnLayer(g, d, c["norm"], "none", False, dtype=dt, flags=flags)
        L.load(c["X"], c["W"], None, c["dOut"])
    else:
        L = HgtLayer(g, d, c["H"], with_mu=False, dtype=dt, flags=flags)
        L.load(c["X"], c["Wk"], c["Wq"], c["Wv"], c["Wo"], c["Watt"], c["Wmsg"], None, c["dOut"])
    return L


def run_oracle(c):
    """-> (dict of expected outputs, seconds forward, seconds backward)."""
    from oracle import layers as O
    N, s, t, r = c["N"], c["src"], c["dst"], c["rel"]
    t0 = time.time()
    if c["layer"] == "rgat" and c["H"] > 1:
        out = O.rgat_heads_fwd(N, s, t, r, c["X"], c["W"], c["w_s"], c["w_t"], c["H"], c["slope"])
        tf = time.time() - t0; t0 = time.time()
        want = O.rgat_heads_bwd(N, s, t, r, c["X"], c["W"], c["w_s"], c["w_t"], c["dOut"], c["H"], c["slope"])
    elif c["layer"] == "rgat":
        out = O.rgat_fwd(N, s, t, r, c["X"], c["W"], c["w_s"], c["w_t"], c["slope"])
        tf = time.time() - t0; t0 = time.time()
        want = O.rgat_bwd(N, s, t, r, c["X"], c["W"], c["w_s"], c["w_t"], c["dOut"], c["slope"])
    elif c["layer"] == "rgcn":
        out = O.rgcn_fwd(N, s, t, r, c["X"], c["W"], None, c["norm"], "none")
        tf = time.time() - t0; t0 = time.time()
        want = {} if c["cid"] == 1 else O.rgcn_bwd(N, s, t, r, c["X"], c["W"], None, c["dOut"], c["norm"], "none", out=out)
        want.pop("dW0", None)
    else:
        names = ("X", "Wk", "Wq", "Wv", "Wo", "Watt", "Wmsg")
        out = O.hgt_fwd(N, s, t, r, c["ntype"], *[c[k] for k in names], None)
        tf = time.time() - t0; t0 = time.time()
        want = O.hgt_bwd(N, s, t, r, c["ntype"], *[c[k] for k in names], None, c["dOut"])
        want.pop("dmu", None)
    tb = time.time() - t0
    want["out"] = out
    return want, tf, tb


def train_step_bench(args):
    """Two-layer RGAT model, full-graph training step (forward, NLL loss, backward, SGD), the
    protocol of the thesis' evaluation section; one JSON line like the layer benchmark."""
    import numpy as np
    import torch
    from paper_2412_04747_amd import synth, binding as B, autograd as A
    c = synth.config(args.config, args.scale)
    if c["layer"] != "rgat":
        sys.exit("bench.py --train: pick an RGAT workload (--config 2 or 3)")
    N, R, E, d = c["N"], c["R"], c["E"], c["d_out"]
    g = A.Graph(N, R, c["src"], c["dst"], c["rel"])
    torch.manual_seed(synth.SEED0)
    layers = [A.RgatConv(R, d, c["slope"]), A.RgatConv(R, d, c["slope"])]
    params = [q for l in layers for q in l.parameters()]
    X = torch.tensor(c["X"], dtype=torch.float32, device="cuda")
    rng = np.random.default_rng(synth.SEED0)
    train = torch.as_tensor(rng.choice(N, max(N // 10, 1), replace=False), device="cuda")
    labels = torch.as_tensor(rng.integers(0, d, len(train)), device="cuda")
    opt = torch.optim.SGD(params, lr=1e-3)

    def step():
        opt.zero_grad(set_to_none=True)
        h = layers[1](g, torch.relu(layers[0](g, X)))
        loss = torch.nn.functional.nll_loss(torch.log_softmax(h[train], dim=1), labels)
        loss.backward()
        opt.step()
        return loss

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    B.rgnn_profile_start()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        loss = step()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    rep = B.rgnn_profile_stop()
    lib_ms = sum(ms for _, ms in rep.values()) / args.steps
    print(f"[bench] train step {dt * 1e3 / args.steps:.3f} ms, of which {lib_ms:.3f} ms in the library's kernels; "
          f"last loss {loss.item():.4f}", file=sys.stderr, flush=True)
    print(json.dumps({
        "metric": "edges/sec for 2-layer RGAT training step (fwd + NLL loss + bwd + SGD)",
        "value": 2 * E * args.steps / dt, "unit": "edges/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": dt * 1e3 / args.steps, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"configs[{args.config - 1}] graph, two RGAT layers of width {d}, N={N}, R={R}, E={E}; "
                               "value counts every edge once per layer"},
        "library_kernel_ms_per_step": lib_ms}))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", type=int, default=3,
                    help="synthetic workload id 1..5 (default 3 = the headline RGAT graph the metric is quoted on)")
    ap.add_argument("--scale", type=float, default=1.0, help="shrink the workload (debugging only)")
    ap.add_argument("--no-oracle", action="store_true", help="skip the CPU oracle leg (no cpu_baseline, no parity)")
    ap.add_argument("--dtype", choices=("f32", "bf16"), default=None,
                    help="override the storage type of the workload's inputs (the values stay the same)")
    ap.add_argument("--heads", type=int, default=0, help="RGAT workloads: number of attention heads (default 1)")
    ap.add_argument("--edge-parallel", action="store_true",
                    help="single-head RGAT: forward aggregation edge by edge with atomic adds (comparison schedule)")
    ap.add_argument("--no-batched", action="store_true", help="force the general walk for every segment (desc.flags)")
    ap.add_argument("--no-row-select", action="store_true",
                    help="write the gradient rows of single-edge pairs per pair instead of reading them through the row selector")
    ap.add_argument("--no-folding", action="store_true", help="HGT: keep node linears and per-relation matrices apart")
    ap.add_argument("--separate-softmax", action="store_true",
                    help="single-head RGAT: edge softmax as a pass of its own with one attention weight per edge")
    ap.add_argument("--fwd-only", action="store_true",
                    help="time the forward call alone (inference: no saved buffer is kept)")
    ap.add_argument("--graph", action="store_true",
                    help="record one step into a HIP graph and time its replays (no per-kernel breakdown: the "
                         "timing events cannot be recorded into a graph)")
    ap.add_argument("--train", action="store_true",
                    help="time a full training step instead: two RGAT layers through the autograd front end, "
                         "log-softmax + NLL loss on 10%% of the nodes, SGD update (RGAT workloads only)")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on one GPU only (--gpus 1); sharding over several GPUs is a design "
                 "note, not code.")

    import numpy as np
    import torch
    from paper_2412_04747_amd import synth, binding as B
    from paper_2412_04747_amd.harness import Graph

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    if args.train:
        return train_step_bench(args)
    t0 = time.time()
    c = synth.config(args.config, args.scale)
    if args.dtype:
        if args.dtype == "bf16" and c["dtype"] != "bf16":
            for k, v in list(c.items()):
                if isinstance(v, np.ndarray) and v.dtype == np.float32:
                    c[k] = synth.round_to_bf16(v)
        c["dtype"] = args.dtype
    if args.heads > 1:
        if c["layer"] != "rgat":
            sys.exit("bench.py --heads: only the RGAT workloads take a head count")
        c["H"] = args.heads
    N, R, E, d, T, H = c["N"], c["R"], c["E"], c["d_out"], c["T"], c["H"]
    fwd_only = c["cid"] == 1 or args.fwd_only
    print(f"[bench] generated config {args.config} ({c['layer']}, {c['dtype']}): N={N} T={T} R={R} E={E} d={d} H={H} "
          f"in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)

    cpu = None
    want = None
    if not args.no_oracle:
        from oracle import layers as O
        # the whole workload, repeated until about ten seconds of CPU work are timed (at most eight times)
        t_f = t_b = 0.0
        reps = 0
        while reps < 8 and (reps == 0 or t_f + t_b < 10.0):
            want, tf1, tb1 = run_oracle(c)
            t_f += tf1
            t_b += 0.0 if fwd_only else tb1
            reps += 1
        cpu = {"value": E * reps / (t_f + t_b), "unit": "edges/s", "cores": O.num_threads(), "kind": "oracle",
               "sample": f"full workload, {reps} repetition{'s' if reps > 1 else ''} (fwd {t_f:.2f}s + bwd {t_b:.2f}s in all)"}
        print(f"[bench] oracle x{reps}: fwd {t_f:.2f}s bwd {t_b:.2f}s on {O.num_threads()} threads", file=sys.stderr, flush=True)

    t0 = time.time()
    g = Graph(N, R, c["src"], c["dst"], c["rel"], c.get("ntype") if T > 1 else None, T,
              c.get("rel_src_ntype"), c.get("rel_dst_ntype"))
    P, Q = g.P, g.Q
    P1 = int(g.info.num_single_pairs) if c["layer"] in ("rgat", "rgcn") else 0
    print(f"[bench] graph index built in {time.time() - t0:.1f}s: P/E={P / E:.3f} Q/E={Q / E:.3f} "
          f"max in-degree {g.info.max_in_degree} index {g.info.index_bytes / 2**20:.0f} MiB", file=sys.stderr, flush=True)
    if (args.edge_parallel or args.separate_softmax) and (c["layer"] != "rgat" or args.heads > 1):
        sys.exit("bench.py --edge-parallel / --separate-softmax: single-head RGAT workloads only")
    flags = ((B.RGNN_FLAG_EDGE_PARALLEL_AGGREGATION if args.edge_parallel else 0) | (B.RGNN_FLAG_NO_BATCHED_WALKS if args.no_batched else 0)
             | (B.RGNN_FLAG_NO_ROW_SELECT if args.no_row_select else 0) | (B.RGNN_FLAG_NO_WEIGHT_FOLDING if args.no_folding else 0)
             | (B.RGNN_FLAG_SEPARATE_SOFTMAX if args.separate_softmax else 0))
    L = make_layer(c, g, args.heads, flags)
    sched = B.rgnn_schedule(g.handle, {"rgcn": B.RGNN_LAYER_RGCN, "rgat": B.RGNN_LAYER_RGAT, "hgt": B.RGNN_LAYER_HGT}[c["layer"]], L.desc)
    n_dst = int(np.count_nonzero(np.bincount(c["dst"], minlength=N)))
    print(f"[bench] schedule picked by the library (flags {flags}): {sched}", file=sys.stderr, flush=True)

    def step():
        L.fwd()
        if not fwd_only:
            L.bwd()

    # One plain 1 GiB device-to-device copy before the timed region: a kernel of known size
    # against which rocprofv3's FETCH_SIZE / WRITE_SIZE counters are calibrated.
    cal = torch.empty(2, 1 << 28, dtype=torch.float32, device="cuda")
    cal[0].fill_(1.0)
    cal[1].copy_(cal[0])
    torch.cuda.synchronize()
    del cal

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    if args.graph:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        hip_graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            step()
            side.synchronize()
            with torch.cuda.graph(hip_graph, stream=side):
                step()
        torch.cuda.synchronize()
        for _ in range(args.warmup):
            hip_graph.replay()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            hip_graph.replay()
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        print(json.dumps({
            "metric": f"edges/sec for {c['layer'].upper()} layer {'fwd' if fwd_only else 'fwd+bwd'} (HIP graph replay)",
            "value": E * args.steps / dt, "unit": "edges/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
            "ms_per_step": dt * 1e3 / args.steps, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "bf16" if c["dtype"] == "bf16" else "f32", "data": "synthetic",
            "config": {"workload": f"configs[{args.config - 1}]: {c['layer'].upper()}, {c['dtype']} inputs, N={N}, R={R}, E={E}, d={d}"},
            "cpu_baseline": cpu}), flush=True)
        return
    # Pass 1 (not the timed region): the same K steps with HIP events around every kernel launch, for the per-kernel
    # table and to find the dominant kernel.
    B.rgnn_profile_select(None)
    B.rgnn_profile_start()
    torch.cuda.synchronize()
    tc = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    all_events_ms = (time.perf_counter() - tc) * 1e3 / args.steps
    rep = B.rgnn_profile_stop()
    dom_name = max(rep.items(), key=lambda kv: kv[1][1])[0]
    # Timed region: K steps, HIP events only around the dominant kernel (two per step), whose average duration over
    # exactly these steps goes into the roofline entry.
    B.rgnn_profile_select(dom_name)
    B.rgnn_profile_start()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    dom_rep = B.rgnn_profile_stop()
    B.rgnn_profile_select(None)
    ms_per_step = dt * 1e3 / args.steps
    dom_n, dom_ms = dom_rep[dom_name]

    parity = None
    if want is not None:
        parity = {}
        got = dict(out=L.out, **({} if fwd_only else L.grads()))
        for k, v in got.items():
            if k not in want:
                continue
            a = v.cpu().numpy().astype(np.float64)
            parity[k] = float(np.abs(a - want[k]).max() / max(np.abs(want[k]).max(), 1e-30))
        print(f"[bench] max relative error vs oracle: {parity}", file=sys.stderr, flush=True)

    half = c["dtype"] == "bf16" and d == 128
    # rows per run instead of per pair: the library's pick on large graphs with fewer runs (a call whose flags bring the rows per pair
    # back leaves the runs' inputs in `saved` as well)
    runs = "run_inputs" in rep and not {"single_logits", "aggregate_bwd_pair"} & set(rep)
    Q1 = int((np.unique(c["dst"].astype(np.int64) * R + c["rel"], return_counts=True)[1] == 1).sum()) if runs else 0

    def work(name):
        if runs and not name.endswith((".reduce", ".combine", ".finish")):
            w = run_row_work(name, E, N, P, Q, Q1, R, d, c["layer"], n_dst)
            if w:
                return w
        w = algorithmic_work(name, E, N, P, Q, R, T, d, H, P1, c["dtype"] == "bf16", c["layer"], sched, n_dst)
        if name == "node_linear_q_bwd" and "node_grad_sum" not in rep and sched.get("hgt_folded") and half:
            w = (w[0], w[1] + P * (d * 2 + 4) + N * 8, w[2] + 1.0 * P * d)      # with the sum over the node's pairs
        return w

    kernels = []
    for name, (n, ms) in rep.items():
        avg_ms = ms / n
        w = work(name)
        row = {"name": name, "launches_per_step": n / args.steps, "avg_ms": avg_ms, "ms_per_step": ms / args.steps}
        if w:
            row["GBps"] = w[1] / avg_ms / 1e6
            row["TFLOPs"] = w[2] / avg_ms / 1e9
            row["bound"] = w[0]
        kernels.append(row)
    kernels.sort(key=lambda r: -r["ms_per_step"])
    for r in kernels:
        print("[bench] {name:28s} {ms_per_step:8.3f} ms/step  avg {avg_ms:8.3f} ms  {gb:>9s} GB/s {tf:>8s} TF/s".format(
            gb=f"{r['GBps']:.0f}" if "GBps" in r else "-", tf=f"{r['TFLOPs']:.1f}" if "TFLOPs" in r else "-", **r),
            file=sys.stderr, flush=True)
    # the dominant kernel's row, re-measured over the timed region
    w = work(dom_name)
    dom = {"name": dom_name, "avg_ms": dom_ms / dom_n}
    if w:
        dom["GBps"] = w[1] / dom["avg_ms"] / 1e6
        dom["TFLOPs"] = w[2] / dom["avg_ms"] / 1e9
    mfma_peak = BF16_MFMA_PEAK_TFLOPS if half else FP32_MFMA_PEAK_TFLOPS
    if w and w[0] == "mfma":
        roof = {"kernel": dom["name"], "bound": "mfma", "achieved": dom["TFLOPs"], "peak": mfma_peak,
                "unit": "TFLOP/s", "frac": dom["TFLOPs"] / mfma_peak, "traffic": None}
    else:
        gb = dom.get("GBps", 0.0)
        roof = {"kernel": dom["name"], "bound": "hbm", "achieved": gb, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": gb / HBM_PEAK_GBS, "traffic": None}
    # HBM bytes per launch from rocprofv3 counters: not measurable from inside this process, so they come from the
    # committed summary of two --pmc runs of this same command (calibrated against the 1 GiB copy above), and only
    # while that summary was taken from the kernel sources this run uses.
    sha = library_sha16()
    default_run = args.config == 3 and args.scale == 1.0 and flags == 0 and args.heads <= 1 and not args.dtype and not fwd_only
    if default_run:
        roof["traffic"], roof["traffic_source"] = counter_traffic(dom["name"], sha)
    else:
        roof["traffic_source"] = "no counter summary is kept for this workload / schedule"
    roof["avg_ms"] = dom["avg_ms"]
    roof["launches_timed"] = dom_n
    roof["algorithmic_bytes"] = w[1] if w else None
    kern_ms = {k["name"]: k["ms_per_step"] for k in kernels}
    steps_roof = None
    if c["layer"] == "rgat" and H == 1 and not fwd_only:
        steps_roof = run_row_steps(kern_ms, E, N, P, Q, Q1, d) if runs else step_rooflines(kern_ms, E, N, P, P1, Q, d)
    if steps_roof:
        for k, v in steps_roof.items():
            print(f"[bench] {k:24s} {v['ms']:.3f} ms  {v['achieved']:.0f} GB/s = {v['frac']:.2f} of HBM peak", file=sys.stderr, flush=True)

    line = {
        "metric": f"edges/sec for {c['layer'].upper()} layer {'fwd' if fwd_only else 'fwd+bwd'}",
        "value": E * args.steps / dt, "unit": "edges/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        # the arithmetic type of the path: fp32 throughout, or bf16 storage / bf16 matrix-core operands with
        # fp32 accumulation for the bfloat16 workloads
        "dtype": "bf16" if c["dtype"] == "bf16" else "f32", "data": "synthetic",
        "config": {"workload": f"configs[{args.config - 1}]: {c['layer'].upper()} {'fwd' if fwd_only else 'fwd+bwd'}, "
                               f"{c['dtype']} inputs, N={N}, T={T}, R={R}, E={E}, d={d}, H={H}"
                               + ("" if args.scale == 1.0 else f" (scale {args.scale})"),
                   "P_over_E": P / E, "Q_over_E": Q / E, "max_in_degree": int(g.info.max_in_degree)},
        "roofline": roof,
        "roofline_steps": steps_roof,
        "schedule": sched,
        "rows_per_run": runs,
        "lib_sha16": sha,
        "cpu_baseline": cpu,
        # the separate pass with events around every kernel, which the `kernels` table and `roofline_steps` come from
        "ms_per_step_with_events_on_every_kernel": all_events_ms,
        "parity_max_rel_err": parity,
        "kernels": kernels,
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
