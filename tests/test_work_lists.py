"""Host planning of the kernels' work lists (tiles/chunks/slots of the typed-linear kernels,
items of the traversal kernels), checked on the CPU against what the kernels rely on.
The planning header is compiled with g++ into a small test library; no GPU is involved."""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
K = dict(tile_rows=0, max_chunks=1, wide_chunks=2, min_chunks=3, chunk_tiles=4, item_max=5, item_target=6, serial_max=7,
         short_len=8)


@pytest.fixture(scope="module")
def wl():
    out = os.path.join(tempfile.mkdtemp(prefix="rgnn_wl_"), "libwl.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-o", out,
                           os.path.join(HERE, "host", "work_lists_shim.cpp")])
    lib = C.CDLL(out)
    lib.wl_item_cut.argtypes = [C.c_longlong]
    return lib


def _field(fn, which, n_hint=1 << 22):
    buf = np.empty(n_hint, np.int32)
    n = fn(which, buf.ctypes.data_as(C.c_void_p), n_hint)
    assert n <= n_hint
    return buf[:n].copy()


def plan_items(lib, ptr, max_len, min_len=0):
    ptr = np.ascontiguousarray(ptr, np.int32)
    n = lib.wl_plan_items(ptr.ctypes.data_as(C.c_void_p), len(ptr) - 1, max_len, min_len)
    names = ("beg", "end", "row", "slot", "split_row", "split_ptr", "part_item", "part_split", "long_item")
    p = {k: _field(lib.wl_items_field, i) for i, k in enumerate(names)}
    sc = np.zeros(6, np.int32)
    lib.wl_items_scalars(sc.ctypes.data_as(C.c_void_p))
    p.update(num_items=n, num_partials=int(sc[0]), num_split=int(sc[1]), first_single=int(sc[2]), num_single=int(sc[3]),
             first_short=int(sc[4]), num_short=int(sc[5]))
    return p


def plan_tiles(lib, seg_ptr, tile_rows, max_chunks):
    seg_ptr = np.ascontiguousarray(seg_ptr, np.int32)
    n = lib.wl_plan_tiles(seg_ptr.ctypes.data_as(C.c_void_p), len(seg_ptr) - 1, tile_rows, max_chunks)
    names = ("tile_seg", "tile_row0", "tile_row1", "chunk_tile", "chunk_slot", "seg_slot_ptr")
    p = {k: _field(lib.wl_tiles_field, i) for i, k in enumerate(names)}
    sc = np.zeros(3, np.int32)
    lib.wl_tiles_scalars(sc.ctypes.data_as(C.c_void_p))
    p.update(num_tiles=n, num_chunks=int(sc[0]), num_slots=int(sc[1]), num_segs=int(sc[2]))
    return p


def _segments(rng, S, hubs):
    """Segment lengths with empty, single-entry, short and a few very long segments."""
    ln = rng.choice([0, 1, 1, 2, 3, 5, 9, 31, 32, 33, 40], size=S)
    for h in hubs:
        ln[rng.integers(0, S)] = h
    return np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)


@pytest.mark.parametrize("max_len,min_len,hubs", [(256, 0, (257, 256, 1000, 5000)), (32, 0, (33, 64, 700)),
                                                   (64, 2, (65, 129, 300)), (1 << 30, 0, (4000,))])
def test_items_cover_each_segment_once(wl, max_len, min_len, hubs):
    rng = np.random.default_rng(7 + max_len % 1000 + min_len)
    ptr = _segments(rng, 3000, hubs)
    p = plan_items(wl, ptr, max_len, min_len)
    serial_max = wl.wl_constant(K["serial_max"])
    n = p["num_items"]
    ln = p["end"] - p["beg"]
    seg_len = np.diff(ptr)
    # every entry of every kept segment lies in exactly one item of that segment; no item is too long
    cover = np.zeros(ptr[-1], np.int32)
    for i in range(n):
        s = p["row"][i]
        assert ptr[s] <= p["beg"][i] <= p["end"][i] <= ptr[s + 1]
        cover[p["beg"][i]:p["end"][i]] += 1
    kept = np.repeat(seg_len >= min_len, seg_len)
    assert (cover[kept] == 1).all() and (cover[~kept] == 0).all()
    assert ln.max() <= max_len
    # whole segments appear once (also the empty ones, which still own an output row), dropped ones never
    whole = p["slot"] < 0
    rows_whole = np.sort(p["row"][whole])
    expect_whole = np.nonzero((seg_len >= min_len) & (seg_len <= max_len))[0]
    assert np.array_equal(rows_whole, expect_whole)
    assert (ln[whole] == seg_len[p["row"][whole]]).all()
    # order: items longer than short_len by length (longest first, pieces before whole segments of the same
    # length), then the short pieces, then the short whole segments by length
    short_len = wl.wl_constant(K["short_len"])
    klass = np.where(ln > short_len, 0, np.where(~(p["slot"] < 0), 1, 2))
    assert (np.diff(klass) >= 0).all()
    for kl in (0, 2):
        sel = np.nonzero(klass == kl)[0]
        assert (np.diff(ln[sel]) <= 0).all()
        same = sel[:-1][np.diff(ln[sel]) == 0]
        assert not ((p["slot"][same] < 0) & (p["slot"][same + 1] >= 0)).any()
    # cut segments: partial rows numbered 0..num_partials-1, grouped per segment in split_ptr order
    cut = np.nonzero(seg_len > max_len)[0]
    assert p["num_split"] == len(cut) and np.array_equal(p["split_row"], cut)
    assert p["split_ptr"][0] == 0 and p["split_ptr"][-1] == p["num_partials"]
    assert np.array_equal(np.sort(p["slot"][~whole]), np.arange(p["num_partials"]))
    for k, s in enumerate(cut):
        a, b = p["split_ptr"][k], p["split_ptr"][k + 1]
        assert b - a == -(-seg_len[s] // max_len)
        items = p["part_item"][a:b]
        assert (p["slot"][items] == np.arange(a, b)).all() and (p["row"][items] == s).all()
        assert (p["part_split"][a:b] == k).all()
        assert p["beg"][items[0]] == ptr[s] and p["end"][items[-1]] == ptr[s + 1]     # pieces in order
        assert (p["beg"][items[1:]] == p["end"][items[:-1]]).all()
    # the single-entry whole segments are one contiguous range
    single = np.nonzero((ln == 1) & whole)[0]
    assert p["num_single"] == len(single)
    if len(single):
        assert p["first_single"] == single[0] and single[-1] == single[0] + len(single) - 1
    # ... preceded directly by the whole segments with 2..short_len entries
    short = np.nonzero((ln >= 2) & (ln <= short_len) & whole)[0]
    assert p["num_short"] == len(short)
    if len(short):
        assert p["first_short"] == short[0] and short[-1] == short[0] + len(short) - 1
        if len(single):
            assert single[0] == short[-1] + 1
    # long items: more than serial_max entries, or any piece of a cut segment
    assert np.array_equal(p["long_item"], np.nonzero((ln > serial_max) | ~whole)[0])


def test_items_keep_segment_order_within_a_length(wl):
    """Stable order: among whole segments of equal length the output rows ascend, which keeps the
    stores of neighbouring lanes close together."""
    rng = np.random.default_rng(3)
    ptr = _segments(rng, 2000, (300,))
    p = plan_items(wl, ptr, 256)
    ln = p["end"] - p["beg"]
    for length in (0, 1, 2, 4, 5):
        rows = p["row"][(ln == length) & (p["slot"] < 0)]
        assert (np.diff(rows) > 0).all()


def test_items_empty_input(wl):
    p = plan_items(wl, np.zeros(1, np.int32), 256)
    assert p["num_items"] == 0 and p["num_partials"] == 0 and p["num_single"] == 0 and list(p["split_ptr"]) == [0]
    p = plan_items(wl, np.zeros(6, np.int32), 256)          # five empty segments
    assert p["num_items"] == 5 and (p["end"] == p["beg"]).all() and p["num_single"] == 0


def test_item_cut_grows_with_the_list(wl):
    lo, hi, target = wl.wl_constant(K["serial_max"]), wl.wl_constant(K["item_max"]), wl.wl_constant(K["item_target"])
    cuts = [wl.wl_item_cut(t) for t in (0, 1, 10_000, 200_000, 3_000_000, 10_000_000, 10**9)]
    assert cuts[0] == lo and cuts[-1] == hi and cuts == sorted(cuts)
    for t, c in zip((200_000, 3_000_000), cuts[3:5]):
        assert c == hi or c * target >= t                   # fine enough to yield `target` items, or at the cap
        assert c & (c - 1) == 0


@pytest.mark.parametrize("S,max_chunks", [(1, 4096), (7, 4096), (200, 4096), (200, 1024), (500, 64)])
def test_tiles_chunks_and_slots(wl, S, max_chunks):
    rng = np.random.default_rng(11 + S)
    ln = rng.choice([0, 1, 63, 64, 65, 200, 5000], size=S)
    ln[rng.integers(0, S)] = 300_000
    seg_ptr = np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)
    T = wl.wl_constant(K["tile_rows"])
    p = plan_tiles(wl, seg_ptr, T, max_chunks)
    nt, nc = p["num_tiles"], p["num_chunks"]
    assert p["num_segs"] == S
    # tiles: in row order, inside one segment, at most T rows, covering every row once
    assert nt == int(np.sum(-(-ln // T)))
    rows = p["tile_row1"] - p["tile_row0"]
    assert (rows > 0).all() and (rows <= T).all()
    assert (seg_ptr[p["tile_seg"]] <= p["tile_row0"]).all() and (p["tile_row1"] <= seg_ptr[p["tile_seg"] + 1]).all()
    assert rows.sum() == seg_ptr[-1] and (p["tile_row0"][1:] >= p["tile_row1"][:-1]).all()
    # chunks: a partition of the tiles into consecutive, nearly equal ranges
    assert nc <= max_chunks and nc <= max(nt, 1)
    ct = p["chunk_tile"]
    assert ct[0] == 0 and ct[-1] == nt and (np.diff(ct) >= 0).all()
    if nc:
        assert np.diff(ct).max() - np.diff(ct).min() <= 1
    # slots: one per (chunk, segment it touches), numbered in chunk order; a segment's slots are consecutive
    slot_of = []
    nxt = 0
    for c in range(nc):
        assert p["chunk_slot"][c] == nxt
        segs = p["tile_seg"][ct[c]:ct[c + 1]]
        for j, s in enumerate(segs):
            if j == 0 or s != segs[j - 1]:
                slot_of.append(s)
                nxt += 1
    assert p["num_slots"] == nxt
    slot_of = np.asarray(slot_of, np.int64)
    assert (np.diff(slot_of) >= 0).all()
    ssp = p["seg_slot_ptr"]
    assert ssp[0] == 0 and ssp[-1] == nxt
    for s in range(S):
        assert (slot_of[ssp[s]:ssp[s + 1]] == s).all()


# ---------------------------------------------------------------- schedule / layout choice per graph

SCHEDULE_FIELDS = ("item_len", "tile_chunks", "wide_chunks", "rows_bf16", "row_select", "hgt_folded", "fused_softmax",
                   "ws_in_lds", "edge_parallel", "dst_batched_single", "dst_batched_short", "pair_walk_multi_only",
                   "pair_batched_single", "pair_batched_short")
LAYER = dict(rgcn=0, rgat=1, hgt=2)


def graph_counts(c):
    """What the choice depends on, counted from the edge list: destinations with one / with 2..4 incoming edges,
    (source, relation) pairs with one / with 2..4 edges, and whether every relation's sources have one node type."""
    N, R = c["N"], c["R"]
    indeg = np.bincount(c["dst"], minlength=N)
    _, outdeg = np.unique(c["rel"].astype(np.int64) * N + c["src"], return_counts=True)
    cnt = lambda deg, lo, hi: int(((deg >= lo) & (deg <= hi)).sum())
    tied = True
    if c["T"] > 1:
        st = c["ntype"][c["src"]]
        tied = all(len(np.unique(st[c["rel"] == r])) <= 1 for r in range(R))
    return dict(dst=(cnt(indeg, 1, 1), cnt(indeg, 2, 4)), pair=(cnt(outdeg, 1, 1), cnt(outdeg, 2, 4)),
                pair_multi=(0, cnt(outdeg, 2, 4)), tied=tied)


def pick(lib, c, k, heads=None, flags=0, dtype=None):
    dt = dtype or c["dtype"]
    a = np.array([LAYER[c["layer"]], 1 if dt == "bf16" else 0, c["d_out"], heads or c["H"], flags, c["R"], int(k["tied"]),
                  c["E"], *k["dst"], *k["pair"], *k["pair_multi"]], dtype=np.int64)
    out = np.zeros(len(SCHEDULE_FIELDS), np.int32)
    lib.wl_pick_schedule(a.ctypes.data_as(C.c_void_p), out.ctypes.data_as(C.c_void_p))
    return dict(zip(SCHEDULE_FIELDS, (int(v) for v in out)))


# The pick for each of the five workloads (tile chunk counts depend on the device's compute-unit count and are
# not part of this table).  Fields not listed are 0.
EXPECTED_PICK = {
    1: dict(item_len=32),
    2: dict(item_len=32, row_select=1, fused_softmax=1, ws_in_lds=1, dst_batched_short=1, pair_walk_multi_only=1,
            pair_batched_short=1),
    3: dict(item_len=256, row_select=1, fused_softmax=1, ws_in_lds=1, dst_batched_single=1, dst_batched_short=1,
            pair_walk_multi_only=1, pair_batched_short=1),
    4: dict(item_len=256, rows_bf16=1, hgt_folded=1, dst_batched_single=1, dst_batched_short=1, pair_batched_single=1,
            pair_batched_short=1),
    5: dict(item_len=256, rows_bf16=1, row_select=1, dst_batched_single=1, dst_batched_short=1, pair_walk_multi_only=1,
            pair_batched_short=1),
}


@pytest.mark.parametrize("cid", [1, 2, 3, 4, 5])
def test_schedule_pick_for_the_five_workloads(wl, cid):
    import sys
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2412_04747_amd import synth
    c = synth.config(cid, graph_only=True)
    got = pick(wl, c, graph_counts(c))
    want = dict.fromkeys(SCHEDULE_FIELDS, 0)
    want.update(EXPECTED_PICK[cid])
    assert got == want, {k: (got[k], want[k]) for k in got if got[k] != want[k]}


def test_schedule_flags_force_the_alternatives(wl):
    import sys
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2412_04747_amd import synth
    c = synth.config(2, graph_only=True)
    k = graph_counts(c)
    k["dst"] = (5000, 5000); k["pair"] = (9000, 7000); k["pair_multi"] = (0, 7000)
    base = pick(wl, c, k)
    assert base["dst_batched_single"] and base["dst_batched_short"] and base["pair_batched_short"] and base["row_select"]
    assert base["fused_softmax"] and base["ws_in_lds"] and not base["edge_parallel"]
    nb = pick(wl, c, k, flags=2)
    assert not any(nb[f] for f in ("dst_batched_single", "dst_batched_short", "pair_batched_single", "pair_batched_short"))
    assert {f: v for f, v in nb.items() if "batched" not in f} == {f: v for f, v in base.items() if "batched" not in f}
    assert not pick(wl, c, k, flags=4)["row_select"] and pick(wl, c, k, flags=4)["pair_walk_multi_only"]
    sep = pick(wl, c, k, flags=16)
    assert not sep["fused_softmax"] and not sep["ws_in_lds"] and not sep["edge_parallel"]
    ep = pick(wl, c, k, flags=1)
    assert ep["edge_parallel"] and not ep["fused_softmax"]
    heads = pick(wl, c, k, heads=4)
    assert heads["fused_softmax"] and heads["row_select"] and heads["pair_walk_multi_only"]
    assert not heads["pair_batched_single"]                 # two or four heads: the row selector serves the single-edge pairs
    eight = pick(wl, c, k, heads=8)
    assert eight["fused_softmax"] and not eight["row_select"] and not eight["pair_walk_multi_only"]
    assert eight["pair_batched_single"]                     # other head counts: the pair-major walk takes every pair
    big_r = dict(c, R=300)                                  # 300 x 64 floats = 75 KB: w_s no longer fits the LDS budget
    assert pick(wl, big_r, k)["fused_softmax"] and not pick(wl, big_r, k)["ws_in_lds"]
    c4 = synth.config(4, scale=0.001, graph_only=True)
    k4 = graph_counts(c4)
    assert k4["tied"] and pick(wl, c4, k4)["hgt_folded"] and not pick(wl, c4, k4, flags=8)["hgt_folded"]
    assert not pick(wl, c4, dict(k4, tied=False))["hgt_folded"]
    assert pick(wl, c4, k4, dtype="f32")["rows_bf16"] == 0


@pytest.mark.parametrize("d,R,singles,want", [
    (64, 4, (19999, 120000), 0), (64, 4, (20000, 120000), 1), (32, 4, (124999, 1000000), 0), (32, 4, (125000, 1000000), 1),
    (128, 4, (5000, 500000), 1),    (32, 7, 19999, 0), (32, 7, 20000, 1), (64, 7, 9999, 0), (64, 7, 10000, 1), (128, 7, 4999, 0), (128, 7, 5000, 1),
    (64, 500, 79999, 0), (64, 500, 80000, 1), (32, 2000, 319999, 0), (32, 2000, 320000, 1), (128, 2000, 100000, 1),
    (64, 4000, 374999, 0), (64, 4000, 375000, 1), (32, 8000, 749999, 0), (32, 8000, 750000, 1)])
def test_row_selector_of_rgcn_where_it_pays(wl, d, R, singles, want):
    """fp32 rows: enough single-edge pairs, enough of them per relation or more rows than the caches hold, and a sixth of the edges in
    them or many (singles: their number, or that and the number of edges)."""
    singles, edges = singles if isinstance(singles, tuple) else (singles, 2 * singles)
    c = dict(layer="rgcn", dtype="f32", d_out=d, H=1, R=R, E=edges)
    k = dict(dst=(0, 0), pair=(singles, 0), pair_multi=(0, 0), tied=True)
    assert pick(wl, c, k)["row_select"] == want
    assert pick(wl, c, k, flags=4)["row_select"] == 0
    if d == 128:
        assert pick(wl, c, k, dtype="bf16")["row_select"] == 1


@pytest.mark.parametrize("R,B,cut,mean", [(1, 1, 256, 900), (7, 5, 256, 40), (40, 23, 64, 100), (300, 16, 1024, 3)])
def test_blocks_cover_each_relation_once(wl, R, B, cut, mean):
    """Every entry in one item of its relation and block, no item above the cut, the pieces of a relation in slots of its own, a relation
    in one item (or without entries) written by an item without a slot, and the items of a block of one chiplet only."""
    rng = np.random.default_rng(R + B)
    cells = rng.poisson(mean, (R, B)) * (rng.random((R, B)) < 0.7)
    cells[R // 2] = 0
    ends = np.cumsum(cells.ravel()).reshape(R, B)
    bound = np.concatenate([ends[:, :1] - cells[:, :1], ends], 1).astype(np.int32)
    n = wl.wl_plan_blocks(bound.ctypes.data_as(C.c_void_p), R, B, cut)
    beg, end, row, slot, split_row, split_ptr = (_field(wl.wl_items_field, i) for i in range(6))
    assert n == len(beg) and n % 8 == 0 and np.all(end - beg <= cut)
    seen, written, of_slot = np.zeros(ends[-1, -1], int), np.zeros(R, int), {}
    for i in range(n):
        if row[i] < 0:
            continue
        seen[beg[i]:end[i]] += 1
        if beg[i] < end[i]:
            b = np.searchsorted(ends[row[i]], beg[i], side="right")
            assert bound[row[i], b] <= beg[i] and end[i] <= bound[row[i], b + 1] and i % 8 == b % 8
        if slot[i] < 0:
            written[row[i]] += 1
        else:
            assert slot[i] not in of_slot
            of_slot[slot[i]] = row[i]
    assert np.all(seen == 1)
    for k, r in enumerate(split_row):
        written[r] += 1
        assert all(of_slot[s] == r for s in range(split_ptr[k], split_ptr[k + 1]))
    assert np.all(written == 1) and len(of_slot) == split_ptr[-1]


@pytest.mark.parametrize("N,R", [(5, 3), (1500, 8), (8192, 8), (14500, 20), (25000, 400), (94000, 20), (200000, 60), (1 << 20, 200)])
def test_blocks_give_every_chiplet_its_share(wl, N, R):
    """Nodes as likely as each other: an eighth of the entries for every chiplet, however few the nodes, and a tenth of that more at most."""
    rng = np.random.default_rng(N)
    E = 300000
    key = np.sort(rng.integers(0, R * N, E))
    B = wl.wl_node_blocks(C.c_longlong(N), R, C.c_longlong(E))
    first = -(-N * np.arange(B + 1) // B)                    # first node of each block
    bound = np.searchsorted(key, np.arange(R)[:, None] * N + first[None]).astype(np.int32)
    wl.wl_plan_blocks(bound.ctypes.data_as(C.c_void_p), R, B, 256)
    beg, end = (_field(wl.wl_items_field, i) for i in range(2))
    share = np.bincount(np.arange(len(beg)) % 8, weights=end - beg, minlength=8) / E
    assert B % 8 == 0 and abs(share.sum() - 1) < 1e-9
    assert share.max() <= 1.1 / 8 or N < 8, share


@pytest.mark.parametrize("E,d,R,rows,want", [
    (131071, 128, 1, 0.6, "000"), (131072, 128, 1, 0.6, "110"), (131072, 128, 1, 0.96, "000"), (240000, 32, 8, 0.6, "000"), (250000, 32, 8, 0.6, "100"),
    (269999, 64, 8, 0.6, "100"), (270000, 64, 8, 0.6, "110"), (1079999, 64, 8, 0.6, "110"), (1080000, 64, 8, 0.6, "111"), (8499999, 32, 400, 0.6, "100"),
    (8500000, 32, 400, 0.6, "110"), (2499999, 128, 400, 0.6, "110"), (2500000, 128, 400, 0.6, "111"), (1 << 30, 64, 1 << 20, 0.6, "100"),
    (2000000000, 128, 209715, 0.6, "111"), (2000000000, 128, 209716, 0.6, "100"), (2000000000, 64, 700000, 0.6, "100")])
def test_rows_per_run_where_they_pay(wl, E, d, R, rows, want):
    """RGCN, RGAT, and RGAT forwards that keep nothing."""
    pick_ = lambda layer, heads=1, flags=0: wl.wl_run_rows(C.c_longlong(E), C.c_longlong(E), C.c_longlong(E), C.c_longlong(int(rows * E)),
                                                           C.c_longlong(int(rows * E)), layer, heads, R, d, flags)
    assert "".join(str(pick_(layer)) for layer in range(3)) == want
    assert "".join(str(pick_(layer, flags=32)) for layer in range(3)) == want                # the accumulation of gradients
    assert not any(pick_(layer, flags=f) for layer in range(3) for f in (1, 2, 4, 8, 16)) and not pick_(1, heads=2)


@pytest.mark.parametrize("S,rows,max_chunks", [(1, 64, 4), (3, 700, 512), (5, 40000, 512), (8, 300000, 512), (2, 20000, 1000)])
def test_chunks_of_like_weight(wl, S, rows, max_chunks):
    """Chunks cover the tiles in order, have a tile each and weigh no more than their share and a tile; the slots follow the chunks."""
    rng = np.random.default_rng(S + rows)
    seg_ptr = np.concatenate([[0], np.cumsum(rng.integers(0, 2 * rows // S + 1, S))]).astype(np.int32)
    seg_ptr[-1] = max(seg_ptr[-1], seg_ptr[-2] + 1)
    tiles = int(np.sum((np.diff(seg_ptr) + 63) // 64))
    weight = np.ascontiguousarray(rng.choice([12, 700, 768, 800, 2000, 5000], tiles), np.int32)
    n = wl.wl_weigh_chunks(seg_ptr.ctypes.data_as(C.c_void_p), S, 64, max_chunks, weight.ctypes.data_as(C.c_void_p))
    seg, chunk_tile, chunk_slot, seg_slot_ptr = (_field(wl.wl_tiles_field, i) for i in (0, 3, 4, 5))
    assert n == len(chunk_tile) - 1 and chunk_tile[0] == 0 and chunk_tile[-1] == tiles and np.all(np.diff(chunk_tile) >= 1)
    sums = np.add.reduceat(weight.astype(np.int64), chunk_tile[:-1])
    assert sums.max() <= weight.sum() / n + weight.max()
    want = [len(set(seg[a:b])) for a, b in zip(chunk_tile[:-1], chunk_tile[1:])]
    assert np.array_equal(np.concatenate([[0], np.cumsum(want)])[:-1], chunk_slot) and seg_slot_ptr[-1] == sum(want)
