// Graph index: destination-major CSR, compact (source, relation) pairs, (destination,
// relation) runs, the pair-major transpose and the work lists the kernels walk.
// Integer bookkeeping only.  Built once per graph (dataset preprocessing in the thesis,
// Ch.3 "Code Generation": transposition, COO -> CSR; Ch.3 "Compact Tensor Materialization
// and Data Layout": the (source node, edge type) -> row mapping, precomputed, CSR-like).
// The index arrays are produced on the device (graph_build.hip); this file derives the small
// work lists from their offset arrays on the host and holds the graph entry points of the ABI.
#include "rgnn_internal.h"
#include "schedule.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>
#include <algorithm>
#include <future>
#include <initializer_list>
#include <map>
#include <mutex>
#include <new>
#include <system_error>

namespace rgnn {

static thread_local char g_err[512] = "";
void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

rgnn_status_t allow_dynamic_lds(const void* kernel, size_t bytes) {
    static std::mutex mu;
    static std::map<std::pair<const void*, int>, size_t> done;   // (kernel, device) -> limit already set
    int dev = 0;
    RGNN_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    size_t& have = done[{kernel, dev}];
    if (have >= bytes) return RGNN_OK;
    RGNN_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    have = bytes;
    return RGNN_OK;
}

rgnn_status_t resident_blocks_per_cu(const void* kernel, int threads, size_t lds, int* out) {
    static std::mutex mu;
    static std::map<std::pair<const void*, std::pair<int, size_t>>, int> done;   // (kernel, (device, lds)) -> blocks
    int dev = 0;
    RGNN_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto key = std::make_pair(kernel, std::make_pair(dev, lds));
    auto it = done.find(key);
    if (it == done.end()) {
        int n = 0;
        RGNN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds));
        it = done.emplace(key, std::max(n, 1)).first;
    }
    *out = it->second;
    return RGNN_OK;
}

// Host arrays to the device.  Several go into one allocation, and while they are small in one copy: an allocation and a copy
// cost the same whatever their size, and a graph has over a hundred arrays (10k edges: 2.1 ms one by one, so 1.1).
struct Uploader {
    rgnn_graph* g;
    rgnn_status_t st = RGNN_OK;
    struct Array { const std::vector<int32_t>* from; int32_t** to; };
    void up(std::initializer_list<Array> list) { up(list.begin(), list.end()); }
    void up(const Array* begin, const Array* end) {
        constexpr size_t kOneCopy = 4 << 20;
        if (st != RGNN_OK) return;
        auto room = [](const Array& a) { return align_up(std::max<size_t>(a.from->size(), 1) * sizeof(int32_t)); };
        size_t bytes = 0;
        for (const Array* a = begin; a != end; ++a) bytes += room(*a);
        void* d = nullptr;
        hipError_t e = hipMalloc(&d, bytes);
        if (e != hipSuccess) {
            set_error("hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
            st = (e == hipErrorOutOfMemory) ? RGNN_ENOMEM : RGNN_EHIP;
            return;
        }
        g->allocs.push_back(d);
        g->index_bytes += bytes;
        std::vector<char> one(bytes <= kOneCopy ? bytes : 0);
        size_t off = 0;
        for (const Array* a = begin; a != end; off += room(*a), ++a) {
            *a->to = reinterpret_cast<int32_t*>(static_cast<char*>(d) + off);
            const size_t n = a->from->size() * sizeof(int32_t);
            if (n == 0) continue;
            if (!one.empty()) memcpy(one.data() + off, a->from->data(), n);
            else if (!copy(*a->to, a->from->data(), n)) return;
        }
        if (!one.empty()) copy(d, one.data(), bytes);
    }
    bool copy(void* d, const void* h, size_t n) {
        const hipError_t e = hipMemcpy(d, h, n, hipMemcpyHostToDevice);
        if (e == hipSuccess) return true;
        set_error("hipMemcpy H2D failed: %s", hipGetErrorString(e));
        st = RGNN_EHIP;
        return false;
    }
};

// Tile lists over one segmentation: the tiles are planned and uploaded once, every list gets its own chunks.
struct Chunking { TileList* list; int max_chunks; };
static void build_tiles(Uploader& U, const std::vector<int32_t>& seg_ptr, int tile_rows, std::initializer_list<Chunking> lists,
                        const std::vector<int32_t>* weight = nullptr) {
    TilePlan p = plan_tiles(seg_ptr, tile_rows);
    std::vector<TilePlan> chunked(lists.size());
    int32_t *seg = nullptr, *row0 = nullptr, *row1 = nullptr;
    std::vector<Uploader::Array> all{{&p.tile_seg, &seg}, {&p.tile_row0, &row0}, {&p.tile_row1, &row1}};
    size_t i = 0;
    for (const Chunking& c : lists) {
        chunk_tiles(p, c.max_chunks, weight);
        TileList& t = *c.list;
        t.tile_rows = p.tile_rows; t.num_tiles = p.num_tiles; t.num_chunks = p.num_chunks; t.num_slots = p.num_slots;
        t.num_segs = p.num_segs; t.max_seg_slots = p.max_seg_slots; t.max_chunk_slots = p.max_chunk_slots;
        TilePlan& k = chunked[i++];
        k.chunk_tile.swap(p.chunk_tile); k.chunk_slot.swap(p.chunk_slot); k.seg_slot_ptr.swap(p.seg_slot_ptr);
        all.insert(all.end(), {{&k.chunk_tile, &t.chunk_tile}, {&k.chunk_slot, &t.chunk_slot}, {&k.seg_slot_ptr, &t.seg_slot_ptr}});
    }
    U.up(all.data(), all.data() + all.size());
    for (const Chunking& c : lists) { c.list->tile_seg = seg; c.list->tile_row0 = row0; c.list->tile_row1 = row1; }
}

// The item lists of a large graph are planned side by side, on threads of their own, while the caller goes on (16M edges: 430 ms for the
// graph without the lists of its runs, with them 305 so; 20M edges 255, so 130).  A list asked for
// is uploaded by the caller, in the order of the requests.
struct ItemPlans {
    struct Request { ItemList* list; std::future<ItemPlan> plan; };
    std::vector<Request> requests;
    bool threads;
    // ptr has to outlive this object.  number: what to call a segment instead of its id (empty: its id)
    void ask(ItemList& list, const std::vector<int32_t>& ptr, int max_len, int min_len = 0, const std::vector<int32_t>* number = nullptr) {
        auto make = [&ptr, max_len, min_len, number] {
            ItemPlan p = plan_items(ptr, max_len, min_len);
            if (number)
                for (std::vector<int32_t>* v : {&p.row, &p.split_row})
                    for (int32_t& s : *v) s = (*number)[s];
            return p;
        };
        std::future<ItemPlan> f;
        if (threads) {
            try { f = std::async(std::launch::async, make); } catch (const std::system_error&) { threads = false; }   // no thread to be had
        }
        if (!f.valid()) f = std::async(std::launch::deferred, make);
        requests.push_back({&list, std::move(f)});
    }
};
static void upload_items(Uploader& U, ItemList& L, const ItemPlan& p) {
    L.num_items = (int32_t)p.beg.size(); L.num_partials = p.num_partials; L.num_split = p.num_split;
    L.first_single = p.first_single; L.num_single = p.num_single;
    L.first_short = p.first_short; L.num_short = p.num_short; L.num_wide = p.num_wide;
    L.num_long = (int32_t)p.long_item.size();
    U.up({{&p.beg, &L.beg}, {&p.end, &L.end}, {&p.row, &L.row}, {&p.slot, &L.slot}, {&p.split_row, &L.split_row},
          {&p.split_ptr, &L.split_ptr}, {&p.part_item, &L.part_item}, {&p.part_split, &L.part_split}, {&p.long_item, &L.long_item}});
}

static void build_long(Uploader& U, LongList& L, const std::vector<int32_t>& ptr) {
    const std::vector<int32_t> ids = long_segments(ptr);
    L.n = (int)ids.size();
    U.up({{&ids, &L.ids}});
}

constexpr int64_t kThreadedPlans = 1 << 17;   // edges

static rgnn_status_t download(std::vector<int32_t>& h, const int32_t* d, size_t n) {
    h.resize(n);
    if (n) RGNN_HIP(hipMemcpy(h.data(), d, n * sizeof(int32_t), hipMemcpyDeviceToHost));
    return RGNN_OK;
}

rgnn_status_t build_index_device(rgnn_graph* g, int format, const int32_t* a, const int32_t* b, const int32_t* relp,
                                 const int32_t* ntypep, const int32_t* rstp, const int32_t* rdtp, int mem);
rgnn_status_t build_run_rows(rgnn_graph* g, std::vector<int32_t>& src_ptr);
rgnn_status_t block_bounds(const rgnn_graph* g, int B, const int32_t* rel_ptr, const int32_t* node, std::vector<int32_t>& bound);

static rgnn_status_t build_blocks(Uploader& U, ItemList& L, int64_t entries, const int32_t* rel_ptr, const int32_t* node) {
    const rgnn_graph* g = U.g;
    const int B = node_blocks(g->N, g->R, entries);
    std::vector<int32_t> bound;
    RGNN_TRY(block_bounds(g, B, rel_ptr, node, bound));
    const BlockPlan p = plan_blocks(bound, g->R, B, block_cut(entries, g->num_cus));
    L.num_items = (int32_t)p.beg.size(); L.num_partials = p.num_partials; L.num_split = (int32_t)p.split_row.size();
    U.up({{&p.beg, &L.beg}, {&p.end, &L.end}, {&p.row, &L.row}, {&p.slot, &L.slot}, {&p.split_row, &L.split_row}, {&p.split_ptr, &L.split_ptr}});
    return U.st;
}

static rgnn_status_t build(rgnn_graph* g, int format, const int32_t* a, const int32_t* b, const int32_t* relp,
                           const int32_t* ntypep, const int32_t* rstp, const int32_t* rdtp, int mem) {
    RGNN_TRY(build_index_device(g, format, a, b, relp, ntypep, rstp, rdtp, mem));
    // offsets back to the host: statistics and the work lists are cheap linear passes over them
    std::vector<int32_t> in_ptr, out_ptr, pair_ptr, relrun_ptr, srcpair_ptr, ntype_ptr, run_ptr, dst_run_ptr, src_ptr, number;
    RGNN_TRY(download(in_ptr, g->idx[RGNN_IDX_IN_PTR], (size_t)g->N + 1));
    RGNN_TRY(download(out_ptr, g->idx[RGNN_IDX_OUT_PTR], (size_t)g->P + 1));
    RGNN_TRY(download(pair_ptr, g->idx[RGNN_IDX_PAIR_PTR], (size_t)g->R + 1));
    RGNN_TRY(download(relrun_ptr, g->idx[RGNN_IDX_RELRUN_PTR], (size_t)g->R + 1));
    RGNN_TRY(download(srcpair_ptr, g->idx[RGNN_IDX_SRCPAIR_PTR], (size_t)g->N + 1));
    RGNN_TRY(download(ntype_ptr, g->idx[RGNN_IDX_NTYPE_PTR], (size_t)g->T + 1));
    RGNN_TRY(download(run_ptr, g->idx[RGNN_IDX_RUN_PTR], (size_t)g->Q + 1));
    ItemPlans plans{{}, g->E >= kThreadedPlans};         // (after the arrays that its threads read)
    plans.ask(g->dst_items, in_ptr, item_cut(g->E));
    plans.ask(g->pair_items, out_ptr, item_cut(g->E));
    plans.ask(g->relrun_items, relrun_ptr, item_cut(g->E));
    plans.ask(g->pair_items_multi, out_ptr, item_cut(g->E), 2);
    plans.ask(g->relpair_items, pair_ptr, item_cut(g->P));
    for (int64_t u = 0; u < g->N; ++u) g->max_node_pairs = std::max(g->max_node_pairs, srcpair_ptr[u + 1] - srcpair_ptr[u]);
    plans.ask(g->srcpair_items, srcpair_ptr, 1 << 30);
    for (int64_t v = 0; v < g->N; ++v) g->max_in_degree = std::max<int64_t>(g->max_in_degree, in_ptr[v + 1] - in_ptr[v]);
    // (only schedules of small graphs ask for it: a destination's runs are dealt to eight half wavefronts in turn)
    for (int64_t v = 0, q = 0; g->Q <= 131072 && v < g->N && q < g->Q; ++v) {
        RunChain half[8];
        for (int h = 0; q < g->Q && run_ptr[q] < in_ptr[v + 1]; ++q, h = (h + 1) % 8) {
            half[h].runs += 1;
            half[h].edges += run_ptr[q + 1] - run_ptr[q];
        }
        for (const RunChain& c : half)
            if (c.length() > g->longest_chain.length()) g->longest_chain = c;
    }
    if (g->Q > 131072) g->longest_chain = RunChain{(int32_t)g->Q, (int32_t)g->E};
    for (int64_t p = 0; p < g->P; ++p) {
        g->max_pair_out_degree = std::max<int64_t>(g->max_pair_out_degree, out_ptr[p + 1] - out_ptr[p]);
        g->num_single_pairs += (out_ptr[p + 1] - out_ptr[p] == 1);
    }
    for (int64_t q = 0; q < g->Q; ++q) g->num_single_runs += run_ptr[q + 1] - run_ptr[q] == 1;
    g->num_multi_runs = g->Q - g->num_single_runs;
    g->rows_saved = 7 * (g->P - g->Q) - 2 * (g->num_single_pairs - g->num_single_runs);
    g->run_rows = sched_run_rows(g->E, g->P, g->num_single_pairs, g->Q, g->num_single_runs);
    if (g->run_rows) {
        number.resize((size_t)g->Q);
        for (int64_t q = 0, n = 0; q < g->Q; ++q) {
            number[q] = (int32_t)n;
            n += run_ptr[q + 1] - run_ptr[q] > 1;
        }
        plans.ask(g->multi_run_items, run_ptr, item_cut(g->E), 2, &number);
        RGNN_TRY(download(dst_run_ptr, g->idx[RGNN_IDX_DST_RUN_PTR], (size_t)g->N + 1));
        plans.ask(g->dstrun_items, dst_run_ptr, item_cut(g->E));
        RGNN_TRY(build_run_rows(g, src_ptr));
        plans.ask(g->src_items, src_ptr, item_cut(g->E));
    }
    Uploader U{g};
    int dev = 0, cus = 0;
    RGNN_HIP(hipGetDevice(&dev));
    RGNN_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    g->num_cus = cus = std::max(cus, 1);
    const int hgt_pairs = pair_share(g->P, g->N, cus, 2), loop_pairs = pair_share(g->P, g->N, cus, 1);
    build_tiles(U, pair_ptr, kTileRows, {{&g->pair_tiles_hgt, hgt_pairs}, {&g->pair_tiles_loop, loop_pairs}, {&g->pair_tiles, kMaxChunks}, {&g->pair_tiles_wide, kWideChunksPerCU * cus},
                                         {&g->pair_tiles_cu2, 2 * cus}, {&g->pair_tiles_cu1, cus}});
    build_tiles(U, ntype_ptr, kTileRows, {{&g->node_tiles_hgt, std::max(cus - 2 * hgt_pairs, 1)}, {&g->node_tiles, kMaxChunks}, {&g->node_tiles_wide, kWideChunksPerCU * cus},
                                          {&g->node_tiles_cu2, 2 * cus}, {&g->node_tiles_cu1, cus}});
    if (g->rel_src_tied && sched_hgt_pairs_with_query(g->N, g->P, g->max_node_pairs)) {
        std::vector<int32_t> perm, weight;
        RGNN_TRY(download(perm, g->idx[RGNN_IDX_NTYPE_PERM], (size_t)g->N));
        for (int t = 0; t < g->T; ++t)
            for (int32_t a = ntype_ptr[t]; a < ntype_ptr[t + 1]; a += kTileRows) {
                const int32_t e = std::min<int32_t>(a + kTileRows, ntype_ptr[t + 1]);
                int32_t pairs = 0;
                for (int32_t i = a; i < e; ++i) pairs += srcpair_ptr[perm[i] + 1] - srcpair_ptr[perm[i]];
                weight.push_back(kSumRowWeight * (e - a) + kSumPairWeight * pairs);
            }
        build_tiles(U, ntype_ptr, kTileRows, {{&g->node_tiles_sum, 2 * cus}}, &weight);
    }
    build_tiles(U, std::vector<int32_t>{0, (int32_t)g->N}, kTileRows, {{&g->all_tiles, kMaxChunks}, {&g->all_tiles_cu1, cus}, {&g->all_tiles_loop, std::max(cus - loop_pairs, 1)}});
    build_long(U, g->long_runs, run_ptr);
    build_long(U, g->long_pairs, out_ptr);
    if (g->run_rows) {
        const int loop_runs = pair_share(g->Q, g->N, cus, 1);
        build_tiles(U, relrun_ptr, kTileRows, {{&g->run_tiles_loop, loop_runs}, {&g->run_tiles_wide, kWideChunksPerCU * cus}, {&g->run_tiles_cu1, cus}});
        build_tiles(U, std::vector<int32_t>{0, (int32_t)g->N}, kTileRows, {{&g->all_tiles_run_loop, std::max(cus - loop_runs, 1)}});
    }
    if (g->run_rows) {
        RGNN_TRY(build_blocks(U, g->pair_blocks, g->P, g->idx[RGNN_IDX_PAIR_PTR], g->idx[RGNN_IDX_PAIR_SRC]));
        RGNN_TRY(build_blocks(U, g->run_blocks, g->Q, g->idx[RGNN_IDX_RELRUN_PTR], g->relrun_dst));
    }
    for (ItemPlans::Request& r : plans.requests) upload_items(U, *r.list, r.plan.get());
    return U.st;
}

}  // namespace rgnn

using namespace rgnn;

extern "C" const char* rgnn_last_error(void) { return g_err; }

extern "C" rgnn_status_t rgnn_graph_create(rgnn_graph_t** gout, int64_t num_nodes, int32_t num_ntypes, int32_t num_rels,
                                           int64_t num_edges, int32_t format, const int32_t* a, const int32_t* b,
                                           const int32_t* rel, const int32_t* ntype, const int32_t* rel_src_ntype,
                                           const int32_t* rel_dst_ntype, int32_t mem) {
    if (!gout) RGNN_FAIL(RGNN_EINVAL, "g is NULL");
    *gout = nullptr;
    if (num_nodes < 0 || num_edges < 0 || num_rels < 1 || num_ntypes < 1)
        RGNN_FAIL(RGNN_EINVAL, "need num_nodes >= 0, num_edges >= 0, num_rels >= 1, num_ntypes >= 1");
    if (format != RGNN_COO && format != RGNN_CSR_DST) RGNN_FAIL(RGNN_EINVAL, "unknown format %d", format);
    if (mem != RGNN_MEM_HOST && mem != RGNN_MEM_DEVICE) RGNN_FAIL(RGNN_EINVAL, "unknown mem %d", mem);
    if (num_edges > 0 && (!a || !rel)) RGNN_FAIL(RGNN_EINVAL, "edge arrays are NULL");
    if ((format == RGNN_CSR_DST || num_edges > 0) && !b) RGNN_FAIL(RGNN_EINVAL, "dst / rowptr array is NULL");
    if (num_ntypes > 1 && !ntype) RGNN_FAIL(RGNN_EINVAL, "ntype is NULL but num_ntypes > 1");
    if ((rel_src_ntype == nullptr) != (rel_dst_ntype == nullptr))
        RGNN_FAIL(RGNN_EINVAL, "rel_src_ntype and rel_dst_ntype must be given together");
    if (num_edges >= (int64_t)1 << 31 || num_nodes >= (int64_t)1 << 31)
        RGNN_FAIL(RGNN_EUNSUPPORTED, "int32 indices: need fewer than 2^31 nodes and edges");
    {
        const long double bound = (long double)std::max<int64_t>(num_nodes, 1) * std::max<int64_t>(num_nodes, 1) * num_rels;
        if (bound >= 9.2e18L) RGNN_FAIL(RGNN_EUNSUPPORTED, "N*N*R must be below 2^63 for the 64-bit sort keys");
    }
    {   // set-up work for the entry point that allocates nothing: its scratch buffer's address on this device
        void* scratch_ptr = nullptr;
        RGNN_TRY(static_scratch(&scratch_ptr));
    }
    rgnn_graph* g = new (std::nothrow) rgnn_graph();
    if (!g) RGNN_FAIL(RGNN_ENOMEM, "out of host memory");
    g->N = num_nodes; g->E = num_edges; g->R = num_rels; g->T = num_ntypes;
    rgnn_status_t st;
    try {
        st = build(g, format, a, b, rel, ntype, ntype ? rel_src_ntype : nullptr, ntype ? rel_dst_ntype : nullptr, mem);
    } catch (const std::bad_alloc&) {
        set_error("out of host memory while building the graph index");
        st = RGNN_ENOMEM;
    }
    if (st == RGNN_OK && hipDeviceSynchronize() != hipSuccess) { set_error("hipDeviceSynchronize failed"); st = RGNN_EHIP; }
    if (st != RGNN_OK) { rgnn_graph_destroy(g); return st; }
    *gout = g;
    return RGNN_OK;
}

extern "C" rgnn_status_t rgnn_graph_destroy(rgnn_graph_t* g) {
    if (!g) return RGNN_OK;
    for (void* p : g->allocs) (void)hipFree(p);
    delete g;
    return RGNN_OK;
}

extern "C" rgnn_status_t rgnn_graph_info(const rgnn_graph_t* g, rgnn_graph_info_t* out) {
    if (!g || !out) RGNN_FAIL(RGNN_EINVAL, "NULL argument");
    out->num_nodes = g->N; out->num_edges = g->E; out->num_pairs = g->P; out->num_runs = g->Q;
    out->max_in_degree = g->max_in_degree; out->max_pair_out_degree = g->max_pair_out_degree;
    out->index_bytes = (int64_t)g->index_bytes; out->num_rels = g->R; out->num_ntypes = g->T;
    out->num_single_pairs = g->num_single_pairs;
    return RGNN_OK;
}

extern "C" rgnn_status_t rgnn_graph_export(const rgnn_graph_t* g, int32_t which, void* host_dst, size_t bytes) {
    if (!g || (!host_dst && bytes)) RGNN_FAIL(RGNN_EINVAL, "NULL argument");
    if (which < 0 || which >= RGNN_IDX_COUNT) RGNN_FAIL(RGNN_EINVAL, "unknown index array %d", which);
    if (bytes != (size_t)g->idx_len[which] * sizeof(int32_t))
        RGNN_FAIL(RGNN_EINVAL, "index array %d holds %lld int32, caller passed %zu bytes", which, (long long)g->idx_len[which], bytes);
    RGNN_HIP(hipDeviceSynchronize());
    if (bytes) RGNN_HIP(hipMemcpy(host_dst, g->idx[which], bytes, hipMemcpyDeviceToHost));
    return RGNN_OK;
}
