// Batched census over many resident graphs: one persistent kernel launch over
// a work-item list (graph, execution mode, dyad range), captured once into a
// HIP graph (zero accumulators -> persistent kernels -> 16 counts per graph to
// pinned host memory) and replayed.  Descriptors and items live in device
// buffers read by the kernel, so another set of graphs that fits the captured
// capacities is served by rewriting those buffers and replaying; the capture is
// redone only when a capacity grows or the tuning changes.  Which hub kernels a
// launch has depends on the set; each of the kinds has a capture of its own, made
// when it is first needed, so that sets of different kinds can alternate.
#include <algorithm>
#include <cstring>

#include "tc_api_internal.h"

namespace tc {

// What a launch holds: hub tasks over forward lists, over dyad records, and of a
// graph with 2^20 hub edges or more.
enum : uint32_t { kHasTri = 1, kHasHub = 2, kHasLarge = 4, kKinds = 8 };

struct batch_plan {
    std::vector<tc_graph> graphs;       // graphs the device buffers currently describe
    uint32_t cap_graphs = 0, cap_items = 0;
    graph_desc* d_desc = nullptr;
    work_item* d_items = nullptr;
    uint32_t* d_num = nullptr;
    unsigned long long* d_accs = nullptr;
    unsigned int* d_ctr = nullptr;
    unsigned long long* h_accs = nullptr;   // pinned
    hipGraph_t graph[kKinds] = {};
    hipGraphExec_t exec[kKinds] = {};
    uint32_t grid = 0, hub_blocks = 0;
    uint32_t hub_tile = 0, batch_tile = 0;  // LDS tiles the captured kernels use
    bool valid = false;                     // buffers describe `graphs`
    bool tri = false;                       // ... through their forward lists
    uint32_t kind = 0;                      // ... whose launch is this one

    void release() {
        for (uint32_t k = 0; k < kKinds; ++k) {
            if (exec[k]) (void)hipGraphExecDestroy(exec[k]);
            if (graph[k]) (void)hipGraphDestroy(graph[k]);
        }
        if (d_desc) (void)hipFree(d_desc);
        if (d_items) (void)hipFree(d_items);
        if (d_num) (void)hipFree(d_num);
        if (d_accs) (void)hipFree(d_accs);
        if (d_ctr) (void)hipFree(d_ctr);
        if (h_accs) (void)hipHostFree(h_accs);
        *this = batch_plan{};
    }
};

void batch_release_all(tc_context_s* ctx) {
    if (ctx->batch) {
        if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
        ctx->batch->release();
        delete ctx->batch;
        ctx->batch = nullptr;
    }
}

void batch_forget_graph_locked(tc_context_s* ctx, tc_graph g) {
    batch_plan* p = ctx->batch;
    if (p && std::find(p->graphs.begin(), p->graphs.end(), g) != p->graphs.end()) {
        p->graphs.clear();
        p->valid = false;
    }
}

graph_desc describe(const device_graph& g) {
    graph_desc d{};
    d.dyads = g.dyads;
    d.nbr = g.nbr;
    d.rinfo = g.rinfo;
    d.n = (uint64_t)g.n;
    d.hub_tasks = g.hub_tasks;
    d.edges = g.tri.edges.recs;
    d.fwd = g.tri.fwd;
    d.edge_tasks = g.tri.edges.tasks;
    d.hub_ntasks = g.n_hub_tasks;
    d.hub_groups = g.n_hub_groups;
    d.asym = g.p - g.mutual;
    d.mutual = g.mutual;
    return d;
}

// Work items of one graph: into it.tri runs of hub tasks of the forward lists,
// or into it.hub the hub task groups of the dyad records; into it.rest the
// chunks of rows, then group-mode records (largest), wave-mode chunks and
// lane-mode chunks, over the forward-list edge records when `tri`.
void append_items(const device_graph& g, uint32_t gi, bool tri, bool served, item_lists& it) {
    std::vector<work_item>& out = it.rest;
    const uint64_t* off = g.bucket_off;
    uint32_t flag = 0;
    if (g.p > 0)
        for (uint64_t x = 0; x < (uint64_t)g.n; x += kBatchRowsPerItem)
            out.push_back(work_item{gi, kItemRows, (uint32_t)x,
                                    (uint32_t)std::min<uint64_t>(x + kBatchRowsPerItem, (uint64_t)g.n)});
    if (tri) {
        off = g.tri.edges.off;
        flag = kItemTri;
        const uint32_t nt = g.tri.edges.n_tasks;
        const uint32_t per = batch_tasks_per_item(g.tri.edges.chunk, nt, served);
        for (uint32_t t = 0; t < nt; t += per)
            it.tri.push_back(work_item{gi, kItemHub | kItemTri, t, std::min(t + per, nt)});
    } else {
        for (uint32_t t = 0; t < g.n_hub_groups; ++t) it.hub.push_back(work_item{gi, kItemHub, t, t + 1});
    }
    for (uint64_t d = off[2]; d < off[3]; ++d)
        out.push_back(work_item{gi, kItemGroup | flag, (uint32_t)d, (uint32_t)d + 1});
    for (uint64_t d = off[1]; d < off[2]; d += kBatchWavePerItem)
        out.push_back(work_item{gi, kItemWave | flag, (uint32_t)d,
                                (uint32_t)std::min<uint64_t>(d + kBatchWavePerItem, off[2])});
    for (uint64_t d = off[0]; d < off[1]; d += kBatchLanePerItem)
        out.push_back(work_item{gi, kItemLane | flag, (uint32_t)d,
                                (uint32_t)std::min<uint64_t>(d + kBatchLanePerItem, off[1])});
}

namespace {

// Whether the buffers' capacities are those of a captured launch.
bool holds(const batch_plan& p, uint32_t graphs, uint32_t items, const tc_tuning& t) {
    return p.d_desc && graphs <= p.cap_graphs && items <= p.cap_items && p.grid == t.batch_blocks &&
           p.hub_blocks == t.hub_blocks && p.hub_tile == t.hub_tile && p.batch_tile == t.batch_tile;
}

hipError_t ensure_capacity(batch_plan* p, uint32_t graphs, uint32_t items, const tc_tuning& t, hipStream_t s) {
    if (holds(*p, graphs, items, t)) return hipSuccess;
    (void)hipStreamSynchronize(s);
    p->release();
    p->cap_graphs = std::max<uint32_t>(graphs + graphs / 4, 16);
    p->cap_items = std::max<uint32_t>(items + items / 4, 1024);
    p->grid = t.batch_blocks;
    p->hub_blocks = t.hub_blocks;
    p->hub_tile = t.hub_tile;
    p->batch_tile = t.batch_tile;
    hipError_t e = device_alloc((void**)&p->d_desc, sizeof(graph_desc) * p->cap_graphs);
    if (e == hipSuccess) e = device_alloc((void**)&p->d_items, sizeof(work_item) * p->cap_items);
    if (e == hipSuccess) e = device_alloc((void**)&p->d_num, 3 * sizeof(uint32_t));
    if (e == hipSuccess) e = device_alloc((void**)&p->d_accs, sizeof(unsigned long long) * kBatchAccWords * p->cap_graphs);
    if (e == hipSuccess) e = device_alloc((void**)&p->d_ctr, sizeof(unsigned int) * 3 * kCounterWords);
    if (e == hipSuccess)
        e = hipHostMalloc((void**)&p->h_accs, sizeof(unsigned long long) * kNumClasses * p->cap_graphs);
    if (e != hipSuccess) p->release();
    return e;
}

// Captures the launch of `kind`: zero accumulators and counters, persistent
// kernels, sums to host memory.
hipError_t ensure_captured(batch_plan* p, uint32_t kind, tc_context_s* ctx) {
    if (p->exec[kind]) return hipSuccess;
    // a hub kernel runs when it has items (one of them also when neither has)
    const uint32_t tri_grid = kind != kHasHub ? tri_blocks(p->hub_blocks, ctx->cu_count, (kind & kHasLarge) != 0) : 0;
    const uint32_t hub_grid = kind & kHasHub ? p->hub_blocks : 0;
    // The branch costs 7 us and gains where there are hub tasks (1 graph
    // without: 46 us with it, 39 without; 4 graphs with 1600 tasks: 60 and 78).
    const hipStream_t s = ctx->stream, side = kind != 0 ? ctx->side : nullptr;
    hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return e;
    const batch_buffers bb{p->d_desc, p->d_items, p->d_num, p->d_accs, p->d_ctr, tri_grid, hub_grid, p->grid,
                           p->cap_graphs, p->h_accs, side, ctx->fork};
    hipError_t el = batch_launch(bb, p->hub_tile, p->batch_tile, s);
    e = hipStreamEndCapture(s, &p->graph[kind]);
    if (el != hipSuccess) e = el;
    if (e == hipSuccess) e = hipGraphInstantiate(&p->exec[kind], p->graph[kind], nullptr, nullptr, 0);
    if (e != hipSuccess) p->release();
    return e;
}

}  // namespace

}  // namespace tc

using namespace tc;

extern "C" int tc_census_batch(tc_context ctx, const tc_graph* graphs, int32_t count, uint64_t* counts) {
    if (!ctx || count < 0 || (count > 0 && (!graphs || !counts))) return TC_ERR_ARG;
    if (count == 0) return TC_OK;
    if (hipSetDevice(ctx->device) != hipSuccess) return TC_ERR_DEVICE;
    std::lock_guard<std::mutex> lk(ctx->mu);
    for (int32_t i = 0; i < count; ++i)
        if (!graphs[i] || !ctx->graphs.count(graphs[i])) return TC_ERR_ARG;
    if (!ctx->batch) ctx->batch = new (std::nothrow) batch_plan();
    if (!ctx->batch) return TC_ERR_NOMEM;
    batch_plan* p = ctx->batch;
    std::vector<tc_graph> want(graphs, graphs + count);
    hipError_t e = hipSuccess;
    const bool tri = ctx->tuning.tri != 0;
    if (!(p->valid && p->graphs == want && holds(*p, 0, 0, ctx->tuning) && p->tri == tri)) {
        item_lists lists;
        std::vector<graph_desc> descs(count);
        bool large = false;
        for (int32_t i = 0; i < count; ++i) {
            const device_graph& g = graphs[i]->g;
            if (!has_records(g, tri && g.tri.fptr)) return TC_ERR_NOMEM;
            descs[i] = describe(g);
            append_items(g, (uint32_t)i, tri && g.tri.fptr, false, lists);
            large = large || (tri && g.tri.edges.n_tasks > 0 && g.tri.edges.chunk == kHubChunk / 2);
        }
        const uint32_t kind = (lists.tri.empty() ? 0u : kHasTri) | (lists.hub.empty() ? 0u : kHasHub) |
                              (large ? kHasLarge : 0u);
        uint32_t nums[3];
        std::vector<work_item>& items = lists.join(nums);
        p->valid = false;   // (until the buffers are written)
        e = ensure_capacity(p, (uint32_t)count, (uint32_t)items.size(), ctx->tuning, ctx->stream);
        if (e == hipSuccess) e = ensure_captured(p, kind, ctx);
        if (e != hipSuccess) return status_from_hip(e);
        uint32_t nitems = (uint32_t)items.size();
        e = hipMemcpyAsync(p->d_desc, descs.data(), sizeof(graph_desc) * count, hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess && nitems)
            e = hipMemcpyAsync(p->d_items, items.data(), sizeof(work_item) * nitems, hipMemcpyHostToDevice,
                               ctx->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(p->d_num, nums, sizeof(nums), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);   // host vectors go out of scope
        if (e != hipSuccess) return status_from_hip(e);
        p->graphs = want;
        p->valid = true;
        p->tri = tri;
        p->kind = kind;
    }
    if (ctx->timing) (void)hipEventRecord(ctx->ev[0], ctx->stream);
    e = hipGraphLaunch(p->exec[p->kind], ctx->stream);
    if (ctx->timing) (void)hipEventRecord(ctx->ev[1], ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return status_from_hip(e);
    if (ctx->timing) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]) == hipSuccess) {
            ctx->kstats.batch_ms += ms;
            ctx->kstats.batch_launches += 1;
        }
    }
    for (int32_t i = 0; i < count; ++i)
        finalize_counts(graphs[i]->g.n, p->h_accs + (size_t)kNumClasses * i, counts + (size_t)kNumClasses * i);
    return TC_OK;
}
