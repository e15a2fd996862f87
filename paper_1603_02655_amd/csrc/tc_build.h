// Device graph storage and the build entry points (definitions in tc_build.hip).
#pragma once
#include <deque>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "tc_internal.h"

namespace tc {

constexpr int kCounters = 16;

// Bucketed task records over one adjacency view: the canonical dyads of the
// neighbour CSR (dyad_rec, hub_task), or the edges of the forward lists
// (edge_rec as uint4, tri_task).
template <class Rec, class Task>
struct rec_set {
    Rec* recs = nullptr;
    Task* tasks = nullptr;
    uint32_t n_tasks = 0;
    uint32_t n_groups = 0;                    // dyads: groups of consecutive tasks (hub_task::group)
    uint32_t n_heavy = 0;                     // edges: tasks up to the last vertex with 64 records or more
    uint32_t chunk = kHubChunk;               // records per task (dyads: and per group)
    uint64_t off[kBuckets + 1] = {0, 0, 0, 0, 0};
    uint64_t cost[kBuckets] = {0, 0, 0, 0};   // sum of the two row lengths per bucket
    uint64_t stream = 0;                      // hub: sum of the entries probed
    uint64_t staged = 0;                      // hub: sum over tasks of the anchor row length
};

// Degree order: x precedes y when (|N(x)|, x) < (|N(y)|, y); the rank of a
// vertex is its place from the end (rank 0 comes last).  The forward list N+(x)
// holds the neighbours that follow x, sorted by rank; every joined pair appears
// in exactly one forward list.  Rows are in rank order; the entry layout and
// what the records hold stand in tc_tri.h.  A triangle in degree order
// x, y, z is found exactly once, at the edge (x, y), as a vertex z of N+(y) that
// stands before y in N+(x).  Edges where no vertex can (N+(y) is empty, or y is
// the first of N+(x)) have no record.
struct forward_lists {
    uint32_t* fwd = nullptr;
    uint32_t* fptr = nullptr;     // n + 1
    uint64_t entries = 0;         // = canonical dyads
    rec_set<uint4, tri_task> edges;
};

// hipMalloc on the calling thread's device.  When the device is full, what the
// contexts on it keep for reuse (their pools' blocks and the scratch of builds
// that are not running) goes back to it first.
hipError_t device_alloc(void** out, uint64_t bytes);

struct build_space;

// Device memory of a context's graphs.  Freed blocks are kept, up to `keep`
// bytes in all, and given to later allocations of about their size; beyond
// that the oldest are returned to the driver, which takes 2-40 ms per graph of
// R-MAT 2^20's size and waits for the whole device.  A block is put back only
// once nothing on the device uses it any more (a graph is freed after the
// streams that ran on it were waited for), so it can serve any stream next.
// The pool also knows the scratch its context keeps (add), so that all of it
// can be given back.  Safe from several threads.
class graph_pool {
public:
    ~graph_pool();
    // Before the first use: the device, and the bytes of freed blocks kept.
    void open(int device, uint64_t keep);
    hipError_t alloc(void** out, uint64_t bytes);
    void put(void* p);
    void add(build_space* sp);
    void remove(build_space* sp);
    // Frees kept memory until at most `to` bytes are left (scratch in use by a
    // running build does not count and stays).
    void give_back(uint64_t to);
    int device() const { return device_; }

private:
    struct block {
        void* p;
        uint64_t bytes;
    };
    void shrink(uint64_t to);      // mu_ held
    int device_ = -1;
    uint64_t keep_ = 0;
    std::mutex mu_;
    std::deque<block> free_;       // oldest first
    std::unordered_map<void*, uint64_t> live_;
    std::vector<build_space*> spaces_;
    uint64_t held_ = 0;            // bytes in free_
};

struct device_graph {
    graph_pool* mem = nullptr;
    int32_t n = 0;
    uint64_t U = 0;            // neighbour entries (2 x canonical dyads)
    uint64_t p = 0;            // canonical dyads
    uint64_t mutual = 0;       // mutual canonical dyads
    uint32_t max_degree = 0;
    int64_t* row_ptr = nullptr;
    uint32_t* nbr = nullptr;
    uint32_t* owner = nullptr; // row of each entry (used to rebuild the buckets)
    uint64_t* tpre = nullptr;
    uint4* rinfo = nullptr;    // per row x: row_ptr[x], row_ptr[x+1] and the prefix counts tpre[row_ptr[x+1]]
    dyad_rec* dyads = nullptr;
    hub_task* hub_tasks = nullptr;
    uint32_t n_hub_tasks = 0;
    uint32_t n_hub_groups = 0;
    uint32_t hub_chunk = kHubChunk;  // records per hub task and per group
    uint64_t bucket_off[kBuckets + 1] = {0, 0, 0, 0, 0};
    uint64_t bucket_cost[kBuckets] = {0, 0, 0, 0};   // sum of |N(u)|+|N(v)| per bucket
    uint64_t hub_stream = 0;   // sum over hub dyads of the non-anchor degree (entries probed)
    uint64_t hub_staged = 0;   // sum over hub tasks of the anchor degree (entries staged)
    bucket_params bp{0, 0, 0, 0, kHubTileEntries, 1};
    bool bucketed = false;     // the records are those of bp (not after a rebucket that failed)
    forward_lists tri;         // built when bp.tri
};

struct build_status {
    bool ok = false;
    bool too_large = false;
    hipError_t hip = hipSuccess;
    int64_t bad_ids = 0, self_loops = 0, duplicates = 0, arcs_kept = 0, max_degree = 0;
    uint64_t sum_d2 = 0;
};

// Device scratch and a page of pinned host memory that builds reuse: grown to
// the largest build, kept between builds up to kSpaceKeep bytes (space_trim)
// and freed with its owner.  One build at a time uses a build_space, and holds
// `busy` meanwhile; the pool it is added to frees the scratch of one that is not.
constexpr uint32_t kSpaceHostWords = 64;
constexpr uint32_t kSpaceHostStats = 32;          // words the build's statistics are published to
constexpr uint64_t kSpaceKeep = 1ull << 30;
// Host arcs are copied to the device through pinned chunks, two per copying
// thread: the runtime's own path for pageable memory pins the caller's pages
// on each call (132 MB from arrays that change from call to call: 2-3 GB/s).
constexpr int kStageThreads = 4;
constexpr uint64_t kStageChunk = 1ull << 20;
struct build_space {
    std::mutex busy;
    graph_pool* pool = nullptr;
    void* base = nullptr;
    uint64_t cap = 0;
    uint64_t* host = nullptr;
    char* stage = nullptr;                        // pinned chunks host arcs go through
    hipEvent_t stage_ev[2 * kStageThreads] = {};  // end of each chunk's last copy
};
hipError_t space_reserve(build_space* sp, uint64_t bytes, hipStream_t s);
void space_trim(build_space* sp, uint64_t keep, hipStream_t s);
void space_free(build_space* sp);

// Arcs on the device, or with host_arcs in host memory.
build_status build_graph_device(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, bool host_arcs,
                                const bucket_params& bp, graph_pool* pool, hipStream_t s, build_space* sp,
                                device_graph* g);
// Device bytes that a build of m arcs over n vertices for one census holds at
// its peak, at most: scratch and graph, through either view.
uint64_t build_footprint(uint64_t n, uint64_t m);
hipError_t bucket_dyads(device_graph* g, const bucket_params& bp, hipStream_t s, build_space* sp);
// Whether g has the records its census reads: the forward lists', or the
// dyads', which a rebucket that failed has given up.
inline bool has_records(const device_graph& g, bool tri) { return g.p == 0 || (tri ? g.tri.fptr != nullptr : g.dyads != nullptr); }
void free_device_graph(device_graph* g);
uint64_t device_graph_bytes(const device_graph& g);

}  // namespace tc
