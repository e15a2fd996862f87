// Census kernel launch interface (definitions in tc_census.hip).
#pragma once
#include <algorithm>

#include "tc_build.h"

namespace tc {

struct census_config {
    uint32_t lane_blocks = 2048;    // grid cap of the lane-per-dyad kernel
    uint32_t wave_blocks = 8192;    // resident one-wave workgroups of the wave kernel
    uint32_t group_blocks = 1024;   // resident workgroups of the group kernel
    uint32_t hub_blocks = 1024;     // resident workgroups of the hub kernel
    uint32_t tri_blocks = 1024;     // the same over edge records, when every workgroup has many tasks
    uint32_t side_blocks = 256;     // workgroups of the totals pass when it runs on the side stream
    uint32_t hub_tile = 1024;       // anchor entries per LDS tile, hub mode (512, 1024, 2048)
    uint32_t wave_tile = 1024;      // row entries staged per round, wave mode (512, 1024, 2048)
    uint32_t group_tile = 4096;     // row entries staged per round, group mode (2048, 4096, 8192)
    uint32_t group_size = 256;      // threads per workgroup, group mode (256, 512)
};

// Workgroups of the hub kernels over edge records with many tasks each: four
// per CU.  Five fit; four are faster, since they leave registers for the lane
// bucket, the terms and a batch's other items that run beside them, and none
// waits for another to end (R-MAT 2^20: 8 per CU 0.894 ms, 5 0.876, 4 0.875, 3
// 0.892; a batch of 512 R-MAT graphs: 0.787, 0.787, 0.757, 0.849).
// A batch with a graph whose tasks have 256 records (2^20 hub edges or more) has
// five: its other items are few beside them (two graphs of R-MAT 2^20 1.61 ms, with
// four 1.74; 512 graphs of 50 to 20000 rows, none so large, 0.71, 0.68).
inline uint32_t tri_blocks(uint32_t hub_blocks, int cu_count, bool large_batch = false) {
    return std::min(hub_blocks, (large_batch ? 5u : 4u) * (uint32_t)(cu_count > 0 ? cu_count : 256));
}

// Whether the kernels are built for these LDS tiles and group size.
bool tile_supported(uint32_t hub_tile, uint32_t wave_tile, uint32_t group_tile, uint32_t group_size,
                    uint32_t batch_tile);

// Per-bucket record slices [begin, end) into g.dyads or the edge records
// (merge buckets); the hub bucket runs its task groups [hub_g0, hub_g1),
// restricted to dyads with u in [u_lo, u_hi).  The terms that need no
// intersection are those of the dyads with u in [u_lo, u_hi), whose rows hold
// the entries [ent_begin, ent_end) (range, dyad records only), or cover the rows
// [row_begin, row_end) and the bases of `asym` and `mutual` pairs.
struct census_slices {
    uint64_t begin[kBuckets];
    uint64_t end[kBuckets];
    uint32_t u_lo = 0, u_hi = 0xffffffffu;
    uint32_t hub_g0 = 0, hub_g1 = 0xffffffffu;
    bool range = false;
    uint64_t ent_begin = 0, ent_end = 0;
    uint32_t row_begin = 0, row_end = 0;
    uint64_t asym = 0, mutual = 0;
};

// ---- batched launch over many graphs ----
struct graph_desc {
    const dyad_rec* dyads;       // dyad records
    const uint32_t* nbr;
    uint64_t n;
    const hub_task* hub_tasks;
    const uint4* edges;          // forward-list edge records (null without forward lists)
    const uint32_t* fwd;
    const tri_task* edge_tasks;
    const uint4* rinfo;          // per row: bounds and prefix counts at its end
    uint32_t hub_ntasks, hub_groups;   // tasks and task groups over the dyad records
    uint64_t asym, mutual;             // joined pairs, one way and both ways
};
// Item kinds: the mode (lane / wave / group / hub), with kItemTri when the item
// indexes the forward-list edge records; kItemRows covers the rows [begin, end)
// of the terms that need no intersection.
enum : uint32_t { kItemLane = 0, kItemWave = 1, kItemGroup = 2, kItemHub = 3, kItemTri = 4, kItemRows = 8 };
struct work_item {
    uint32_t graph, kind, begin, end;   // records [begin, end) of graph `graph`'s record array;
                                        // hub items: task groups [begin, end) of the graph, or with
                                        // kItemTri its hub tasks [begin, end)
};
// Hub tasks of the forward lists per item, of a graph whose tasks have up to
// `chunk` records.  Tasks of 256 are those of a graph with 2^20 hub edges or
// more, which has to fill the chip by itself: a task per wavefront (one random
// graph of 5000 vertices and 500 neighbours each: 32 tasks 414 us, 8 156, 4 130;
// a complete one of 1500: 1736, 512, 355; R-MAT 2^20 1066, 881, 885).  Of shorter
// tasks and of fewer, 32 (256 R-MAT graphs of up to 20000 rows: 355 us, 8 tasks of 64 389).
// In the serving loop also of many tasks: its one thread makes and copies the
// items of every round, other rounds fill the chip, and 8000 requests/s waited 14
// to 21 ms (median) with 4 tasks of every large graph in an item, 4.7 so.
inline uint32_t batch_tasks_per_item(uint32_t chunk, uint32_t tasks, bool served) {
    return chunk == kHubChunk / 2 && !(served && tasks > 16384) ? 4 : 32;
}
constexpr uint32_t kBatchRowsPerItem = 4096;   // rows per rows item
// (1024, four per thread: 0.96 ms instead of 0.92 for 512 graphs of up to 20 k
// vertices, and 3.9 instead of 3.5 ms for 48 served ones of up to 10^6)
constexpr uint32_t kBatchLanePerItem = 256;   // one record per thread of a 256-thread workgroup
constexpr uint32_t kBatchWavePerItem = 16;    // four wavefronts, four dyads each

// Zeroes the accumulators and the work counters, then runs the persistent
// kernels: over the items items[0..nums[0]) (hub tasks of forward lists) with
// tri_grid workgroups, over those up to nums[1] (dyad hub task groups, LDS tile
// of hub_tile anchor entries) with hub_grid, and over those up to nums[2]
// (wave-mode tile batch_tile, group-mode tile 4 x batch_tile) with grid, and
// writes every graph's sums to `out`.  A hub kernel with a grid of 0 is left out.  hipErrorInvalidValue for a tile the
// kernels are not built for.
constexpr uint32_t kBatchCopies = 8;          // of a graph's accumulators
constexpr uint64_t kBatchAccWords = (uint64_t)kNumClasses * kBatchCopies;
struct batch_buffers {
    const graph_desc* descs;
    const work_item* items;
    const uint32_t* nums;           // 3 words of device memory
    unsigned long long* accs;       // kBatchAccWords per graph
    unsigned int* counters;         // 3 x kCounterWords
    uint32_t tri_grid, hub_grid, grid;
    uint32_t graphs;
    unsigned long long* out;        // pinned: 16 sums per graph
    hipStream_t side = nullptr;     // a second stream and two events: the kernel of the other items runs there
    hipEvent_t* fork = nullptr;
};
hipError_t batch_launch(const batch_buffers& b, uint32_t hub_tile, uint32_t batch_tile, hipStream_t s);

// Copies the 16-class table into the constant table the batch kernel reads.
hipError_t census_upload_table();
// One census on stream s: the bucket kernels over the given slices with
// `table` (64 bytes of device memory: the bin of every code, kNumClasses for
// codes that are not counted), the terms that need no intersection, and a last
// kernel that writes the sums to `out` (pinned host memory) and leaves acc
// (kAccCopies x 16 u64, x 64 for kLabelled) and counters (kBuckets x kCounterWords)
// zero, as they have to be before.  With `tri` the slices index the
// forward-list edge records (g.tri.edges).  When `side` is given
// (with two events in `fork`) and the hub bucket streams more entries than the
// graph has, these terms run on `side`, followed there by the lane bucket,
// beside the other bucket kernels; s waits for it at the end.  ev, when not
// null, holds 2*kBuckets + 2 events: around each bucket's launch, then around
// the terms.
// kClasses: 16 sums by a class table.  kLabelledPass: 16 sums by one of the
// labelled census's pass tables (dyad records).  kLabelled: all 64 code sums
// (forward lists; the table maps every code to itself).
enum census_kind { kClasses, kLabelledPass, kLabelled };
constexpr int kAccWords = 64 * kAccCopies;
hipError_t census_launch(const device_graph& g, const census_slices& sl, bool tri, const uint8_t* table,
                         census_kind kind, unsigned long long* acc, unsigned int* counters, unsigned long long* out,
                         const census_config& cfg, hipStream_t s, hipEvent_t* ev, hipStream_t side = nullptr,
                         hipEvent_t* fork = nullptr);
// Zeroes `words` accumulators and the counters (before the first census that uses them, or after a
// failed launch).
hipError_t census_clear(unsigned long long* acc, int words, unsigned int* counters, hipStream_t s);

}  // namespace tc
