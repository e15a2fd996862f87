// Graph build on the device: canonicalise arcs, sort, merge direction flags,
// CSR of undirected neighbours with two direction bits per entry, prefix
// counts of the direction bits, and the bucketed canonical-dyad task records.
//
// Follows the thesis's input model (section "Triad Census Algorithm"): a strict
// digraph G = [V, E] with E a set of ordered pairs and N(u) the undirected
// neighbourhood; and its adjacency-array (CRS) representation (section
// "Graph Data Structures").  Canonical dyads are the connected pairs u < v; the
// bucket key |N(u)| + |N(v)| - 2 is the workload estimate of the
// "Canonical Dyad (uniform distr.)" task-queue generation.
#include "tc_build.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <thread>

namespace tc {

namespace {

constexpr int kT = 256;            // threads per block for build kernels
constexpr int kI = 8;              // items per thread
constexpr int kTile = kT * kI;     // 2048 items per block

inline uint32_t blocks_for(uint64_t n) { return (uint32_t)((n + kTile - 1) / kTile); }

__device__ inline uint64_t lanemask_lt() {
    return (1ull << __lane_id()) - 1ull;
}

// ---- block-wide exclusive scan of one uint64 per thread (256 threads) ----
__device__ uint64_t block_exclusive_scan(uint64_t x, uint64_t* sh_warp /*[4]*/, uint64_t* block_total) {
    const int lane = __lane_id();
    const int wid = threadIdx.x >> 6;
    uint64_t incl = x;
    for (int off = 1; off < 64; off <<= 1) {
        uint64_t y = __shfl_up((unsigned long long)incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) sh_warp[wid] = incl;
    __syncthreads();
    uint64_t base = 0, tot = 0;
    for (int w = 0; w < kT / 64; ++w) {
        if (w < wid) base += sh_warp[w];
        tot += sh_warp[w];
    }
    __syncthreads();
    if (block_total) *block_total = tot;
    return base + incl - x;
}

template <class T>
__global__ __launch_bounds__(kT) void k_scan_reduce(const T* __restrict__ in, uint64_t n, uint64_t* __restrict__ sums) {
    __shared__ uint64_t sh[kT / 64];
    uint64_t base = (uint64_t)blockIdx.x * kTile, s = 0;
    for (int k = 0; k < kI; ++k) {
        uint64_t i = base + (uint64_t)k * kT + threadIdx.x;
        if (i < n) s += in[i];
    }
    uint64_t tot;
    block_exclusive_scan(s, sh, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// single workgroup: exclusive scan of in[0..n) to out (they may be one array),
// total to *total; the tile sums of a larger scan, or a whole small one
constexpr int kSpineT = 1024;
constexpr int kSpineI = 4;
template <class T>
__global__ __launch_bounds__(kSpineT) void k_scan_spine(const T* in, T* out, uint64_t n, T* __restrict__ total) {
    __shared__ uint64_t sh[kSpineT / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    uint64_t carry = 0;
    for (uint64_t base = 0; base < n; base += kSpineT * kSpineI) {
        uint64_t loc[kSpineI], s = 0;
        for (int k = 0; k < kSpineI; ++k) {
            const uint64_t i = base + tid * kSpineI + k;
            loc[k] = s;
            s += i < n ? (uint64_t)in[i] : 0;
        }
        uint64_t incl = s;
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t y = __shfl_up((unsigned long long)incl, off, 64);
            if ((int)lane >= off) incl += y;
        }
        if (lane == 63) sh[wid] = incl;
        __syncthreads();
        uint64_t ex = carry + incl - s;
        for (uint32_t w = 0; w < kSpineT / 64; ++w) {
            if (w < wid) ex += sh[w];
            carry += sh[w];
        }
        for (int k = 0; k < kSpineI; ++k) {
            const uint64_t i = base + tid * kSpineI + k;
            if (i < n) out[i] = (T)(ex + loc[k]);
        }
        __syncthreads();
    }
    if (tid == 0 && total) *total = (T)carry;
}

template <class T>
__global__ __launch_bounds__(kT) void k_scan_apply(const T* in, T* out, uint64_t n,
                                                    const uint64_t* __restrict__ sums) {
    __shared__ uint64_t sh[kT / 64];
    __shared__ uint64_t vals[kTile];
    uint64_t base = (uint64_t)blockIdx.x * kTile;
    for (int k = 0; k < kI; ++k) {
        uint64_t i = base + (uint64_t)k * kT + threadIdx.x;
        vals[k * kT + threadIdx.x] = i < n ? in[i] : 0;
    }
    __syncthreads();
    uint64_t loc[kI], s = 0;
    for (int k = 0; k < kI; ++k) { loc[k] = s; s += vals[threadIdx.x * kI + k]; }
    uint64_t ex = block_exclusive_scan(s, sh, nullptr);
    uint64_t off = sums[blockIdx.x];
    for (int k = 0; k < kI; ++k) vals[threadIdx.x * kI + k] = off + ex + loc[k];
    __syncthreads();
    for (int k = 0; k < kI; ++k) {
        uint64_t i = base + (uint64_t)k * kT + threadIdx.x;
        if (i < n) out[i] = (T)vals[k * kT + threadIdx.x];
    }
}

// ---- canonicalise: two keys per arc (one per orientation) -----------------
// key = owner << (bits + 2) | w << 2 | flag, flag 1 = owner->w, 2 = w->owner.
// Loops and bad ids become the sentinel (all sort bits set; as a key it would
// be a loop of the last id, which never occurs), which sorts last.
// The keys with flag 1 stand before all those with flag 2.  The sort looks at
// the bits above the flags and is stable, so among the equal pairs of the
// sorted keys the flags rise: what a pair's run holds shows at its ends.
//
// Bound by memory (8 bytes in, 16 out per arc).  The two counters get one
// atomic per workgroup of a small fixed grid: atomics on one address take about
// 12 ns each here whoever issues them, so one per wavefront with a loop cost
// 0.20 ms on 16.6 M arcs with one loop in 1000; now 0.08 ms.
constexpr uint32_t kStatBlocks = 1024;   // workgroups of the kernels that end with atomics on shared counters

__device__ inline unsigned long long block_sum(unsigned long long x, unsigned long long* sh /*[kT / 64]*/) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    if (__lane_id() == 0) sh[threadIdx.x >> 6] = x;
    __syncthreads();
    unsigned long long s = 0;
    for (int w = 0; w < kT / 64; ++w) s += sh[w];
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(kT) void k_canon(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                               uint64_t m, int32_t n, uint32_t bits, uint64_t* __restrict__ keys,
                                               unsigned long long* __restrict__ counters) {
    __shared__ unsigned long long sh[kT / 64];
    const uint64_t sentinel = (1ull << (2 * bits + 2)) - 1ull;
    unsigned long long loops = 0, bads = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * kT + threadIdx.x; i < m; i += (uint64_t)gridDim.x * kT) {
        const int32_t s = src[i], d = dst[i];
        const bool bad = s < 0 || s >= n || d < 0 || d >= n;
        const bool loop = !bad && s == d;
        uint64_t k0 = sentinel, k1 = sentinel;
        if (!bad && !loop) {
            k0 = ((uint64_t)s << (bits + 2)) | ((uint64_t)d << 2) | 1ull;
            k1 = ((uint64_t)d << (bits + 2)) | ((uint64_t)s << 2) | 2ull;
        }
        keys[i] = k0;
        keys[m + i] = k1;
        loops += loop ? 1u : 0u;
        bads += bad ? 1u : 0u;
    }
    loops = block_sum(loops, sh);
    bads = block_sum(bads, sh);
    if (threadIdx.x == 0) {
        if (bads) atomicAdd(&counters[0], bads);
        if (loops) atomicAdd(&counters[1], loops);
    }
}

// ---- LSD radix sort, digits of at most 9 bits starting at bit 2 -------------
// Per pass: a digit histogram per tile, one scan of the (digit, tile) counts,
// and a stable scatter.  A tile's keys are first put in digit order in LDS, so
// that the writes of a tile are runs of the keys of one digit instead of
// single keys.  Bound by memory (8 bytes read for the counts, 16 moved by the
// scatter); tiles of 4096 keys make runs of 16 keys (128 bytes) with 8-bit
// digits and 42 KiB of LDS, three workgroups per CU.
constexpr int kDigitBits = 9;
constexpr int kDigits = 1 << kDigitBits;
constexpr int kSortI = 16;                  // keys per thread
constexpr int kSortISmall = 4;              // ... below kSortSmall keys: four times the workgroups, a quarter
constexpr uint64_t kSortSmall = 1ull << 21; // of the serial rounds (20 k keys: 16 us a pass less 5)
constexpr int kSortWaves = kT / 64;

// O: 32-bit key positions, or 64-bit for 2^32 keys or more.  I: keys per thread.
template <class O, int I>
__global__ __launch_bounds__(kT) void k_radix_hist(const uint64_t* __restrict__ keys, uint64_t count, uint32_t shift,
                                                    uint32_t nbins, O* __restrict__ hist, uint32_t nblocks) {
    __shared__ uint32_t h[kDigits];
    for (uint32_t d = threadIdx.x; d < nbins; d += kT) h[d] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * (kT * I);
#pragma unroll
    for (int k = 0; k < I; ++k) {
        const uint64_t i = base + (uint64_t)k * kT + threadIdx.x;
        if (i < count) atomicAdd(&h[(keys[i] >> shift) & (nbins - 1)], 1u);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < nbins; d += kT) hist[(uint64_t)d * nblocks + blockIdx.x] = h[d];
}

// Wavefront w of a workgroup holds the tile's keys [w, w + 1) * 64 * kSortI, 64
// consecutive ones per round; the rank of a key among the equal digits before
// it in its wavefront comes from ballots, those of earlier wavefronts from the
// wavefronts' digit counts.
template <class O, int I>
__global__ __launch_bounds__(kT) void k_radix_scatter(const uint64_t* __restrict__ in, uint64_t* __restrict__ out,
                                                       uint64_t count, uint32_t shift, uint32_t dbits,
                                                       const O* __restrict__ offsets, uint32_t nblocks) {
    constexpr int kKeys = kT * I;
    __shared__ uint64_t stage[kKeys];
    __shared__ uint16_t wcnt[kSortWaves][kDigits];
    __shared__ O to_out[kDigits];            // global offset of the digit's run minus its start in the tile
    __shared__ uint64_t wsum[kT / 64];
    const uint32_t nbins = 1u << dbits, lane = __lane_id(), wid = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kKeys;
    const uint32_t here = (uint32_t)(count - base < (uint64_t)kKeys ? count - base : (uint64_t)kKeys);
    for (uint32_t d = threadIdx.x; d < nbins; d += kT)
        for (int w = 0; w < kSortWaves; ++w) wcnt[w][d] = 0;
    __syncthreads();
    uint64_t key[I];
    uint32_t pos[I];    // rank inside the wavefront's equal digits
#pragma unroll
    for (int r = 0; r < I; ++r) {
        const uint32_t i = wid * 64 * I + (uint32_t)r * 64 + lane;
        key[r] = i < here ? in[base + i] : 0;
    }
#pragma unroll
    for (int r = 0; r < I; ++r) {
        const uint32_t i = wid * 64 * I + (uint32_t)r * 64 + lane;
        const bool valid = i < here;
        const uint32_t dg = (uint32_t)(key[r] >> shift) & (nbins - 1);
        uint64_t peers = __ballot(valid);
        for (uint32_t b = 0; b < dbits; ++b) {
            const uint64_t bb = __ballot((dg >> b) & 1u);
            peers &= ((dg >> b) & 1u) ? bb : ~bb;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t prev = valid ? wcnt[wid][dg] : 0u;
        pos[r] = prev + before;
        // (the fences keep the read above and the write below in order for the lanes of the wavefront)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) wcnt[wid][dg] = (uint16_t)(prev + (uint32_t)__popcll(peers));
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread t takes the digits 2t and 2t + 1: their starts in the tile, and
    // per wavefront the number of equal digits in earlier wavefronts
    uint32_t tot[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t d = 2 * threadIdx.x + q;
        if (d < nbins)
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = wcnt[w][d];
                wcnt[w][d] = (uint16_t)tot[q];
                tot[q] += c;
            }
    }
    const uint32_t start = (uint32_t)block_exclusive_scan(tot[0] + tot[1], wsum, nullptr);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t d = 2 * threadIdx.x + q, s0 = start + (q ? tot[0] : 0u);
        if (d < nbins) {
            to_out[d] = offsets[(uint64_t)d * nblocks + blockIdx.x] - s0;
            for (int w = 0; w < kSortWaves; ++w) wcnt[w][d] = (uint16_t)(wcnt[w][d] + s0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < I; ++r) {
        const uint32_t i = wid * 64 * I + (uint32_t)r * 64 + lane;
        const uint32_t dg = (uint32_t)(key[r] >> shift) & (nbins - 1);
        if (i < here) stage[wcnt[wid][dg] + pos[r]] = key[r];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < I; ++k) {
        const uint32_t i = (uint32_t)k * kT + threadIdx.x;
        if (i < here) {
            const uint64_t x = stage[i];
            out[(O)(to_out[(uint32_t)(x >> shift) & (nbins - 1)] + i)] = x;
        }
    }
}

// ---- unique (owner, w) pairs with OR-ed direction flags --------------------
// The sorted keys of one (owner, w) pair are adjacent; the first of them is
// its head and becomes a neighbour entry.  A tile is kT * kI keys, wavefront w
// holding 64 * kI consecutive ones, 64 per round, so that every running count
// (entries, direction bits) is a ballot and a lane count.
//
// Both passes are bound by reading the keys.  They take the place of a head
// flag per key, a scan of the flags, an atomic per entry on its row's degree
// and a second scan for the direction bits.
//
// The flags of a run rise, so a run that starts with 2 holds 2 only, and one
// that starts with 1 holds 2 too if its last key does: found by doubling steps
// and halving them again, 40 reads for 10^6 repeats (a build of 1.8 M arcs with
// such a pair took 248 ms when a lane walked the run in each pass, 1.2 now).
struct run_of {
    bool head;
    uint32_t f;
};
__device__ inline run_of run_at(const uint64_t* __restrict__ keys, uint64_t i, uint64_t count, uint64_t sentinel) {
    const uint64_t k = keys[i], before = keys[i ? i - 1 : 0], after = keys[i + 1 < count ? i + 1 : i];
    if ((i != 0 && (before >> 2) == (k >> 2)) || (k >> 2) == (sentinel >> 2)) return run_of{false, 0u};
    const bool more = i + 1 < count && (after >> 2) == (k >> 2);
    uint32_t f = (uint32_t)(k & 3u) | (more ? (uint32_t)(after & 3u) : 0u);
    if (more && f == 1u) {
        uint64_t last = i + 1, step = 1;   // keys[last] is in the run
        while (last + step < count && (keys[last + step] >> 2) == (k >> 2)) {
            last += step;
            step *= 2;
        }
        for (step /= 2; step != 0; step /= 2)
            if (last + step < count && (keys[last + step] >> 2) == (k >> 2)) last += step;
        f |= (uint32_t)(keys[last] & 3u);
    }
    return run_of{true, f};
}

// Per tile: entries, and the two direction-bit counts (as in tpre).
__global__ __launch_bounds__(kT) void k_runs_count(const uint64_t* __restrict__ keys, uint64_t count, uint32_t bits,
                                                   uint64_t* __restrict__ ents, uint64_t* __restrict__ types) {
    __shared__ unsigned long long sh[kT / 64];
    const uint64_t sentinel = (1ull << (2 * bits + 2)) - 1ull;
    unsigned long long e = 0, t = 0;
    for (int r = 0; r < kI; ++r) {
        const uint64_t i = (uint64_t)blockIdx.x * kTile + (threadIdx.x >> 6) * 64 * kI + r * 64 + __lane_id();
        if (i < count) {
            const run_of q = run_at(keys, i, count, sentinel);
            if (q.head) {
                e += 1;
                t += (unsigned long long)(q.f & 1u) | ((unsigned long long)(q.f >> 1) << 32);
            }
        }
    }
    e = block_sum(e, sh);
    t = block_sum(t, sh);
    if (threadIdx.x == 0) {
        ents[blockIdx.x] = e;
        types[blockIdx.x] = t;
    }
}

// Scans both per-tile counts in place on one workgroup; the totals go to the
// host (pinned memory), with the counters of k_canon.
__global__ __launch_bounds__(1024) void k_runs_spine(uint64_t* __restrict__ ents, uint64_t* __restrict__ types,
                                                     uint64_t nb, const unsigned long long* __restrict__ counters,
                                                     uint64_t* __restrict__ host) {
    __shared__ uint64_t sa[16], sb[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    uint64_t ca = 0, cb = 0;
    for (uint64_t base = 0; base < nb; base += 4096) {
        uint64_t a[4], b[4], xa = 0, xb = 0;
        for (uint32_t k = 0; k < 4; ++k) {
            const uint64_t i = base + 4 * tid + k;
            const uint64_t va = i < nb ? ents[i] : 0, vb = i < nb ? types[i] : 0;
            a[k] = xa;
            b[k] = xb;
            xa += va;
            xb += vb;
        }
        uint64_t ia = xa, ib = xb;
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t ya = __shfl_up((unsigned long long)ia, off, 64), yb = __shfl_up((unsigned long long)ib, off, 64);
            if ((int)lane >= off) { ia += ya; ib += yb; }
        }
        if (lane == 63) { sa[wid] = ia; sb[wid] = ib; }
        __syncthreads();
        uint64_t pa = ca + ia - xa, pb = cb + ib - xb;
        for (uint32_t w = 0; w < 16; ++w) {
            if (w < wid) { pa += sa[w]; pb += sb[w]; }
            ca += sa[w];
            cb += sb[w];
        }
        for (uint32_t k = 0; k < 4; ++k) {
            const uint64_t i = base + 4 * tid + k;
            if (i < nb) {
                ents[i] = pa + a[k];
                types[i] = pb + b[k];
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        host[0] = ca;
        host[1] = cb;
        host[2] = counters[0];
        host[3] = counters[1];
    }
}

// ptr[x] = e for the rows x in (before, upto]: the lanes with a few rows each
// write their own, and a longer gap (vertices without entries) is written by
// the whole wavefront.  Called by all lanes; `on` lanes have a range.
template <class P>
__device__ inline void fill_rows(bool on, int64_t before, int64_t upto, uint64_t e, P* __restrict__ ptr) {
    const bool wide = on && upto - before > 8;
    if (on && !wide)
        for (int64_t x = before + 1; x <= upto; ++x) ptr[x] = (P)e;
    uint64_t todo = __ballot(wide);
    while (todo) {
        const int l = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        const int64_t b = __shfl((long long)before, l, 64), u = __shfl((long long)upto, l, 64);
        const P v = (P)__shfl((unsigned long long)e, l, 64);
        for (int64_t x = b + 1 + __lane_id(); x <= u; x += 64) ptr[x] = v;
    }
}

// Writes the entries, their owners, the exclusive direction-bit prefix and the
// row starts.
__global__ __launch_bounds__(kT) void k_runs_emit(const uint64_t* __restrict__ keys, uint64_t count, uint32_t bits,
                                                  const uint64_t* __restrict__ ents, const uint64_t* __restrict__ types,
                                                  uint64_t U, uint64_t total_types, int32_t n,
                                                  uint32_t* __restrict__ nbr, uint32_t* __restrict__ owner,
                                                  uint64_t* __restrict__ tpre, int64_t* __restrict__ row_ptr) {
    __shared__ uint32_t se[kT / 64], so[kT / 64], si[kT / 64];
    const uint64_t sentinel = (1ull << (2 * bits + 2)) - 1ull;
    const uint32_t lane = __lane_id(), wid = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kTile + wid * 64 * kI;
    run_of q[kI];
    uint32_t ne = 0, no = 0, ni = 0;
#pragma unroll
    for (int r = 0; r < kI; ++r) {
        const uint64_t i = base + r * 64 + lane;
        q[r] = i < count ? run_at(keys, i, count, sentinel) : run_of{false, 0u};
        ne += (uint32_t)__popcll(__ballot(q[r].head));
        no += (uint32_t)__popcll(__ballot(q[r].head && (q[r].f & 1u)));
        ni += (uint32_t)__popcll(__ballot(q[r].head && (q[r].f >> 1)));
    }
    if (lane == 0) { se[wid] = ne; so[wid] = no; si[wid] = ni; }
    __syncthreads();
    uint64_t e0 = ents[blockIdx.x], t0 = types[blockIdx.x];
    for (uint32_t w = 0; w < wid; ++w) {
        e0 += se[w];
        t0 += (uint64_t)so[w] | ((uint64_t)si[w] << 32);
    }
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < kI; ++r) {
        const uint64_t i = base + r * 64 + lane;
        const uint64_t mh = __ballot(q[r].head), mo = __ballot(q[r].head && (q[r].f & 1u)),
                       mi = __ballot(q[r].head && (q[r].f >> 1));
        const uint64_t e = e0 + (uint32_t)__popcll(mh & lt);
        int64_t before = -1, o = -1;
        if (q[r].head) {
            const uint64_t k = keys[i];
            o = (int64_t)(k >> (bits + 2));
            before = i == 0 ? -1 : (int64_t)(keys[i - 1] >> (bits + 2));
            nbr[e] = ((uint32_t)((k >> 2) & ((1ull << bits) - 1ull)) << 2) | q[r].f;
            owner[e] = (uint32_t)o;
            tpre[e] = t0 + ((uint64_t)__popcll(mo & lt) | ((uint64_t)__popcll(mi & lt) << 32));
        }
        fill_rows(q[r].head, before, o, e, row_ptr);
        // the last entry: the rows after its own, and the ends of the prefix
        const bool last = q[r].head && e + 1 == U;
        if (last) tpre[U] = total_types;
        fill_rows(last, o, (int64_t)n, U, row_ptr);
        e0 += (uint32_t)__popcll(mh);
        t0 += (uint64_t)__popcll(mo) | ((uint64_t)__popcll(mi) << 32);
    }
}

// Per row: its degree, and its bounds with the direction-bit prefix counts at
// its end; the largest degree and the sum of the squares, one atomic per
// workgroup of a small grid (one per wavefront: 1.39 ms on 3.8 M rows, now
// 0.05 ms for both).
__global__ __launch_bounds__(kT) void k_row_info(const int64_t* __restrict__ row_ptr, int32_t n,
                                                 const uint64_t* __restrict__ tpre, uint4* __restrict__ rinfo,
                                                 uint32_t* __restrict__ deg, uint2* __restrict__ rows,
                                                 unsigned long long* __restrict__ counters) {
    __shared__ unsigned long long sh[kT / 64], shm[kT / 64];
    unsigned long long sq = 0, mx = 0;
    for (int64_t x = (int64_t)blockIdx.x * kT + threadIdx.x; x < n; x += (int64_t)gridDim.x * kT) {
        const uint64_t rb = (uint64_t)row_ptr[x], re = (uint64_t)row_ptr[x + 1], t = tpre[re];
        rinfo[x] = make_uint4((uint32_t)rb, (uint32_t)re, (uint32_t)t, (uint32_t)(t >> 32));
        const unsigned long long d = re - rb;
        deg[x] = (uint32_t)d;
        rows[x] = make_uint2((uint32_t)rb, (uint32_t)d);
        sq += d * d;
        mx = d > mx ? d : mx;
    }
    sq = block_sum(sq, sh);
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(mx, off, 64);
        mx = o > mx ? o : mx;
    }
    if (__lane_id() == 0) shm[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kT / 64; ++w) mx = shm[w] > mx ? shm[w] : mx;
        if (sq) atomicAdd(&counters[3], sq);
        if (mx) atomicMax(&counters[4], mx);
    }
}

// ---- dyads: buckets, stable partition, hub tasks --------------------------
// Every connected pair is emitted once.  A pair whose larger degree is at
// least t_hub is a hub dyad, emitted from its anchor's row (the endpoint of
// larger degree, ties to the larger id), so the hub bucket is anchor-major;
// any other pair is emitted from the row of its smaller id (u-major) into the
// lane / wave / group bucket by k = |N(u)| + |N(v)| - 2.
// Bucket of the neighbour entry (o, w): the dyad is emitted once, from its
// first vertex, or from its anchor in the hub bucket.  The other row's length
// is looked up only where the entry can be the emitting one: an entry below the
// diagonal emits only as the anchor of a hub dyad, and so not from a row
// shorter than t_hub (citation graph: half of the look-ups).
// len_of(w): the length of row w.
template <class F>
__device__ inline int rec_bucket(uint32_t o, uint32_t w, uint32_t d_o, const bucket_params& bp, F len_of,
                                 uint64_t* cost, uint64_t* stream) {
    if (o > w && d_o < bp.t_hub) return kBuckets;
    const uint64_t d_w = len_of(w);
    *cost = d_o + d_w;
    if ((d_o > d_w ? d_o : d_w) >= bp.t_hub) {
        const bool o_anchor = d_o > d_w || (d_o == d_w && o > w);
        if (!o_anchor) return kBuckets;
        *stream = d_w;
        return kBucketHub;
    }
    if (!(o < w)) return kBuckets;
    const uint64_t k = d_o + d_w - 2;
    return k < bp.t0 ? 0 : (k < bp.t1 ? 1 : 2);
}

// Per tile: the records of each bucket (counts, bucket-major), and the sums
// of kPartWords quantities (part, quantity-major): the cost of each bucket,
// the hub stream, the mutual pairs.  The tiles' sums are added up by
// k_bucket_sums: eight atomics per tile on shared counters took 1.4 of the
// kernel's 1.5 ms on 29.5 M entries.
constexpr uint32_t kPartWords = kBuckets + 2;
__device__ inline void store_tile_sums(const uint32_t (&my)[kBuckets], const unsigned long long (&mycost)[kBuckets],
                                       unsigned long long mystream, unsigned long long mut,
                                       uint64_t* __restrict__ counts, uint64_t* __restrict__ part, uint32_t nblocks,
                                       unsigned long long* sh) {
#pragma unroll
    for (int q = 0; q < kBuckets; ++q) {
        const unsigned long long c = block_sum(my[q], sh), x = block_sum(mycost[q], sh);
        if (threadIdx.x == 0) {
            counts[(uint64_t)q * nblocks + blockIdx.x] = c;
            part[(uint64_t)q * nblocks + blockIdx.x] = x;
        }
    }
    const unsigned long long st = block_sum(mystream, sh), mu = block_sum(mut, sh);
    if (threadIdx.x == 0) {
        part[(uint64_t)kBuckets * nblocks + blockIdx.x] = st;
        part[(uint64_t)(kBuckets + 1) * nblocks + blockIdx.x] = mu;
    }
}

__global__ __launch_bounds__(kT) void k_dyad_count(const uint32_t* __restrict__ nbr, const uint32_t* __restrict__ owner,
                                                    const uint32_t* __restrict__ len, uint64_t U, bucket_params bp,
                                                    uint64_t* __restrict__ counts, uint32_t nblocks,
                                                    uint64_t* __restrict__ part, uint8_t* __restrict__ bucket) {
    __shared__ unsigned long long sh[kT / 64];
    uint64_t base = (uint64_t)blockIdx.x * kTile;
    uint32_t my[kBuckets] = {0, 0, 0, 0}, mut = 0;
    unsigned long long mycost[kBuckets] = {0, 0, 0, 0}, mystream = 0;
    for (int k = 0; k < kI; ++k) {
        uint64_t e = base + (uint64_t)k * kT + threadIdx.x;
        uint64_t cost = 0, stream = 0;
        int b = kBuckets;
        uint32_t ent = 0;
        if (e < U) {
            ent = nbr[e];
            const uint32_t o = owner[e];
            b = rec_bucket(o, ent >> 2, len[o], bp, [&](uint32_t w) { return len[w]; }, &cost, &stream);
            bucket[e] = (uint8_t)b;
        }
#pragma unroll
        for (int q = 0; q < kBuckets; ++q) {
            my[q] += b == q ? 1u : 0u;
            mycost[q] += b == q ? cost : 0ull;
        }
        if (b < kBuckets) {
            mut += ((ent & 3u) == 3u) ? 1u : 0u;
            if (b == kBucketHub) mystream += stream;
        }
    }
    store_tile_sums(my, mycost, mystream, mut, counts, part, nblocks, sh);
}

// One workgroup per quantity of `part`: its sum over the tiles to
// host[kBuckets + 1 + quantity]; one more writes the bucket starts (the scanned
// counts at each bucket's first tile, and the total) to host[0 .. kBuckets].
__global__ __launch_bounds__(kT) void k_bucket_sums(const uint64_t* __restrict__ part, const uint64_t* __restrict__ counts,
                                                    uint32_t nblocks, uint64_t* __restrict__ host) {
    __shared__ unsigned long long sh[kT / 64];
    const uint32_t q = blockIdx.x;
    if (q == kPartWords) {
        if (threadIdx.x <= kBuckets) host[threadIdx.x] = counts[(uint64_t)threadIdx.x * nblocks];
        return;
    }
    unsigned long long s = 0;
    for (uint32_t i = threadIdx.x; i < nblocks; i += kT) s += part[(uint64_t)q * nblocks + i];
    s = block_sum(s, sh);
    if (threadIdx.x == 0) host[kBuckets + 1 + q] = s;
}

// Writes the records in entry order through a stable per-bucket ranking:
// lane / wave / group records are u-major, and hub records, which come from
// their anchor's row, anchor-major.
// Every wavefront holds 64 * kI consecutive entries, 64 per round, so that
// ranks are ballots and lane counts and one barrier per tile is enough.  The
// buckets come from the counting pass, so that a row is looked up only for a
// record.
__global__ __launch_bounds__(kT) void k_dyad_scatter(const uint32_t* __restrict__ nbr, const uint32_t* __restrict__ owner,
                                                      const uint2* __restrict__ rows, uint64_t U,
                                                      const uint8_t* __restrict__ bucket,
                                                      const uint64_t* __restrict__ offsets, uint32_t nblocks,
                                                      uint64_t hub_begin, uint32_t* __restrict__ anchors,
                                                      dyad_rec* __restrict__ out) {
    __shared__ uint32_t wcnt[kT / 64][kBuckets];
    const uint32_t lane = __lane_id(), wid = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kTile + wid * 64 * kI;
    uint32_t mine[kBuckets] = {0, 0, 0, 0};
    int b[kI];
#pragma unroll
    for (int k = 0; k < kI; ++k) {
        const uint64_t e = base + k * 64 + lane;
        b[k] = e < U ? (int)bucket[e] : kBuckets;
#pragma unroll
        for (int q = 0; q < kBuckets; ++q) mine[q] += (uint32_t)__popcll(__ballot(b[k] == q));
    }
    if (lane == 0)
        for (int q = 0; q < kBuckets; ++q) wcnt[wid][q] = mine[q];
    __syncthreads();
    uint64_t at[kBuckets];
#pragma unroll
    for (int q = 0; q < kBuckets; ++q) {
        at[q] = offsets[(uint64_t)q * nblocks + blockIdx.x];
        for (uint32_t w = 0; w < wid; ++w) at[q] += wcnt[w][q];
    }
#pragma unroll
    for (int k = 0; k < kI; ++k) {
        uint64_t to = 0;
#pragma unroll
        for (int q = 0; q < kBuckets; ++q) {
            const uint64_t m = __ballot(b[k] == q);
            if (b[k] == q) to = at[q] + (uint32_t)__popcll(m & lanemask_lt());
            at[q] += (uint32_t)__popcll(m);
        }
        if (b[k] < kBuckets) {
            const uint64_t e = base + k * 64 + lane;
            const uint32_t ent = nbr[e], o = owner[e], w = ent >> 2, f = ent & 3u;
            const bool up = o < w;
            const uint2 ro = rows[o], rw = rows[w], ru = up ? ro : rw, rv = up ? rw : ro;
            dyad_rec rec;
            rec.bu = ru.x;
            rec.eu = ru.x + ru.y;
            rec.bv = rv.x;
            rec.ev = rv.x + rv.y;
            rec.u = up ? o : w;
            rec.vf = up ? (w << 2) | f : (o << 2) | ((f & 1u) << 1) | (f >> 1);
            out[to] = rec;
            if (b[k] == kBucketHub) anchors[to - hub_begin] = o;
        }
    }
}

// ---- forward lists ----------------------------------------------------------
// Ranks: the vertices sorted by falling degree, ties by falling id (a stable
// sort of the degrees alone, from the ids in falling order).
__global__ __launch_bounds__(kT) void k_vertex_keys(const uint32_t* __restrict__ deg, int32_t n, uint32_t max_degree,
                                                    uint64_t* __restrict__ keys) {
    const int32_t i = (int32_t)(blockIdx.x * kT + threadIdx.x);
    if (i >= n) return;
    const uint32_t v = (uint32_t)(n - 1 - i);
    keys[i] = ((uint64_t)(max_degree - deg[v]) << 32) | v;
}

__global__ __launch_bounds__(kT) void k_ranks(const uint64_t* __restrict__ keys, int32_t n, uint32_t* __restrict__ rank) {
    const int32_t r = (int32_t)(blockIdx.x * kT + threadIdx.x);
    if (r < n) rank[(uint32_t)keys[r]] = (uint32_t)r;
}

// One key per joined pair {x, y}, rank y < rank x: rank x << (bits + 3) |
// rank y << 3 | f_xy << 1 | [id y > id x], from the neighbour entry above the
// diagonal (one look-up of a rank per pair).  The keys are sorted next, so
// their order does not matter: a workgroup takes the place of its keys from a
// counter, one atomic per 8192 entries.
constexpr int kPairT = 512;
constexpr int kPairI = 16;
constexpr int kPairTile = kPairT * kPairI;
__global__ __launch_bounds__(kPairT) void k_pair_keys(const uint32_t* __restrict__ nbr, const uint32_t* __restrict__ owner,
                                                      const uint32_t* __restrict__ rank, uint64_t U, uint32_t bits,
                                                      unsigned long long* __restrict__ counter,
                                                      uint64_t* __restrict__ keys) {
    __shared__ uint32_t sw[kPairT / 64];
    __shared__ unsigned long long s_at;
    const uint32_t lane = __lane_id(), wid = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kPairTile + wid * 64 * kPairI;
    uint32_t ent[kPairI], o[kPairI], mine = 0;
#pragma unroll
    for (int r = 0; r < kPairI; ++r) {
        const uint64_t e = base + r * 64 + lane;
        ent[r] = e < U ? nbr[e] : 0u;
        o[r] = e < U ? owner[e] : 0xffffffffu;
        mine += (uint32_t)__popcll(__ballot(e < U && (ent[r] >> 2) > o[r]));
    }
    if (lane == 0) sw[wid] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kPairT / 64; ++w) t += sw[w];
        s_at = atomicAdd(counter, (unsigned long long)t);
    }
    __syncthreads();
    uint64_t at = s_at;
    for (uint32_t w = 0; w < wid; ++w) at += sw[w];
#pragma unroll
    for (int r = 0; r < kPairI; ++r) {
        const uint64_t e = base + r * 64 + lane;
        const uint32_t w = ent[r] >> 2, f = ent[r] & 3u;
        const bool on = e < U && w > o[r];
        const uint64_t m = __ballot(on);
        if (on) {
            const uint32_t ro = rank[o[r]], rw = rank[w];
            const bool owner_x = rw < ro;   // the owner plays x (then id y > id x)
            const uint32_t fxy = owner_x ? f : ((f & 1u) << 1) | (f >> 1);
            const uint64_t x = owner_x ? ro : rw, y = owner_x ? rw : ro;
            keys[at + (uint32_t)__popcll(m & lanemask_lt())] =
                (x << (bits + 3)) | (y << 3) | (fxy << 1) | (owner_x ? 1u : 0u);
        }
        at += (uint32_t)__popcll(m);
    }
}

// The forward lists and their row starts from the sorted keys.
// fptr holds `count` in every row before: the rows after the last key's, the
// vertices without any neighbour among them (R-MAT 2^20: 0.4 M, 0.11 ms for one
// wavefront), are right so.
__global__ __launch_bounds__(kT) void k_fwd_emit(const uint64_t* __restrict__ keys, uint64_t count, uint32_t bits,
                                                 uint32_t* __restrict__ fwd, uint32_t* __restrict__ fptr) {
#pragma unroll
    for (int r = 0; r < kI; ++r) {
        const uint64_t i = (uint64_t)blockIdx.x * kTile + (uint64_t)r * kT + threadIdx.x;
        int64_t before = -1, x = -1;
        const bool on = i < count;
        if (on) {
            const uint64_t k = keys[i];
            x = (int64_t)(k >> (bits + 3));
            before = i == 0 ? -1 : (int64_t)(keys[i - 1] >> (bits + 3));
            fwd[i] = ((uint32_t)(k & 7u) << 29) | ((uint32_t)((k >> 3) & ((1ull << bits) - 1ull)) << 1);
        }
        fill_rows(on && x != before, before, x, i, fptr);
    }
}

// Bucket of the edge of sorted key i (x, y): hub when the longer of the two
// forward lists reaches t_hub, else by their joint length; kBuckets for an
// edge that closes no triangle with a smaller rank.
//
// A hub edge is found at y (its prefix of N+(x) streams against a table of
// N+(y)) or, `at_x`, at x (N+(y) streams against a table of N+(x); x and y
// change their roles in the record, so the kernels see no difference).  The
// prefix is seldom much longer than N+(y), which is all ranks below y that y is
// joined to, and the choice is y; but where y has few neighbours of smaller
// rank and x many (items of a user, both sides of a bipartite graph with a
// vertex joined to all), the prefixes add up to the square of the row lengths.
// x takes the edge when that more than halves the blocks of 16 to stream: never
// on R-MAT, random, complete or citation graphs (there finding an edge at x for
// one block less gains 0.5 % of the blocks or, random graph of 200 neighbours
// per vertex, 2.4 %, for a third of the edges moved).  4000 vertices joined to each
// of 2000 and one vertex to all: 2.20 ms, now 0.20; 20000 users with 1000 of 6000
// items each, a few links among the items: 2.98 ms, now 0.21.
struct edge_at {
    uint32_t bx, by, dy, y, pos, bits;
    uint64_t cost;
    int bucket;
    __device__ inline bool at_x() const { return (pos + 15u) >> 4 > 2u * ((dy + 15u) >> 4); }
};
__device__ inline edge_at edge_bucket(const uint64_t* __restrict__ keys, uint64_t i, uint64_t count, uint32_t bits,
                                      const uint32_t* __restrict__ fptr, const bucket_params& bp) {
    edge_at r{};
    r.bucket = kBuckets;
    if (i >= count) return r;
    const uint64_t k = keys[i];
    const uint32_t x = (uint32_t)(k >> (bits + 3));
    r.y = (uint32_t)((k >> 3) & ((1ull << bits) - 1ull));
    r.bx = fptr[x];
    r.pos = (uint32_t)i - r.bx;
    if (r.pos == 0) return r;
    r.by = fptr[r.y];
    r.dy = fptr[r.y + 1] - r.by;
    r.bits = (uint32_t)(k & 7u);
    const uint64_t dx = fptr[x + 1] - r.bx, dy = r.dy;
    if (dy == 0) return r;
    r.cost = dx + dy;
    r.bucket = (dx > dy ? dx : dy) >= bp.t_hub ? kBucketHub : r.cost < bp.t0 ? 0 : r.cost < bp.t1 ? 1 : 2;
    return r;
}

__global__ __launch_bounds__(kT) void k_edge_count(const uint64_t* __restrict__ keys, uint64_t count, uint32_t bits,
                                                   const uint32_t* __restrict__ fptr, bucket_params bp,
                                                   uint64_t* __restrict__ counts, uint32_t nblocks,
                                                   uint64_t* __restrict__ part) {
    __shared__ unsigned long long sh[kT / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kTile;
    uint32_t my[kBuckets] = {0, 0, 0, 0};
    unsigned long long mycost[kBuckets] = {0, 0, 0, 0}, mystream = 0;
    for (int k = 0; k < kI; ++k) {
        const edge_at r = edge_bucket(keys, base + (uint64_t)k * kT + threadIdx.x, count, bits, fptr, bp);
#pragma unroll
        for (int q = 0; q < kBuckets; ++q) {
            my[q] += r.bucket == q ? 1u : 0u;
            mycost[q] += r.bucket == q ? r.cost : 0ull;
        }
        if (r.bucket == kBucketHub) mystream += r.at_x() ? r.dy : r.pos;
    }
    store_tile_sums(my, mycost, mystream, 0ull, counts, part, nblocks, sh);
}

// A hub edge's record needs i, the start bx of x's row, the code bits, and
// whether the prefix has entries not below kCore (`tail`).  Where they fit
// beside y in 64 bits, the key the edges are sorted by holds them all: y, i, the
// place of y in the row (i - bx, below sqrt(2 F): the d neighbours after x have
// degree d or more), tail, bits.  Otherwise the key holds y and i, and the
// record gathers the rest by i (R-MAT 2^20, 14 M hub edges: 0.37 ms for the
// gathers, which miss the L2 at 55 G lines/s, 0.15 ms without).  An edge found
// at x has x in the place of y, and a place of 0 (which no hub edge has), or
// the top bit, to tell it by; its record gathers y by i either way.
struct hub_key {
    uint32_t ibits, pbits;   // pbits 0: y << 32 | i
    __host__ __device__ uint32_t y_shift() const { return pbits ? 4 + pbits + ibits : 32; }
};
constexpr uint64_t kFoundAtX = 1ull << 63;

// Lane / wave / group records in x-major order; for the hub edges a key, in
// x-major order too (sorted by y next, or x).  Without room in the key, keys[i]
// becomes bx << 4 | tail << 3 | bits, except for an edge found at x.
// (five wavefronts per SIMD: with the two registers more that four allow 131 us
// on R-MAT 2^20, 123 so)
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(5))) void k_edge_scatter(uint64_t* keys, uint64_t count, uint32_t bits,
                                                     const uint32_t* __restrict__ fptr, bucket_params bp,
                                                     const uint64_t* __restrict__ offsets, uint32_t nblocks,
                                                     uint64_t hub_begin, hub_key hk, const uint32_t* __restrict__ fwd,
                                                     uint64_t* __restrict__ hubkeys, uint4* __restrict__ out) {
    __shared__ uint32_t wcnt[kT / 64][kBuckets];
    const uint32_t lane = __lane_id(), wid = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kTile + wid * 64 * kI;   // the wavefront's keys
    uint32_t mine[kBuckets] = {0, 0, 0, 0};
    edge_at r[kI];
#pragma unroll
    for (int k = 0; k < kI; ++k) {
        r[k] = edge_bucket(keys, base + k * 64 + lane, count, bits, fptr, bp);
#pragma unroll
        for (int q = 0; q < kBuckets; ++q) mine[q] += (uint32_t)__popcll(__ballot(r[k].bucket == q));
    }
    if (lane == 0)
        for (int q = 0; q < kBuckets; ++q) wcnt[wid][q] = mine[q];
    __syncthreads();
    uint64_t at[kBuckets];
#pragma unroll
    for (int q = 0; q < kBuckets; ++q) {
        at[q] = offsets[(uint64_t)q * nblocks + blockIdx.x];
        for (uint32_t w = 0; w < wid; ++w) at[q] += wcnt[w][q];
    }
#pragma unroll
    for (int k = 0; k < kI; ++k) {
        const uint64_t i = base + k * 64 + lane;
#pragma unroll
        for (int q = 0; q < kBuckets; ++q) {
            const uint64_t m = __ballot(r[k].bucket == q);
            if (r[k].bucket == q) {
                const uint64_t to = at[q] + (uint32_t)__popcll(m & lanemask_lt());
                if (q == kBucketHub) {
                    const uint32_t low = ((fwd[i - 1] & 0x00fffffeu) >= 2u * kCore ? 8u : 0u) | r[k].bits;
                    if (r[k].at_x()) {
                        const uint64_t x = keys[i] >> (bits + 3);
                        hubkeys[to - hub_begin] = hk.pbits ? (x << hk.y_shift()) | (i << (4 + hk.pbits))
                                                           : kFoundAtX | (x << 32) | i;
                    } else if (hk.pbits) {
                        hubkeys[to - hub_begin] = ((uint64_t)r[k].y << hk.y_shift()) | (i << (4 + hk.pbits)) |
                                                  ((uint64_t)r[k].pos << 4) | low;
                    } else {
                        hubkeys[to - hub_begin] = ((uint64_t)r[k].y << 32) | i;
                        keys[i] = ((uint64_t)r[k].bx << 4) | low;
                    }
                } else out[to] = make_uint4(r[k].bx, (uint32_t)i, r[k].by, (r[k].bits << 29) | r[k].dy);
            }
            at[q] += (uint32_t)__popcll(m);
        }
    }
}

// Hub records from the keys sorted by y, and the run of each y (first and one
// past the last record, zero elsewhere); x in the place of y where the edge is
// found at x.  fptr, bits: for the records of these.
__global__ __launch_bounds__(kT) void k_edge_hub(const uint64_t* __restrict__ hubkeys, uint64_t hubs, hub_key hk,
                                                 const uint64_t* __restrict__ edges, const uint32_t* __restrict__ fwd,
                                                 const uint32_t* __restrict__ fptr, uint32_t bits,
                                                 uint32_t* __restrict__ first, uint32_t* __restrict__ past,
                                                 uint4* __restrict__ out) {
    const uint32_t ys = hk.y_shift();
    const uint64_t idmask = (1ull << bits) - 1ull;
    uint64_t key[kI], ed[kI];
#pragma unroll
    for (int r = 0; r < kI; ++r) {
        const uint64_t j = (uint64_t)blockIdx.x * kTile + (uint64_t)r * kT + threadIdx.x;
        key[r] = j < hubs ? hubkeys[j] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < kI; ++r) {
        const uint64_t j = (uint64_t)blockIdx.x * kTile + (uint64_t)r * kT + threadIdx.x;
        ed[r] = j < hubs && !hk.pbits ? edges[(uint32_t)key[r]] : 0ull;
    }
    auto run = [&](uint64_t k) { return (uint32_t)((k >> ys) & idmask); };
#pragma unroll
    for (int r = 0; r < kI; ++r) {
        const uint64_t j = (uint64_t)blockIdx.x * kTile + (uint64_t)r * kT + threadIdx.x;
        if (j >= hubs) continue;
        const uint32_t y = run(key[r]);
        uint32_t i, bx, low;
        bool at_x;
        if (hk.pbits) {
            i = (uint32_t)((key[r] >> (4 + hk.pbits)) & ((1ull << hk.ibits) - 1ull));
            bx = i - (uint32_t)((key[r] >> 4) & ((1ull << hk.pbits) - 1ull));
            low = (uint32_t)key[r] & 15u;
            at_x = bx == i;
        } else {
            i = (uint32_t)key[r];
            bx = (uint32_t)(ed[r] >> 4);
            low = (uint32_t)ed[r] & 15u;
            at_x = (key[r] & kFoundAtX) != 0;
        }
        if (at_x) {   // the pair as (y, x): its arcs the other way, the order of the ids turned
            const uint64_t e = hk.pbits ? edges[i] : ed[r];
            const uint32_t other = (uint32_t)((e >> 3) & idmask), b = (uint32_t)e & 7u;
            bx = fptr[other];
            i = fptr[other + 1];
            low = ((fwd[i - 1] & 0x00fffffeu) >= 2u * kCore ? 8u : 0u) | ((b & 2u) << 1) | ((b & 4u) >> 1) |
                  ((b & 1u) ^ 1u);
        }
        uint32_t core = i;
        if (low & 8u) {
            uint32_t lo = bx, hi = i - 1;
            while (lo < hi) {
                const uint32_t mid = lo + ((hi - lo) >> 1);
                if ((fwd[mid] & 0x00fffffeu) < 2u * kCore) lo = mid + 1; else hi = mid;
            }
            core = lo;
        }
        out[j] = make_uint4(bx, core, i, low & 7u);
        if (j == 0 || run(hubkeys[j - 1]) != y) first[y] = (uint32_t)j;
        if (j + 1 == hubs || run(hubkeys[j + 1]) != y) past[y] = (uint32_t)j + 1;
    }
}

__global__ __launch_bounds__(kT) void k_tri_ntasks(const uint32_t* __restrict__ first, const uint32_t* __restrict__ past,
                                                   int32_t n, const uint32_t* __restrict__ fptr, uint32_t chunk,
                                                   uint64_t* __restrict__ ntask, unsigned long long* __restrict__ sums) {
    __shared__ unsigned long long sh[kT / 64];
    __shared__ uint32_t s_heavy;
    if (threadIdx.x == 0) s_heavy = 0;
    __syncthreads();
    unsigned long long staged = 0;
    for (int64_t y = (int64_t)blockIdx.x * kT + threadIdx.x; y < n; y += (int64_t)gridDim.x * kT) {
        const uint64_t t = (past[y] - first[y] + chunk - 1) / chunk;
        ntask[y] = t;
        staged += t * (unsigned long long)(fptr[y + 1] - fptr[y]);
        if (past[y] - first[y] >= 64) atomicMax(&s_heavy, (uint32_t)y + 1u);
    }
    staged = block_sum(staged, sh);
    if (threadIdx.x == 0 && staged) {
        atomicAdd(&sums[0], staged);
        if (s_heavy) atomicMax(&sums[1], (unsigned long long)s_heavy);
    }
}

__global__ void k_tri_publish(const uint64_t* __restrict__ task_off, int32_t n, const unsigned long long* __restrict__ sums,
                              uint64_t* __restrict__ host) {
    if (threadIdx.x == 0) {
        host[0] = task_off[n];
        host[1] = sums[0];
        host[2] = task_off[sums[1]];
    }
}

// Tasks in rank order: the vertices with the most records come first.
__global__ __launch_bounds__(kT) void k_tri_tasks(const uint32_t* __restrict__ first, const uint32_t* __restrict__ past,
                                                  int32_t n, const uint32_t* __restrict__ fptr, uint32_t chunk,
                                                  const uint64_t* __restrict__ task_off, uint32_t hub_begin,
                                                  tri_task* __restrict__ tasks) {
    const int32_t y = (int32_t)(blockIdx.x * kT + threadIdx.x);
    if (y >= n) return;
    const uint32_t a = first[y], b = past[y];
    uint64_t t = task_off[y];
    for (uint32_t j = a; j < b; j += chunk, ++t)
        tasks[t] = tri_task{hub_begin + j, hub_begin + (b - j < chunk ? b : j + chunk), fptr[y], fptr[y + 1]};
}

__global__ __launch_bounds__(kT) void k_row_len(const int64_t* __restrict__ row_ptr, int32_t n,
                                                uint32_t* __restrict__ len, uint2* __restrict__ rows) {
    const int64_t x = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (x >= n) return;
    const uint32_t b = (uint32_t)row_ptr[x], l = (uint32_t)row_ptr[x + 1] - b;
    len[x] = l;
    rows[x] = make_uint2(b, l);
}

// The run of hub records of each anchor: first and one past the last, from
// the records' anchors in record order (zero for the other vertices).
__global__ __launch_bounds__(kT) void k_hub_runs(const uint32_t* __restrict__ anchors, uint32_t count,
                                                 uint32_t* __restrict__ first, uint32_t* __restrict__ past) {
    const uint32_t i = blockIdx.x * kT + threadIdx.x;
    if (i >= count) return;
    const uint32_t a = anchors[i];
    if (i == 0 || anchors[i - 1] != a) first[a] = i;
    if (i + 1 == count || anchors[i + 1] != a) past[a] = i + 1;
}

// Hub tasks: the hub records of anchor row h are contiguous, [first[h],
// past[h]) inside the hub bucket; they are cut into runs of `chunk`.  Tasks of
// anchors whose row is longer than `big_row` are placed first (they are the
// longest), the others after them: their numbers are counted in the high and
// the low 32 bits of one word per row, so that one scan places both.
__global__ __launch_bounds__(kT) void k_hub_ntasks(const uint32_t* __restrict__ first, const uint32_t* __restrict__ past,
                                                    int32_t n, const uint32_t* __restrict__ len,
                                                    uint64_t* __restrict__ ntask, uint32_t big_row, uint32_t chunk,
                                                    unsigned long long* __restrict__ staged_sum) {
    __shared__ unsigned long long sh[kT / 64];
    unsigned long long staged = 0;
    for (int64_t h = (int64_t)blockIdx.x * kT + threadIdx.x; h < n; h += (int64_t)gridDim.x * kT) {
        const uint32_t d = len[h];
        const uint64_t t = (past[h] - first[h] + chunk - 1) / chunk;
        ntask[h] = d > big_row ? t << 32 : t;
        staged += t * (unsigned long long)d;
    }
    staged = block_sum(staged, sh);
    if (threadIdx.x == 0 && staged) atomicAdd(staged_sum, staged);
}

__global__ __launch_bounds__(kT) void k_hub_emit(const uint32_t* __restrict__ first, const uint32_t* __restrict__ past,
                                                  int32_t n, const uint32_t* __restrict__ len,
                                                  const uint64_t* __restrict__ task_off, uint32_t big_row,
                                                  uint32_t chunk, uint64_t hub_begin, hub_task* __restrict__ tasks) {
    int32_t h = (int32_t)(blockIdx.x * kT + threadIdx.x);
    if (h >= n) return;
    const uint64_t c = past[h] - first[h], base = hub_begin + first[h], off = task_off[h];
    const uint64_t t0 = len[h] > big_row ? off >> 32 : (task_off[n] >> 32) + (off & 0xffffffffull);
    for (uint64_t j = 0; j * chunk < c; ++j) {
        hub_task t;
        t.begin = (uint32_t)(base + j * chunk);
        t.end = (uint32_t)(base + (c < (j + 1) * chunk ? c : (j + 1) * chunk));
        t.anchor = (uint32_t)h;
        t.group = 0;
        tasks[t0 + j] = t;
    }
}

// Groups of consecutive hub tasks that one workgroup runs with a single LDS
// tile: each window of kHubGroupTasks tasks is cut greedily before a task whose
// records would take the group past `chunk` or whose anchor row would take
// the group's rows past `tile` entries (a row longer than that stays alone).
// Without goff, counts the groups of every window into gcount; with goff (the
// scanned counts), stores the first task of each group in tasks[g].group.
__global__ __launch_bounds__(kT) void k_hub_group(hub_task* __restrict__ tasks, const dyad_rec* __restrict__ recs,
                                                  uint64_t ntasks, const uint64_t* __restrict__ goff,
                                                  uint64_t* __restrict__ gcount, uint32_t tile, uint32_t chunk) {
    const uint64_t w = (uint64_t)blockIdx.x * kT + threadIdx.x;
    const uint64_t t0 = w * kHubGroupTasks;
    if (t0 >= ntasks) return;
    const uint32_t nt = (uint32_t)(ntasks - t0 < kHubGroupTasks ? ntasks - t0 : kHubGroupTasks);
    uint32_t starts[kHubGroupTasks];
    uint32_t ng = 0, gs = 0, sr = 0, se = 0;
    for (uint32_t j = 0; j < nt; ++j) {
        const uint32_t b = tasks[t0 + j].begin, e = tasks[t0 + j].end, a = tasks[t0 + j].anchor;
        const dyad_rec r0 = recs[b];
        const uint32_t l = r0.u == a ? r0.eu - r0.bu : r0.ev - r0.bv, r = e - b;
        if (j > gs && (l > tile || sr + r > chunk || se + l > tile)) {
            starts[ng++] = gs;
            gs = j;
            sr = 0;
            se = 0;
        }
        sr += r;
        se += l;
    }
    starts[ng++] = gs;
    if (goff == nullptr) {
        gcount[w] = ng;
    } else {
        for (uint32_t k = 0; k < ng; ++k) tasks[goff[w] + k].group = (uint32_t)t0 + starts[k];
    }
}

// Words of device memory to pinned host memory (read after the next synchronisation).
__global__ void k_publish(const uint64_t* __restrict__ a, uint64_t* __restrict__ host, int count) {
    if ((int)threadIdx.x < count) host[threadIdx.x] = a[threadIdx.x];
}

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u64(uint64_t* p, uint64_t n, uint64_t v) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

inline uint32_t grid1(uint64_t n) { return (uint32_t)((n + kT - 1) / kT); }


// Device scratch of a build, taken front to back; all of it belongs to the
// build's stream, so memory handed back by a rewind is reused in stream order.
class arena {
public:
    arena(const build_space& sp) : base_((char*)sp.base), cap_(sp.cap) {}
    template <class T>
    T* take(uint64_t count) {
        const size_t b = (count * sizeof(T) + 255) & ~(size_t)255;
        if (b > cap_ - used_) { full = true; return nullptr; }
        T* p = (T*)(base_ + used_);
        used_ += b;
        return p;
    }
    size_t mark() const { return used_; }
    void rewind(size_t m) { used_ = m; }
    bool full = false;

private:
    char* base_;
    size_t cap_, used_ = 0;
};

inline uint32_t sort_digit_bits(uint32_t sort_bits) {
    const uint32_t passes = (sort_bits + kDigitBits - 1) / kDigitBits;
    return passes ? (sort_bits + passes - 1) / passes : 1;
}
inline int sort_items(uint64_t count) { return count < kSortSmall ? kSortISmall : kSortI; }
inline uint64_t sort_tiles(uint64_t count) {
    const uint64_t t = (uint64_t)kT * sort_items(count);
    return (count + t - 1) / t;
}
inline uint64_t scan_scratch_words(uint64_t count) { return (count + kTile - 1) / kTile + 1; }

// Scratch words and bytes of the two phases of a build: sorting 2 m keys, and
// bucketing U <= 2 m entries of n rows (tasks of at least kHubChunk / 2 records).
inline uint64_t sort_space_bytes(uint64_t m, uint32_t bits) {
    const uint64_t keys = 2 * m, wide = keys >= (1ull << 32) ? 8 : 4;
    const uint64_t hist = (1ull << sort_digit_bits(2 * bits)) * sort_tiles(keys);
    return 2 * 8 * keys + wide * hist + 8 * scan_scratch_words(hist) + 16 * ((keys + kTile - 1) / kTile) + 16 * 256;
}
inline uint64_t bucket_space_bytes(uint64_t U, uint64_t n) {
    const uint64_t nb = (U + kTile - 1) / kTile + 1, p = U / 2, tasks = std::min(n, p) + p / (kHubChunk / 2) + 1;
    return 8 * (kBuckets * nb + 1) + 8 * kPartWords * nb + 8 * scan_scratch_words(std::max(U + 1, n + 1)) +
           4 * 3 * (n + 2) + 4 * p + U + 2 * 8 * (n + 1) + 8 * (tasks / kHubGroupTasks + 2) +
           8 * scan_scratch_words(tasks) + 32 * 256;
}
inline uint64_t forward_space_bytes(uint64_t U, uint64_t n) {
    const uint64_t F = U / 2, nb = (U + kTile - 1) / kTile + 1;
    // (hub keys and vertices may be few: tiles of the small size)
    const uint64_t hist = (uint64_t)kDigits * (std::max(F, n) / (kT * kSortISmall) + 1);
    return 3 * 8 * F + 4 * hist + 8 * scan_scratch_words(std::max(hist, n + 1)) + 2 * 8 * n + 4 * n + 8 * nb +
           8 * (kBuckets * nb + 1) + 8 * kPartWords * nb + 4 * 2 * (n + 2) + 8 * (n + 1) + 32 * 256;
}
inline uint64_t view_space_bytes(uint64_t U, uint64_t n, bool tri) {
    return std::max(bucket_space_bytes(U, n), tri ? forward_space_bytes(U, n) : 0);
}
// Scratch of a whole build: the counters and per-row words, then the larger phase.
inline uint64_t build_space_bytes(uint64_t n, uint64_t m, uint32_t bits, bool tri) {
    return 4096 + (sizeof(uint32_t) + sizeof(uint2)) * (n + 1) +
           std::max(sort_space_bytes(m, bits), view_space_bytes(2 * m, n, tri));
}
// Ids below 2^bits.
inline uint32_t id_bits(uint64_t n) {
    uint32_t b = 1;
    while ((1ull << b) < n) ++b;
    return b;
}

}  // namespace

uint64_t build_footprint(uint64_t n, uint64_t m) {
    const uint64_t base = sizeof(int64_t) * (n + 1) + 2 * m * (2 * sizeof(uint32_t) + sizeof(uint64_t)) +
                          sizeof(uint4) * (n + 1) + sizeof(uint32_t) * kRowPad + sizeof(uint64_t);
    const uint64_t runs = std::min(n, m);   // (a vertex's last hub task is short)
    const uint64_t dyads = sizeof(dyad_rec) * m + sizeof(hub_task) * (runs + m / kHubChunk);
    const uint64_t tri = sizeof(uint32_t) * (n + 1 + m + kRowPad) + sizeof(uint4) * m +
                         sizeof(tri_task) * (runs + m / 64);
    const uint64_t graph = base + std::max(dyads, tri);
    // (a reused block may be a quarter larger than asked for)
    return build_space_bytes(n, m, id_bits(n), true) + graph + graph / 4;
}

hipError_t fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(grid1(n)), dim3(kT), 0, s, p, n, v);
    return hipGetLastError();
}

namespace {

// The pools of every context, for give-backs to a device that is full.  Lock
// order: the registry, a pool, a build_space (tried only); hipMalloc runs under none.
std::mutex g_pools_mu;
std::vector<graph_pool*> g_pools;

}  // namespace

hipError_t device_alloc(void** out, uint64_t bytes) {
    hipError_t e = hipMalloc(out, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> lk(g_pools_mu);
        for (graph_pool* p : g_pools)
            if (p->device() == device) p->give_back(0);
    }
    e = hipMalloc(out, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

void graph_pool::open(int device, uint64_t keep) {
    device_ = device;
    keep_ = keep;
    std::lock_guard<std::mutex> lk(g_pools_mu);
    g_pools.push_back(this);
}

void graph_pool::add(build_space* sp) {
    std::lock_guard<std::mutex> lk(mu_);
    spaces_.push_back(sp);
    sp->pool = this;
}

void graph_pool::remove(build_space* sp) {
    std::lock_guard<std::mutex> lk(mu_);
    spaces_.erase(std::remove(spaces_.begin(), spaces_.end(), sp), spaces_.end());
}

void graph_pool::give_back(uint64_t to) {
    std::lock_guard<std::mutex> lk(mu_);
    uint64_t scratch = 0;
    for (build_space* sp : spaces_) {
        std::unique_lock<std::mutex> idle(sp->busy, std::try_to_lock);
        if (idle) scratch += sp->cap;
    }
    shrink(to > scratch ? to - scratch : 0);
    for (build_space* sp : spaces_) {
        if (scratch + held_ <= to) break;
        std::unique_lock<std::mutex> idle(sp->busy, std::try_to_lock);
        if (!idle || !sp->cap) continue;
        scratch -= std::min(scratch, sp->cap);
        (void)hipFree(sp->base);   // (its last build ended with a wait)
        sp->base = nullptr;
        sp->cap = 0;
    }
}

graph_pool::~graph_pool() {
    {
        std::lock_guard<std::mutex> lk(g_pools_mu);
        g_pools.erase(std::remove(g_pools.begin(), g_pools.end(), this), g_pools.end());
    }
    shrink(0);
    for (auto& b : live_) (void)hipFree(b.first);
}

void graph_pool::shrink(uint64_t to) {
    while (held_ > to && !free_.empty()) {
        held_ -= free_.front().bytes;
        (void)hipFree(free_.front().p);
        free_.pop_front();
    }
}

hipError_t graph_pool::alloc(void** out, uint64_t bytes) {
    *out = nullptr;
    // sizes in steps of an eighth of their power of two, so that graphs of
    // about one size reuse each other's blocks; a block too large to be kept
    // has its own size, and so has one that only fits without the rest
    const uint64_t exact = std::max<uint64_t>(bytes, 1);
    uint64_t step = 4096;
    while (16 * step < bytes) step *= 2;
    bytes = (exact + step - 1) / step * step;
    if (bytes > keep_) bytes = exact;
    void* p = nullptr;
    try {
        {
            std::lock_guard<std::mutex> lk(mu_);
            size_t best = free_.size();
            for (size_t i = 0; i < free_.size(); ++i)
                if (free_[i].bytes >= bytes && free_[i].bytes <= bytes + bytes / 4 &&
                    (best == free_.size() || free_[i].bytes < free_[best].bytes))
                    best = i;
            if (best < free_.size()) {
                const block b = free_[best];
                live_.emplace(b.p, b.bytes);
                free_.erase(free_.begin() + (std::ptrdiff_t)best);
                held_ -= b.bytes;
                *out = b.p;
                return hipSuccess;
            }
        }
        hipError_t e = device_alloc(&p, bytes);
        if (e != hipSuccess && exact < bytes) e = device_alloc(&p, bytes = exact);
        if (e != hipSuccess) return e;
        std::lock_guard<std::mutex> lk(mu_);
        live_.emplace(p, bytes);
        *out = p;
        return hipSuccess;
    } catch (...) {
        if (p) (void)hipFree(p);
        return hipErrorOutOfMemory;
    }
}

void graph_pool::put(void* p) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(mu_);
    const auto it = live_.find(p);
    if (it == live_.end()) return;
    const uint64_t bytes = it->second;
    live_.erase(it);
    if (bytes <= keep_) {
        try {
            free_.push_back(block{p, bytes});
            held_ += bytes;
            shrink(keep_);
            return;
        } catch (...) {
        }
    }
    (void)hipFree(p);
}

hipError_t space_reserve(build_space* sp, uint64_t bytes, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (!sp->host) e = hipHostMalloc((void**)&sp->host, sizeof(uint64_t) * kSpaceHostWords);
    if (e == hipSuccess && bytes > sp->cap) {
        (void)hipStreamSynchronize(s);
        if (sp->base) (void)hipFree(sp->base);
        sp->base = nullptr;
        sp->cap = 0;
        e = device_alloc(&sp->base, bytes);
        if (e == hipSuccess) sp->cap = bytes;
    }
    return e;
}

void space_trim(build_space* sp, uint64_t keep, hipStream_t s) {
    if (sp->cap <= keep) return;
    (void)hipStreamSynchronize(s);
    (void)hipFree(sp->base);
    sp->base = nullptr;
    sp->cap = 0;
}

namespace {

hipError_t stage_reserve(build_space* sp) {
    hipError_t e = hipSuccess;
    if (!sp->stage) e = hipHostMalloc((void**)&sp->stage, 2 * kStageThreads * kStageChunk);
    for (int k = 0; k < 2 * kStageThreads && e == hipSuccess; ++k)
        if (!sp->stage_ev[k]) e = hipEventCreateWithFlags(&sp->stage_ev[k], hipEventDisableTiming);
    return e;
}

// Copies bytes [begin, end) of `from` to `to` on stream s through the two
// chunks of thread t.
hipError_t stage_range(build_space* sp, int device, int t, const char* from, char* to, uint64_t begin, uint64_t end,
                       hipStream_t s) {
    hipError_t e = hipSetDevice(device);
    for (uint64_t b = begin, k = 0; b < end && e == hipSuccess; b += kStageChunk, ++k) {
        const uint64_t len = std::min(kStageChunk, end - b);
        const int c = 2 * t + (int)(k & 1);
        char* chunk = sp->stage + (uint64_t)c * kStageChunk;
        e = hipEventSynchronize(sp->stage_ev[c]);   // (an event never recorded has ended)
        if (e != hipSuccess) break;
        std::memcpy(chunk, from + b, len);
        e = hipMemcpyAsync(to + b, chunk, len, hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipEventRecord(sp->stage_ev[c], s);
    }
    return e;
}

// Host bytes to device memory on stream s; the source is not read after the
// return.  Arrays of 16 MiB or more are copied by kStageThreads threads, since
// one thread's copy into the chunks is slower than the bus.
hipError_t stage_copy(build_space* sp, const void* from, void* to, uint64_t bytes, hipStream_t s) {
    hipError_t e = stage_reserve(sp);
    int device = 0;
    if (e == hipSuccess) e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const char* f = (const char*)from;
    char* d = (char*)to;
    if (bytes < (16ull << 20)) return stage_range(sp, device, 0, f, d, 0, bytes, s);
    const uint64_t part = ((bytes + kStageThreads - 1) / kStageThreads + 255) & ~255ull;
    hipError_t got[kStageThreads];
    std::thread th[kStageThreads];
    for (int t = 1; t < kStageThreads; ++t) {
        const uint64_t b = std::min(bytes, part * t), n = std::min(bytes, part * (t + 1));
        try {
            th[t] = std::thread([=, &got] { got[t] = stage_range(sp, device, t, f, d, b, n, s); });
        } catch (...) {
            got[t] = stage_range(sp, device, t, f, d, b, n, s);
        }
    }
    got[0] = stage_range(sp, device, 0, f, d, 0, std::min(bytes, part), s);
    for (int t = 1; t < kStageThreads; ++t)
        if (th[t].joinable()) th[t].join();
    for (int t = 0; t < kStageThreads; ++t)
        if (got[t] != hipSuccess) e = got[t];
    return e;
}

}  // namespace

void space_free(build_space* sp) {
    if (sp->pool) sp->pool->remove(sp);
    sp->pool = nullptr;
    if (sp->stage) (void)hipHostFree(sp->stage);
    for (hipEvent_t& ev : sp->stage_ev) {
        if (ev) (void)hipEventDestroy(ev);
        ev = nullptr;
    }
    if (sp->base) (void)hipFree(sp->base);
    if (sp->host) (void)hipHostFree(sp->host);
    sp->stage = nullptr;
    sp->base = nullptr;
    sp->host = nullptr;
    sp->cap = 0;
}

namespace {

// Exclusive scan of in[0..count) to out (they may be one array); *total (device
// memory, 64-bit scans only) receives the sum.  Up to kScanDirect values are
// scanned by one workgroup in one launch.
constexpr uint64_t kScanDirect = 16384;
template <class T>
hipError_t scan_exclusive(const T* in, T* out, uint64_t count, T* total, arena& ar, hipStream_t s) {
    static_assert(sizeof(T) == 8 || sizeof(T) == 4, "32- or 64-bit scans");
    if (sizeof(T) == 4 && total) return hipErrorInvalidValue;
    if (count <= kScanDirect) {
        hipLaunchKernelGGL(k_scan_spine<T>, dim3(1), dim3(kSpineT), 0, s, in, out, count, total);
        return hipGetLastError();
    }
    const uint32_t nb = blocks_for(count);
    const size_t mark = ar.mark();
    uint64_t* sums = ar.take<uint64_t>(nb);
    if (!sums) return hipErrorOutOfMemory;
    hipLaunchKernelGGL(k_scan_reduce<T>, dim3(nb), dim3(kT), 0, s, in, count, sums);
    hipLaunchKernelGGL(k_scan_spine<uint64_t>, dim3(1), dim3(kSpineT), 0, s, (const uint64_t*)sums, sums, (uint64_t)nb,
                       (uint64_t*)total);
    hipLaunchKernelGGL(k_scan_apply<T>, dim3(nb), dim3(kT), 0, s, in, out, count, (const uint64_t*)sums);
    ar.rewind(mark);
    return hipGetLastError();
}

template <class O, int I>
hipError_t radix_pass(const uint64_t* in, uint64_t* out, uint64_t count, uint32_t shift, uint32_t dbits, O* hist,
                      arena& ar, hipStream_t s) {
    const uint32_t nb = (uint32_t)sort_tiles(count), nbins = 1u << dbits;
    hipLaunchKernelGGL((k_radix_hist<O, I>), dim3(nb), dim3(kT), 0, s, in, count, shift, nbins, hist, nb);
    hipError_t e = scan_exclusive<O>(hist, hist, (uint64_t)nbins * nb, nullptr, ar, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_radix_scatter<O, I>), dim3(nb), dim3(kT), 0, s, in, out, count, shift, dbits, (const O*)hist, nb);
    return hipGetLastError();
}

// Sorts `count` keys on bits [first, first + sort_bits); result in *keys (buffers swapped as needed).
hipError_t radix_sort(uint64_t** keys, uint64_t** tmp, uint64_t count, uint32_t first, uint32_t sort_bits, arena& ar,
                      hipStream_t s) {
    if (count <= 1 || sort_bits == 0) return hipSuccess;
    const uint32_t dbits = sort_digit_bits(sort_bits);
    const size_t mark = ar.mark();
    const uint64_t words = (1ull << dbits) * sort_tiles(count);
    const bool wide = count >= (1ull << 32);
    void* hist = wide ? (void*)ar.take<uint64_t>(words) : (void*)ar.take<uint32_t>(words);
    if (!hist) return hipErrorOutOfMemory;
    hipError_t e = hipSuccess;
    for (uint32_t done = 0; done < sort_bits && e == hipSuccess; done += dbits) {
        const uint32_t b = std::min(dbits, sort_bits - done);
        if (wide) e = radix_pass<uint64_t, kSortI>(*keys, *tmp, count, first + done, b, (uint64_t*)hist, ar, s);
        else if (sort_items(count) == kSortI)
            e = radix_pass<uint32_t, kSortI>(*keys, *tmp, count, first + done, b, (uint32_t*)hist, ar, s);
        else e = radix_pass<uint32_t, kSortISmall>(*keys, *tmp, count, first + done, b, (uint32_t*)hist, ar, s);
        std::swap(*keys, *tmp);
    }
    ar.rewind(mark);
    return e;
}

uint32_t bit_width_u32(uint32_t x) {
    uint32_t b = 0;
    while (x) { ++b; x >>= 1; }
    return b;
}

hipError_t bucket_all(device_graph* g, const bucket_params& bp, const uint32_t* deg, const uint2* rows, bool fresh,
                      build_space* sp, arena& ar, hipStream_t s);

}  // namespace

#define TRY(x) do { hipError_t _e = (x); if (_e != hipSuccess) { err = _e; goto done; } } while (0)
#define TAKE(p, T, count) do { p = ar.take<T>(count); if (!p) { err = hipErrorOutOfMemory; goto done; } } while (0)

build_status build_graph_device(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, bool host_arcs,
                                const bucket_params& bp, graph_pool* pool, hipStream_t s, build_space* sp,
                                device_graph* g) {
    build_status st{};
    hipError_t err = hipSuccess;
    // ids below 2^bits; the sentinel key is a loop of id 2^bits - 1
    const uint32_t bits = id_bits((uint64_t)n);
    const uint64_t keys_n = 2ull * (uint64_t)m;
    *g = device_graph{};
    g->n = n;
    g->mem = pool;
    const uint64_t need = build_space_bytes((uint64_t)n, (uint64_t)m, bits, bp.tri != 0);
    if ((err = space_reserve(sp, need, s)) != hipSuccess) {
        st.hip = err;
        return st;
    }
    arena ar(*sp);
    unsigned long long* counters = nullptr;
    uint32_t* deg = nullptr;
    uint2* rows = nullptr;
    uint64_t *keys = nullptr, *tmp = nullptr, *ents = nullptr, *types = nullptr, U = 0, total_types = 0;
    const uint64_t tiles = (keys_n + kTile - 1) / kTile;
    size_t mark = 0;
    TAKE(counters, unsigned long long, kCounters);
    TAKE(deg, uint32_t, (uint64_t)n + 1);
    TAKE(rows, uint2, (uint64_t)n + 1);
    mark = ar.mark();
    TRY(fill_u64((uint64_t*)counters, kCounters, 0, s));
    if (keys_n > 0) {
        TAKE(keys, uint64_t, keys_n);
        TAKE(tmp, uint64_t, keys_n);
        TAKE(ents, uint64_t, tiles);
        TAKE(types, uint64_t, tiles);
        if (host_arcs) {   // the second key buffer holds the arcs until the first sort pass
            int32_t* a = (int32_t*)tmp;
            TRY(stage_copy(sp, src, a, sizeof(int32_t) * (uint64_t)m, s));
            TRY(stage_copy(sp, dst, a + m, sizeof(int32_t) * (uint64_t)m, s));
            src = a;
            dst = a + m;
        }
        hipLaunchKernelGGL(k_canon, dim3((uint32_t)std::min<uint64_t>(((uint64_t)m + kT - 1) / kT, kStatBlocks)), dim3(kT),
                           0, s, src, dst, (uint64_t)m, n, bits, keys, counters);
        TRY(hipGetLastError());
        TRY(radix_sort(&keys, &tmp, keys_n, 2, 2 * bits, ar, s));
        hipLaunchKernelGGL(k_runs_count, dim3((uint32_t)tiles), dim3(kT), 0, s, keys, keys_n, bits, ents, types);
        hipLaunchKernelGGL(k_runs_spine, dim3(1), dim3(1024), 0, s, ents, types, tiles, counters, sp->host);
        TRY(hipGetLastError());
        TRY(hipStreamSynchronize(s));
        U = sp->host[0];
        total_types = sp->host[1];
        st.bad_ids = (int64_t)sp->host[2];
        st.self_loops = (int64_t)sp->host[3];
        if (st.bad_ids) goto done;
    }
    if (U >= (1ull << 32)) { st.too_large = true; goto done; }
    g->U = U;
    g->p = U / 2;
    g->mutual = (total_types & 0xffffffffull) - U / 2;   // a mutual pair holds two arcs
    st.arcs_kept = (int64_t)(total_types & 0xffffffffull);
    st.duplicates = m - st.self_loops - st.arcs_kept;
    TRY(g->mem->alloc((void**)&g->row_ptr, sizeof(int64_t) * ((size_t)n + 1)));
    TRY(g->mem->alloc((void**)&g->nbr, sizeof(uint32_t) * (U + kRowPad)));
    TRY(g->mem->alloc((void**)&g->owner, sizeof(uint32_t) * (U ? U : 1)));
    TRY(g->mem->alloc((void**)&g->tpre, sizeof(uint64_t) * (U + 1)));
    TRY(g->mem->alloc((void**)&g->rinfo, sizeof(uint4) * ((size_t)n + 1)));
    if (U > 0) {
        hipLaunchKernelGGL(k_runs_emit, dim3((uint32_t)tiles), dim3(kT), 0, s, keys, keys_n, bits, ents, types, U,
                           total_types, n, g->nbr, g->owner, g->tpre, g->row_ptr);
    } else {
        TRY(fill_u64((uint64_t*)g->row_ptr, (uint64_t)n + 1, 0, s));
        TRY(fill_u64(g->tpre, 1, 0, s));
    }
    if (n > 0)
        hipLaunchKernelGGL(k_row_info, dim3(std::min(grid1((uint64_t)n), kStatBlocks)), dim3(kT), 0, s,
                           (const int64_t*)g->row_ptr, n, (const uint64_t*)g->tpre, g->rinfo, deg, rows, counters);
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, (const uint64_t*)counters + 3, sp->host + kSpaceHostStats, 2);
    TRY(hipGetLastError());
    ar.rewind(mark);   // (the keys are read by then, in stream order)
    TRY(bucket_all(g, bp, deg, rows, true, sp, ar, s));
    st.sum_d2 = sp->host[kSpaceHostStats];
    st.max_degree = (int64_t)g->max_degree;
    st.ok = true;
done:
    (void)hipStreamSynchronize(s);
    st.hip = err;
    if (!st.ok) free_device_graph(g);
    return st;
}

namespace {

// Cuts the hub records of each anchor ([first, past) inside the hub bucket)
// into tasks of at most `chunk` records, anchors whose rows span several LDS
// tiles first, and the tasks into groups (k_hub_group).  *staged_out: the
// sum over the tasks of the anchor-row length.
hipError_t cut_hub_tasks(const uint32_t* first, const uint32_t* past, int32_t n, const uint32_t* len,
                         uint64_t hub_begin, const dyad_rec* recs, const bucket_params& bp, uint32_t chunk,
                         graph_pool* mem, build_space* sp, arena& ar, hipStream_t s, hub_task** tasks_out, uint32_t* ntasks_out,
                         uint32_t* ngroups_out, uint64_t* staged_out) {
    hipError_t err = hipSuccess;
    const size_t mark = ar.mark();
    uint64_t *task_off = nullptr, *gcount = nullptr;
    unsigned long long* staged = nullptr;
    hub_task* tasks = nullptr;
    uint64_t ntasks = 0, windows = 0;
    const uint32_t stat_grid = std::min(grid1((uint64_t)n), kStatBlocks);
    TAKE(task_off, uint64_t, (uint64_t)n + 1);
    TAKE(staged, unsigned long long, 1);
    TRY(fill_u64((uint64_t*)staged, 1, 0, s));
    hipLaunchKernelGGL(k_hub_ntasks, dim3(stat_grid), dim3(kT), 0, s, first, past, n, len, task_off, bp.hub_tile, chunk,
                       staged);
    TRY(scan_exclusive<uint64_t>(task_off, task_off, (uint64_t)n, task_off + n, ar, s));
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, (const uint64_t*)task_off + n, sp->host, 1);
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, (const uint64_t*)staged, sp->host + 1, 1);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(s));
    ntasks = (sp->host[0] >> 32) + (sp->host[0] & 0xffffffffull);
    *staged_out = sp->host[1];
    TRY(mem->alloc((void**)&tasks, sizeof(hub_task) * (ntasks ? ntasks : 1)));
    hipLaunchKernelGGL(k_hub_emit, dim3(grid1((uint64_t)n)), dim3(kT), 0, s, first, past, n, len,
                       (const uint64_t*)task_off, bp.hub_tile, chunk, hub_begin, tasks);
    windows = (ntasks + kHubGroupTasks - 1) / kHubGroupTasks;
    TAKE(gcount, uint64_t, windows + 1);
    hipLaunchKernelGGL(k_hub_group, dim3(grid1(windows)), dim3(kT), 0, s, tasks, recs, ntasks,
                       (const uint64_t*)nullptr, gcount, bp.hub_tile, chunk);
    TRY(scan_exclusive<uint64_t>(gcount, gcount, windows, gcount + windows, ar, s));
    hipLaunchKernelGGL(k_hub_group, dim3(grid1(windows)), dim3(kT), 0, s, tasks, recs, ntasks,
                       (const uint64_t*)gcount, (uint64_t*)nullptr, bp.hub_tile, chunk);
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, (const uint64_t*)gcount + windows, sp->host, 1);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(s));
    *tasks_out = tasks;
    tasks = nullptr;
    *ntasks_out = (uint32_t)ntasks;
    *ngroups_out = (uint32_t)sp->host[0];
done:
    if (tasks) (void)hipStreamSynchronize(s);   // (an error: what was launched may still write them)
    mem->put(tasks);
    ar.rewind(mark);
    return err;
}

// Gives up g's dyad records (nothing on the device uses them).
void drop_dyads(device_graph* g) {
    g->mem->put(g->dyads);
    g->mem->put(g->hub_tasks);
    g->dyads = nullptr;
    g->hub_tasks = nullptr;
    g->n_hub_tasks = 0;
    g->n_hub_groups = 0;
    g->hub_stream = 0;
    g->hub_staged = 0;
    for (uint64_t& o : g->bucket_off) o = 0;
    for (uint64_t& c : g->bucket_cost) c = 0;
}

// The dyad view: records of g's canonical dyads by bucket, hub tasks and the
// per-bucket sums.  deg: the rows' lengths.
hipError_t bucket_dyad_records(device_graph* g, const bucket_params& bp, const uint32_t* deg, const uint2* rows,
                               build_space* sp, arena& ar, hipStream_t s) {
    hipError_t err = hipSuccess;
    const size_t mark = ar.mark();
    const uint64_t U = g->U;
    const int32_t n = g->n;
    graph_pool* mem = g->mem;
    uint64_t *counts = nullptr, *part = nullptr;
    uint32_t *first = nullptr, *past = nullptr, *anchors = nullptr;
    uint8_t* bucket = nullptr;
    uint64_t hubs = 0;
    const uint32_t nb = blocks_for(U ? U : 1);
    drop_dyads(g);
    TAKE(counts, uint64_t, (uint64_t)kBuckets * nb + 1);
    TAKE(part, uint64_t, (uint64_t)kPartWords * nb);
    TAKE(bucket, uint8_t, U);
    hipLaunchKernelGGL(k_dyad_count, dim3(nb), dim3(kT), 0, s, g->nbr, g->owner, deg, U, bp, counts, nb, part, bucket);
    TRY(scan_exclusive<uint64_t>(counts, counts, (uint64_t)kBuckets * nb, counts + (uint64_t)kBuckets * nb, ar, s));
    hipLaunchKernelGGL(k_bucket_sums, dim3(kPartWords + 1), dim3(kT), 0, s, (const uint64_t*)part,
                       (const uint64_t*)counts, nb, sp->host);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(s));
    for (int b = 0; b <= kBuckets; ++b) g->bucket_off[b] = sp->host[b];
    for (int b = 0; b < kBuckets; ++b) g->bucket_cost[b] = sp->host[kBuckets + 1 + b];
    g->hub_stream = sp->host[2 * kBuckets + 1];
    hubs = g->bucket_off[kBucketHub + 1] - g->bucket_off[kBucketHub];
    TRY(mem->alloc((void**)&g->dyads, sizeof(dyad_rec) * (g->p ? g->p : 1)));
    if (hubs > 0) {
        // (an even number of words each, so that they can be cleared 8 bytes at a time)
        TAKE(first, uint32_t, ((uint64_t)n + 2) & ~1ull);
        TAKE(past, uint32_t, ((uint64_t)n + 2) & ~1ull);
        TAKE(anchors, uint32_t, hubs);
        TRY(fill_u64((uint64_t*)first, ((uint64_t)n + 2) / 2, 0, s));
        TRY(fill_u64((uint64_t*)past, ((uint64_t)n + 2) / 2, 0, s));
    }
    if (g->p > 0) {
        hipLaunchKernelGGL(k_dyad_scatter, dim3(nb), dim3(kT), 0, s, g->nbr, g->owner, rows, U,
                           (const uint8_t*)bucket, (const uint64_t*)counts, nb, g->bucket_off[kBucketHub], anchors, g->dyads);
        TRY(hipGetLastError());
    }
    if (hubs > 0) {
        hipLaunchKernelGGL(k_hub_runs, dim3(grid1(hubs)), dim3(kT), 0, s, (const uint32_t*)anchors, (uint32_t)hubs, first,
                           past);
        TRY(cut_hub_tasks(first, past, n, deg, g->bucket_off[kBucketHub], g->dyads, bp, kHubChunk, mem, sp, ar, s,
                          &g->hub_tasks, &g->n_hub_tasks, &g->n_hub_groups, &g->hub_staged));
    }
done:
    ar.rewind(mark);
    return err;
}

void free_forward(graph_pool* mem, forward_lists* t) {
    mem->put(t->fwd);
    mem->put(t->fptr);
    mem->put(t->edges.recs);
    mem->put(t->edges.tasks);
    *t = forward_lists{};
}

constexpr uint32_t hub_key_bits = 64;

// Forward lists of g (degree order), their edge records and hub tasks.
hipError_t build_forward(device_graph* g, const bucket_params& bp, const uint32_t* deg, build_space* sp, arena& ar,
                         hipStream_t s) {
    hipError_t err = hipSuccess;
    const size_t mark = ar.mark();
    const uint64_t U = g->U, F = U / 2;   // every joined pair is in one forward list
    const int32_t n = g->n;
    const uint32_t bits = id_bits((uint64_t)n);
    graph_pool* mem = g->mem;
    forward_lists& t = g->tri;
    auto& out = t.edges;
    uint64_t *vk = nullptr, *vt = nullptr, *keys = nullptr, *tmp = nullptr, *hk = nullptr, *counts = nullptr,
             *part = nullptr, *task_off = nullptr;
    uint32_t *rank = nullptr, *first = nullptr, *past = nullptr;
    unsigned long long *staged = nullptr, *counter = nullptr;
    uint64_t hubs = 0, total = 0;
    hub_key hkey{0, 0};
    size_t inner = 0;
    const uint32_t nb = blocks_for(F ? F : 1);
    t.entries = F;
    TRY(mem->alloc((void**)&t.fptr, sizeof(uint32_t) * ((size_t)n + 1)));
    TRY(mem->alloc((void**)&t.fwd, sizeof(uint32_t) * (F + kRowPad)));
    out.chunk = kHubChunk;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid1((uint64_t)n + 1)), dim3(kT), 0, s, t.fptr, (uint64_t)n + 1, (uint32_t)F);
    TRY(hipGetLastError());
    if (F == 0) {
        TRY(mem->alloc((void**)&out.recs, sizeof(uint4)));
        goto done;
    }
    TAKE(rank, uint32_t, n);
    TAKE(keys, uint64_t, F);
    TAKE(tmp, uint64_t, F);
    inner = ar.mark();
    TAKE(vk, uint64_t, n);
    TAKE(vt, uint64_t, n);
    hipLaunchKernelGGL(k_vertex_keys, dim3(grid1((uint64_t)n)), dim3(kT), 0, s, deg, n, g->max_degree, vk);
    TRY(radix_sort(&vk, &vt, (uint64_t)n, 32, bit_width_u32(g->max_degree), ar, s));
    hipLaunchKernelGGL(k_ranks, dim3(grid1((uint64_t)n)), dim3(kT), 0, s, (const uint64_t*)vk, n, rank);
    TRY(hipGetLastError());
    ar.rewind(inner);
    TAKE(counter, unsigned long long, 1);
    TRY(fill_u64((uint64_t*)counter, 1, 0, s));
    hipLaunchKernelGGL(k_pair_keys, dim3((uint32_t)((U + kPairTile - 1) / kPairTile)), dim3(kPairT), 0, s, g->nbr, g->owner,
                       (const uint32_t*)rank, U, bits, counter, keys);
    TRY(hipGetLastError());
    TRY(radix_sort(&keys, &tmp, F, 3, 2 * bits, ar, s));
    hipLaunchKernelGGL(k_fwd_emit, dim3(blocks_for(F)), dim3(kT), 0, s, (const uint64_t*)keys, F, bits, t.fwd, t.fptr);
    TAKE(counts, uint64_t, (uint64_t)kBuckets * nb + 1);
    TAKE(part, uint64_t, (uint64_t)kPartWords * nb);
    hipLaunchKernelGGL(k_edge_count, dim3(nb), dim3(kT), 0, s, (const uint64_t*)keys, F, bits, (const uint32_t*)t.fptr,
                       bp, counts, nb, part);
    TRY(scan_exclusive<uint64_t>(counts, counts, (uint64_t)kBuckets * nb, counts + (uint64_t)kBuckets * nb, ar, s));
    hipLaunchKernelGGL(k_bucket_sums, dim3(kPartWords + 1), dim3(kT), 0, s, (const uint64_t*)part,
                       (const uint64_t*)counts, nb, sp->host);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(s));
    for (int b = 0; b <= kBuckets; ++b) out.off[b] = sp->host[b];
    for (int b = 0; b < kBuckets; ++b) out.cost[b] = sp->host[kBuckets + 1 + b];
    out.stream = sp->host[2 * kBuckets + 1];
    total = out.off[kBuckets];
    hubs = out.off[kBucketHub + 1] - out.off[kBucketHub];
    out.chunk = hubs >= kHubSplitRecords ? kHubChunk / 2 : hubs >= kHubSmallRecords ? 64 : kHubChunk;
    TRY(mem->alloc((void**)&out.recs, sizeof(uint4) * (total ? total : 1)));
    if (total == 0) goto done;
    hkey.ibits = bit_width_u32((uint32_t)F);
    hkey.pbits = bit_width_u32((uint32_t)std::sqrt(2.0 * (double)F) + 1u);
    if (bits + hkey.ibits + hkey.pbits + 4 > hub_key_bits) hkey.pbits = 0;
    // (the second key buffer is free: it takes the hub keys)
    hipLaunchKernelGGL(k_edge_scatter, dim3(nb), dim3(kT), 0, s, keys, F, bits,
                       (const uint32_t*)t.fptr, bp, (const uint64_t*)counts, nb, out.off[kBucketHub], hkey,
                       (const uint32_t*)t.fwd, tmp, out.recs);
    TRY(hipGetLastError());
    if (hubs == 0) goto done;
    TAKE(hk, uint64_t, hubs);
    TAKE(first, uint32_t, ((uint64_t)n + 2) & ~1ull);
    TAKE(past, uint32_t, ((uint64_t)n + 2) & ~1ull);
    TAKE(task_off, uint64_t, (uint64_t)n + 1);
    TAKE(staged, unsigned long long, 2);
    TRY(fill_u64((uint64_t*)first, ((uint64_t)n + 2) / 2, 0, s));
    TRY(fill_u64((uint64_t*)past, ((uint64_t)n + 2) / 2, 0, s));
    TRY(fill_u64((uint64_t*)staged, 2, 0, s));
    TRY(radix_sort(&tmp, &hk, hubs, hkey.y_shift(), bits, ar, s));
    hipLaunchKernelGGL(k_edge_hub, dim3(blocks_for(hubs)), dim3(kT), 0, s, (const uint64_t*)tmp, hubs, hkey,
                       (const uint64_t*)keys, (const uint32_t*)t.fwd, (const uint32_t*)t.fptr, bits, first, past,
                       out.recs + out.off[kBucketHub]);
    hipLaunchKernelGGL(k_tri_ntasks, dim3(std::min(grid1((uint64_t)n), kStatBlocks)), dim3(kT), 0, s,
                       (const uint32_t*)first, (const uint32_t*)past, n, (const uint32_t*)t.fptr, out.chunk, task_off,
                       staged);
    TRY(scan_exclusive<uint64_t>(task_off, task_off, (uint64_t)n, task_off + n, ar, s));
    hipLaunchKernelGGL(k_tri_publish, dim3(1), dim3(64), 0, s, (const uint64_t*)task_off, n,
                       (const unsigned long long*)staged, sp->host);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(s));
    out.n_heavy = (uint32_t)sp->host[2];
    out.n_tasks = (uint32_t)sp->host[0];
    out.n_groups = out.n_tasks;
    out.staged = sp->host[1];
    TRY(mem->alloc((void**)&out.tasks, sizeof(tri_task) * (out.n_tasks ? out.n_tasks : 1)));
    hipLaunchKernelGGL(k_tri_tasks, dim3(grid1((uint64_t)n)), dim3(kT), 0, s, (const uint32_t*)first,
                       (const uint32_t*)past, n, (const uint32_t*)t.fptr, out.chunk, (const uint64_t*)task_off,
                       (uint32_t)out.off[kBucketHub], out.tasks);
    TRY(hipGetLastError());
done:
    ar.rewind(mark);
    return err;
}

// Both views of g.  `fresh`: the largest degree is on its way to the host, and
// there once the dyad records' synchronisation has passed.  The old records
// are given up before the new ones are built (there may not be room for both),
// so an error leaves g without the view that failed: no null pointer with a
// count beside it, and `bucketed` false, so that the next rebucket builds.
hipError_t bucket_all(device_graph* g, const bucket_params& bp, const uint32_t* deg, const uint2* rows, bool fresh,
                      build_space* sp, arena& ar, hipStream_t s) {
    g->bucketed = false;
    hipError_t err = bp.dyads ? bucket_dyad_records(g, bp, deg, rows, sp, ar, s) : hipStreamSynchronize(s);
    if (err != hipSuccess) {
        (void)hipStreamSynchronize(s);
        drop_dyads(g);
        return err;
    }
    if (fresh) g->max_degree = (uint32_t)sp->host[kSpaceHostStats + 1];
    g->bp = bp;
    free_forward(g->mem, &g->tri);
    if (bp.tri) err = build_forward(g, bp, deg, sp, ar, s);
    if (err != hipSuccess) {
        (void)hipStreamSynchronize(s);
        free_forward(g->mem, &g->tri);
        return err;
    }
    g->bucketed = true;
    return hipSuccess;
}

}  // namespace

#undef TAKE
#undef TRY

hipError_t bucket_dyads(device_graph* g, const bucket_params& bp, hipStream_t s, build_space* sp) {
    hipError_t e = space_reserve(sp, 4096 + (sizeof(uint32_t) + sizeof(uint2)) * ((uint64_t)g->n + 1) +
                                     view_space_bytes(g->U, (uint64_t)g->n, bp.tri != 0), s);
    if (e != hipSuccess) return e;
    arena ar(*sp);
    uint32_t* deg = ar.take<uint32_t>((uint64_t)g->n + 1);
    uint2* rows = ar.take<uint2>((uint64_t)g->n + 1);
    if (!deg || !rows) return hipErrorOutOfMemory;
    if (g->n > 0) {
        hipLaunchKernelGGL(k_row_len, dim3(grid1((uint64_t)g->n)), dim3(kT), 0, s, (const int64_t*)g->row_ptr, g->n, deg,
                           rows);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = bucket_all(g, bp, deg, rows, false, sp, ar, s);
    (void)hipStreamSynchronize(s);
    return e;
}

void free_device_graph(device_graph* g) {
    graph_pool* mem = g->mem;
    const int32_t n = g->n;
    if (!mem) return;   // nothing was allocated
    free_forward(mem, &g->tri);
    mem->put(g->row_ptr);
    mem->put(g->nbr);
    mem->put(g->owner);
    mem->put(g->tpre);
    mem->put(g->rinfo);
    mem->put(g->dyads);
    mem->put(g->hub_tasks);
    *g = device_graph{};
    g->n = n;
}

uint64_t device_graph_bytes(const device_graph& g) {
    uint64_t b = sizeof(int64_t) * ((uint64_t)g.n + 1) + (sizeof(uint32_t) * 2 + sizeof(uint64_t)) * g.U +
                 sizeof(uint32_t) * kRowPad + sizeof(uint4) * ((uint64_t)g.n + 1) +
                 sizeof(uint64_t) + sizeof(dyad_rec) * (g.dyads ? g.p : 0) + sizeof(hub_task) * (uint64_t)g.n_hub_tasks;
    if (g.tri.fptr)
        b += sizeof(uint32_t) * ((uint64_t)g.n + 1 + g.tri.entries + kRowPad) +
             sizeof(uint4) * g.tri.edges.off[kBuckets] + sizeof(tri_task) * (uint64_t)g.tri.edges.n_tasks;
    return b;
}

}  // namespace tc
