// Census kernels: one canonical dyad (u, v), u < v, per task, following the
// subquadratic census (section "Triad Census Algorithm", figure "Subquadratic
// Triad Census Algorithm") with the pre-computed dyad type of the v0.4 change.
//
// Per dyad with f = IsEdge(u,v) + 2 IsEdge(v,u):
//   * dyadic triads:  n - |S| - 2 = n - |N(u)| - |N(v)| + |N(u) ^ N(v)| go to
//     class 102 if f == 3, else 012;
//   * a third vertex w in S is counted (the canonical condition
//     v < w  or  (u < w < v and w not adjacent to u)) exactly when
//       w in N(u) and w > v            (code f | f_uw << 2 | f_vw << 4), or
//       w in N(v) \ N(u) and w > u     (code f | f_vw << 4);
//   * classes come from the 64 -> 16 table.
// Non-shared third vertices never need to be visited one by one: the number
// of entries of each direction type in a row range is a difference of the
// row's prefix counts (tpre), so a dyad adds those totals once and the merge of
// N(u) and N(v) only has to find the shared vertices, each of which moves one
// count from its single-list class to its full-code class.
//
// Four execution modes over the buckets (key |N(u)| + |N(v)| - 2, and the
// longer row for the hub bucket):
//   lane  : one lane per record, the two rows compared 8 entries at a time;
//   wave  : one 64-lane wavefront per record, merge path over LDS-staged tiles;
//   group : one 256-lane workgroup per record, merge path over larger tiles;
//   hub   : one workgroup per group of runs of records that share an
//           endpoint (anchor), whose rows are staged in an LDS hash table and
//           probed by the other rows.
// These run over the dyad records.  The forward-list path has kernels of the
// same four modes over its edge records (k_tri_*, tc_tri.h), where a shared
// vertex closes a triangle that is credited to its three dyads (on_triangle),
// and the terms without intersection come from a pass over the rows
// (k_census_rows) or, labelled, over the entries (k_census_totals).  Most
// censuses on that path are one launch of all of them (k_tri_one).
// Counts accumulate in LDS bins (per lane, per wavefront, or per signature in
// the hub mode); each workgroup adds its 16 sums to the graph's accumulators
// with one 64-bit global atomic per class when it finishes.
//
// The class of every code comes from a 64-entry table staged in LDS.  The
// single-graph kernels take the table as an argument: the 16-class table; for
// the labelled (64-class) census on the forward-list path a table that keeps all
// codes apart, over the dyad records one of three pass tables that send the codes
// whose (u, v) part is f to bin (code >> 2) and every other code to the discard
// bin (index kNumClasses), which is never flushed.
#include "tc_census.h"
#include "tc_tri.h"

namespace tc {

namespace {

__constant__ uint8_t c_table[64];

constexpr int kBins = kNumClasses + 1;     // 16 classes and the discard bin (kNumClasses)

// ---- class histograms in LDS ------------------------------------------------
// wave_bins: one row per wavefront updated with LDS atomics (shared neighbours
// are rare next to the work that finds them).
// block_bins: one row shared by the workgroup (LDS atomics; used where updates
// are rare next to the work that produces them).
template <int B>
struct block_bins {
    static constexpr int kWords = kBins;
    unsigned long long* bins;
    __device__ inline void add(uint32_t cls, unsigned long long x) { atomicAdd(&bins[cls], x); }
    __device__ inline void clear() {
        for (int i = threadIdx.x; i < kWords; i += B) bins[i] = 0;
    }
    __device__ inline void flush(unsigned long long* acc) {
        __syncthreads();
        if (threadIdx.x < kNumClasses && bins[threadIdx.x] != 0) atomicAdd(&acc[threadIdx.x], bins[threadIdx.x]);
    }
};

// The forward-list kernels' bins: 16 classes or 64 codes, one row per workgroup.
template <bool Lab>
struct tri_bins {
    static constexpr uint32_t kWords = Lab ? 64 : kNumClasses;
    unsigned long long* bins;
    __device__ inline void add(uint32_t bin, unsigned long long x) { atomicAdd(&bins[bin], x); }
};

template <int B>
struct wave_bins {
    static constexpr int kWords = kBins * (B / 64);
    unsigned long long* bins;
    __device__ inline void add(uint32_t cls, unsigned long long x) {
        atomicAdd(&bins[(threadIdx.x >> 6) * kBins + cls], x);
    }
    __device__ inline void clear() {
        for (int i = threadIdx.x; i < kWords; i += B) bins[i] = 0;
    }
    __device__ inline void flush(unsigned long long* acc) {
        __syncthreads();
        if (threadIdx.x < kNumClasses) {
            unsigned long long s = 0;
            for (int w = 0; w < B / 64; ++w) s += bins[w * kBins + threadIdx.x];
            if (s != 0) atomicAdd(&acc[threadIdx.x], s);
        }
    }
};

// First position in [lo, hi) of a sorted row whose vertex is >= w.
__device__ inline uint32_t find_first_ge(const uint32_t* __restrict__ nbr, uint32_t lo, uint32_t hi, uint32_t w) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if ((nbr[mid] >> 2) < w) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// A vertex w adjacent to both u (entry flags fa) and v (flags fb).
template <class H>
__device__ inline void on_common(uint32_t w, uint32_t fa, uint32_t fb, uint32_t u, uint32_t v, uint32_t f,
                                 const uint8_t* T, H& h) {
    h.add(T[f], 1ull);                                    // |S| is one smaller
    if (w > v) {                                          // counted with its full code
        h.add(T[f | (fa << 2) | (fb << 4)], 1ull);
        h.add(T[f | (fa << 2)], ~0ull);                   // not a u-only vertex
    }
    if (w > u) h.add(T[f | (fb << 4)], ~0ull);            // not a v-only vertex
}

// The copy of the accumulators (16, or 64 for the labelled census) this
// workgroup adds to.
__device__ inline unsigned long long* acc_copy(unsigned long long* acc, uint32_t words = kNumClasses) {
    return acc + words * (blockIdx.x % kAccCopies);
}

__device__ inline uint32_t swap_dir(uint32_t f) { return ((f & 1u) << 1) | (f >> 1); }

// A triangle {u, v, w}, u < v, found once (from the forward lists of its two
// first vertices in degree order): w is a shared vertex of each of its three
// dyads.  f = f_uv relative to u, fa = f_uw relative to u, fb = f_vw relative
// to v.
template <class H>
__device__ inline void on_triangle(uint32_t w, uint32_t fa, uint32_t fb, uint32_t u, uint32_t v, uint32_t f,
                                   const uint8_t* T, H& h) {
    const uint32_t sa = swap_dir(fa), sb = swap_dir(fb), sf = swap_dir(f);
    on_common(w, fa, fb, u, v, f, T, h);                      // dyad (u, v), third vertex w
    if (u < w) on_common(v, f, sb, u, w, fa, T, h);           // dyad (u, w), third vertex v
    else on_common(v, sb, f, w, u, sa, T, h);                 // dyad (w, u)
    if (v < w) on_common(u, sf, sa, v, w, fb, T, h);          // dyad (v, w), third vertex u
    else on_common(u, sa, sf, w, v, sb, T, h);                // dyad (w, v)
}

// Scales every update of one signature by its count.
template <class H>
struct scaled_bins {
    H& h;
    unsigned long long c;
    __device__ inline void add(uint32_t cls, unsigned long long x) { h.add(cls, x * c); }
};

// Turns the signature counts of a workgroup of `threads` into updates of h and
// clears them.  Labelled signatures hold the order of the three ids.
template <bool Lab, class H>
__device__ inline void tri_flush(tri_sig<Lab>& sig, uint32_t threads, const uint8_t* T, H& h) {
    constexpr uint32_t kB = tri_sig<Lab>::kBits, kM = (1u << kB) - 1u;
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (what follows from it stays out of a caller's loop, whose registers it would take)
    __syncthreads();
    for (uint32_t k = tid; k < tri_sig<Lab>::kSlots; k += threads) {
        const unsigned long long c = sig.n[k];
        if (c == 0) continue;
        sig.n[k] = 0;
        scaled_bins<H> sh{h, c};
        uint32_t xy = k & kM, xz = (k >> kB) & kM, yz = k >> (2 * kB);
        uint32_t px = 0, py = 1, pz = 2;
        if (Lab) {
            const uint32_t gxy = xy & 1u, gxz = xz & 1u, gyz = yz & 1u;
            px = 2u - gxy - gxz;
            py = gxy + 1u - gyz;
            pz = gxz + gyz;
            xy >>= 1;
            xz >>= 1;
            yz >>= 1;
        }
        if (px < py) on_triangle(pz, xz, yz, px, py, xy, T, sh);
        else on_triangle(pz, yz, xz, py, px, swap_dir(xy), T, sh);
    }
    __syncthreads();
}

__device__ inline dyad_rec load_rec(const dyad_rec* p) {
    const uint4 a = *reinterpret_cast<const uint4*>(p);
    const uint2 c = *reinterpret_cast<const uint2*>(&p->u);
    dyad_rec r;
    r.bu = a.x; r.eu = a.y; r.bv = a.z; r.ev = a.w;
    r.u = c.x; r.vf = c.y;
    return r;
}

// Entries are (w << 2) | f with w < 2^23, so the all-ones word never occurs
// and serves as the end-of-list sentinel.  Comparing vertices of two entries:
//   w(a) <= w(b)  <=>  a <= (b | 3),      w(a) == w(b)  <=>  (a ^ b) < 4.
constexpr uint32_t kSentinel = 0xffffffffu;

// ---------------------------------------------------------------- lane ----
// One lane per record: the two rows, read from global memory (L1/L2 resident
// for the short rows of this bucket), compared in chunks.
constexpr int kLaneB = 256;

// The two rows are compared kLaneChunk entries at a time: a chunk of each is
// loaded with independent loads and every pair of the two chunks compared in
// registers; then the chunk whose last vertex is smaller is replaced.  No pair
// is compared twice and no shared vertex is missed: the chunk left in place
// holds no vertex below the last one of the chunk that is replaced, and the
// next chunk of a row starts above its current one.
constexpr uint32_t kLaneChunk = 8;

__device__ inline void load_chunk(const uint32_t* __restrict__ nbr, uint32_t pos, uint32_t end, uint32_t pad,
                                  uint32_t (&c)[kLaneChunk]) {
#pragma unroll
    for (uint32_t k = 0; k < kLaneChunk; ++k) c[k] = pos + k < end ? nbr[pos + k] : pad;
}

template <class H>
__device__ inline void lane_dyad(const dyad_rec& r, const uint32_t* __restrict__ nbr, const uint8_t* T, H& h) {
    const uint32_t u = r.u, v = r.vf >> 2, f = r.vf & 3u;
    // pads: never equal to an entry or to each other (entries are below 2^25)
    constexpr uint32_t kPadA = 0xffffffffu, kPadB = 0xfffffff0u;
    uint32_t i = r.bu, j = r.bv;
    uint32_t A[kLaneChunk], B[kLaneChunk];
    load_chunk(nbr, i, r.eu, kPadA, A);
    load_chunk(nbr, j, r.ev, kPadB, B);
    for (;;) {
#pragma unroll
        for (uint32_t p = 0; p < kLaneChunk; ++p)
#pragma unroll
            for (uint32_t q = 0; q < kLaneChunk; ++q)
                if ((A[p] ^ B[q]) < 4u) on_common(A[p] >> 2, A[p] & 3u, B[q] & 3u, u, v, f, T, h);
        const uint32_t la = min(kLaneChunk, r.eu - i), lb = min(kLaneChunk, r.ev - j);
        uint32_t lastA = A[0], lastB = B[0];
#pragma unroll
        for (uint32_t k = 1; k < kLaneChunk; ++k) {
            lastA = k < la ? A[k] : lastA;
            lastB = k < lb ? B[k] : lastB;
        }
        if (lastA <= (lastB | 3u)) {
            i += kLaneChunk;
            if (i >= r.eu) break;
            load_chunk(nbr, i, r.eu, kPadA, A);
        } else {
            j += kLaneChunk;
            if (j >= r.ev) break;
            load_chunk(nbr, j, r.ev, kPadB, B);
        }
    }
}

__global__ __launch_bounds__(kLaneB) void k_census_lane(census_args L) {
    __shared__ uint8_t T[64];
    __shared__ unsigned long long wbins[wave_bins<kLaneB>::kWords];
    if (threadIdx.x < 64) T[threadIdx.x] = L.table[threadIdx.x];
    wave_bins<kLaneB> h{wbins};
    h.clear();
    __syncthreads();
    for (uint64_t d = (uint64_t)blockIdx.x * kLaneB + threadIdx.x; d < L.count; d += (uint64_t)gridDim.x * kLaneB)
        lane_dyad(load_rec(L.dyads + d), L.nbr, T, h);
    h.flush(acc_copy(L.acc));
}

// The per-dyad terms that need no intersection, of a whole graph, for the 16
// classes, which do not depend on the vertices' names: with a, b and m the
// numbers of vertices that x is joined to by an arc out, an arc in and both
// ways (d = a + b + m), every unordered pair of x's neighbours is one path of
// two joined pairs centred at x, counted once in the class of its two types
// (a (a - 1) / 2, a b, a m, ...), and the dyadic base of the pairs of x is
// n - d per pair, of which n per pair is added once for the whole graph
// (asym and mutual pairs) and -d (a + b) and -d m here.
//
// Reads 16 bytes per row where the pass over the entries (k_census_totals)
// reads 16 per entry: 3.8 M rows take 0.02 ms instead of 0.25 for 33 M entries.
constexpr uint32_t kRowSums = 8;
__device__ const uint8_t kRowCode[kRowSums] = {1, 3, 1 | 4, 2 | 8, 3 | 12, 1 | 8, 1 | 12, 2 | 12};

__device__ inline void row_add(const uint4* __restrict__ rinfo, uint32_t x, unsigned long long (&s)[kRowSums]) {
    const uint4 r = rinfo[x];
    uint2 before = make_uint2(0u, 0u);
    if (x != 0) before = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint32_t*>(rinfo + x) - 2);
    const uint32_t d = r.y - r.x, m = (r.z - before.x) + (r.w - before.y) - d, a = (r.z - before.x) - m,
                   b = (r.w - before.y) - m;
    const unsigned long long A = a, B = b, M = m, D = d;
    s[0] -= D * (A + B);
    s[1] -= D * M;
    s[2] += A * (A - 1) / 2;
    s[3] += B * (B - 1) / 2;
    s[4] += M * (M - 1) / 2;
    s[5] += A * B;
    s[6] += A * M;
    s[7] += B * M;
}

// Sums over the wavefront; lane 0 adds them to h.
template <class H>
__device__ inline void row_flush(unsigned long long (&s)[kRowSums], const uint8_t* T, H& h) {
#pragma unroll
    for (uint32_t k = 0; k < kRowSums; ++k) {
        for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_xor(s[k], o, 64);
        if (__lane_id() == 0 && s[k] != 0) h.add(T[kRowCode[k]], s[k]);
    }
}

// Rows [x0, x1), and the base of asym one-way and mutual two-way pairs.
__global__ __launch_bounds__(kLaneB) void k_census_rows(const uint4* __restrict__ rinfo, uint32_t x0, uint32_t x1,
                                                        uint64_t n, uint64_t asym, uint64_t mutual,
                                                        const uint8_t* __restrict__ table,
                                                        unsigned long long* __restrict__ acc) {
    __shared__ unsigned long long wbins[wave_bins<kLaneB>::kWords];
    __shared__ uint8_t T[64];
    if (threadIdx.x < 64) T[threadIdx.x] = table[threadIdx.x];
    wave_bins<kLaneB> h{wbins};
    h.clear();
    __syncthreads();
    unsigned long long s[kRowSums] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        s[0] = n * asym;
        s[1] = n * mutual;
    }
    for (uint64_t x = (uint64_t)x0 + (uint64_t)blockIdx.x * kLaneB + threadIdx.x; x < x1; x += (uint64_t)gridDim.x * kLaneB)
        row_add(rinfo, (uint32_t)x, s);
    row_flush(s, T, h);
    h.flush(acc_copy(acc));
}

// The same terms for the labelled census, whose codes depend on the ids, for
// every dyad at once, one lane per neighbour entry: entry y of row x, with
// the prefix counts of the direction bits, gives the typed counts of the
// entries after y in row x.  When y > x these are the entries of N(u) above v
// for the dyad (u, v) = (x, y); when y < x they are the entries of N(v) above
// u for the dyad (y, x).  The dyadic base n - |N(u)| - |N(v)| is split the
// same way: n - |N(x)| from the first side, -|N(x)| from the second.  The
// entry arrays are read coalesced, and the row's bounds and prefix counts at
// its end come in one 16-byte record shared by the row's entries.
//
// totals_entries: entries base + k * B + threadIdx.x (k < kPer) below `end`,
// their loads issued before any is used.
// Part: only of the dyads (u, v) with u in [u_lo, u_hi).
template <uint32_t kPer, uint32_t B, bool Part, class H>
__device__ inline void totals_entries(uint64_t base, uint64_t end, const uint32_t* __restrict__ nbr,
                                      const uint32_t* __restrict__ owner, const uint4* __restrict__ rinfo,
                                      const uint64_t* __restrict__ tpre, uint64_t n, const uint8_t* T, H& h,
                                      uint32_t u_lo = 0, uint32_t u_hi = 0) {
    uint32_t x[kPer], ent[kPer];
    uint64_t rb[kPer], re[kPer], pend[kPer], pnext[kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint64_t e = base + k * B + threadIdx.x;
        x[k] = e < end ? owner[e] : 0u;
        ent[k] = e < end ? nbr[e] : 0u;
        pnext[k] = e < end ? tpre[e + 1] : 0ull;
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint4 ri = rinfo[x[k]];
        rb[k] = ri.x;
        re[k] = ri.y;
        pend[k] = (uint64_t)ri.z | ((uint64_t)ri.w << 32);
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint64_t e = base + k * B + threadIdx.x;
        if (e >= end) continue;
        const uint32_t y = ent[k] >> 2, fxy = ent[k] & 3u;
        if (Part && min(x[k], y) - u_lo >= u_hi - u_lo) continue;
        const uint64_t pc = pend[k] - pnext[k];                 // direction bits after e in row x
        const uint64_t tot = re[k] - e - 1, out = pc & 0xffffffffull, in = pc >> 32;
        const uint64_t mut = out + in - tot;
        const bool first = y > x[k];                            // x plays u, else v
        const uint32_t f = first ? fxy : swap_dir(fxy);
        const uint32_t sh = first ? 2u : 4u;
        h.add(T[f], (unsigned long long)((first ? n : 0ull) - (re[k] - rb[k])));
        h.add(T[f | (1u << sh)], out - mut);
        h.add(T[f | (2u << sh)], in - mut);
        h.add(T[f | (3u << sh)], mut);
    }
}

constexpr uint32_t kTotalsPer = 4;   // entries per thread and step
// Distinct bins the totals pass can reach: at most 8 with a pass table of the
// dyad path, and the 21 codes themselves on the forward-list path, which keeps
// all 64 codes in one pass.
template <bool Lab>
constexpr uint32_t totals_slot_count() { return Lab ? 21 : 8; }

// Adds straight to a graph's 16 accumulators in global memory.
struct global_bins {
    unsigned long long* acc;
    __device__ inline void add(uint32_t cls, unsigned long long x) { atomicAdd(&acc[cls], x); }
};

// Per-lane bins over a few slots: the totals pass reaches only the bins of the
// codes f, f | t << 2 and f | t << 4 (f, t in 1..3), so a lane keeps one 64-bit
// slot per reachable bin (or two lanes of a workgroup share one: COLS columns).
// The codes are remapped to slots in a table.
template <uint32_t COLS>
struct slot_bins {
    unsigned long long* bins;   // slots x COLS
    __device__ inline void add(uint32_t slot, unsigned long long x) {
        atomicAdd(&bins[slot * COLS + (threadIdx.x & (COLS - 1))], x);
    }
};

// The k-th of the 21 reachable codes: f, f | t << 2 (t = 1..3), f | t << 4.
__device__ inline uint32_t totals_code(uint32_t k) {
    const uint32_t f = 1 + k / 7, j = k % 7;
    return j == 0 ? f : (j <= 3 ? f | (j << 2) : f | ((j - 3) << 4));
}

// Fills TS (code -> slot) and bin_of_slot for the reachable codes of table T;
// returns the number of slots (on thread 0).  A thread per code, since one that
// looks for equal bins takes 12 us, as long as the entries of a small graph.  The
// forward-list path's table tells all codes apart; with the other tables codes
// share bins, and the first lane that holds a bin has its slot.
template <bool Lab>
__device__ inline uint32_t totals_slots(const uint8_t* T, uint8_t* TS, uint32_t* bin_of_slot) {
    constexpr uint32_t kSlots = totals_slot_count<Lab>();
    if constexpr (Lab) {
        if (threadIdx.x < kSlots) {
            const uint32_t c = totals_code(threadIdx.x);
            TS[c] = (uint8_t)threadIdx.x;
            bin_of_slot[threadIdx.x] = T[c];
        }
        return kSlots;
    } else {
        if (threadIdx.x >= 64) return 0;
        const uint32_t k = threadIdx.x;
        const bool in = k < 21;
        const uint32_t c = totals_code(in ? k : 0u), bin = T[c];
        uint32_t first = k;
        for (uint32_t j = 0; j < 21; ++j)
            if ((uint32_t)__builtin_amdgcn_readlane((int)bin, (int)j) == bin && j < first) first = j;
        const uint64_t firsts = __ballot(in && first == k);
        const uint32_t slot = (uint32_t)__popcll(firsts & ((1ull << first) - 1ull));
        if (in && slot < kSlots) {
            TS[c] = (uint8_t)slot;
            bin_of_slot[slot] = bin;
        }
        return (uint32_t)__popcll(firsts);
    }
}

// Sums the per-lane slots over a kLaneB workgroup into h (wavefront w takes
// slots w, w + 4), without those of bins from `bins` on (the discard bin).
template <uint32_t COLS, class H>
__device__ inline void slots_flush(unsigned long long* sbins, const uint32_t* bin_of_slot, uint32_t nslots,
                                   uint32_t bins, H& h) {
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t sl = threadIdx.x >> 6; sl < nslots; sl += kLaneB / 64) {
        unsigned long long v = 0;
        for (uint32_t i = lane; i < COLS; i += 64) v += sbins[sl * COLS + i];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0 && v != 0 && bin_of_slot[sl] < bins) h.add(bin_of_slot[sl], v);
    }
}

// Over all U neighbour entries.
template <bool Lab>
__global__ __launch_bounds__(kLaneB) void k_census_totals(const uint32_t* __restrict__ nbr,
                                                          const uint32_t* __restrict__ owner,
                                                          const uint4* __restrict__ rinfo,
                                                          const uint64_t* __restrict__ tpre, uint64_t U,
                                                          uint64_t n, const uint8_t* __restrict__ table,
                                                          unsigned long long* __restrict__ acc) {
    constexpr uint32_t kSlots = totals_slot_count<Lab>(), kWords = tri_bins<Lab>::kWords;
    __shared__ unsigned long long sbins[kSlots * kLaneB];
    __shared__ uint8_t T[64], TS[64];
    __shared__ uint32_t bin_of_slot[kSlots], s_nslots;
    if (threadIdx.x < 64) T[threadIdx.x] = table[threadIdx.x];
    __syncthreads();
    const uint32_t ns = totals_slots<Lab>(T, TS, bin_of_slot);
    if (threadIdx.x == 0) s_nslots = ns;
    for (uint32_t k = threadIdx.x; k < kSlots * kLaneB; k += kLaneB) sbins[k] = 0;
    __syncthreads();
    slot_bins<kLaneB> hs{sbins};
    for (uint64_t base = (uint64_t)blockIdx.x * kLaneB * kTotalsPer; base < U;
         base += (uint64_t)gridDim.x * kLaneB * kTotalsPer)
        totals_entries<kTotalsPer, kLaneB, false>(base, U, nbr, owner, rinfo, tpre, n, TS, hs);
    global_bins g{acc_copy(acc, kWords)};
    slots_flush<kLaneB>(sbins, bin_of_slot, s_nslots, kWords, g);
}

// The terms of the dyads (u, v) with u in [u_lo, u_hi), for a census of a range.
// All: from the entries of the whole graph, as above; the rest are skipped.
// Otherwise from the entries [e0, e1) of the rows of the range above the
// diagonal, each of which looks its own place up in the row of v: log2 |N(v)|
// reads at random instead of 16 bytes in turn per entry of the graph (the choice
// between the two: range_terms).
template <bool All>
__global__ __launch_bounds__(kLaneB) void k_range_terms(const uint32_t* __restrict__ nbr,
                                                        const uint32_t* __restrict__ owner,
                                                        const uint4* __restrict__ rinfo,
                                                        const uint64_t* __restrict__ tpre, uint64_t e0, uint64_t e1,
                                                        uint32_t u_lo, uint32_t u_hi, uint64_t n,
                                                        const uint8_t* __restrict__ table,
                                                        unsigned long long* __restrict__ acc) {
    constexpr uint32_t kSlots = totals_slot_count<false>();
    __shared__ unsigned long long sbins[kSlots * kLaneB];
    __shared__ uint8_t T[64], TS[64];
    __shared__ uint32_t bin_of_slot[kSlots], s_nslots;
    if (threadIdx.x < 64) T[threadIdx.x] = table[threadIdx.x];
    __syncthreads();
    const uint32_t ns = totals_slots<false>(T, TS, bin_of_slot);
    if (threadIdx.x == 0) s_nslots = ns;
    for (uint32_t k = threadIdx.x; k < kSlots * kLaneB; k += kLaneB) sbins[k] = 0;
    __syncthreads();
    slot_bins<kLaneB> h{sbins};
    if constexpr (All) {
        for (uint64_t base = (uint64_t)blockIdx.x * kLaneB * kTotalsPer; base < e1;
             base += (uint64_t)gridDim.x * kLaneB * kTotalsPer)
            totals_entries<kTotalsPer, kLaneB, true>(base, e1, nbr, owner, rinfo, tpre, n, TS, h, u_lo, u_hi);
    } else {
        for (uint64_t e = e0 + (uint64_t)blockIdx.x * kLaneB + threadIdx.x; e < e1; e += (uint64_t)gridDim.x * kLaneB) {
            const uint32_t u = owner[e], v = nbr[e] >> 2, f = nbr[e] & 3u;
            if (v < u) continue;
            // after place i of a row, the entries of each direction type
            auto after = [&](const uint4& row, uint64_t i, uint32_t sh) {
                const uint64_t pc = ((uint64_t)row.z | ((uint64_t)row.w << 32)) - tpre[i + 1];
                const uint64_t tot = row.y - i - 1, out = pc & 0xffffffffull, in = pc >> 32, mut = out + in - tot;
                h.add(TS[f | (1u << sh)], out - mut);
                h.add(TS[f | (2u << sh)], in - mut);
                h.add(TS[f | (3u << sh)], mut);
            };
            const uint4 ru = rinfo[u], rv = rinfo[v];
            h.add(TS[f], (unsigned long long)(n - (ru.y - ru.x) - (rv.y - rv.x)));
            after(ru, e, 2u);
            after(rv, find_first_ge(nbr, rv.x, rv.y, u), 4u);
        }
    }
    global_bins g{acc_copy(acc)};
    slots_flush<kLaneB>(sbins, bin_of_slot, s_nslots, kNumClasses, g);
}

// ---------------------------------------------------------- merge path ----
// Group-cooperative intersection of rows [bu, eu) and [bv, ev) in rounds.  A
// round stages the next TW entries of each row in LDS (followed by a
// sentinel), produces the first min(TW, na + nb) outputs of the merged order
// (ties: the N(u) copy first), and lane l handles outputs [l*PER, (l+1)*PER)
// after locating its start on the merge path by binary search (co-rank).  A
// shared vertex is seen when its N(u) copy is taken while the N(v) head holds
// the same vertex.  The lane that produces the round's last output publishes
// how many N(u) entries the round consumed.
// P says how two entries compare (le, eq; the sentinel is above every entry)
// and what a shared vertex means (shared).
template <class P>
__device__ inline uint32_t co_rank(const uint32_t* sA, uint32_t na, const uint32_t* sB, uint32_t nb, uint32_t d) {
    uint32_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    while (lo < hi) {
        uint32_t mid = (lo + hi + 1) >> 1;
        if (P::le(sA[mid - 1], sB[d - mid])) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Synchronisation of the group that shares a dyad: the whole workgroup, or a
// single wavefront (whose lanes run in lockstep, LDS accesses in order; the
// fences keep the compiler from moving LDS accesses across the point).
struct block_sync {
    __device__ inline void operator()() const { __syncthreads(); }
};
struct wave_sync {
    __device__ inline void operator()() const {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

// Dyad records: a shared neighbour of the dyad.
template <class H>
struct dyad_rows {
    const dyad_rec& r;
    const uint8_t* T;
    H& h;
    __device__ static inline bool le(uint32_t a, uint32_t b) { return a <= (b | 3u); }
    __device__ static inline bool eq(uint32_t a, uint32_t b) { return (a ^ b) < 4u; }
    __device__ inline void shared(uint32_t a, uint32_t b) {
        on_common(a >> 2, a & 3u, b & 3u, r.u, r.vf >> 2, r.vf & 3u, T, h);
    }
};
// Edge records: a triangle.
template <bool Lab>
struct edge_rows {
    uint32_t xy;
    tri_sig<Lab>& sig;
    __device__ static inline bool le(uint32_t a, uint32_t b) { return (a & kRankMask) <= (b & kRankMask); }
    __device__ static inline bool eq(uint32_t a, uint32_t b) { return ((a ^ b) & kRankMask) == 0u; }
    __device__ inline void shared(uint32_t a, uint32_t b) {
        sig.hit(xy, tri_sig<Lab>::code(a), tri_sig<Lab>::code(b));
    }
};

template <int G, int TW, class Sync, class P>
__device__ inline void merge_path(uint32_t bu, uint32_t eu, uint32_t bv, uint32_t ev, const uint32_t* __restrict__ nbr,
                                  uint32_t* sA, uint32_t* sB, uint32_t* s_xt, uint32_t lane, P rows) {
    constexpr uint32_t PER = TW / G;
    static_assert(TW % G == 0, "tile is a multiple of the group");
    const Sync sync{};
    const uint32_t la = eu - bu, lb = ev - bv;
    uint32_t a_pos = 0, b_pos = 0;
    while (a_pos < la && b_pos < lb) {
        const uint32_t na = min((uint32_t)TW, la - a_pos), nb = min((uint32_t)TW, lb - b_pos);
        uint32_t ra[PER], rb[PER];
#pragma unroll
        for (uint32_t t = 0; t < PER; ++t) {
            const uint32_t k = lane + t * G;
            ra[t] = k < na ? nbr[bu + a_pos + k] : kSentinel;
            rb[t] = k < nb ? nbr[bv + b_pos + k] : kSentinel;
        }
#pragma unroll
        for (uint32_t t = 0; t < PER; ++t) {
            sA[lane + t * G] = ra[t];
            sB[lane + t * G] = rb[t];
        }
        if (lane == 0) {
            sA[TW] = kSentinel;
            sB[TW] = kSentinel;
        }
        sync();
        const uint32_t total = min((uint32_t)TW, na + nb);
        const uint32_t d0 = lane * PER;
        if (d0 < total) {
            const uint32_t steps = min(PER, total - d0);
            uint32_t i = co_rank<P>(sA, na, sB, nb, d0);
            uint32_t j = d0 - i;
            uint32_t a = sA[i], b = sB[j];
#pragma unroll
            for (uint32_t t = 0; t < PER; ++t) {
                if (t < steps) {
                    if (P::eq(a, b) && a != kSentinel) rows.shared(a, b);
                    const bool ta = P::le(a, b);
                    i += ta ? 1u : 0u;
                    j += ta ? 0u : 1u;
                    const uint32_t x = ta ? sA[i] : sB[j];
                    a = ta ? x : a;
                    b = ta ? b : x;
                }
            }
            if (d0 + steps == total) *s_xt = i;
        }
        sync();
        const uint32_t xt = *s_xt;
        a_pos += xt;
        b_pos += total - xt;
    }
}

// ------------------------------------------------------ work distribution ----
// Dyads are handed out in chunks of CH through eight counters, one per XCD
// (workgroup b runs on XCD b % 8 on this part), so that the atomics stay in
// one L2: counter x hands out the chunk indices x, x + 8, x + 16, ... (x, x + g,
// x + 2 g, ... in a grid of g < 8 workgroups, which uses only g counters).
__device__ inline uint32_t take_chunk(unsigned int* ctr, uint32_t xcd, uint32_t blocks) {
    return xcd + min(blocks, (uint32_t)kXcds) * atomicAdd(&ctr[xcd * kCounterStride], 1u);
}

// ---------------------------------------------------------------- wave ----
constexpr int kWaveB = 64;
constexpr uint32_t kWaveChunk = 16;

// TW: entries of each row staged per round (the tunable LDS tile).
template <int TW>
__global__ __launch_bounds__(kWaveB) void k_census_wave(census_args L, unsigned int* ctr) {
    __shared__ unsigned long long bins[wave_bins<kWaveB>::kWords];
    __shared__ uint8_t T[64];
    __shared__ uint32_t sA[TW + 1], sB[TW + 1];
    __shared__ uint32_t s_xt;
    T[threadIdx.x] = L.table[threadIdx.x];
    wave_bins<kWaveB> h{bins};
    h.clear();
    __syncthreads();
    const uint32_t xcd = blockIdx.x % kXcds;
    uint32_t c = 0;
    if (threadIdx.x == 0) c = take_chunk(ctr, xcd, gridDim.x);
    c = __shfl(c, 0, 64);
    while ((uint64_t)c * kWaveChunk < L.count) {
        uint32_t cn = 0;
        if (threadIdx.x == 0) cn = take_chunk(ctr, xcd, gridDim.x);      // next chunk, fetched early
        const uint32_t end = min((uint32_t)L.count, (c + 1) * kWaveChunk);
        for (uint32_t d = c * kWaveChunk; d < end; ++d) {
            const dyad_rec r = load_rec(L.dyads + d);
            merge_path<kWaveB, TW, block_sync>(r.bu, r.eu, r.bv, r.ev, L.nbr, sA, sB, &s_xt, threadIdx.x,
                                               dyad_rows<wave_bins<kWaveB>>{r, T, h});
        }
        c = __shfl(cn, 0, 64);
    }
    h.flush(acc_copy(L.acc));
}

// --------------------------------------------------------------- group ----
constexpr uint32_t kGroupChunk = 2;

// B: workgroup size; TW: entries of each row staged per round (both tunable).
template <int B, int TW>
__global__ __launch_bounds__(B) void k_census_group(census_args L, unsigned int* ctr) {
    __shared__ unsigned long long bins[wave_bins<B>::kWords];
    __shared__ uint8_t T[64];
    __shared__ uint32_t sA[TW + 1], sB[TW + 1];
    __shared__ uint32_t s_xt, s_next;
    if (threadIdx.x < 64) T[threadIdx.x] = L.table[threadIdx.x];
    wave_bins<B> h{bins};
    h.clear();
    const uint32_t xcd = blockIdx.x % kXcds;
    if (threadIdx.x == 0) s_next = take_chunk(ctr, xcd, gridDim.x);
    __syncthreads();
    uint32_t c = s_next;
    __syncthreads();
    while ((uint64_t)c * kGroupChunk < L.count) {
        if (threadIdx.x == 0) s_next = take_chunk(ctr, xcd, gridDim.x);  // next chunk, fetched early
        const uint32_t end = min((uint32_t)L.count, (c + 1) * kGroupChunk);
        for (uint32_t d = c * kGroupChunk; d < end; ++d) {
            const dyad_rec r = load_rec(L.dyads + d);
            merge_path<B, TW, block_sync>(r.bu, r.eu, r.bv, r.ev, L.nbr, sA, sB, &s_xt, threadIdx.x,
                                          dyad_rows<wave_bins<B>>{r, T, h});
        }
        __syncthreads();
        c = s_next;
        __syncthreads();
    }
    h.flush(acc_copy(L.acc));
}


// ----------------------------------------------------------------- hub ----
// Hub records, grouped by anchor (their endpoint with the longer row) into
// hub tasks of up to kHubChunk records that share the anchor.  A workgroup
// takes kHubGroupTasks consecutive tasks at a time, stages the anchor rows into
// an LDS hash table (kHubTile entries in 4-slot buckets, the next bucket on
// overflow) -- the rows of several tasks together when they fit one tile, a
// longer row tile by tile -- and streams the other endpoint's row of every
// record against it: each entry of that row is probed once, in the tile whose
// vertex range holds it.  The anchor row is thus read once per task instead of
// once per record, and the work per record is proportional to the shorter row.
constexpr int kHubB = 256;
constexpr uint32_t kEmpty = 0xffffffffu;                 // never an entry (w < 2^23)
constexpr uint32_t kHubGather = 8;
constexpr uint32_t kHubFlushAfter = (1u << 24) - 1u;      // kHubB times this stays below 2^32

// Geometry of one LDS tile of TILE anchor entries (the tunable hub tile): a
// hash table of TILE / 2 buckets of 4 slots (mean load 2 entries) and a filter
// of 8 bits per staged entry.  The table hashes a key (m << 23) | w (m the
// task's place in its group, w the vertex) folded to 24 bits, w + (m << 20),
// with a 24 x 24-bit multiply and keeps the top bits of the low 32 bits of the
// product (a full 32-bit multiply issues at a quarter of the rate).  The
// filter position of (m, w) is w * C + mix(m) (one multiply-add, mix(m)
// computed once per record): its top bits pick the filter word and its low
// five bits the bit, which is the shift count a 32-bit shift takes as it is.
// Only the placement depends on the hashes: a probe compares whole keys.
constexpr uint32_t kHubBucketMul = 0x9E3779u;            // odd 24-bit multipliers
constexpr uint32_t kHubFilterMul = 0x85EBCBu;
constexpr uint32_t kHubMemberMul = 0x9E3779B1u;          // odd 32-bit multiplier of the member index
__device__ inline uint32_t hub_fold(uint32_t key) { return (key & ((1u << 23) - 1u)) + ((key >> 23) << 20); }
// Low 32 bits of the product of the low 24 bits of a and b, unsigned (HIP's
// __umul24 returns a signed int, whose right shifts would be arithmetic).
__device__ inline uint32_t mul24(uint32_t a, uint32_t b) { return (uint32_t)__umul24(a, b); }
__device__ inline uint32_t hub_member_mix(uint32_t m) { return m * kHubMemberMul; }
template <uint32_t TILE>
struct hub_geom {
    static constexpr uint32_t kBuckets = TILE / 2;
    static constexpr uint32_t kSlots = 4 * kBuckets;
    static constexpr int kBucketBits = __builtin_ctz(kBuckets);
    static constexpr int kFilterLog = __builtin_ctz(TILE) + 3;
    static constexpr uint32_t kFilterBits = 1u << kFilterLog;
    static constexpr uint32_t kWordShift = 32 - (kFilterLog - 5);   // position >> kWordShift: the filter word
    static_assert((TILE & (TILE - 1)) == 0 && TILE >= 256 && TILE <= 4096, "power-of-two tile");
    static_assert(kFilterBits / 32 >= (uint32_t)kHubB / 8, "filter words");
    // from a folded key
    __device__ static inline uint32_t bucket_of(uint32_t fold) { return mul24(fold, kHubBucketMul) >> (32 - kBucketBits); }
    // vertex w (< 2^23) of the member whose hub_member_mix is mix
    __device__ static inline uint32_t filter_pos(uint32_t w, uint32_t mix) { return mul24(w, kHubFilterMul) + mix; }
};

// Buckets fill their slots in order, so a bucket whose last slot is empty
// ends the probe sequence of every vertex that hashes to it or before it.
template <uint32_t TILE>
__device__ inline void hub_insert(uint32_t* hash, uint32_t e) {
    using G = hub_geom<TILE>;
    uint32_t b = G::bucket_of(hub_fold(e >> 2));
    for (;;) {
        for (uint32_t s = 0; s < 4; ++s)
            if (atomicCAS(&hash[4 * b + s], kEmpty, e) == kEmpty) return;
        b = (b + 1) & (G::kBuckets - 1);
    }
}

// The whole bucket is read at once and its four slots compared without
// branches; the next bucket is read only when this one is full and holds no
// match.  key4 is the stored word with its direction bits cleared,
// (m << 25) | (w << 2), and fold the folded key.  A slot XOR key4 is below 4
// exactly when the slot holds the key (a key is stored at most once), and is
// then the slot's direction bits: the smallest of the four, clamped to 4, is
// the hit's direction bits, or 4 for no hit.
template <uint32_t TILE>
__device__ inline uint32_t hub_probe(const uint32_t* hash, uint32_t key4, uint32_t fold) {
    using G = hub_geom<TILE>;
    const uint4* h4 = reinterpret_cast<const uint4*>(hash);
    uint32_t b = G::bucket_of(fold);
    for (;;) {
        const uint4 q = h4[b];
        const uint32_t r = min(min(min(q.x ^ key4, q.y ^ key4), q.z ^ key4), min(q.w ^ key4, 4u));
        if (r < 4u || q.w == kEmpty) return r;
        b = (b + 1) & (G::kBuckets - 1);
    }
}

// Exclusive scan of a[0..count) in place on a 256-thread block (count <=
// 4 * 256); a[count .. count + kScanPad) receive the total.  wsum holds 4 words
// of LDS.
constexpr uint32_t kScanPad = 8;
__device__ inline void block_scan_u32(uint32_t* a, uint32_t count, uint32_t* wsum) {
    constexpr uint32_t kPer = kHubChunk / kHubB;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    uint32_t loc[kPer], s = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t i = tid * kPer + k;
        loc[k] = s;
        s += i < count ? a[i] : 0u;
    }
    uint32_t incl = s;
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(incl, o, 64);
        if ((int)lane >= o) incl += y;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    uint32_t base = 0, tot = 0;
    for (uint32_t w = 0; w < kHubB / 64; ++w) {
        base += w < wid ? wsum[w] : 0u;
        tot += wsum[w];
    }
    base += incl - s;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t i = tid * kPer + k;
        if (i < count) a[i] = base + loc[k];
    }
    if (tid < kScanPad) a[count + tid] = tot;
    __syncthreads();
}

// What a shared vertex w of the dyad (or edge record) (u, v), u < v, adds to
// the census depends only on the direction bits f = f_uv, fa = f_uw, fb = f_vw
// (each 1, 2 or 3: the pairs are joined) and on where w lies: below u, between
// u and v, or above v (where = [w > u] + [w > v]).  The hub mode counts shared
// vertices per signature f | fa << 2 | fb << 4 | where << 6 (192 slots, 81 of
// them reachable) in one 32-bit LDS histogram per workgroup and turns the
// counts into class updates when it flushes.
constexpr uint32_t kSigs = 192;

// Aligned blocks of kHubGather entries that hold the entries [p0, p1) of a row
// (row arrays are padded so that the last block is readable).
static_assert(kHubGather == 8, "a block is read as two 16-byte loads");
__device__ inline uint32_t hub_blocks(uint32_t p0, uint32_t p1) {
    return p1 > p0 ? (p1 + kHubGather - 1) / kHubGather - p0 / kHubGather : 0u;
}

// LDS of the hub mode: the hash table, one candidate ring per wavefront, four
// per-record arrays, scan scratch, the signature histogram, the filter and the
// task words.
constexpr uint32_t kHubRing = 128;   // candidates a wavefront holds between probe rounds
struct hub_lds {
    uint32_t* hash;   // hub_geom::kSlots, 16-byte aligned
    uint32_t* ring_e; // kHubRing x (kHubB / 64) candidates: the entry
    uint32_t* ring_m; // ... and the meta word of its record
    uint32_t* pos;    // next unprobed position in the other endpoint's row
    uint32_t* end;    // end of that row's entries in the current tile
    uint32_t* meta;   // (m << 26) | (x << 3) | (anchor is u) << 2 | f_uv, m the task's place in its group
    uint32_t* off;    // blocks of this tile, then their exclusive scan and kScanPad copies of the total
    uint32_t* wsum;   // 4 words
    uint32_t* sig;    // kSigs counts shared by the workgroup
    uint32_t* filt;   // hub_geom::kFilterBits bits: a vertex whose bit is clear is not in the tile
    uint32_t* tk;     // kHubTkWords: the tasks of the current chunk and their groups
};
// Words of hub_lds::tk: per task of the chunk its first record, record count,
// anchor-row start, anchor-row length and anchor; the group boundaries and
// their count; the record and row prefixes of the current group's members.
constexpr uint32_t kTkBegin = 0, kTkNrec = 8, kTkHb = 16, kTkLen = 24, kTkAnchor = 32, kTkGroups = 40,
                   kTkNGroups = 49, kTkRb = 50, kTkEb = 59, kHubTkWords = 68;
static_assert(kHubGroupTasks == 8, "the task words hold eight tasks");
template <uint32_t TILE>
constexpr uint32_t hub_lds_words() {
    return hub_geom<TILE>::kSlots + 2 * kHubRing * (kHubB / 64) + 3 * kHubChunk + (kHubChunk + kScanPad) + 4 + kSigs +
           hub_geom<TILE>::kFilterBits / 32 + kHubTkWords;
}

// Wavefronts per SIMD the hub kernels are compiled for: seven (the best
// measured with 1024-entry tiles), or as many workgroups as the LDS of a CU
// (160 KiB) holds for larger tiles (the kernels' other LDS takes < 256 bytes).
template <uint32_t TILE>
constexpr uint32_t hub_waves_per_simd() {
    return (163840u / (4u * hub_lds_words<TILE>() + 256u)) < 7u ? (163840u / (4u * hub_lds_words<TILE>() + 256u))
                                                                   : 7u;
}

template <uint32_t TILE>
__device__ inline hub_lds hub_carve(uint32_t* base) {
    uint32_t* p = base;
    hub_lds S;
    S.hash = p;  p += hub_geom<TILE>::kSlots;
    S.ring_e = p;  p += kHubRing * (kHubB / 64);
    S.ring_m = p;  p += kHubRing * (kHubB / 64);
    S.pos = p;   p += kHubChunk;
    S.end = p;   p += kHubChunk;
    S.meta = p;  p += kHubChunk;
    S.off = p;   p += kHubChunk + kScanPad;
    S.wsum = p;  p += 4;
    S.sig = p;   p += kSigs;
    S.filt = p;  p += hub_geom<TILE>::kFilterBits / 32;
    S.tk = p;
    return S;
}

__device__ inline void hub_bins_clear(const hub_lds& S) {
    for (uint32_t k = threadIdx.x; k < kSigs; k += kHubB) S.sig[k] = 0;
}

// Adds the signature counts to h (one thread per signature) and clears them.
template <class H>
__device__ inline void hub_bins_flush(const hub_lds& S, const uint8_t* T, H& h) {
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < kSigs; k += kHubB) {
        const uint32_t c = S.sig[k];
        if (c == 0) continue;
        S.sig[k] = 0;
        const uint32_t f = k & 3u, fa = (k >> 2) & 3u, fb = (k >> 4) & 3u, where = k >> 6;
        if (f == 0 || fa == 0 || fb == 0) continue;   // never counted
        // ids that put w below u, between u and v, or above v
        const uint32_t u = 1u, v = 3u, w = where * 2u;
        scaled_bins<H> sh{h, (unsigned long long)c};
        on_common(w, fa, fb, u, v, f, T, sh);
    }
    __syncthreads();
}

// One group of hub tasks on the whole workgroup (kHubB threads): members
// [js, js + M) of the chunk's tasks, whose anchor rows together fit one tile
// unless the group is a single task.  Per tile of the members' concatenated
// anchor rows: clear and fill the hash table (an entry of member m is stored
// with m above its 25 bits, so each record matches its own anchor only);
// count, for every record, the aligned blocks of kHubGather entries that hold
// the entries of the other row in the tile's vertex range; scan the counts;
// then each wavefront walks a quarter of the flattened block list, one block
// per lane, and probes the entries that pass the tile's filter 64 at a time.
// A hit adds one to the workgroup's count of the hit's signature.
template <uint32_t TILE, class H>
__device__ inline void hub_group_run(uint32_t js, uint32_t M, const dyad_rec* __restrict__ dyads,
                                     const uint32_t* __restrict__ nbr, uint32_t u_lo, uint32_t u_hi, const hub_lds& S,
                                     const uint8_t* T, H& h, uint32_t& since) {
    using G = hub_geom<TILE>;
    const uint32_t tid = threadIdx.x;
    const uint32_t* rb = S.tk + kTkRb;   // record prefix of the members (M + 1 words)
    const uint32_t* eb = S.tk + kTkEb;   // anchor-row prefix of the members (M + 1 words)
    const uint32_t nrec = rb[M], total = eb[M];
    const bool multi_tile = total > TILE;   // a single task
    for (uint32_t i = tid; i < nrec; i += kHubB) {
        uint32_t m = 0;
        while (m + 1 < M && rb[m + 1] <= i) ++m;
        const uint32_t a = S.tk[kTkAnchor + js + m];
        const dyad_rec r = load_rec(dyads + S.tk[kTkBegin + js + m] + (i - rb[m]));
        const bool anchor_u = r.u == a;
        const uint32_t x = anchor_u ? (r.vf >> 2) : r.u;
        const uint32_t xb = anchor_u ? r.bv : r.bu, xe = anchor_u ? r.ev : r.eu;
        const bool in = r.u >= u_lo && r.u < u_hi;
        const uint32_t p0 = in ? xb : xe;   // outside the requested range: nothing to probe
        S.pos[i] = p0;
        S.meta[i] = (m << 26) | (x << 3) | (anchor_u ? 4u : 0u) | (r.vf & 3u);
        if (!multi_tile) {
            S.end[i] = xe;
            S.off[i] = hub_blocks(p0, xe);
        }
    }
    for (uint32_t tb = 0; tb < total; tb += TILE) {
        const uint32_t te = min(total, tb + TILE);
        for (uint32_t k = tid; k < G::kSlots; k += kHubB) S.hash[k] = kEmpty;
        for (uint32_t k = tid; k < G::kFilterBits / 32; k += kHubB) S.filt[k] = 0;
        __syncthreads();
        for (uint32_t f = tb + tid; f < te; f += kHubB) {
            uint32_t m = 0;
            while (m + 1 < M && eb[m + 1] <= f) ++m;
            const uint32_t v = nbr[S.tk[kTkHb + js + m] + (f - eb[m])];
            hub_insert<TILE>(S.hash, (m << 25) | v);
            const uint32_t fp = G::filter_pos(v >> 2, hub_member_mix(m));
            atomicOr(&S.filt[fp >> G::kWordShift], 1u << (fp & 31u));
        }
        if (multi_tile) {
            const uint32_t hb = S.tk[kTkHb + js], a = S.tk[kTkAnchor + js];
            const uint32_t w_end = te < total ? (nbr[hb + te] >> 2) : kEmpty;
            for (uint32_t i = tid; i < nrec; i += kHubB) {
                const uint32_t p0 = S.pos[i];
                uint32_t xe = p0;
                if (p0 != 0xffffffffu) {
                    const dyad_rec r = load_rec(dyads + S.tk[kTkBegin + js] + i);
                    xe = r.u == a ? r.ev : r.eu;
                }
                const uint32_t p1 = w_end == kEmpty ? xe : find_first_ge(nbr, p0, xe, w_end);
                S.end[i] = p1;
                S.off[i] = hub_blocks(p0, p1);
            }
        }
        __syncthreads();
        block_scan_u32(S.off, nrec, S.wsum);
        const uint32_t P = S.off[nrec];
        // The shared 32-bit signature counts grow by at most kHubGather * P in
        // this tile: they are flushed first when the tiles since the last flush
        // could take them past 2^32 (`per` is the same on every thread).
        const uint32_t per = (uint32_t)min((uint64_t)kHubGather * P / kHubB + 1, (uint64_t)kHubFlushAfter);
        if (since + per > kHubFlushAfter) {
            hub_bins_flush(S, T, h);
            since = 0;
        }
        since += per;
        // The rows to probe are cut into aligned blocks of kHubGather entries
        // (a row's first and last block masked to the row).  Wavefront w takes
        // the w-th quarter [q0, q1) of the flattened list of blocks and walks it
        // 64 blocks at a time, one block per lane, read with two 16-byte loads.
        // A lane finds the record of its next block from the four record
        // starts after its current one (by bisection beyond).  Entries that
        // pass the filter are appended to the wavefront's ring of candidates,
        // and every 64 candidates are probed together, one per lane.
        const uint32_t lane = tid & 63u, wid = tid >> 6;
        constexpr uint32_t kWaves = kHubB / 64;
        const uint32_t q0 = (uint32_t)(((uint64_t)P * wid) / kWaves), q1 = (uint32_t)(((uint64_t)P * (wid + 1)) / kWaves);
        uint32_t* ring_e = S.ring_e + wid * kHubRing;
        uint32_t* ring_m = S.ring_m + wid * kHubRing;
        uint32_t cnt = 0;   // the same on every lane: ring[0, cnt) waits to be probed
        // Probes ring[l] on the lanes l < c (c <= 64): a hit adds one to the
        // count of its signature.  The hit's direction bits fh are relative
        // to the anchor a, the candidate's fx to the other endpoint x; the
        // anchor is u (then fa = fh, fb = fx) or v (fa = fx, fb = fh).
        auto probe_round = [&](uint32_t c) {
            wave_sync{}();
            if (lane < c) {
                const uint32_t qe = ring_e[lane], qm = ring_m[lane];
                const uint32_t w = qe >> 2, mm = qm >> 26;
                const uint32_t fh = hub_probe<TILE>(S.hash, (qe & ~3u) | (mm << 25), w + (mm << 20));
                if (fh < 4u) {
                    const uint32_t a = S.tk[kTkAnchor + js + mm];
                    const uint32_t x = (qm >> 3) & ((1u << 23) - 1u);
                    const uint32_t sx = (qm & 4u) ? 4u : 2u;
                    const uint32_t code = (qm & 3u) | ((qe & 3u) << sx) | (fh << (6u - sx));
                    const uint32_t where = (w > a ? 1u : 0u) + (w > x ? 1u : 0u);
                    atomicAdd(&S.sig[code | (where << 6)], 1u);
                }
            }
            wave_sync{}();
        };
        if (q0 < q1) {
            uint32_t i = 0;
            {
                // lanes past the quarter's end take its last record and gather nothing
                const uint32_t first = min(q0 + lane, q1 - 1u);
                uint32_t hi = nrec;                     // record holding `first`: off[i] <= first < off[i+1]
                while (hi - i > 1) {
                    const uint32_t mid = (i + hi) >> 1;
                    if (S.off[mid] <= first) i = mid; else hi = mid;
                }
            }
            uint32_t next = S.off[i + 1], p0 = S.pos[i], p1 = S.end[i], m = S.meta[i];
            uint32_t mix = hub_member_mix(m >> 26);
            uint32_t bb = p0 / kHubGather - S.off[i];   // block of flattened index f: bb + f (mod 2^32)
            for (uint32_t win = q0; win < q1; win += 64u) {
                // lanes past the quarter's end read its last block and keep no entry of it
                const uint32_t f = min(win + lane, q1 - 1u);
                if (f >= next) {
                    // The record of f from the next four record starts
                    // (off[nrec ..] = P > f past the last record), and by
                    // bisection when it lies further ahead.
                    const uint32_t o2 = S.off[i + 2], o3 = S.off[i + 3], o4 = S.off[i + 4], o5 = S.off[i + 5];
                    i += 1u + (f >= o2 ? 1u : 0u) + (f >= o3 ? 1u : 0u) + (f >= o4 ? 1u : 0u) + (f >= o5 ? 1u : 0u);
                    next = S.off[i + 1];
                    if (f >= next) {
                        uint32_t hi = nrec;
                        while (hi - i > 1) {
                            const uint32_t mid = (i + hi) >> 1;
                            if (S.off[mid] <= f) i = mid; else hi = mid;
                        }
                        next = S.off[i + 1];
                    }
                    p0 = S.pos[i];
                    p1 = S.end[i];
                    m = S.meta[i];
                    mix = hub_member_mix(m >> 26);
                    bb = p0 / kHubGather - S.off[i];
                }
                const uint32_t b0 = (bb + f) * kHubGather;   // first entry of the block: b0 < p1, p0 < b0 + 8
                const uint4* src = reinterpret_cast<const uint4*>(nbr + b0);
                const uint4 lo4 = src[0], hi4 = src[1];
                const uint32_t e[kHubGather] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
                const uint32_t klo = p0 > b0 ? p0 - b0 : 0u, khi = min(p1 - b0, kHubGather);
                // bit k: word k is an entry of the row (none past the quarter's end)
                const uint32_t vm = win + lane < q1 ? ((1u << khi) - 1u) & ~((1u << klo) - 1u) : 0u;
                // Filter: the word of every entry first, then the bits.
                uint32_t fp[kHubGather], fw[kHubGather];
#pragma unroll
                for (uint32_t k = 0; k < kHubGather; ++k) {
                    fp[k] = G::filter_pos(e[k] >> 2, mix);
                    fw[k] = S.filt[fp[k] >> G::kWordShift];
                }
                // appends: the entries that pass go to ring[cnt ..] in lane order
#pragma unroll
                for (uint32_t k = 0; k < kHubGather; ++k) {
                    const bool pass = ((fw[k] >> (fp[k] & 31u)) & (vm >> k) & 1u) != 0u;
                    const unsigned long long bal = __builtin_amdgcn_ballot_w64(pass);
                    // (the lanes of the mask: the same lanes as pass, without a second compare)
                    if (__builtin_amdgcn_inverse_ballot_w64(bal)) {
                        const uint32_t r = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)bal, cnt));
                        ring_e[r] = e[k];
                        ring_m[r] = m;
                    }
                    cnt += (uint32_t)__popcll(bal);
                    if (cnt >= 64u) {
                        probe_round(64u);
                        cnt -= 64u;
                        // the rest moves to the front
                        uint32_t te = 0, tm = 0;
                        if (lane < cnt) {
                            te = ring_e[64u + lane];
                            tm = ring_m[64u + lane];
                        }
                        wave_sync{}();
                        if (lane < cnt) {
                            ring_e[lane] = te;
                            ring_m[lane] = tm;
                        }
                    }
                }
            }
            if (cnt != 0) probe_round(cnt);
        }
        __syncthreads();
        if (multi_tile)
            for (uint32_t i = tid; i < nrec; i += kHubB) S.pos[i] = S.end[i];
        __syncthreads();
    }
}

// Hub tasks [t0, t1) (at most kHubGroupTasks) on the whole workgroup: their
// descriptors and anchor rows are read once, and runs of consecutive tasks
// whose records fit one chunk and whose anchor rows fit one tile are processed together; a task whose anchor
// row spans several tiles runs alone.
template <uint32_t TILE, class H>
__device__ inline void hub_chunk_run(const hub_task* __restrict__ tasks, uint32_t t0, uint32_t t1,
                                     const dyad_rec* __restrict__ dyads, const uint32_t* __restrict__ nbr,
                                     uint32_t u_lo, uint32_t u_hi, const hub_lds& S, const uint8_t* T, H& h,
                                     uint32_t& since) {
    const uint32_t tid = threadIdx.x, nt = t1 - t0;
    if (tid < nt) {
        const hub_task tk = tasks[t0 + tid];
        const dyad_rec r0 = load_rec(dyads + tk.begin);
        const bool au = r0.u == tk.anchor;
        const uint32_t hb = au ? r0.bu : r0.bv, he = au ? r0.eu : r0.ev;
        S.tk[kTkBegin + tid] = tk.begin;
        S.tk[kTkNrec + tid] = tk.end - tk.begin;
        S.tk[kTkHb + tid] = hb;
        S.tk[kTkLen + tid] = he - hb;
        S.tk[kTkAnchor + tid] = tk.anchor;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t ng = 0, sr = 0, se = 0;
        S.tk[kTkGroups] = 0;
        for (uint32_t j = 0; j < nt; ++j) {
            const uint32_t r = S.tk[kTkNrec + j], l = S.tk[kTkLen + j];
            if (j > S.tk[kTkGroups + ng] && (l > TILE || sr + r > kHubChunk || se + l > TILE)) {
                S.tk[kTkGroups + ++ng] = j;
                sr = 0;
                se = 0;
            }
            sr += r;
            se += l;
        }
        S.tk[kTkGroups + ++ng] = nt;
        S.tk[kTkNGroups] = ng;
    }
    __syncthreads();
    const uint32_t ng = S.tk[kTkNGroups];
    for (uint32_t g = 0; g < ng; ++g) {
        const uint32_t js = S.tk[kTkGroups + g], M = S.tk[kTkGroups + g + 1] - js;
        if (tid == 0) {
            uint32_t r = 0, e = 0;
            for (uint32_t m = 0; m < M; ++m) {
                S.tk[kTkRb + m] = r;
                S.tk[kTkEb + m] = e;
                r += S.tk[kTkNrec + js + m];
                e += S.tk[kTkLen + js + m];
            }
            S.tk[kTkRb + M] = r;
            S.tk[kTkEb + M] = e;
        }
        __syncthreads();
        hub_group_run<TILE>(js, M, dyads, nbr, u_lo, u_hi, S, T, h, since);
        __syncthreads();
    }
}

template <uint32_t TILE>
__global__ __launch_bounds__(kHubB)
__attribute__((amdgpu_waves_per_eu(hub_waves_per_simd<TILE>(), hub_waves_per_simd<TILE>()))) void k_census_hub(
    census_args L, const hub_task* __restrict__ tasks, uint32_t ntasks, uint32_t ngroups, uint32_t g0, uint32_t g1,
    unsigned int* ctr) {
    __shared__ __attribute__((aligned(16))) uint32_t hub_words[hub_lds_words<TILE>()];
    __shared__ unsigned long long bins[block_bins<kHubB>::kWords];
    __shared__ uint8_t T[64];
    __shared__ uint32_t s_next;
    if (threadIdx.x < 64) T[threadIdx.x] = L.table[threadIdx.x];
    block_bins<kHubB> h{bins};
    h.clear();
    const hub_lds S = hub_carve<TILE>(hub_words);
    hub_bins_clear(S);
    __syncthreads();
    uint32_t since = 0;
    const uint32_t xcd = blockIdx.x % kXcds;
    // task groups g0 + k, k taken from the counters, below g1 (<= ngroups)
    if (threadIdx.x == 0) s_next = g0 + take_chunk(ctr, xcd, gridDim.x);
    __syncthreads();
    uint32_t c = s_next;
    __syncthreads();
    while (c < g1) {
        if (threadIdx.x == 0) s_next = g0 + take_chunk(ctr, xcd, gridDim.x);
        const uint32_t t0 = tasks[c].group, t1 = c + 1 < ngroups ? tasks[c + 1].group : ntasks;
        hub_chunk_run<TILE>(tasks, t0, t1, L.dyads, L.nbr, L.u_lo, L.u_hi, S, T, h, since);
        c = s_next;
        __syncthreads();
    }
    hub_bins_flush(S, T, h);
    h.flush(acc_copy(L.acc));
}

// ------------------------------------------------------- forward lists ----
// The four modes over the edge records (tc_tri.h).  Every workgroup counts
// triangle signatures and turns them into class updates when it ends.
template <bool Lab>
__device__ inline void tri_end(tri_sig<Lab>& sig, uint32_t threads, unsigned long long* bins, const uint8_t* T,
                               unsigned long long* acc) {
    constexpr uint32_t kWords = tri_bins<Lab>::kWords;
    for (uint32_t k = threadIdx.x; k < kWords; k += threads) bins[k] = 0;
    tri_bins<Lab> h{bins};
    tri_flush<Lab>(sig, threads, T, h);
    unsigned long long* to = acc_copy(acc, kWords);
    for (uint32_t k = threadIdx.x; k < kWords; k += threads)
        if (bins[k] != 0) atomicAdd(&to[k], bins[k]);
}

template <bool Lab>
__global__ __launch_bounds__(kLaneB) void k_tri_lane(tri_args L) {
    __shared__ unsigned long long n[tri_sig<Lab>::kSlots], bins[tri_bins<Lab>::kWords];
    __shared__ uint8_t T[64];
    if (threadIdx.x < 64) T[threadIdx.x] = L.table[threadIdx.x];
    tri_sig<Lab> sig{n};
    sig.clear(kLaneB);
    __syncthreads();
    for (uint64_t d = (uint64_t)blockIdx.x * kLaneB + threadIdx.x; d < L.count; d += (uint64_t)gridDim.x * kLaneB)
        lane_edge<Lab>(load_edge(L.recs + d), L.fwd, sig);
    tri_end<Lab>(sig, kLaneB, bins, T, L.acc);
}

template <bool Lab, int TW>
__global__ __launch_bounds__(kWaveB) void k_tri_wave(tri_args L, unsigned int* ctr) {
    __shared__ unsigned long long n[tri_sig<Lab>::kSlots], bins[tri_bins<Lab>::kWords];
    __shared__ uint8_t T[64];
    __shared__ uint32_t sA[TW + 1], sB[TW + 1];
    __shared__ uint32_t s_xt;
    T[threadIdx.x] = L.table[threadIdx.x];
    tri_sig<Lab> sig{n};
    sig.clear(kWaveB);
    __syncthreads();
    const uint32_t xcd = blockIdx.x % kXcds;
    uint32_t c = 0;
    if (threadIdx.x == 0) c = take_chunk(ctr, xcd, gridDim.x);
    c = __shfl(c, 0, 64);
    while ((uint64_t)c * kWaveChunk < L.count) {
        uint32_t cn = 0;
        if (threadIdx.x == 0) cn = take_chunk(ctr, xcd, gridDim.x);      // next chunk, fetched early
        const uint32_t end = min(L.count, (c + 1) * kWaveChunk);
        for (uint32_t d = c * kWaveChunk; d < end; ++d) {
            const edge_rec r = load_edge(L.recs + d);
            merge_path<kWaveB, TW, block_sync>(r.bx, r.ex, r.by, r.ey, L.fwd, sA, sB, &s_xt, threadIdx.x,
                                               edge_rows<Lab>{r.code<Lab>(), sig});
        }
        c = __shfl(cn, 0, 64);
    }
    tri_end<Lab>(sig, kWaveB, bins, T, L.acc);
}

template <bool Lab, int B, int TW>
__global__ __launch_bounds__(B) void k_tri_group(tri_args L, unsigned int* ctr) {
    __shared__ unsigned long long n[tri_sig<Lab>::kSlots], bins[tri_bins<Lab>::kWords];
    __shared__ uint8_t T[64];
    __shared__ uint32_t sA[TW + 1], sB[TW + 1];
    __shared__ uint32_t s_xt, s_next;
    if (threadIdx.x < 64) T[threadIdx.x] = L.table[threadIdx.x];
    tri_sig<Lab> sig{n};
    sig.clear(B);
    const uint32_t xcd = blockIdx.x % kXcds;
    if (threadIdx.x == 0) s_next = take_chunk(ctr, xcd, gridDim.x);
    __syncthreads();
    uint32_t c = s_next;
    __syncthreads();
    while ((uint64_t)c * kGroupChunk < L.count) {
        if (threadIdx.x == 0) s_next = take_chunk(ctr, xcd, gridDim.x);  // next chunk, fetched early
        const uint32_t end = min(L.count, (c + 1) * kGroupChunk);
        for (uint32_t d = c * kGroupChunk; d < end; ++d) {
            const edge_rec r = load_edge(L.recs + d);
            merge_path<B, TW, block_sync>(r.bx, r.ex, r.by, r.ey, L.fwd, sA, sB, &s_xt, threadIdx.x,
                                          edge_rows<Lab>{r.code<Lab>(), sig});
        }
        __syncthreads();
        c = s_next;
        __syncthreads();
    }
    tri_end<Lab>(sig, B, bins, T, L.acc);
}

// Hub tasks, a wavefront each.  The first `heavy` tasks are handed out one at a
// time, those after them (of vertices with few records) in runs of
// kTriLightTasks, so that handing out does not bound them.
constexpr uint32_t kTriLightTasks = 8;
constexpr int kTriB = 256;
constexpr uint32_t kTriWaves = kTriB / 64;
// Wavefronts per SIMD the hub kernels are compiled for: five or six (96 or 80
// registers) measured the same, seven spill (R-MAT 2^20 with eight workgroups per
// CU: 0.89, 0.89, 0.93 ms).
constexpr int kTriWavesPerSimd = 5;

// The LDS of a hub workgroup.
template <bool Lab>
struct tri_lds {
    uint4 tab[kTriWaves][tri_table<Lab>::kWords / 4];
    uint32_t starts[kTriWaves][kTriSegment / 32];
};

// The tasks that this wavefront of workgroup `block` (of `blocks`) takes.
template <bool Lab>
__device__ inline void tri_tasks(const uint4* __restrict__ recs, const uint32_t* __restrict__ fwd,
                                 const tri_task* __restrict__ tasks, uint32_t ntasks, uint32_t heavy,
                                 unsigned int* ctr, uint32_t block, uint32_t blocks, tri_lds<Lab>& S,
                                 tri_sig<Lab>& sig) {
    const uint32_t wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    tri_counts cnt;
    cnt.clear();
    const uint32_t xcd = block % kXcds, waves = blocks * kTriWaves;
    uint32_t u = block * kTriWaves + wid;                     // the first unit needs no counter
    const uint32_t units = heavy + (ntasks - heavy + kTriLightTasks - 1) / kTriLightTasks;
    while (u < units) {
        uint32_t next = 0;
        if (__lane_id() == 0) next = waves + take_chunk(ctr, xcd, blocks);    // fetched early
        uint32_t k = u < heavy ? u : heavy + (u - heavy) * kTriLightTasks;
        const uint32_t last = u < heavy ? u + 1 : min(k + kTriLightTasks, ntasks);
        for (; k < last; ++k) {
            const tri_task t = tasks[k];
            tri_run<Lab>(recs, fwd, t.begin, t.end, t.by, t.ey, reinterpret_cast<uint32_t*>(S.tab[wid]),
                         S.starts[wid], sig, cnt);
        }
        u = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
    }
    if constexpr (!Lab) cnt.flush(sig);
}

template <bool Lab>
__global__ __launch_bounds__(kTriB) __attribute__((amdgpu_waves_per_eu(Lab ? 4 : kTriWavesPerSimd))) void k_tri_hub(
    tri_args L, const tri_task* __restrict__ tasks, uint32_t ntasks, uint32_t heavy, unsigned int* ctr) {
    __shared__ tri_lds<Lab> S;
    __shared__ unsigned long long n[tri_sig<Lab>::kSlots], bins[tri_bins<Lab>::kWords];
    __shared__ uint8_t T[64];
    if (threadIdx.x < 64) T[threadIdx.x] = L.table[threadIdx.x];
    tri_sig<Lab> sig{n};
    sig.clear(kTriB);
    __syncthreads();
    tri_tasks<Lab>(L.recs, L.fwd, tasks, ntasks, heavy, ctr, blockIdx.x, gridDim.x, S, sig);
    tri_end<Lab>(sig, kTriB, bins, T, L.acc);
}

// A whole census in one launch: the first workgroups run the hub tasks, the
// next the lane bucket, the others the terms without intersection, and the last
// one to end writes the sums.  A small census is bound by its launches (of three
// or four, 24 us for 2000 vertices and 8000 arcs, 19 in one; the copy-free
// launch and wait for one kernel is most of it); beside the hub tasks the other
// ranges start as soon as a CU has room for them, without events.  The rule of
// its use and more times: launch_one.
struct one_args {
    tri_args lane;               // its accumulators and table serve all
    const uint4* recs;           // hub records
    const tri_task* tasks;
    uint32_t ntasks, heavy, hub_blocks, lane_blocks;
    const uint4* rinfo;
    uint32_t x0, x1;             // rows of the terms (16 classes)
    const uint32_t* nbr;         // entries of the terms (64 codes)
    const uint32_t* owner;
    const uint64_t* tpre;
    uint64_t U;
    uint64_t n, asym, mutual;
    unsigned int* counters;
    unsigned long long* out;
};

// True in the workgroup that calls it last.  Two levels of counters, since
// adds to one line take about 12 ns each.  Nobody waits.
__device__ inline bool last_to_end(unsigned int* ctr, unsigned int* top) {
    __shared__ uint32_t s_last;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t g = blockIdx.x % kXcds, members = (gridDim.x - g + kXcds - 1) / kXcds;
        bool last = atomicAdd(&ctr[g * kCounterStride], 1u) + 1 == members;
        if (last) last = atomicAdd(top, 1u) + 1 == min(gridDim.x, (uint32_t)kXcds);
        s_last = last;
    }
    __syncthreads();
    return s_last != 0;
}

// The labelled terms' slots take the place of the hub tables (two lanes to a
// column, 21 KB).
constexpr uint32_t kOneCols = kTriB / 2;
static_assert(kTriB == kLaneB, "the terms' steps are of kLaneB threads");

template <bool Lab>
__global__ __launch_bounds__(kTriB) __attribute__((amdgpu_waves_per_eu(Lab ? 4 : kTriWavesPerSimd))) void k_tri_one(
    one_args A) {
    constexpr uint32_t kWords = tri_bins<Lab>::kWords, kSlots = totals_slot_count<Lab>();
    __shared__ tri_lds<Lab> S;
    __shared__ unsigned long long n[tri_sig<Lab>::kSlots], bins[kWords], sums[kTriB];
    __shared__ uint8_t T[64];
    if (threadIdx.x < 64) T[threadIdx.x] = A.lane.table[threadIdx.x];
    if (threadIdx.x < kWords) bins[threadIdx.x] = 0;
    tri_sig<Lab> sig{n};
    sig.clear(kTriB);
    tri_bins<Lab> h{bins};
    __syncthreads();
    const uint32_t terms = A.hub_blocks + A.lane_blocks;
    if (blockIdx.x < terms) {
        if (blockIdx.x < A.hub_blocks) {
            tri_tasks<Lab>(A.recs, A.lane.fwd, A.tasks, A.ntasks, A.heavy, A.counters + kBucketHub * kCounterWords,
                           blockIdx.x, A.hub_blocks, S, sig);
        } else {
            for (uint64_t d = (uint64_t)(blockIdx.x - A.hub_blocks) * kTriB + threadIdx.x; d < A.lane.count;
                 d += (uint64_t)A.lane_blocks * kTriB)
                lane_edge<Lab>(load_edge(A.lane.recs + d), A.lane.fwd, sig);
        }
        tri_flush<Lab>(sig, kTriB, T, h);
    } else if constexpr (Lab) {
        static_assert(sizeof(S.tab) >= sizeof(unsigned long long) * kSlots * kOneCols, "the slots fit");
        __shared__ uint8_t TS[64];
        __shared__ uint32_t bin_of_slot[kSlots];
        unsigned long long* sbins = reinterpret_cast<unsigned long long*>(S.tab);
        (void)totals_slots<true>(T, TS, bin_of_slot);
        for (uint32_t k = threadIdx.x; k < kSlots * kOneCols; k += kTriB) sbins[k] = 0;
        __syncthreads();
        slot_bins<kOneCols> hs{sbins};
        for (uint64_t base = (uint64_t)(blockIdx.x - terms) * kTriB * kTotalsPer; base < A.U;
             base += (uint64_t)(gridDim.x - terms) * kTriB * kTotalsPer)
            totals_entries<kTotalsPer, kTriB, false>(base, A.U, A.nbr, A.owner, A.rinfo, A.tpre, A.n, TS, hs);
        slots_flush<kOneCols>(sbins, bin_of_slot, kSlots, kWords, h);
        __syncthreads();
    } else {
        unsigned long long s[kRowSums] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (blockIdx.x == terms && threadIdx.x == 0) {
            s[0] = A.n * A.asym;
            s[1] = A.n * A.mutual;
        }
        for (uint64_t x = (uint64_t)A.x0 + (uint64_t)(blockIdx.x - terms) * kTriB + threadIdx.x; x < A.x1;
             x += (uint64_t)(gridDim.x - terms) * kTriB)
            row_add(A.rinfo, (uint32_t)x, s);
        row_flush(s, T, h);
        __syncthreads();
    }
    // The old value is waited for, so that the sum is in place before the
    // workgroup says that it has ended; the last one reads with atomics too.
    if (threadIdx.x < kWords && bins[threadIdx.x] != 0) {
        const unsigned long long old = atomicAdd(&acc_copy(A.lane.acc, kWords)[threadIdx.x], bins[threadIdx.x]);
        asm volatile("" ::"v"(old) : "memory");
    }
    if (!last_to_end(A.counters, A.counters + kCounterWords)) return;
    unsigned long long v = 0;
    for (uint32_t k = threadIdx.x; k < kWords * kAccCopies; k += kTriB) v += atomicExch(&A.lane.acc[k], 0ull);
    sums[threadIdx.x] = v;
    if (threadIdx.x < kBuckets * kXcds) A.counters[threadIdx.x * kCounterStride] = 0;
    __syncthreads();
    if (threadIdx.x < kWords) {
        unsigned long long s = 0;
        for (uint32_t c = threadIdx.x; c < kTriB; c += kWords) s += sums[c];
        A.out[threadIdx.x] = s;
    }
}

// --------------------------------------------------------------- batch ----
// Persistent launches over the work items of many resident graphs: the hub
// tasks of every graph's forward lists (k_tri_batch), the hub task groups of
// the graphs that run their dyad records (k_census_batch_hub), then the other
// items (k_census_batch).  A
// workgroup takes items one at a time (per-XCD counters); an item is a slice
// of one graph's bucket, over its dyad records or its forward-list edge
// records: up to 256 lane-mode records (one per thread), up to
// 4 * kBatchWavePerItem wave-mode records (wavefront w takes every fourth), one
// group-mode record, one group of hub tasks, or a chunk of the rows.  Counts go
// to per-wavefront bins that are flushed into the graph's 16 accumulators
// whenever the workgroup moves to another graph.
constexpr int kBatchB = 256;
// The tile area of k_census_batch for wave-mode tile TW (the tunable batch
// tile; the group-mode tile is 4 TW): four wavefronts' pairs of TW-entry
// tiles, or one pair of 4 TW-entry tiles.
template <int TW>
constexpr int batch_tile_words() {
    return (4 * 2 * (TW + 1) > 2 * (4 * TW + 1)) ? 4 * 2 * (TW + 1) : 2 * (4 * TW + 1);
}

// The copy of a graph's accumulators this workgroup adds to.  A workgroup adds
// its sums whenever it moves on to another graph, and the workgroups at one
// graph are many (13 atomics each on one line, about 12 ns apiece).
__device__ inline unsigned long long* batch_acc(unsigned long long* accs, uint32_t graph) {
    return accs + (uint64_t)kNumClasses * ((uint64_t)kBatchCopies * graph + blockIdx.x % kBatchCopies);
}

// The hub tasks of the forward lists: an item is a run of tasks of one graph,
// which its four wavefronts take in turn.
__global__ __launch_bounds__(kTriB) __attribute__((amdgpu_waves_per_eu(kTriWavesPerSimd))) void k_tri_batch(const graph_desc* __restrict__ G,
                                                     const work_item* __restrict__ items,
                                                     const uint32_t* __restrict__ nums,
                                                     unsigned long long* __restrict__ accs,
                                                     unsigned int* __restrict__ ctr) {
    __shared__ uint4 tab[kTriWaves][tri_table<false>::kWords / 4];
    __shared__ uint32_t starts[kTriWaves][kTriSegment / 32];
    __shared__ unsigned long long n[tri_sig<false>::kSlots], bins[kNumClasses];
    __shared__ uint8_t T[64];
    __shared__ uint32_t s_next;
    const uint32_t wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x < 64) T[threadIdx.x] = c_table[threadIdx.x];
    tri_sig<false> sig{n};
    sig.clear(kTriB);
    tri_counts cnt;
    cnt.clear();
    const uint32_t count = nums[0], xcd = blockIdx.x % kXcds;
    uint32_t cur = 0xffffffffu;
    auto flush = [&] {
        cnt.flush(sig);
        if (threadIdx.x < kNumClasses) bins[threadIdx.x] = 0;
        tri_bins<false> h{bins};
        tri_flush<false>(sig, kTriB, T, h);
        if (threadIdx.x < kNumClasses && bins[threadIdx.x] != 0)
            atomicAdd(&batch_acc(accs, cur)[threadIdx.x], bins[threadIdx.x]);
        __syncthreads();
    };
    if (threadIdx.x == 0) s_next = take_chunk(ctr, xcd, gridDim.x);
    __syncthreads();
    uint32_t idx = s_next;
    __syncthreads();
    while (idx < count) {
        if (threadIdx.x == 0) s_next = take_chunk(ctr, xcd, gridDim.x);
        const work_item it = items[idx];
        if (it.graph != cur) {
            if (cur != 0xffffffffu) flush();
            cur = it.graph;
        }
        const graph_desc& g = G[it.graph];
        const uint4* recs = g.edges;
        const uint32_t* fwd = g.fwd;
        const tri_task* tasks = g.edge_tasks;
        for (uint32_t k = it.begin + wid; k < it.end; k += kTriWaves) {
            const tri_task t = tasks[k];
            tri_run<false>(recs, fwd, t.begin, t.end, t.by, t.ey, reinterpret_cast<uint32_t*>(tab[wid]), starts[wid], sig,
                           cnt);
        }
        __syncthreads();
        idx = s_next;
        __syncthreads();
    }
    if (cur != 0xffffffffu) flush();
}

template <uint32_t TILE>
__global__ __launch_bounds__(kHubB)
__attribute__((amdgpu_waves_per_eu(hub_waves_per_simd<TILE>(), hub_waves_per_simd<TILE>()))) void
k_census_batch_hub(
    const graph_desc* __restrict__ G, const work_item* __restrict__ items, const uint32_t* __restrict__ nums,
    unsigned long long* __restrict__ accs, unsigned int* __restrict__ ctr) {
    __shared__ __attribute__((aligned(16))) uint32_t hub_words[hub_lds_words<TILE>()];
    __shared__ unsigned long long bins[block_bins<kHubB>::kWords];
    __shared__ uint8_t T[64];
    __shared__ uint32_t s_next;
    if (threadIdx.x < 64) T[threadIdx.x] = c_table[threadIdx.x];
    block_bins<kHubB> h{bins};
    h.clear();
    const hub_lds S = hub_carve<TILE>(hub_words);
    hub_bins_clear(S);
    __syncthreads();
    const uint32_t item0 = nums[0], count = nums[1];
    const uint32_t xcd = blockIdx.x % kXcds;
    uint32_t cur = 0xffffffffu, since = 0;
    if (threadIdx.x == 0) s_next = item0 + take_chunk(ctr, xcd, gridDim.x);
    __syncthreads();
    uint32_t idx = s_next;
    __syncthreads();
    while (idx < count) {
        if (threadIdx.x == 0) s_next = item0 + take_chunk(ctr, xcd, gridDim.x);
        const work_item it = items[idx];
        if (it.graph != cur) {
            if (cur != 0xffffffffu) {
                hub_bins_flush(S, T, h);
                h.flush(batch_acc(accs, cur));
                __syncthreads();
                h.clear();
            }
            cur = it.graph;
            since = 0;
            __syncthreads();
        }
        const graph_desc g = G[it.graph];
        for (uint32_t k = it.begin; k < it.end; ++k) {
            const uint32_t t0 = g.hub_tasks[k].group;
            const uint32_t t1 = k + 1 < g.hub_groups ? g.hub_tasks[k + 1].group : g.hub_ntasks;
            hub_chunk_run<TILE>(g.hub_tasks, t0, t1, g.dyads, g.nbr, 0u, 0xffffffffu, S, T, h, since);
        }
        idx = s_next;
        __syncthreads();
    }
    if (cur != 0xffffffffu) {
        hub_bins_flush(S, T, h);
        h.flush(batch_acc(accs, cur));
    }
}

// One item in the wave or group mode: records [it.begin, it.end) with the
// lists of `list`, by wavefronts in turn or one record by the workgroup.
// rows(d, bu, eu, bv, ev) gives record d's rows and what a shared vertex means.
template <int TW, class F>
__device__ inline void batch_merge(bool group, const work_item& it, const uint32_t* __restrict__ list, uint32_t* tiles,
                                   uint32_t* s_xt, F rows) {
    const uint32_t tid = threadIdx.x, wid = tid >> 6, lane = tid & 63u;
    uint32_t bu, eu, bv, ev;
    if (group) {
        auto r = rows(it.begin, bu, eu, bv, ev);
        merge_path<kBatchB, 4 * TW, block_sync>(bu, eu, bv, ev, list, tiles, tiles + 4 * TW + 1, &s_xt[0], tid, r);
        return;
    }
    uint32_t* sA = tiles + wid * 2 * (TW + 1);
    uint32_t* sB = sA + TW + 1;
    for (uint32_t d = it.begin + wid; d < it.end; d += kBatchB / 64) {
        auto r = rows(d, bu, eu, bv, ev);
        merge_path<64, TW, wave_sync>(bu, eu, bv, ev, list, sA, sB, &s_xt[wid], lane, r);
    }
}

// Compiled for seven wavefronts per SIMD with 512-entry tiles (72 VGPRs; the
// few values that no longer fit are reloaded once per item): the kernel waits
// on memory, and more resident waves hide more of it than the spills cost.
// Larger tiles are held to fewer waves by their LDS and keep their registers.
template <int TW>
constexpr int batch_min_waves() { return TW <= 512 ? 7 : 1; }
template <int TW>
__global__ __launch_bounds__(kBatchB) __attribute__((amdgpu_waves_per_eu(batch_min_waves<TW>()))) void k_census_batch(
    const graph_desc* __restrict__ G, const work_item* __restrict__ items, const uint32_t* __restrict__ nums,
    unsigned long long* __restrict__ accs, unsigned int* __restrict__ ctr) {
    __shared__ __attribute__((aligned(16))) uint32_t tiles[batch_tile_words<TW>()];
    __shared__ unsigned long long bins[wave_bins<kBatchB>::kWords], n[tri_sig<false>::kSlots];
    __shared__ uint8_t T[64];
    __shared__ uint32_t s_xt[kBatchB / 64], s_next;
    if (threadIdx.x < 64) T[threadIdx.x] = c_table[threadIdx.x];
    wave_bins<kBatchB> h{bins};
    h.clear();
    tri_sig<false> sig{n};
    sig.clear(kBatchB);
    const uint32_t first = nums[1], count = nums[2];
    const uint32_t xcd = blockIdx.x % kXcds;
    const uint32_t tid = threadIdx.x;
    uint32_t cur = 0xffffffffu;
    if (tid == 0) s_next = first + take_chunk(ctr, xcd, gridDim.x);
    __syncthreads();
    uint32_t idx = s_next;
    __syncthreads();
    while (idx < count) {
        if (tid == 0) s_next = first + take_chunk(ctr, xcd, gridDim.x);
        const work_item it = items[idx];
        if (it.graph != cur) {
            if (cur != 0xffffffffu) {
                tri_flush<false>(sig, kBatchB, T, h);
                h.flush(batch_acc(accs, cur));
                __syncthreads();
                h.clear();
            }
            cur = it.graph;
            __syncthreads();
        }
        const graph_desc& g = G[it.graph];
        if (it.kind == kItemRows) {
            unsigned long long rs[kRowSums] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (it.begin == 0 && tid == 0) {
                rs[0] = g.n * g.asym;
                rs[1] = g.n * g.mutual;
            }
            for (uint32_t x = it.begin + tid; x < it.end; x += kBatchB) row_add(g.rinfo, x, rs);
            row_flush(rs, T, h);
        } else if (it.kind & kItemTri) {
            const uint4* recs = g.edges;
            const uint32_t* fwd = g.fwd;
            if ((it.kind & 3u) == kItemLane) {
                if (it.begin + tid < it.end) lane_edge<false>(load_edge(recs + it.begin + tid), fwd, sig);
            } else {
                batch_merge<TW>((it.kind & 3u) == kItemGroup, it, fwd, tiles, s_xt,
                                [&](uint32_t d, uint32_t& bu, uint32_t& eu, uint32_t& bv, uint32_t& ev) {
                                    const edge_rec r = load_edge(recs + d);
                                    bu = r.bx;
                                    eu = r.ex;
                                    bv = r.by;
                                    ev = r.ey;
                                    return edge_rows<false>{r.code<false>(), sig};
                                });
            }
        } else {
            const dyad_rec* recs = g.dyads;
            const uint32_t* nbr = g.nbr;
            if (it.kind == kItemLane) {
                if (it.begin + tid < it.end) lane_dyad(load_rec(recs + it.begin + tid), nbr, T, h);
            } else {
                dyad_rec r;
                batch_merge<TW>(it.kind == kItemGroup, it, nbr, tiles, s_xt,
                                [&](uint32_t d, uint32_t& bu, uint32_t& eu, uint32_t& bv, uint32_t& ev) {
                                    r = load_rec(recs + d);
                                    bu = r.bu;
                                    eu = r.eu;
                                    bv = r.bv;
                                    ev = r.ev;
                                    return dyad_rows<wave_bins<kBatchB>>{r, T, h};
                                });
            }
        }
        __syncthreads();
        idx = s_next;
        __syncthreads();
    }
    if (cur != 0xffffffffu) {
        tri_flush<false>(sig, kBatchB, T, h);
        h.flush(batch_acc(accs, cur));
    }
}

// The sums of every graph's copies, to pinned host memory.
__global__ __launch_bounds__(256) void k_batch_finish(const unsigned long long* __restrict__ accs, uint32_t graphs,
                                                      unsigned long long* __restrict__ out) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x, graph = i / kNumClasses, cls = i % kNumClasses;
    if (graph >= graphs) return;
    unsigned long long s = 0;
    for (uint32_t c = 0; c < kBatchCopies; ++c)
        s += accs[(uint64_t)kNumClasses * ((uint64_t)kBatchCopies * graph + c) + cls];
    out[i] = s;
}

__global__ void k_fill_u64_grid(unsigned long long* p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__global__ void k_zero_counters(unsigned int* p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x * kCounterStride] = 0;
}

// End of a census: the sums of the accumulators' copies go to `out` (pinned
// host memory), and accumulators and work counters are zero again for the next
// census, which so needs no clearing launches and no copy.
constexpr int kFinishT = 512;
template <int W>
__global__ __launch_bounds__(kFinishT) void k_census_finish(unsigned long long* __restrict__ acc,
                                                            unsigned int* __restrict__ counters,
                                                            unsigned long long* __restrict__ out) {
    static_assert(kFinishT % W == 0, "a thread's accumulators belong to one bin");
    __shared__ unsigned long long sh[kFinishT];
    unsigned long long v = 0;
    for (int k = threadIdx.x; k < W * kAccCopies; k += kFinishT) {
        v += acc[k];
        acc[k] = 0;
    }
    sh[threadIdx.x] = v;
    if (threadIdx.x < kBuckets * kXcds) counters[threadIdx.x * kCounterStride] = 0;
    __syncthreads();
    if (threadIdx.x < W) {
        unsigned long long s = 0;
        for (int c = threadIdx.x; c < kFinishT; c += W) s += sh[c];
        out[threadIdx.x] = s;
    }
}

__global__ __launch_bounds__(kFinishT) void k_census_clear(unsigned long long* __restrict__ acc, int words,
                                                           unsigned int* __restrict__ counters) {
    for (int k = threadIdx.x; k < words; k += kFinishT) acc[k] = 0;
    if (threadIdx.x < kBuckets * kXcds) counters[threadIdx.x * kCounterStride] = 0;
}

}  // namespace

bool tile_supported(uint32_t hub_tile, uint32_t wave_tile, uint32_t group_tile, uint32_t group_size,
                    uint32_t batch_tile) {
    const bool hub = hub_tile == 512 || hub_tile == 1024 || hub_tile == 2048;
    const bool wave = wave_tile == 512 || wave_tile == 1024 || wave_tile == 2048;
    const bool group = group_tile == 2048 || group_tile == 4096 || group_tile == 8192;
    const bool gsize = group_size == 256 || group_size == 512;
    const bool batch = batch_tile == 512 || batch_tile == 1024 || batch_tile == 2048;
    return hub && wave && group && gsize && batch;
}

namespace {

template <uint32_t HT, int BT>
hipError_t launch_batch_kernels(const batch_buffers& b, hipStream_t s) {
    // The other items' kernel gets a branch of its own: it fills what the hub
    // kernels leave, above all their ends.  512 R-MAT graphs of 50 to 20000 rows:
    // 0.88 ms one after the other, 0.75 ms side by side; 16 of them 124 and 97 us.
    hipStream_t rest = s;
    if (b.side) {
        hipError_t e = hipEventRecord(b.fork[0], s);
        if (e == hipSuccess) e = hipStreamWaitEvent(b.side, b.fork[0], 0);
        if (e != hipSuccess) return e;
        rest = b.side;
    }
    if (b.tri_grid)
        hipLaunchKernelGGL(k_tri_batch, dim3(b.tri_grid), dim3(kTriB), 0, s, b.descs, b.items, b.nums, b.accs,
                           b.counters);
    if (b.hub_grid)
        hipLaunchKernelGGL((k_census_batch_hub<HT>), dim3(b.hub_grid), dim3(kHubB), 0, s, b.descs, b.items, b.nums,
                           b.accs, b.counters + kCounterWords);
    hipLaunchKernelGGL(k_census_batch<BT>, dim3(b.grid), dim3(kBatchB), 0, rest, b.descs, b.items, b.nums, b.accs,
                       b.counters + 2 * kCounterWords);
    if (b.side) {
        hipError_t e = hipEventRecord(b.fork[1], b.side);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, b.fork[1], 0);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_batch_finish, dim3((b.graphs * kNumClasses + 255) / 256), dim3(256), 0, s, b.accs, b.graphs,
                       b.out);
    return hipGetLastError();
}

template <uint32_t HT>
hipError_t launch_batch_bt(uint32_t bt, const batch_buffers& b, hipStream_t s) {
    if (bt == 512) return launch_batch_kernels<HT, 512>(b, s);
    if (bt == 1024) return launch_batch_kernels<HT, 1024>(b, s);
    return launch_batch_kernels<HT, 2048>(b, s);
}

}  // namespace

hipError_t batch_launch(const batch_buffers& b, uint32_t hub_tile, uint32_t batch_tile, hipStream_t s) {
    if (!tile_supported(hub_tile, 1024, 4096, 256, batch_tile) || b.graphs == 0) return hipErrorInvalidValue;
    const uint64_t acc_words = kBatchAccWords * b.graphs;
    uint32_t zb = (uint32_t)std::min<uint64_t>((acc_words + 255) / 256, 1024);
    hipLaunchKernelGGL(k_fill_u64_grid, dim3(zb ? zb : 1), dim3(256), 0, s, b.accs, acc_words);
    hipLaunchKernelGGL(k_zero_counters, dim3(1), dim3(64), 0, s, b.counters, 3 * kXcds);
    if (hub_tile == 512) return launch_batch_bt<512>(batch_tile, b, s);
    if (hub_tile == 1024) return launch_batch_bt<1024>(batch_tile, b, s);
    return launch_batch_bt<2048>(batch_tile, b, s);
}

hipError_t census_upload_table() {
    return hipMemcpyToSymbol(HIP_SYMBOL(c_table), kTable.t, sizeof(kTable.t));
}

namespace {

void launch_bucket(int b, const census_args& L, uint64_t cnt, const census_config& cfg, unsigned int* counters,
                   hipStream_t s) {
    if (b == 0) {
        uint32_t grid = (uint32_t)std::min<uint64_t>((cnt + kLaneB - 1) / kLaneB, cfg.lane_blocks);
        hipLaunchKernelGGL(k_census_lane, dim3(grid), dim3(kLaneB), 0, s, L);
    } else if (b == 1) {
        const dim3 grid((uint32_t)std::min<uint64_t>(cnt, cfg.wave_blocks));
        unsigned int* c = counters + kCounterWords;
        if (cfg.wave_tile == 512) hipLaunchKernelGGL((k_census_wave<512>), grid, dim3(kWaveB), 0, s, L, c);
        else if (cfg.wave_tile == 1024) hipLaunchKernelGGL((k_census_wave<1024>), grid, dim3(kWaveB), 0, s, L, c);
        else hipLaunchKernelGGL((k_census_wave<2048>), grid, dim3(kWaveB), 0, s, L, c);
    } else if (b == 2) {
        const dim3 grid((uint32_t)std::min<uint64_t>(cnt, cfg.group_blocks));
        unsigned int* c = counters + 2 * kCounterWords;
        if (cfg.group_size == 256) {
            if (cfg.group_tile == 2048) hipLaunchKernelGGL((k_census_group<256, 2048>), grid, dim3(256), 0, s, L, c);
            else if (cfg.group_tile == 4096) hipLaunchKernelGGL((k_census_group<256, 4096>), grid, dim3(256), 0, s, L, c);
            else hipLaunchKernelGGL((k_census_group<256, 8192>), grid, dim3(256), 0, s, L, c);
        } else {
            if (cfg.group_tile == 2048) hipLaunchKernelGGL((k_census_group<512, 2048>), grid, dim3(512), 0, s, L, c);
            else if (cfg.group_tile == 4096) hipLaunchKernelGGL((k_census_group<512, 4096>), grid, dim3(512), 0, s, L, c);
            else hipLaunchKernelGGL((k_census_group<512, 8192>), grid, dim3(512), 0, s, L, c);
        }
    }
}

// Dyad task groups [g0, g1) of the ngroups.
void launch_hub(const census_args& L, const hub_task* tasks, uint32_t ntasks, uint32_t ngroups, uint32_t g0,
                uint32_t g1, const census_config& cfg, unsigned int* counters, hipStream_t s) {
    unsigned int* c = counters + 3 * kCounterWords;
    const dim3 grid((uint32_t)std::min<uint64_t>(g1 - g0, cfg.hub_blocks));
    if (cfg.hub_tile == 512)
        hipLaunchKernelGGL((k_census_hub<512>), grid, dim3(kHubB), 0, s, L, tasks, ntasks, ngroups, g0, g1, c);
    else if (cfg.hub_tile == 1024)
        hipLaunchKernelGGL((k_census_hub<1024>), grid, dim3(kHubB), 0, s, L, tasks, ntasks, ngroups, g0, g1, c);
    else
        hipLaunchKernelGGL((k_census_hub<2048>), grid, dim3(kHubB), 0, s, L, tasks, ntasks, ngroups, g0, g1, c);
}

// Workgroups for nt hub tasks of the edge records.  Below 16 tasks per wave of
// tri_blocks, more of them even out the ends (R-MAT 50021 with 3.8 tasks per
// wave: 0.093 ms and 0.0905 ms).
uint32_t tri_grid(uint32_t nt, const census_config& cfg) {
    const uint32_t wgs = (nt + kTriWaves - 1) / kTriWaves;
    return std::min(wgs, wgs >= 16 * (uint64_t)cfg.tri_blocks ? cfg.tri_blocks : cfg.hub_blocks);
}

// Edge records of bucket b; for the hub bucket, the tasks [g0, g1).
template <bool Lab>
void launch_tri(int b, const tri_args& L, const rec_set<uint4, tri_task>& edges, uint32_t g0, uint32_t g1,
                const census_config& cfg, unsigned int* counters, hipStream_t s) {
    unsigned int* c = counters + b * kCounterWords;
    if (b == 0) {
        const uint32_t grid = (uint32_t)std::min<uint64_t>((L.count + kLaneB - 1) / kLaneB, cfg.lane_blocks);
        hipLaunchKernelGGL((k_tri_lane<Lab>), dim3(grid), dim3(kLaneB), 0, s, L);
    } else if (b == 1) {
        const dim3 grid(std::min(L.count, cfg.wave_blocks));
        if (cfg.wave_tile == 512) hipLaunchKernelGGL((k_tri_wave<Lab, 512>), grid, dim3(kWaveB), 0, s, L, c);
        else if (cfg.wave_tile == 1024) hipLaunchKernelGGL((k_tri_wave<Lab, 1024>), grid, dim3(kWaveB), 0, s, L, c);
        else hipLaunchKernelGGL((k_tri_wave<Lab, 2048>), grid, dim3(kWaveB), 0, s, L, c);
    } else if (b == 2) {
        const dim3 grid(std::min(L.count, cfg.group_blocks));
        if (cfg.group_size == 256) {
            if (cfg.group_tile == 2048) hipLaunchKernelGGL((k_tri_group<Lab, 256, 2048>), grid, dim3(256), 0, s, L, c);
            else if (cfg.group_tile == 4096) hipLaunchKernelGGL((k_tri_group<Lab, 256, 4096>), grid, dim3(256), 0, s, L, c);
            else hipLaunchKernelGGL((k_tri_group<Lab, 256, 8192>), grid, dim3(256), 0, s, L, c);
        } else {
            if (cfg.group_tile == 2048) hipLaunchKernelGGL((k_tri_group<Lab, 512, 2048>), grid, dim3(512), 0, s, L, c);
            else if (cfg.group_tile == 4096) hipLaunchKernelGGL((k_tri_group<Lab, 512, 4096>), grid, dim3(512), 0, s, L, c);
            else hipLaunchKernelGGL((k_tri_group<Lab, 512, 8192>), grid, dim3(512), 0, s, L, c);
        }
    } else {
        const uint32_t nt = g1 - g0, heavy = std::min(nt, edges.n_heavy > g0 ? edges.n_heavy - g0 : 0u);
        const dim3 grid(tri_grid(nt, cfg));
        hipLaunchKernelGGL((k_tri_hub<Lab>), grid, dim3(kTriB), 0, s, L, (const tri_task*)edges.tasks + g0, nt, heavy, c);
    }
}

// Launches k_tri_one if the census is one for it: whole rows' terms, no wave or
// group records and no events between the kernels.  Without hub work the lane
// bucket is the census, and runs eight waves per SIMD in its own kernel, five in
// this one: up to 4096 workgroups the launches cost more (sparse graphs of 4
// arcs per vertex, separate and one: 2000 vertices 22.8 and 19.2 us, 60 k 23.5
// and 20.3, 150 k with 1650 lane workgroups 26.4 and 24.1, 400 k with 4402 37.2
// and 36.5, 3 M 192 and 198).  When the hub tasks stream more than the graph has
// entries the lane bucket runs beside them, and one launch needs no second
// stream and no events for that (skewed graphs of 12 arcs per vertex: 20 k
// vertices 50.3 and 31.4 us, 150 k 115 and 86.5, 1 M 416 and 397; R-MAT 50021 88
// and 62, 2^20 881 and 863; labelled, 131071 vertices 152 and 103, 2.5 M 1595 and
// 1332).
constexpr uint32_t kOneLanes = 4096;
bool launch_one(bool lab, const device_graph& g, const census_slices& sl, uint32_t g0, uint32_t g1,
                const uint8_t* table, unsigned long long* acc, unsigned int* counters, unsigned long long* out, const census_config& cfg,
                hipEvent_t* ev, hipStream_t s) {
    const uint64_t lanes = sl.end[0] > sl.begin[0] ? sl.end[0] - sl.begin[0] : 0;
    if (ev || sl.range || g.p == 0 || sl.end[1] > sl.begin[1] || sl.end[2] > sl.begin[2] ||
        (lanes > kOneLanes * (uint64_t)kTriB && g.tri.edges.stream <= g.U))
        return false;
    const rec_set<uint4, tri_task>& edges = g.tri.edges;
    one_args A{};
    A.lane = tri_args{edges.recs + sl.begin[0], (uint32_t)lanes, g.tri.fwd, acc, table};
    A.recs = edges.recs;
    A.tasks = (const tri_task*)edges.tasks + g0;
    A.ntasks = g1 - g0;
    A.heavy = std::min(A.ntasks, edges.n_heavy > g0 ? edges.n_heavy - g0 : 0u);
    A.hub_blocks = A.ntasks ? tri_grid(A.ntasks, cfg) : 0;
    A.lane_blocks = (uint32_t)std::min<uint64_t>((lanes + kTriB - 1) / kTriB, cfg.lane_blocks);
    A.rinfo = g.rinfo;
    A.x0 = sl.row_begin;
    A.x1 = sl.row_end;
    A.n = (uint64_t)g.n;
    A.asym = sl.asym;
    A.mutual = sl.mutual;
    A.counters = counters;
    A.out = out;
    if (lab) {
        A.nbr = g.nbr;
        A.owner = g.owner;
        A.tpre = g.tpre;
        A.U = g.U;
        // (four per CU, what fits: one and two take 105 to 112 us where four take
        // 103 on 131071 skewed vertices, 1642 and 1429 where four take 1332 on 2.5 M)
        const uint32_t tw = (uint32_t)std::min<uint64_t>((g.U + kTotalsPer * kTriB - 1) / (kTotalsPer * kTriB),
                                                         4 * (uint64_t)cfg.side_blocks);
        hipLaunchKernelGGL(k_tri_one<true>, dim3(A.hub_blocks + A.lane_blocks + tw), dim3(kTriB), 0, s, A);
    } else {
        const uint64_t rows = sl.row_end - sl.row_begin;
        const uint32_t rw =
            (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((rows + kTriB - 1) / kTriB, cfg.side_blocks));
        hipLaunchKernelGGL(k_tri_one<false>, dim3(A.hub_blocks + A.lane_blocks + rw), dim3(kTriB), 0, s, A);
    }
    return true;
}

}  // namespace

hipError_t census_clear(unsigned long long* acc, int words, unsigned int* counters, hipStream_t s) {
    hipLaunchKernelGGL(k_census_clear, dim3(1), dim3(kFinishT), 0, s, acc, words, counters);
    return hipGetLastError();
}

namespace {

// The terms of a census of a range: from all entries of the graph where the
// range's rows hold a sixteenth of them or more.  A share of 1, 1/4, 1/16 and
// 1/32 of 10^5 vertices with 200 neighbours each takes 1.35, 0.55, 0.35 and 0.31
// ms so, and 2.42, 0.77, 0.38 and 0.30 with look-ups; of a citation graph of 10^6
// vertices 317, 177, 146, 139 us and 556, 219, 145, 128.  (Two look-ups per dyad
// in the bucket kernels, whose lanes wait for one another: 2.11, 0.68, 0.41,
// 0.35 ms on the former.)
constexpr uint64_t kRangeEntries = 16;
void range_terms(const device_graph& g, const census_slices& sl, const uint8_t* table, unsigned long long* acc,
                 const census_config& cfg, hipStream_t s) {
    const uint64_t mine = sl.ent_end - sl.ent_begin;
    if (mine == 0) return;
    const bool all = mine * kRangeEntries >= g.U;
    const uint64_t per = all ? kTotalsPer * kLaneB : kLaneB, count = all ? g.U : mine;
    const dim3 grid((uint32_t)std::min<uint64_t>((count + per - 1) / per, 8 * (uint64_t)cfg.side_blocks));
    if (all)
        hipLaunchKernelGGL(k_range_terms<true>, grid, dim3(kLaneB), 0, s, g.nbr, g.owner, g.rinfo, g.tpre, 0ull, g.U,
                           sl.u_lo, sl.u_hi, (uint64_t)g.n, table, acc);
    else
        hipLaunchKernelGGL(k_range_terms<false>, grid, dim3(kLaneB), 0, s, g.nbr, g.owner, g.rinfo, g.tpre,
                           sl.ent_begin, sl.ent_end, sl.u_lo, sl.u_hi, (uint64_t)g.n, table, acc);
}

}  // namespace

hipError_t census_launch(const device_graph& g, const census_slices& sl, bool tri, const uint8_t* table,
                         census_kind kind, unsigned long long* acc, unsigned int* counters, unsigned long long* out,
                         const census_config& cfg, hipStream_t s, hipEvent_t* ev, hipStream_t side, hipEvent_t* fork) {
    if (!tile_supported(cfg.hub_tile, cfg.wave_tile, cfg.group_tile, cfg.group_size, 1024))
        return hipErrorInvalidValue;
    const bool lab = tri && kind == kLabelled;
    const uint32_t ngroups = tri ? g.tri.edges.n_tasks : g.n_hub_groups;
    const uint32_t hg0 = std::min(sl.hub_g0, ngroups), hg1 = std::max(hg0, std::min(sl.hub_g1, ngroups));
    if (tri && kind != kLabelledPass && launch_one(lab, g, sl, hg0, hg1, table, acc, counters, out, cfg, ev, s))
        return hipGetLastError();
    // The terms without intersection and the lane bucket wait on memory:
    // beside the hub kernel, they use what it leaves (only when the hub kernel
    // has more to stream than the graph has entries).
    const bool beside = tri && side != nullptr && fork != nullptr && g.tri.edges.stream > g.U;
    hipStream_t ts = s;
    if (beside) {
        hipError_t e = hipEventRecord(fork[0], s);
        if (e == hipSuccess) e = hipStreamWaitEvent(side, fork[0], 0);
        if (e != hipSuccess) return e;
        ts = side;
    }
    auto terms = [&] {
        if (ev) (void)hipEventRecord(ev[2 * kBuckets], ts);
        if (sl.range) {
            range_terms(g, sl, table, acc, cfg, ts);
        } else if (g.p > 0) {
            if (kind != kClasses) {
                const uint32_t grid = (uint32_t)std::min<uint64_t>(
                    (g.U + kTotalsPer * kLaneB - 1) / (kTotalsPer * kLaneB), beside ? cfg.side_blocks : cfg.lane_blocks);
                if (lab)
                    hipLaunchKernelGGL(k_census_totals<true>, dim3(grid), dim3(kLaneB), 0, ts, g.nbr, g.owner, g.rinfo,
                                       g.tpre, g.U, (uint64_t)g.n, table, acc);
                else
                    hipLaunchKernelGGL(k_census_totals<false>, dim3(grid), dim3(kLaneB), 0, ts, g.nbr, g.owner, g.rinfo,
                                       g.tpre, g.U, (uint64_t)g.n, table, acc);
            } else {
                // (few workgroups: each ends with eight atomics)
                const uint64_t rows = sl.row_end - sl.row_begin;
                const uint32_t grid = (uint32_t)std::max<uint64_t>(
                    1, std::min<uint64_t>((rows + kLaneB - 1) / kLaneB, 4 * (uint64_t)cfg.side_blocks));
                hipLaunchKernelGGL(k_census_rows, dim3(grid), dim3(kLaneB), 0, ts, g.rinfo, sl.row_begin, sl.row_end,
                                   (uint64_t)g.n, sl.asym, sl.mutual, table, acc);
            }
        }
        if (ev) (void)hipEventRecord(ev[2 * kBuckets + 1], ts);
    };
    // (dyad records, and forward lists with events between the kernels or with
    // wave or group records)
    // Beside the hub kernel, a lane bucket of more than two workgroups per CU
    // is launched after it: workgroups that come first keep the hub kernel's
    // waiting (R-MAT 2^20, 1000 lane workgroups: 1.82 ms first, 1.73 after).  A
    // smaller one leaves the hub kernel its places and ends under it when it
    // comes first (50 k vertices, 170 workgroups: 0.20 ms first, 0.24 after).
    const uint64_t lanes = sl.end[0] > sl.begin[0] ? sl.end[0] - sl.begin[0] : 0;
    const bool hub_first = beside && lanes > 2 * (uint64_t)kLaneB * cfg.side_blocks;
    if (!hub_first) terms();
    for (int q = 0; q < kBuckets; ++q) {
        const int b = !hub_first ? q : q == 0 ? kBucketHub : q == kBucketHub ? 0 : q;
        if (hub_first && b == 0) terms();
        uint64_t cnt = sl.end[b] > sl.begin[b] ? sl.end[b] - sl.begin[b] : 0;
        if (b == kBucketHub) cnt = hg1 - hg0;
        // beside the hub kernel, the lane bucket follows the terms on the side stream
        const hipStream_t bs = beside && b == 0 ? side : s;
        if (ev) (void)hipEventRecord(ev[2 * b], bs);
        if (cnt > 0 && tri) {
            const tri_args L{g.tri.edges.recs + (b == kBucketHub ? 0 : sl.begin[b]), (uint32_t)cnt, g.tri.fwd, acc, table};
            if (lab) launch_tri<true>(b, L, g.tri.edges, hg0, hg1, cfg, counters, bs);
            else launch_tri<false>(b, L, g.tri.edges, hg0, hg1, cfg, counters, bs);
        } else if (cnt > 0) {
            census_args L{g.dyads + sl.begin[b], (uint32_t)cnt, g.nbr, acc, sl.u_lo, sl.u_hi, table};
            if (b == kBucketHub) {
                L.dyads = g.dyads;
                launch_hub(L, g.hub_tasks, g.n_hub_tasks, ngroups, hg0, hg1, cfg, counters, s);
            } else {
                launch_bucket(b, L, cnt, cfg, counters, bs);
            }
        }
        if (ev) (void)hipEventRecord(ev[2 * b + 1], bs);
    }
    if (beside) {
        hipError_t e = hipEventRecord(fork[1], side);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, fork[1], 0);
        if (e != hipSuccess) return e;
    }
    if (lab) hipLaunchKernelGGL(k_census_finish<64>, dim3(1), dim3(kFinishT), 0, s, acc, counters, out);
    else hipLaunchKernelGGL(k_census_finish<kNumClasses>, dim3(1), dim3(kFinishT), 0, s, acc, counters, out);
    return hipGetLastError();
}

}  // namespace tc
