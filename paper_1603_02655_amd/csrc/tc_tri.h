// Device code of the forward-list path: triangles of a graph, each once.
//
// Vertices are numbered by rank (rank 0: the largest degree, ties to the larger
// id).  The forward list N+(x) holds the neighbours of smaller rank, sorted by
// rank; an entry is (f << 30) | (g << 29) | (rank << 1) with f = IsEdge(x, y) +
// 2 IsEdge(y, x) and g = [id(y) > id(x)].  A triangle {x, y, z}, z < y < x by
// rank, is found at the edge (x, y), as an entry z of N+(y) that is also in
// N+(x), where it stands before y: the part of N+(x) before y (its prefix) is
// all of N+(x) an edge has to look at.  A hub record may have x and y the other
// way round (all of N+(y) against N+(x), where y's list is much the shorter):
// what follows holds for it with the two names exchanged.
//
// What a triangle adds to the census depends on the direction codes of its
// three pairs only (with g, the order of the three ids): a kernel counts
// signatures in LDS and turns the counts into class updates when it ends.
#pragma once
#include "tc_internal.h"

namespace tc {

constexpr uint32_t kRankMask = 0x00fffffeu;     // the rank bits of an entry
__device__ inline uint32_t rank_of(uint32_t e) { return (e & kRankMask) >> 1; }

// Signature of a triangle: the codes of (x, y), (x, z) and (y, z), each
// relative to the first vertex.  Unlabelled: 2 bits each (f).  Labelled: 3 bits
// each (f << 1 | g, the top bits of an entry).
template <bool Lab>
struct tri_sig {
    static constexpr uint32_t kBits = Lab ? 3 : 2;
    static constexpr uint32_t kSlots = 1u << (3 * kBits);
    __device__ static inline uint32_t code(uint32_t e) { return e >> (32 - kBits); }
    __device__ static inline uint32_t slot(uint32_t xy, uint32_t xz, uint32_t yz) {
        return xy | (xz << kBits) | (yz << (2 * kBits));
    }
    unsigned long long* n;   // kSlots counts in LDS
    __device__ inline void hit(uint32_t xy, uint32_t xz, uint32_t yz) { atomicAdd(&n[slot(xy, xz, yz)], 1ull); }
    __device__ inline void clear(uint32_t threads) {
        for (uint32_t k = threadIdx.x; k < kSlots; k += threads) n[k] = 0;
    }
};

// Loads of several entries from any 4-byte position.
struct __attribute__((packed, aligned(4))) entries4 {
    uint32_t a, b, c, d;
};
__device__ inline void load_entries4(const uint32_t* __restrict__ p, uint32_t* e) {
    const entries4 q = *reinterpret_cast<const entries4*>(p);
    e[0] = q.a;
    e[1] = q.b;
    e[2] = q.c;
    e[3] = q.d;
}

// First position in [lo, hi) of a row whose rank (its bits in place) is >= key.
__device__ inline uint32_t rank_bound(const uint32_t* __restrict__ fwd, uint32_t lo, uint32_t hi, uint32_t key) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if ((fwd[mid] & kRankMask) < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Edge record: the prefix of N+(x), [bx, ex) (ex is also the position of y's
// entry in N+(x)), N+(y), [by, ey), and the top three bits of y's entry; in
// memory {bx, ex, by, bits << 29 | ey - by}.  Hub records hold {bx, core, ex,
// bits} instead: core is the end of the prefix's entries below kCore.
struct edge_rec {
    uint32_t bx, ex, by, ey, xy;
    template <bool Lab>
    __device__ inline uint32_t code() const { return Lab ? xy : xy >> 1; }
};
__device__ inline edge_rec load_edge(const uint4* __restrict__ p) {
    const uint4 q = *p;
    return edge_rec{q.x, q.y, q.z, q.z + (q.w & 0x1fffffffu), q.w >> 29};
}

// One lane per edge: the prefix of x, kEdgeA entries at a time, against N+(y),
// kEdgeB at a time; all pairs of two chunks are compared in registers, then the
// chunk whose last rank is smaller is replaced.  The lists are short: bound by
// the L2 misses of the rows of y (citation graph, 12.2 M edges: 14.8 M lines of
// 64 bytes in 0.27 ms; records read ahead change nothing).  Comparing whole
// 32-byte rows of id-ordered lists took 0.52 ms; the rows of popular vertices
// now lie side by side, and one branch tests all 32 pairs (a branch per pair:
// as many scalar instructions as vector ones).
constexpr uint32_t kEdgeA = 4, kEdgeB = 8;

template <bool Lab>
__device__ inline void lane_edge(const edge_rec& r, const uint32_t* __restrict__ fwd, tri_sig<Lab>& sig) {
    using S = tri_sig<Lab>;
    constexpr uint32_t kPadA = 0x01000000u, kPadB = 0x02000000u;   // above every rank, never equal
    uint32_t i = r.bx, j = r.by;
    uint32_t a[kEdgeA], b[kEdgeB], ka[kEdgeA], kb[kEdgeB];
    auto load_a = [&] {
        load_entries4(fwd + i, a);
#pragma unroll
        for (uint32_t k = 0; k < kEdgeA; ++k) ka[k] = i + k < r.ex ? a[k] & kRankMask : kPadA;
    };
    auto load_b = [&] {
        load_entries4(fwd + j, b);
        load_entries4(fwd + j + 4, b + 4);
#pragma unroll
        for (uint32_t k = 0; k < kEdgeB; ++k) kb[k] = j + k < r.ey ? b[k] & kRankMask : kPadB;
    };
    const uint32_t xy = r.code<Lab>();
    load_a();
    load_b();
    for (;;) {
        // 0 when some pair is equal: one branch for all pairs
        uint32_t d = 0xffffffffu;
#pragma unroll
        for (uint32_t p = 0; p < kEdgeA; ++p)
#pragma unroll
            for (uint32_t q = 0; q < kEdgeB; q += 2) d = min(d, min(ka[p] ^ kb[q], ka[p] ^ kb[q + 1]));
        if (d == 0) {
#pragma unroll
            for (uint32_t p = 0; p < kEdgeA; ++p) {
                uint32_t yz = 0;
#pragma unroll
                for (uint32_t q = 0; q < kEdgeB; ++q) yz = ka[p] == kb[q] ? b[q] : yz;
                if (yz) sig.hit(xy, S::code(a[p]), S::code(yz));
            }
        }
        uint32_t la = ka[0], lb = kb[0];   // the last rank of each chunk
#pragma unroll
        for (uint32_t k = 1; k < kEdgeA; ++k) la = ka[k] < kPadA ? ka[k] : la;
#pragma unroll
        for (uint32_t k = 1; k < kEdgeB; ++k) lb = kb[k] < kPadA ? kb[k] : lb;
        if (la <= lb) {
            i += kEdgeA;
            if (i >= r.ex) break;
            load_a();
        } else {
            j += kEdgeB;
            if (j >= r.ey) break;
            load_b();
        }
    }
}

// ------------------------------------------------------------ hub records ----
// One wavefront per task: a run of edges with one y.  N+(y) is put into a
// table in the wavefront's own LDS, kBits bits per rank below kCore (the
// direction code, 0 where a rank is not in N+(y)), and the prefixes of the
// edges stream against it, 16 entries per lane and step; a table read answers
// with the code at once, and the codes of 16 entries are packed into one word
// and counted with AND and bit counts.  No hashing, no candidates, no barriers.
//
// What bounds it: no unit by itself (R-MAT 2^20, 0.82 ms for 1.09e9 entries:
// vector units 59 % busy, texture units 61 %, LDS 31 %, 6.1 TB/s of L2 misses, most
// served before HBM), but the chain of a window (marks, record, entries, table)
// at four wavefronts per SIMD, and a task's start (table and records) on graphs with many short ones.
// The hash table with candidate rings that it replaces took 1.70 ms there (32
// vector instructions per entry and lane, now 17) and streamed the whole shorter list
// of an edge, 1.75e9 entries.
//
// kCore = 16384 ranks are 4 KiB of table: 32 wavefronts per CU.  On skewed
// graphs nearly all of the stream lies below it (R-MAT 2^20: 99.0 %).  In further
// passes, over the rest of the prefixes, the same LDS holds kTail entries of N+(y)
// from kCore on, as codes modulo kCore / 2 and in a hash table of buckets of four:
// where few entries hit a code, a lane looks its hits up one after the other,
// where many do, all its entries.  (Hits looked up in N+(y) itself, by halving:
// 200 complete graphs of 300 took 6.2 ms, now 1.03; 60000 vertices with 300 random
// neighbours 0.92, now 0.75; 100000 on a ring with the 80 nearest 0.71, now 0.24.)
constexpr int kFewHits = 4;               // hits among a lane's 16 entries up to which it looks them up one by one
constexpr uint32_t kTriSegment = 1024;    // blocks whose row starts are marked in LDS at a time

template <bool Lab>
struct tri_table {
    static constexpr uint32_t kBits = Lab ? 4 : 2;
    static constexpr uint32_t kPer = 32 / kBits;                 // ranks per word
    static constexpr uint32_t kWords = kCore / kPer;
    static constexpr uint32_t kTop = Lab ? 3 : 2;                // code bits at the top of a field
    // Word of an entry's rank (modulo kCore), and the left shift that brings
    // its code to the word's top bits.
    __device__ static inline uint32_t word(uint32_t e) { return (e >> (Lab ? 4 : 5)) & (kWords - 1); }
    __device__ static inline uint32_t shift(uint32_t e) { return Lab ? (e << 1) & 28u : e & 31u; }
    __device__ static inline uint32_t field(uint32_t e) { return (e >> (32 - kTop)) << (32 - kTop); }

    // The tables of ranks from kCore on: codes modulo kCore / 2 in the first half
    // of the words, where an answer may be another rank's, and a hash table of the
    // entries in the second.  Slots of a bucket fill in order, and a full bucket
    // goes on in the next; half the slots at most are taken, so a search ends.
    static constexpr uint32_t kHalf = kWords / 2;
    static constexpr uint32_t kBuckets = kHalf / 4;
    static constexpr uint32_t kTail = kHalf / 2;
    static_assert(kBuckets == (Lab ? 256 : 128), "the bits of a bucket");
    __device__ static inline uint32_t tail_word(uint32_t e) { return word(e) & (kHalf - 1); }
    __device__ static inline uint32_t bucket(uint32_t key) {   // the top bits of a 24 x 24-bit product
        return (uint32_t)__umul24(key, 0x9E3779u) >> (32 - (Lab ? 8 : 7));
    }
    __device__ static inline void insert(uint32_t* tab, uint32_t e) {
        atomicOr(&tab[tail_word(e)], field(e) >> shift(e));
        for (uint32_t b = bucket(e & kRankMask);; b = (b + 1) & (kBuckets - 1))
            for (uint32_t s = 0; s < 4; ++s)
                if (atomicCAS(&tab[kHalf + 4 * b + s], 0u, e) == 0u) return;
    }
    // The entry of e's rank, or 0.
    __device__ static inline uint32_t find(const uint32_t* tab, uint32_t e) {
        const uint32_t key = e & kRankMask;
        for (uint32_t b = bucket(key);; b = (b + 1) & (kBuckets - 1)) {
            const uint4 q = reinterpret_cast<const uint4*>(tab + kHalf)[b];
            uint32_t f = (q.x & kRankMask) == key ? q.x : 0u;
            f = (q.y & kRankMask) == key ? q.y : f;
            f = (q.z & kRankMask) == key ? q.z : f;
            f = (q.w & kRankMask) == key ? q.w : f;
            if (f != 0u || q.w == 0u) return f;
        }
    }
};

// Sums over the wavefront's lanes, inclusive (lane 63 holds the whole sum).
// (DPP adds: a scan through LDS permutes takes about 100 cycles a step.)
__device__ inline uint32_t wave_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return x;
}

// Packed counts of the nine pairs of codes (of (y, z) and (x, z)) of the
// unlabelled census, one 10-bit field for each code of (x, y).
struct tri_counts {
    uint32_t c[3][3];
    uint32_t steps;        // steps since the last flush: at most 63 keep a field below 2^10
    __device__ inline void clear() {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) c[i][j] = 0;
        steps = 0;
    }
    // The wavefront's sums go to the signature counts in LDS.
    __device__ inline void flush(tri_sig<false>& sig) {
        uint32_t lane = __lane_id();
        asm volatile("" : "+v"(lane));   // (addresses are made here, not kept in registers through the stream)
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i)
#pragma unroll
            for (uint32_t j = 0; j < 3; ++j) {
                // 64 lanes of fields below 2^10: sums below 2^16
                uint32_t a = wave_scan((c[i][j] & 1023u) | (((c[i][j] >> 20) & 1023u) << 16));
                uint32_t b = wave_scan((c[i][j] >> 10) & 1023u);
                a = (uint32_t)__builtin_amdgcn_readlane((int)a, 63);
                b = (uint32_t)__builtin_amdgcn_readlane((int)b, 63);
                if (lane < 3) {
                    const uint32_t s = lane == 0 ? a & 0xffffu : lane == 1 ? b : a >> 16;
                    if (s) atomicAdd(&sig.n[tri_sig<false>::slot(lane + 1, j + 1, i + 1)], (unsigned long long)s);
                }
            }
        clear();
    }
};

struct tri_wave_sync {
    __device__ inline void operator()() const {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

// The value of lane k of each quad of lanes (k a constant after unrolling).
__device__ inline uint32_t quad_lane(uint32_t x, uint32_t k) {
    switch (k) {
        case 0: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x00, 0xf, 0xf, true);
        case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x55, 0xf, 0xf, true);
        case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xaa, 0xf, 0xf, true);
        default: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xff, 0xf, 0xf, true);
    }
}
// Byte 3 - j of lane k goes to byte 3 - k of lane j, in each quad of lanes.
__device__ inline uint32_t quad_transpose(uint32_t x) {
    const uint32_t s = 3u - (__lane_id() & 3u);
    const uint32_t hi = __builtin_amdgcn_perm(quad_lane(x, 0), quad_lane(x, 1), ((4u + s) << 24) | (s << 16) | 0x0c0cu);
    const uint32_t lo = __builtin_amdgcn_perm(quad_lane(x, 2), quad_lane(x, 3), 0x0c0c0000u | ((4u + s) << 8) | s);
    return hi | lo;
}

// The part of the records' lists that a table answers for: entries below kCore
// (Tail false), or from kCore on, of those with ranks from `key0` (if cut_lo) and
// below `key1` (if cut_hi; ranks with their bits in place).
struct tri_part {
    bool none, cut_lo, cut_hi;   // none: the table is empty
    uint32_t key0, key1;
};

// Streams that part of the records [begin, end) against the table in tab; `first`
// is the lane's first record.  True if some record has entries from kCore on.
template <bool Lab, bool Tail>
__device__ inline bool tri_stream(const uint4* __restrict__ recs, const uint32_t* __restrict__ fwd, uint32_t begin,
                                  uint32_t end, const uint4& first, const tri_part& part, const uint32_t* tab,
                                  uint32_t* starts, tri_sig<Lab>& sig, tri_counts& cnt) {
    using TB = tri_table<Lab>;
    using S = tri_sig<Lab>;
    const uint32_t lane = __lane_id();
    const tri_wave_sync sync{};
    // The lanes of a quad take blocks q, 16 + q, 32 + q and 48 + q of a window.
    const uint32_t block = ((lane & 3u) << 4) | (lane >> 2);
    const uint64_t upto = (2ull << block) - 1ull;
    const uint4 none = make_uint4(0, 0, 0, 0);
    bool tails = false;
    for (uint32_t b = begin; b < end; b += 64) {
        // 64 records, one per lane: their parts in blocks of 16 entries
        const uint4 r = b == begin ? first : b + lane < end ? recs[b + lane] : none;
        if (!Tail) tails = tails || __ballot(r.y != r.z) != 0;
        uint32_t p0 = Tail ? r.y : r.x, p1 = Tail ? r.z : r.y;
        if (!Tail && part.none) continue;
        if (Tail && part.cut_lo) p0 = rank_bound(fwd, p0, p1, part.key0);
        if (Tail && part.cut_hi) p1 = rank_bound(fwd, p0, p1, part.key1);
        const uint32_t nb = (p1 - p0 + 15u) >> 4;
        const uint32_t incl = wave_scan(nb), start = incl - nb;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (total == 0) continue;
        uint32_t q_base = p0 - 16u * start, q_end = p1, q_code = r.w;
        const uint64_t some = __ballot(nb != 0);
        if ((some & (some + 1ull)) != 0) {
            // the records with blocks move to the first lanes: lane j holds
            // the j-th of them (first entry minus 16 x its first block, end,
            // code); the others go to the places above
            const uint32_t to = (uint32_t)__popcll(some & ((1ull << lane) - 1ull));
            const int dst = (int)(4u * (nb != 0 ? to : (uint32_t)__popcll(some) + (lane - to)));
            q_base = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)q_base);
            q_end = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)q_end);
            q_code = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)q_code);
        }
        uint32_t before = 0;   // records that start before the window
        for (uint32_t seg = 0; seg < total; seg += kTriSegment) {
            // one bit per block: a record starts there
            sync();
            if (lane < kTriSegment / 32) starts[lane] = 0;
            sync();
            if (nb != 0 && start >= seg && start < seg + kTriSegment)
                atomicOr(&starts[(start - seg) >> 5], 1u << ((start - seg) & 31u));
            sync();
            const uint32_t stop = min(total, seg + kTriSegment);
            for (uint32_t win = seg; win < stop; win += 64) {
                const uint32_t wi = (win - seg) >> 5;
                const uint32_t m0 = __builtin_amdgcn_readfirstlane((int)starts[wi]),
                               m1 = __builtin_amdgcn_readfirstlane((int)starts[wi + 1]);
                const uint64_t m = (uint64_t)m0 | ((uint64_t)m1 << 32);
                // the record of the lane's block: the last that starts at or before it
                const uint32_t at = before + (uint32_t)__popcll(m & upto) - 1u;
                before += (uint32_t)__popcll(m);
                const int src = (int)(4u * at);
                const uint32_t base = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)q_base);
                const uint32_t pe = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)q_end);
                const uint32_t xy3 = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)q_code);
                const uint32_t t = win + block;
                const bool on = t < total;
                const uint32_t e0 = on ? base + 16u * t : 0u;       // (entries 0..15 are readable)
                const uint32_t ne = on ? min(pe - e0, 16u) : 0u;    // entries of the row in the block
                // Load k reads blocks 16 k .. 16 k + 15 of the window, four lanes the
                // quarters of one block, so that it touches no line that another
                // of the four loads does: lane l gets entries 4 (l % 4) .. + 3
                // of the four blocks of its quad.
                uint32_t e[16];
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    load_entries4(fwd + quad_lane(e0, k) + 4u * (lane & 3u), e + 4 * k);
                if (!Lab) {
                    // codes of (y, z) and (x, z), first entry in the top bits
                    // (all table reads are issued before the first is used)
                    uint32_t A = 0, B = 0, w[16];
#pragma unroll
                    for (uint32_t k = 0; k < 16; ++k) w[k] = tab[Tail ? TB::tail_word(e[k]) : TB::word(e[k])];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (uint32_t k = 0; k < 16; ++k) {
                        A = __builtin_amdgcn_alignbit(A, w[k] << TB::shift(e[k]), 30);
                        B = __builtin_amdgcn_alignbit(B, e[k], 30);
                    }
                    const bool many = Tail && __any(__popc((A | (A >> 1)) & 0x55555555u) > kFewHits);
                    if (many) {
#pragma unroll
                        for (uint32_t k = 0; k < 16; ++k) {
                            A = __builtin_amdgcn_alignbit(A, TB::find(tab, e[k]), 30);
                            __builtin_amdgcn_sched_barrier(0);   // (their buckets would take 64 registers)
                        }
                    }
                    // byte 3 - k is this lane's quarter of the quad's block k:
                    // the lanes of the quad exchange them, each for its own block
                    A = quad_transpose(A);
                    B = quad_transpose(B);
                    A &= (uint32_t)(0xffffffff00000000ull >> (2u * ne));
                    if (Tail && !many) {
                        uint32_t h = (A | (A >> 1)) & 0x55555555u;
                        while (h) {
                            const uint32_t k = (uint32_t)__clz((int)h) >> 1, at_k = 30u - 2u * k;
                            h &= ~(1u << at_k);
                            const uint32_t yz = TB::find(tab, fwd[e0 + k]);
                            A = (A & ~(3u << at_k)) | (S::code(yz) << at_k);
                        }
                    }
                    constexpr uint32_t kOdd = 0x55555555u;
                    const uint32_t a1 = A & kOdd, a2 = (A >> 1) & kOdd, a3 = a1 & a2;
                    const uint32_t b1 = B & kOdd, b2 = (B >> 1) & kOdd, b3 = b1 & b2;
                    const uint32_t av[3] = {a1 ^ a3, a2 ^ a3, a3}, bv[3] = {b1 ^ b3, b2 ^ b3, b3};
                    const uint32_t mul = 1u << (10u * ((xy3 >> 1) - 1u));
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int j = 0; j < 3; ++j)
                            cnt.c[i][j] += (uint32_t)__umul24(__popc(av[i] & bv[j]), mul);
                    if (++cnt.steps == 63) {
                        if constexpr (!Lab) cnt.flush(sig);
                    }
                } else {
#pragma unroll
                    for (uint32_t k = 0; k < 16; ++k) {
                        const uint32_t n_k = quad_lane(ne, k / 4), xy_k = quad_lane(xy3, k / 4);
                        const bool in = 4u * (lane & 3u) + k % 4 < n_k;
                        uint32_t yz = tab[Tail ? TB::tail_word(e[k]) : TB::word(e[k])] << TB::shift(e[k]);   // (code in the top bits)
                        if (in && yz >= 0x20000000u) {
                            if (Tail) yz = TB::find(tab, e[k]);
                            if (yz != 0u) sig.hit(xy_k, S::code(e[k]), S::code(yz));
                        }
                    }
                }
            }
        }
    }
    return tails;
}

// Runs the records [begin, end) of a task on one wavefront.  tab: kWords of
// LDS, starts: kTriSegment / 32 words, both the wavefront's own.  The pass over
// the ranks below kCore and those over the others are two instances of the stream:
// as one, the tests for the others cost the former 1 to 5 %.
template <bool Lab>
__device__ inline void tri_run(const uint4* __restrict__ recs, const uint32_t* __restrict__ fwd, uint32_t begin,
                               uint32_t end, uint32_t by, uint32_t ey, uint32_t* tab, uint32_t* starts,
                               tri_sig<Lab>& sig, tri_counts& cnt) {
    using TB = tri_table<Lab>;
    const uint32_t lane = __lane_id();
    const tri_wave_sync sync{};
    const uint4 none = make_uint4(0, 0, 0, 0);
    const uint4 first = begin + lane < end ? recs[begin + lane] : none;   // (read beside the table's entries)
    auto clear = [&] {
        sync();
        uint32_t zero = 0;
        asm volatile("" : "+v"(zero));   // (not kept in registers through the stream)
        for (uint32_t k = lane; k < TB::kWords / 4; k += 64) reinterpret_cast<uint4*>(tab)[k] = make_uint4(zero, zero, zero, zero);
        sync();
    };
    clear();
    uint32_t ty = by;   // end of the entries of N+(y) below kCore
    for (uint32_t k = by; k < ey; k += 64) {
        const uint32_t p = k + lane;
        const uint32_t e = p < ey ? fwd[p] : 0u;
        const bool core = p < ey && rank_of(e) < kCore;
        if (core) atomicOr(&tab[TB::word(e)], TB::field(e) >> TB::shift(e));
        const uint32_t n = (uint32_t)__popcll(__ballot(core));
        ty += n;
        if (n != 64) break;   // (ranks rise)
    }
    sync();
    const bool tails = tri_stream<Lab, false>(recs, fwd, begin, end, first, tri_part{ty == by, false, false, 0u, 0u}, tab,
                                              starts, sig, cnt);
    if (!tails) return;
    // The others, kTail to a table: met by the part of a prefix from the table's
    // first rank to the first of the next.
    for (uint32_t from = ty; from < ey; from += TB::kTail) {
        const uint32_t past = min(from + TB::kTail, ey);
        clear();
        for (uint32_t p = from + lane; p < past; p += 64) TB::insert(tab, fwd[p]);
        sync();
        const bool cut_lo = from > ty, cut_hi = past < ey;
        (void)tri_stream<Lab, true>(recs, fwd, begin, end, first,
                                    tri_part{false, cut_lo, cut_hi, cut_lo ? fwd[from] & kRankMask : 0u,
                                             cut_hi ? fwd[past] & kRankMask : 0u},
                                    tab, starts, sig, cnt);
    }
}

}  // namespace tc
