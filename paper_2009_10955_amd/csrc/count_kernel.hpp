// Persistent counting kernel for gfx950.
//
// What it computes: the number of embeddings of a pattern under one
// configuration (schedule + restriction closure), i.e. the nested-loop search
// of Section II-B / IV-B with candidate sets formed by intersecting sorted
// neighbor lists and cut by the restrictions (the generated code of Fig.
// pseudocode_performance), with every level's injectivity enforced
// (Section II-A requires a bijection). Optionally the innermost 2 to 4
// pairwise non-adjacent levels are not enumerated but counted by
// inclusion-exclusion (Section IV-D, Algorithm 2).
//
// How it maps to the machine:
//   * Tasks are root edges (v0, v1) = the first two loops fused, taken in
//     chunks from a device-wide queue of kCursors cursors (the fine-grained task
//     partitioning of Section IV-E, as a lock-free queue instead of a master
//     thread). Root arrays are ordered by their smaller (higher-degree)
//     endpoint, so hubs go first, and the heaviest roots can be split over
//     their level-2 candidates into several tasks.
//   * A group of G lanes (G in {64, 32, 16, 8}) of one wavefront shares one
//     search path. Intersections are group-cooperative (each lane
//     binary-searches one element of the smaller list in the larger one;
//     ballot + popcount compact the hits). G < 64 runs 64/G independent paths
//     per wavefront, which pays on graphs whose lists are short.
//   * Intersection results ("tmp" sets) live in a per-group scratch region in
//     HBM; they are written and re-read while hot in L2. (A variant with the
//     buffers in LDS was measured slower and turned every buffer access into
//     a flat access; it is not kept.)
//   * The second-to-last level is spread over the lanes (leaf mode 1: each
//     lane counts the last level for its own candidate), walked with the
//     group counting each last level together (leaf mode 2), flattened with
//     the level above it into one balanced batch (leaf mode 3), or spread over
//     the lanes with long hub-tested lists walked by the whole group (leaf
//     mode 4).
//   * Hub vertices carry dense neighbor bitmaps: a membership test against a
//     hub's list is one word load.
//   * The last level is never enumerated: its count is
//     |C ∩ [lo, hi)| minus the earlier bound vertices that fall in it.
//   * Counts: a 64-bit total and a carry count per lane, an exact 128-bit
//     wavefront sum, one pair of atomics per wavefront into one of kSlots
//     128-bit device totals; a last step adds these, divides the sum by the
//     IEP over-count and flags a quotient that does not fit in 64 bits.
//   * Byte accounting (MODE_ACCOUNT) is the same search, leaf mode and memo
//     with a per-lane byte counter added where memory is touched: it measures
//     the bytes of the path the timed launch takes.
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

#include "internal.hpp"
#include "sets.hpp"

namespace gpcount {

using namespace gpdev;

constexpr int kBlock = 256;

// The table kernel's blocks: 16 wavefronts with a table of 32,768 vertices, or
// 4 with one of 8,192 (16-bit counts, 64 or 16 KB of LDS: 32 wavefronts per CU).
constexpr int table_max(int waves) { return waves * 2048; }
// Words of the filter of N(p) that the table kernel for IEP keeps: bit y mod
// 32 * kFiltWords is set for every y in N(p).
constexpr int kFiltWords = 2048;
constexpr int kIepTableWaves = 8;  // its blocks: 32 KB of table, 8 of filter, three blocks per CU

// Kernel modes: plain count, per-root counts, accounting of the bytes the
// search reads and writes (never timed), or (table kernels: clocks in the plain one cost a
// small 4-cycle count 3 of 55 us) a plain count that reports its busy time.
enum { MODE_PLAIN = 0, MODE_PER_ROOT = 1, MODE_ACCOUNT = 2, MODE_SAMPLE = 3 };

// Inclusion-exclusion over at most this many innermost levels.
constexpr int kIepMaxN = GP_IEP_MAX_INNER;

// A launch's queue: kSlots slots of kSlotWords words (256 bytes, so that slots
// lie in different memory channels). Every slot holds a partial 128-bit total
// and, in batches, busy clock ticks; every kCursorStep-th also a task cursor.
// Chunk q of the task space belongs to cursor q mod kCursors, so all cursors
// together still walk the tasks in order, heaviest first.
//
// Why many: atomics with a return value on one address complete one after
// another at the memory side, 12 ns each, whoever issues them. One cursor
// bounded every launch of small tasks (R-MAT 18 4-clique per root, 488K grabs:
// 6.0 ms, 5.9 of them the cursor), and 8,192 wavefronts ending against it, and
// adding their totals to one word, cost 0.1 ms each even on the smallest
// graph. Why not more cursors: a group that finds its own dry reads all of
// them, and thousands of groups do so as a launch ends (a batch of small
// launches: 47 ms with one cursor per plan, 63 with 64).
constexpr int kSlots = 64;
constexpr int kSlotWords = 32;
constexpr int kQueueWords = kSlots * kSlotWords;
constexpr int kCursors = 16;
constexpr int kCursorStep = kSlots / kCursors;
enum { SLOT_CURSOR = 0, SLOT_LO = 1, SLOT_HI = 2, SLOT_BUSY = 3 };
// set once every cursor is exhausted (a word of a slot without a cursor)
constexpr int kDoneWord = 2 * kSlotWords + 4;

struct CountArgs {
    const int64_t* row_ptr;
    const int32_t* col;
    const int2* roots;
    int64_t n_roots;      // sampled roots: roots[root_offset + r * root_stride], r < n_roots
    int64_t root_offset;
    int64_t root_stride;
    // The first split_roots sampled roots (the heaviest: root arrays are
    // ordered by their hub endpoint) are each split into split_ways tasks, the
    // j-th of which binds only every split_ways-th level-2 candidate from j on.
    // Tasks: split_roots * split_ways split ones, then one per remaining root.
    int64_t n_tasks;
    int64_t n_chunks;  // ceil(n_tasks / chunk)
    int64_t split_roots;
    int32_t split_ways;
    const uint32_t* hub_bits;  // n_hubs dense bitmaps of hub_words words
    int64_t hub_words;
    int32_t n_hubs;
    int32_t* scratch;
    int64_t buf_cap;
    unsigned long long* queue;     // kQueueWords words; with xcd_block > 0 cursor x is XCD x's
    unsigned long long* result;    // {count (low word, set by finish_count), flags, bytes}
    unsigned long long* per_root;  // optional, indexed by CSR entry of (v0, v1)
    // optional {sum over wavefronts of active clock ticks, wavefronts, longest
    // chunk of tasks in ticks}: the balanced run time of a sample and its tail
    unsigned long long* busy;
    // with busy: stop taking tasks once a wavefront has run this many clock
    // ticks (0: no limit); the count is then incomplete and flagged (bit 2)
    uint64_t budget_ticks;
    // optional (leaf mode 4, plans the host found eligible): per group,
    // n_hubs words {root tag, |N(x) & pre & cut|} for hub candidates x
    // or (IEP plans the host found eligible) one table for the launch of
    // 2^memo_ways_log2 rows of n_hubs words {a + 1 with the high bit set, |N(a) & N(x)|}
    unsigned long long* memo;
    int32_t chunk;
    int32_t memo_ways_log2;
    // > 0: the task space is dealt to the XCDs in blocks of xcd_block tasks
    // (a multiple of chunk): block b goes to XCD b mod kXcds, each XCD takes
    // its blocks in order from its own cursor and then helps the others; 0:
    // one cursor for the device
    int64_t xcd_block;
    int32_t tab_n;  // table kernel: vertices its table covers
    int32_t whole_chunk;  // table kernel, with busy: tasks per grab of a whole count
};

typedef void (*KernelFn)(GpPlanDesc, CountArgs);

// Batched launch: one entry per plan. Each plan has its own launch shape
// (lanes per group, leaf mode, tasks per grab) and its own task cursor.
constexpr int kBatchMaxPlans = 64;

struct BatchPlan {
    const int2* roots;    // this plan's whole root array (cut already applied)
    int64_t root_offset;  // sampled roots: roots[root_offset + r * root_stride]
    int64_t root_stride;
    int64_t n_tasks;      // tasks of this plan in the launch
    int64_t n_chunks;     // wavefront grabs: ceil(n_tasks / (64 / group * chunk))
    int64_t task_offset;  // where in the plan's own task space the launch starts
    int64_t split_roots;  // as in CountArgs: the first split_roots roots run as
    int32_t split_ways;   // split_ways tasks each
    int32_t group;        // lanes per group: 64, 32 or 16
    int32_t leaf;         // 1, 3 or 4
    int32_t chunk;        // tasks per group per grab
    uint32_t tag_base;    // leaf-4 memo tags are tag_base + root + 1; 0: no memo
    int32_t pad;
};


// The descriptors and task ranges of one batched launch's plans, in the order
// waves take them, passed by value: kernel arguments live in constant memory,
// so every field is a scalar load, where a table read from global memory costs
// a vector load and registers at every use.
constexpr int kRunMaxPlans = 8;
struct RunDescs {
    GpPlanDesc d[kRunMaxPlans];
    BatchPlan bp[kRunMaxPlans];
};

struct BatchArgs {
    const int64_t* row_ptr;
    const int32_t* col;
    int32_t np;
    const uint32_t* hub_bits;
    int64_t hub_words;
    int32_t n_hubs;
    int32_t* scratch;        // per wavefront: slots_per_wave groups x nbuf slots x buf_cap
    int64_t buf_cap;
    int32_t nbuf;            // buffer slots per group (max over plans)
    int32_t slots_per_wave;  // 64 / (the smallest group of any plan)
    unsigned long long* memo;     // leaf mode 4: per wavefront slots_per_wave x n_hubs words; IEP: one table (or null)
    int32_t iep_memo_log2;        // IEP: log2 of the table's rows of n_hubs words; -1: none
    unsigned long long* queues;   // per plan: kSlots slots
};

typedef void (*BatchFn)(BatchArgs, RunDescs);

// Where a group's root tasks come from.
struct TaskSpace {
    const int2* roots;
    int64_t offset, stride;  // root r is roots[offset + r * stride]
    int64_t split_roots;     // task -> root as in CountArgs
    int32_t split_ways;
    uint32_t tag_base;       // memo tag of root r: tag_base + r + 1
};

// Root of task t, and the level-2 slice it binds: the first split_roots roots
// are split_ways tasks each, the rest one task each.
__device__ __forceinline__ int64_t task_root(int64_t t, int64_t split_roots, int32_t split_ways, int32_t& sj,
                                             int32_t& sJ) {
    const int64_t split_tasks = split_roots * (int64_t)split_ways;
    if (t < split_tasks) {
        const int64_t r = t / split_ways;
        sj = (int32_t)(t - r * split_ways);
        sJ = split_ways;
        return r;
    }
    sj = 0;
    sJ = 1;
    return t - split_tasks + split_roots;
}

// Values equal in every lane of a group. With 64-lane groups they are
// wavefront-uniform: readfirstlane lets the compiler keep them, and what is
// computed from them (bound vertices, set bounds, loop counters), in scalar
// registers, which leaves vector registers for more resident wavefronts.
template <int G>
__device__ __forceinline__ int32_t uni(int32_t x) {
    if constexpr (G == 64) return __builtin_amdgcn_readfirstlane(x);
    else return x;
}
template <int G>
__device__ __forceinline__ int64_t uni64(int64_t x) {
    if constexpr (G == 64) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)x);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)x >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    } else {
        return x;
    }
}
// Cut a group-uniform set to [lo, hi) (lo, hi group-uniform).
template <int G>
__device__ __forceinline__ Set trim_u(Set s, int32_t lo, int32_t hi) {
    const Group<G> g;
    int32_t b = lo > 0 ? uni<G>(lower_bound_group<G>(g, s.p, s.n, lo)) : 0;
    int32_t e = hi < 0x7fffffff ? uni<G>(lower_bound_group<G>(g, s.p, s.n, hi)) : s.n;
    if (e < b) e = b;
    return Set{s.p + b, e - b, s.bits};
}

struct FlatRoot;

template <int G>
struct Ctx {
    const int64_t* row_ptr;
    const int32_t* col;
    int32_t* bufs;
    int64_t cap;
    int32_t* lens;  // LDS: length per buffer slot
    uint64_t* bytes;  // accounting mode: per-lane bytes
    const uint32_t* hub_bits;
    int64_t hub_words;
    int32_t n_hubs;
    int32_t sj, sJ;     // level-2 slice of the current task: candidates sj, sj + sJ, ...
    uint64_t deadline;  // clock tick after which every search loop stops (0: none)
    unsigned long long* memo;  // this group's last-level memo, or the launch's IEP memo (null: none)
    uint32_t tag;              // memo validity tag of the current root
    int32_t memo_log2;         // IEP memo: log2 of its rows
    uint32_t* cnt;             // IEP: this lane's subset sizes in LDS, kBlock words apart
    const uint16_t* tab;       // leaf mode 5: the block's path table in LDS, of vertices [0, tab_n)
    int32_t tab_n;
    int32_t out;               // leaf mode 5: the root endpoint left out of the table, a neighbor of p (-1: none)
    const uint32_t* filt;      // IEP with the table: N(p) hashed to kFiltWords words of bits in LDS
    FlatRoot* flat;               // k = 3: 64 edges' walks and the flags of their starts in LDS (null: none)
    int32_t* starts;
    Group<G> g;

    __device__ __forceinline__ bool expired() const {
        return deadline != 0 && wall_clock64() > deadline;
    }

    __device__ __forceinline__ Set nbr(int32_t v) const {
        int64_t b = row_ptr[v], e = row_ptr[v + 1];
        return Set{col + b, (int32_t)(e - b), v < n_hubs ? hub_bits + (int64_t)v * hub_words : nullptr};
    }
    // whether u and v are adjacent: a bit of the higher-degree one's bitmap, else
    // a search in the shorter list
    __device__ __forceinline__ bool edge(int32_t u, int32_t v) const {
        const int32_t h = min(u, v), o = max(u, v);
        if (h < n_hubs) return (hub_bits[(int64_t)h * hub_words + (o >> 5)] >> (o & 31)) & 1u;
        const Set s = nbr(o);
        return contains(s.p, s.n, h);
    }
    __device__ __forceinline__ Set buf(int slot) const {
        return Set{bufs + (int64_t)slot * cap, lens[slot], nullptr};
    }
    // the same for a group-uniform vertex or slot
    __device__ __forceinline__ Set nbr_u(int32_t v) const {
        const int64_t b = uni64<G>(row_ptr[v]), e = uni64<G>(row_ptr[v + 1]);
        return Set{col + b, (int32_t)(e - b), v < n_hubs ? hub_bits + (int64_t)v * hub_words : nullptr};
    }
    __device__ __forceinline__ Set buf_u(int slot) const {
        return Set{bufs + (int64_t)slot * cap, uni<G>(lens[slot]), nullptr};
    }
};

// v[idx] for a runtime idx without dynamic register indexing.
// Up to five vertices the selected values are ORed (no chain of selects: 2-3%
// of the R-MAT 17 5-cycle and house); from six on that holds too many registers: 6-cycle
// per root on Chung-Lu (1,989 vertices, 32 lanes) 61.4 ms ORed, 55.4 by selects.
template <int K>
__device__ __forceinline__ int32_t pick(const int32_t (&v)[K], int idx) {
    if constexpr (K >= 6) {
        int32_t r = v[0];
#pragma unroll
        for (int j = 1; j < K; ++j) r = (idx == j) ? v[j] : r;
        return r;
    }
    int32_t r = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) r |= (idx == j) ? v[j] : 0;
    return r;
}

template <int K>
__device__ __forceinline__ void bounds(uint32_t hi_src, uint32_t lo_src, const int32_t (&v)[K],
                                       int32_t& lo, int32_t& hi) {
    lo = 0;
    hi = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if ((hi_src >> j) & 1u) hi = min(hi, v[j]);
        if ((lo_src >> j) & 1u) lo = max(lo, v[j] + 1);
    }
}

template <int K>
__device__ __forceinline__ bool inj_hit(uint32_t inj, const int32_t (&v)[K], int32_t x) {
    bool hit = false;
#pragma unroll
    for (int j = 0; j < K; ++j)
        if ((inj >> j) & 1u) hit |= (v[j] == x);
    return hit;
}

// acc += c, counting wrap-arounds of the low word in carry: (carry, acc) is
// the lane's exact 128-bit total.
__device__ __forceinline__ void add_count(uint64_t& acc, uint64_t c, uint64_t& carry) {
    const uint64_t s = acc + c;
    carry += (s < acc) ? 1u : 0u;
    acc = s;
}

// (carry, acc) += (hi, lo).
__device__ __forceinline__ void add_count128(uint64_t& acc, uint64_t& carry, uint64_t lo, uint64_t hi) {
    const uint64_t s = acc + lo;
    carry += hi + ((s < acc) ? 1u : 0u);
    acc = s;
}

// Wavefront sum of the lanes' 128-bit totals (hi, lo); every lane gets it.
__device__ __forceinline__ void wave_sum128(uint64_t& lo, uint64_t& hi) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint64_t tlo = __shfl_xor(lo, off, 64);
        const uint64_t thi = __shfl_xor(hi, off, 64);
        const uint64_t u = lo + tlo;
        hi += thi + (u < lo ? 1u : 0u);
        lo = u;
    }
}

// Add a 128-bit value to a total in device memory held as two words: the low
// word at *lo_word, the high word at *hi_word. Called by one lane.
__device__ __forceinline__ void publish128(unsigned long long* lo_word, unsigned long long* hi_word, uint64_t lo,
                                           uint64_t hi) {
    if (lo) {
        const unsigned long long old = atomicAdd(lo_word, (unsigned long long)lo);
        hi += (old + lo < old) ? 1u : 0u;
    }
    if (hi) atomicAdd(hi_word, (unsigned long long)hi);
}

// Sum of a queue's kSlots 128-bit totals; every lane of the wavefront gets it.
__device__ __forceinline__ void slot_sum128(const unsigned long long* queue, uint64_t& lo, uint64_t& hi) {
    static_assert(kSlots == 64, "one slot per lane");
    const unsigned long long* s = queue + (int64_t)__lane_id() * kSlotWords;
    lo = s[SLOT_LO];
    hi = s[SLOT_HI];
    wave_sum128(lo, hi);
}

// The end of every count: the 128-bit total (hi, *lo_word) divided by div
// (the IEP over-count, 1 otherwise). *lo_word receives the quotient's low 64
// bits; flags: bit 0 if the quotient does not fit in 64 bits, bit 1 if div
// does not divide the total (an internal error). Shift-and-subtract long
// division by one lane: it runs once per count.
__device__ __forceinline__ void finish128(unsigned long long* lo_word, unsigned long long* flags, uint64_t hi,
                                          uint64_t div) {
    const uint64_t lo = *lo_word;
    if (div <= 1) {
        if (hi) *flags |= 1ull;
        return;
    }
    uint64_t qhi = 0, qlo = 0, r = 0;
    for (int i = 127; i >= 0; --i) {
        const uint64_t bit = i >= 64 ? (hi >> (i - 64)) & 1u : (lo >> i) & 1u;
        const bool top = (r >> 63) != 0;  // r < div < 2^64, so 2r + bit may need 65 bits
        r = (r << 1) | bit;
        if (top || r >= div) {
            r -= div;
            if (i >= 64) qhi |= 1ull << (i - 64);
            else qlo |= 1ull << i;
        }
    }
    if (r) *flags |= 2ull;
    if (qhi) *flags |= 1ull;
    *lo_word = qlo;
}

// Bytes read by one binary search in a sorted list of n int32.
__device__ __forceinline__ uint64_t probe_bytes(int32_t n) {
    return 4ull * (uint64_t)(32 - __clz(n > 0 ? n : 1));
}
// Bytes of one membership test in s: a bitmap word, or a binary search.
__device__ __forceinline__ uint64_t test_bytes(const Set& s) {
    return s.bits ? 4ull : probe_bytes(s.n);
}
// Bytes of cutting s to [lo, hi): one binary search per bound applied.
__device__ __forceinline__ uint64_t cut_bytes(const Set& s, int32_t lo, int32_t hi) {
    return probe_bytes(s.n) * (uint64_t)((lo > 0) + (hi < 0x7fffffff));
}
// Bytes of a test-based intersection (group or galloping): every element of
// the smaller operand read and tested in the larger one.
__device__ __forceinline__ uint64_t probe_isect_bytes(Set a, Set b) {
    if (a.n > b.n) {
        const Set t = a;
        a = b;
        b = t;
    }
    return (uint64_t)a.n * (4ull + test_bytes(b));
}
// Bytes of intersect_count_serial: bitmap tests, galloping or a merge.
__device__ __forceinline__ uint64_t serial_isect_bytes(Set a, Set b) {
    if (a.n > b.n) {
        const Set t = a;
        a = b;
        b = t;
    }
    if (a.n == 0) return 0;
    if (b.bits || a.n * 16 < b.n) return probe_isect_bytes(a, b);
    return 4ull * (uint64_t)(a.n + b.n);
}

__device__ __forceinline__ void group_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Builds scheduled right after level h is bound. False once one comes out empty:
// every buffer holds a superset of some level's candidates, so nothing below
// this binding is an embedding (with inclusion-exclusion, no tuple either), and
// the remaining builds and levels are skipped.
template <int K, int G, int MODE>
__device__ __forceinline__ bool run_builds(const GpPlanDesc& d, const Ctx<G>& c, int h,
                                           const int32_t (&v)[K]) {
    const int b0 = d.build_begin[h], b1 = d.build_end[h];
    for (int t = b0; t < b1; ++t) {
        const GpBuild& b = d.b[t];
        int32_t lo, hi;
        bounds<K>(b.hi_src, b.lo_src, v, lo, hi);
        Set A = b.src_buf >= 0 ? c.buf_u(b.src_buf) : c.nbr_u(pick<K>(v, b.src_list));
        Set B = c.nbr_u(pick<K>(v, b.with_list));
        // The shorter operand is walked and the other tested whole. Only the
        // walk is cut, and a walk of a few steps not even that: its elements are
        // compared with the bounds. Each cut left out is two or more dependent
        // loads less before the first element.
        if (B.n < A.n) {
            const Set t = A;
            A = B;
            B = t;
        }
        if (A.n > 4 * G && (b.hi_src | b.lo_src)) {
            if constexpr (MODE == MODE_ACCOUNT)
                if (c.g.gl == 0) *c.bytes += cut_bytes(A, lo, hi);
            A = trim_u<G>(A, lo, hi);
        }
        int32_t n = uni<G>(intersect_into<G>(c.g, A, B, lo, hi, c.bufs + (int64_t)b.dst * c.cap));
        if constexpr (MODE == MODE_ACCOUNT)
            if (c.g.gl == 0) *c.bytes += (uint64_t)A.n * (4 + test_bytes(B)) + 4ull * (uint64_t)n;
        if (n == 0) return false;
        group_fence();
        c.lens[b.dst] = n;
        group_fence();
    }
    return true;
}

// Count of the last level for bound values v[0..K-2], by one lane. at: index of
// v[K-2] in its level's whole candidate set (used where GpLevel::pre_below).
template <int K, int G, int MODE>
__device__ __forceinline__ uint32_t leaf_serial(const GpPlanDesc& d, const Ctx<G>& c,
                                                const int32_t (&v)[K], int32_t at = 0) {
    const GpLevel& lv = d.lv[K - 1];
    int32_t lo, hi;
    bounds<K>(lv.hi_src, lv.lo_src, v, lo, hi);
    if (lv.last_list < 0) {
        Set S = lv.list >= 0 ? c.nbr(pick<K>(v, lv.list)) : c.buf(lv.buf);
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(S, lo, hi);
        S = trim(S, lo, hi);
        uint32_t cnt = (uint32_t)S.n;
#pragma unroll
        for (int j = 0; j < K - 1; ++j) {
            if ((lv.inj >> j) & 1u) {
                int32_t y = v[j];
                if (y >= lo && y < hi) {
                    if constexpr (MODE == MODE_ACCOUNT) *c.bytes += test_bytes(S);
                    if (member(S, y)) --cnt;
                }
            }
        }
        return cnt;
    }
    Set A = lv.pre_buf >= 0 ? c.buf(lv.pre_buf) : c.nbr(pick<K>(v, lv.pre_list));
    Set B = c.nbr(pick<K>(v, lv.last_list));
    // injectivity folded into the intersection: matches equal to an earlier
    // image are not counted
    const uint32_t inj = lv.inj;
    auto skip = [&](int32_t x) { return inj_hit<K>(inj, v, x); };
    if (lv.pre_below) {
        // the cliques: the part of A below v[K-2], with no search for where it
        // ends, tested in N(v[K-2]); B is cut by being tested
        A.n = at;
        if (B.bits) {
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8ull * (uint64_t)A.n;
            return count_bits(A, B.bits, skip);
        }
        if (B.n <= A.n) B = trim(B, lo, hi);
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += serial_isect_bytes(A, B);
        return intersect_count_serial(A, B, skip);
    }
    // a hub operand is tested by bits, so only the other operand is cut; a
    // short list is range-tested element by element instead of cut
    if (B.bits && A.n <= kShortList && A.n * 4 <= B.n) {
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8ull * (uint64_t)A.n;
        return count_bits_range(A, lo, hi, B.bits, skip);
    }
    if (A.bits && B.n <= kShortList && B.n * 4 <= A.n) {
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8ull * (uint64_t)B.n;
        return count_bits_range(B, lo, hi, A.bits, skip);
    }
    if (B.bits) {
        const Set Ac = trim(A, lo, hi);
        if (Ac.n * 4 <= B.n) {
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(A, lo, hi) + 8ull * (uint64_t)Ac.n;
            return count_bits(Ac, B.bits, skip);
        }
    } else if (A.bits) {
        const Set Bc = trim(B, lo, hi);
        if (Bc.n * 4 <= A.n) {
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(B, lo, hi) + 8ull * (uint64_t)Bc.n;
            return count_bits(Bc, A.bits, skip);
        }
    }
    if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(A, lo, hi) + cut_bytes(B, lo, hi);
    A = trim(A, lo, hi);
    B = trim(B, lo, hi);
    if constexpr (MODE == MODE_ACCOUNT) *c.bytes += serial_isect_bytes(A, B);
    return intersect_count_serial(A, B, skip);
}

// Count of the last level, computed by the whole group (same value in every lane).
template <int K, int G, int MODE>
__device__ __forceinline__ uint32_t leaf_group(const GpPlanDesc& d, const Ctx<G>& c,
                                               const int32_t (&v)[K]) {
    const GpLevel& lv = d.lv[K - 1];
    if (lv.last_list < 0) {
        // every lane computes the same count; only lane 0 keeps the bytes
        uint64_t keep = 0;
        if constexpr (MODE == MODE_ACCOUNT) keep = *c.bytes;
        uint32_t r = leaf_serial<K, G, MODE>(d, c, v);
        if constexpr (MODE == MODE_ACCOUNT)
            if (c.g.gl != 0) *c.bytes = keep;
        return r;
    }
    int32_t lo, hi;
    bounds<K>(lv.hi_src, lv.lo_src, v, lo, hi);
    Set A = lv.pre_buf >= 0 ? c.buf_u(lv.pre_buf) : c.nbr_u(pick<K>(v, lv.pre_list));
    Set B = c.nbr_u(pick<K>(v, lv.last_list));
    uint64_t cb = 0;
    if constexpr (MODE == MODE_ACCOUNT) cb = cut_bytes(A, lo, hi) + cut_bytes(B, lo, hi);
    A = trim_u<G>(A, lo, hi);
    B = trim_u<G>(B, lo, hi);
    if constexpr (MODE == MODE_ACCOUNT)
        if (c.g.gl == 0) *c.bytes += cb + probe_isect_bytes(A, B);
    const uint32_t inj = lv.inj;
    return intersect_count_group<G>(c.g, A, B, [&](int32_t x) { return inj_hit<K>(inj, v, x); });
}

// Counting with inclusion-exclusion over the N innermost levels (Section
// IV-D). For bound values v[0..K-N-1] every inner level j has a candidate set
// S_j: its parents' common neighbors (all parents are outer levels: the inner
// pattern vertices are pairwise non-adjacent), cut by the restrictions to
// outer levels and without the outer images. The number of N-tuples with
// y_j in S_j and all y_j distinct is the inclusion-exclusion sum over the
// "y_a = y_b" conditions; Algorithm 2 evaluates each term as a product over
// the components of the conditions' graph of |intersection of the
// component's sets|. Terms whose graphs have the same components are
// collected here: a partition of the N levels into blocks contributes
// prod over blocks B of (-1)^(|B|-1) (|B|-1)! |∩_{j in B} S_j| (the sum of
// (-1)^edges over the connected graphs on |B| vertices). The value fits
// in 128 bits (each |S_j| < 2^31, N <= 4).
//
// How |∩_{j in M} S_j| is computed is laid down per subset M by the planner
// (GpIepTerm): the fewest operands that cover the parents (a set built from
// N(v0) needs no test against N(v0)), the outer images that may lie in the
// intersection and are subtracted, and an earlier subset with the same set
// (inner levels with the same parents: one walk instead of three for N = 2,
// seven for N = 3). One loop over the subsets, not unrolled: the kernel carries
// one copy of the walk, where a copy per subset for lanes and for groups spilled
// up to 3.6 KB per lane.
//
// Every lane holds one binding. A lane walks the shorter operand alone when it
// has at most kIepLaneWork elements; longer walks are taken by the whole group,
// one lane's after another, and only those: the lane keeps its binding and the
// other subsets' sizes.
//
// The memo: one table per launch, shared by every group, of W = 2^l rows of
// n_hubs words (l = CountArgs::memo_ways_log2). Word (a mod W) * n_hubs + x
// holds {a + 1 with the high bit set (apart from leaf mode 4's root tags),
// |N(a) & N(x)|} for hubs a and x: a size that depends on (a, x) alone, the
// same for every plan, group and launch on the graph. Rows by a, the endpoint
// bound first: the lanes look up ascending x of one a, in neighbouring words
// that stay in L2 while groups work on roots of a (rows by x: every lookup a
// line of its own, 512 KB apart). Tag and size share one 64-bit word, written
// and read whole, so a word another group overwrote, or one not yet visible,
// only ever reads as a miss. The host takes the most ways, up to
// kIepMemoWaysMax, whose table fits kIepMemoBytes (or the room left).
constexpr int64_t kIepMemoWaysMax = 4096;
constexpr int64_t kIepMemoBytes = int64_t(2) << 30;
constexpr int32_t kIepLaneWork = 96;

// The memo word of hubs (a, x), or null.
template <int G>
__device__ __forceinline__ unsigned long long* iep_memo_word(const Ctx<G>& c, int32_t a, int32_t x) {
    if (!c.memo || a >= c.n_hubs || x >= c.n_hubs) return nullptr;
    return c.memo + (int64_t)(a & ((int32_t(1) << c.memo_log2) - 1)) * c.n_hubs + x;
}

template <int G, int MODE>
__device__ __forceinline__ bool adjacent(const Ctx<G>& c, int32_t u, int32_t v) {
    if constexpr (MODE == MODE_ACCOUNT) {
        const int32_t o = max(u, v);
        *c.bytes += min(u, v) < c.n_hubs ? 4 : probe_bytes((int32_t)(c.row_ptr[o + 1] - c.row_ptr[o]));
    }
    return c.edge(u, v);
}

// What one pair_count call counts: |A & B & E1 & E2 & [lo, hi)|, A and B per
// lane, E1 and E2 group-uniform and ne of them used (ne < 0: A alone); cut:
// whether lo, hi restrict. memo: the word that keeps the size (uncut pairs),
// or null, its tag alongside.
struct PairOps {
    Set A, B, E1, E2;
    int ne;
    bool cut;
    int32_t lo, hi;
    unsigned long long* memo;
    uint32_t tag;
};

// The size of every active lane's p. Called by all lanes of the group together.
template <int G, int MODE>
__device__ __forceinline__ uint32_t pair_count(const Ctx<G>& c, const PairOps& p, bool active) {
    Set A = p.A, B = p.B;
    const Set &E1 = p.E1, &E2 = p.E2;
    const int ne = p.ne;
    const bool cut = p.cut;
    const int32_t lo = p.lo, hi = p.hi;
    unsigned long long* memo = p.memo;
    const uint32_t tag = p.tag;
    uint32_t r = 0;
    bool longw = false;
    if (ne < 0) {
        if (active) {
            if (cut) {
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(A, lo, hi);
                A = trim(A, lo, hi);
            }
            r = (uint32_t)A.n;
        }
        return r;
    }
    if (active) {
        bool walk = true;
        if (memo) {
            const unsigned long long e = __hip_atomic_load(memo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
            if ((uint32_t)(e >> 32) == tag) {
                r = (uint32_t)e;
                memo = nullptr;
                walk = false;
            }
        }
        if (walk) {
            if (B.n < A.n) {
                const Set t = A;
                A = B;
                B = t;
            }
            if (cut) {
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(A, lo, hi);
                A = trim(A, lo, hi);
            }
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += (uint64_t)A.n * (4 + test_bytes(B));
            if (A.n > kIepLaneWork) {
                longw = true;
            } else if (ne == 0) {
                r = intersect_count_serial(A, B);
            } else {
                for (int32_t i = 0; i < A.n; ++i) {
                    const int32_t y = A.p[i];
                    r += member(B, y) && member(E1, y) && (ne < 2 || member(E2, y));
                }
            }
        }
    }
    uint64_t m = c.g.ballot(longw);
    while (m) {
        const int src = __builtin_ctzll(m);
        m &= m - 1;
        const int32_t* ap = (const int32_t*)uni64<G>(c.g.bcast((long long)A.p, src));
        const int32_t* bp = (const int32_t*)uni64<G>(c.g.bcast((long long)B.p, src));
        const uint32_t* bb = (const uint32_t*)uni64<G>(c.g.bcast((long long)B.bits, src));
        const int32_t an = uni<G>(c.g.bcast(A.n, src)), bn = uni<G>(c.g.bcast(B.n, src));
        const Set W{bp, bn, bb};
        uint32_t mine = 0;
        if (ne == 0 && bb) {
            // four elements per lane in flight
            int32_t i = c.g.gl;
            for (; i + 3 * G < an; i += 4 * G) {
                const int32_t y0 = ap[i], y1 = ap[i + G], y2 = ap[i + 2 * G], y3 = ap[i + 3 * G];
                const uint32_t w0 = bb[y0 >> 5], w1 = bb[y1 >> 5], w2 = bb[y2 >> 5], w3 = bb[y3 >> 5];
                mine += ((w0 >> (y0 & 31)) & 1u) + ((w1 >> (y1 & 31)) & 1u) + ((w2 >> (y2 & 31)) & 1u) +
                        ((w3 >> (y3 & 31)) & 1u);
            }
            for (; i < an; i += G) {
                const int32_t y = ap[i];
                mine += (bb[y >> 5] >> (y & 31)) & 1u;
            }
        } else {
            for (int32_t i = c.g.gl; i < an; i += G) {
                const int32_t y = ap[i];
                mine += member(W, y) && (ne < 1 || member(E1, y)) && (ne < 2 || member(E2, y));
            }
        }
        const uint32_t tot = c.g.sum(mine);
        if (c.g.gl == src) r = tot;
    }
    if (memo) {
        __hip_atomic_store(memo, ((unsigned long long)tag << 32) | r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
    }
    return r;
}

template <int K, int G>
__device__ __forceinline__ Set iep_operand(const Ctx<G>& c, const int32_t (&w)[K], int op) {
    return op >= 0 ? c.nbr(pick<K>(w, op)) : c.buf(-1 - op);
}

// The outer images among w[0..F-1] that lie in a term's set, of the levels in
// t.inj: w[o] is in the cut and adjacent to every parent's image (those the
// pattern makes adjacent are not tested).
template <int K, int G, int MODE, int F>
__device__ __forceinline__ uint32_t iep_images(const GpPlanDesc& d, const Ctx<G>& c, const GpIepTerm& t, uint32_t inj,
                                               const int32_t (&w)[K], int32_t lo, int32_t hi) {
    uint32_t n = 0;
#pragma unroll
    for (int o = 0; o < F; ++o) {
        if (!((inj >> o) & 1u)) continue;
        const int32_t y = w[o];
        bool in = y >= lo && y < hi;
        uint32_t need = t.pm & ~(uint32_t)d.adj[o];
        while (need) {
            const int p = __builtin_ctz(need);
            need &= need - 1;
            if (in) in = adjacent<G, MODE>(c, y, pick<K>(w, p));
        }
        n += in ? 1u : 0u;
    }
    return n;
}

// The operands of term t for an active lane's binding w.
template <int K, int G>
__device__ __forceinline__ void iep_operands(const Ctx<G>& c, const GpIepTerm& t, const int32_t (&w)[K], bool active,
                                             PairOps& p) {
    bounds<K>(t.hi_src, t.lo_src, w, p.lo, p.hi);
    p.cut = (t.hi_src | t.lo_src) != 0;
    p.ne = t.n_op - 2;
    p.memo = nullptr;
    p.tag = 0;
    p.A = p.B = p.E1 = p.E2 = Set{nullptr, 0, nullptr};
    // in every lane, active or not: the group's walks test their elements in them
    if (t.n_op > 2) p.E1 = iep_operand<K, G>(c, w, t.op[1]);
    if (t.n_op > 3) p.E2 = iep_operand<K, G>(c, w, t.op[2]);
    if (!active) return;
    p.A = iep_operand<K, G>(c, w, t.op[0]);
    if (t.n_op < 2) return;
    p.B = iep_operand<K, G>(c, w, t.op[t.n_op - 1]);
    if (t.memo) {
        const int32_t a = pick<K>(w, t.op[0]);
        p.memo = iep_memo_word<G>(c, a, pick<K>(w, t.op[1]));
        p.tag = 0x80000000u | (uint32_t)(a + 1);
    }
}

// Terms of the sum over partitions from the sizes cnt[(M - 1) * kBlock].
template <int N>
__device__ __forceinline__ unsigned __int128 iep_combine(const uint32_t* cnt) {
    typedef unsigned __int128 u128;
    auto P = [&](int a) { return (u128)cnt[(a - 1) * kBlock]; };
    if constexpr (N == 2) {
        return P(1) * P(2) - P(3);
    } else if constexpr (N == 3) {
        return P(1) * P(2) * P(4) - P(3) * P(4) - P(5) * P(2) - P(6) * P(1) + 2 * P(7);
    } else {
        // blocks: singles 1 2 4 8; pairs 3 5 9 6 10 12; triples 7 11 13 14; all 15
        return P(1) * P(2) * P(4) * P(8) -
               (P(3) * P(4) * P(8) + P(5) * P(2) * P(8) + P(9) * P(2) * P(4) + P(6) * P(1) * P(8) +
                P(10) * P(1) * P(4) + P(12) * P(1) * P(2)) +
               (P(3) * P(12) + P(5) * P(10) + P(9) * P(6)) +
               2 * (P(7) * P(8) + P(11) * P(4) + P(13) * P(2) + P(14) * P(1)) - 6 * P(15);
    }
}

// The inclusion-exclusion value of every active lane's binding w (outer
// levels 0 .. K-N-1). Called by all lanes of the group together.
template <int K, int G, int MODE, int N>
__device__ __forceinline__ unsigned __int128 iep_value(const GpPlanDesc& d, const Ctx<G>& c, const int32_t (&w)[K],
                                                       bool active) {
    static_assert(N >= 2 && N <= kIepMaxN && N <= K - 2, "IEP inner levels");
#pragma unroll 1
    for (int m = 0; m < (1 << N) - 1; ++m) {
        const GpIepTerm& t = d.it[m];
        if (t.alias >= 0) {
            c.cnt[m * kBlock] = c.cnt[t.alias * kBlock];
            continue;
        }
        PairOps p;
        iep_operands<K, G>(c, t, w, active, p);
        uint32_t r = pair_count<G, MODE>(c, p, active);
        if (active && t.inj) r -= iep_images<K, G, MODE, K - N>(d, c, t, t.inj, w, p.lo, p.hi);
        c.cnt[m * kBlock] = r;
    }
    return iep_combine<N>(c.cnt);
}

// The last two enumerated levels flattened into one load-balanced batch
// (leaf mode 3): each lane takes a candidate x of level K-3 and cuts its
// level-(K-2) candidate list; a group prefix sum over the list lengths then
// deals every (x, y) pair to a lane, which counts the last level alone. This
// keeps all G lanes busy when the per-candidate lists are short (sparse
// graphs), where leaf mode 1 leaves most lanes idle. Only used when no build
// runs after level K-3 is bound.
template <int K, int G, int MODE>
__device__ void flat_leaf(const GpPlanDesc& d, const Ctx<G>& c, const int32_t (&v)[K], Set S,
                          int32_t st, uint32_t inj_l, uint64_t& acc, uint64_t& carry) {
    constexpr int L = K - 3;
    const GpLevel& l2 = d.lv[K - 2];
    for (int32_t base = 0; base < S.n; base += G) {
        if (c.expired()) break;
        const int32_t i = base + c.g.gl;
        int32_t x2 = 0;
        Set C{nullptr, 0, nullptr};
        if (i < S.n) {
            x2 = S.p[(int64_t)i * st];
            if (!inj_hit<K>(inj_l, v, x2)) {
                int32_t w[K];
#pragma unroll
                for (int j = 0; j < K; ++j) w[j] = v[j];
                w[L] = x2;
                int32_t lo, hi;
                bounds<K>(l2.hi_src, l2.lo_src, w, lo, hi);
                C = l2.list >= 0 ? c.nbr(pick<K>(w, l2.list)) : c.buf(l2.buf);
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(C, lo, hi);
                C = trim(C, lo, hi);
            }
        }
        // inclusive prefix sum of the list lengths over the group
        int32_t incl = C.n;
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {
            int32_t t = __shfl_up(incl, off, G);
            if (c.g.gl >= off) incl += t;
        }
        const int32_t total = __shfl(incl, G - 1, G);
        const int32_t excl = incl - C.n;
        const long long cp = (long long)C.p;
        if constexpr (MODE == MODE_ACCOUNT)
            if (c.g.gl == 0) *c.bytes += 4ull * (uint64_t)total;
        for (int32_t t0 = 0; t0 < total; t0 += G) {
            const int32_t item = t0 + c.g.gl;
            // owner: the last lane whose exclusive prefix is <= item
            int32_t o = 0;
#pragma unroll
            for (int step = G / 2; step >= 1; step >>= 1) {
                const int32_t e2 = __shfl(excl, o + step, G);
                if (e2 <= item) o += step;
            }
            const int32_t ox = __shfl(x2, o, G);
            const int32_t oex = __shfl(excl, o, G);
            const int32_t* op = (const int32_t*)__shfl(cp, o, G);
            if (item < total) {
                const int32_t y = op[item - oex];
                int32_t w[K];
#pragma unroll
                for (int j = 0; j < K; ++j) w[j] = v[j];
                w[L] = ox;
                if (!inj_hit<K>(l2.inj, w, y)) {
                    w[K - 2] = y;
                    // pre_below sets are cut at their build: op is the whole buffer
                    add_count(acc, leaf_serial<K, G, MODE>(d, c, w, item - oex), carry);
                }
            }
        }
    }
}

// Leaf mode 4: lanes take different second-to-last candidates x as in leaf
// mode 1, except that where the last level is pre & N(x) with a group-uniform
// pre that is a hub bitmap, a long N(x) (more than kCoopList elements after the
// cut) is walked by the whole group: one hub candidate otherwise keeps one
// lane busy for thousands of elements while the other lanes of its wavefront
// idle. The group takes the long lists one after another (ballot), each lane
// every G-th element (coalesced loads), and each element costs one bit test
// in the shared bitmap. Returns false (nothing done) when the last level has
// another form; the caller then counts it as in leaf mode 1.
//
// With a memo (c.memo), the count |N(x) & pre & [lo, hi)| of a hub candidate
// x is kept per root edge: the host enables it only when pre and the cut come
// from the two root levels, so for one root they are fixed and the count
// depends on x alone, however the levels between were bound (split tasks of
// one root that a group takes in a row share it). The earlier
// images the last level must avoid are then all parents of x, so each lies
// in N(x), and whether it falls in the set is its pre bit and the cut: they
// are subtracted per lane.
constexpr int32_t kCoopList = 64;

template <int K, int G, int MODE>
__device__ bool coop_bits_leaf(const GpPlanDesc& d, const Ctx<G>& c, const int32_t (&v)[K], Set S, int32_t st,
                               uint32_t inj_l, uint64_t& acc, uint64_t& carry) {
    const GpLevel& ll = d.lv[K - 1];
    if (ll.last_list != K - 2) return false;
    const Set A = ll.pre_buf >= 0 ? c.buf_u(ll.pre_buf) : c.nbr_u(pick<K>(v, ll.pre_list));
    if (!A.bits) return false;
    const uint32_t* bits = A.bits;
    for (int32_t base = 0; base < S.n; base += G) {
        if (c.expired()) break;
        const int32_t i = base + c.g.gl;
        int32_t x = -1;
        Set B{nullptr, 0, nullptr};
        bool longl = false;
        if (i < S.n) {
            x = S.p[(int64_t)i * st];
            if (!inj_hit<K>(inj_l, v, x)) {
                int32_t w[K];
#pragma unroll
                for (int j = 0; j < K; ++j) w[j] = v[j];
                w[K - 2] = x;
                int32_t lo, hi;
                bounds<K>(ll.hi_src, ll.lo_src, w, lo, hi);
                auto skip = [&](int32_t y) { return inj_hit<K>(ll.inj, w, y); };
                if (c.memo && x < c.n_hubs) {
                    // earlier images in the set: parents of x, so in N(x)
                    uint32_t corr = 0;
#pragma unroll
                    for (int j = 0; j < K - 1; ++j)
                        if ((ll.inj >> j) & 1u) {
                            const int32_t y = w[j];
                            if (y >= lo && y < hi) {
                                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 4;
                                corr += ((bits[y >> 5] >> (y & 31)) & 1u) ? 1u : 0u;
                            }
                        }
                    const unsigned long long e = c.memo[x];
                    if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
                    if ((uint32_t)(e >> 32) == c.tag) {
                        add_count(acc, (uint32_t)e - corr, carry);
                    } else {
                        const Set Bn = c.nbr(x);
                        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(Bn, lo, hi);
                        B = trim(Bn, lo, hi);
                        if (B.n <= kCoopList) {
                            const uint32_t all = count_bits(B, bits, [](int32_t) { return false; });
                            c.memo[x] = ((unsigned long long)c.tag << 32) | all;
                            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8ull * (uint64_t)B.n + 8;
                            add_count(acc, all - corr, carry);
                        } else {
                            longl = true;
                        }
                    }
                } else {
                    B = c.nbr(x);
                    if (B.n <= kShortList) {
                        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8ull * (uint64_t)B.n;
                        add_count(acc, count_bits_range(B, lo, hi, bits, skip), carry);
                    } else {
                        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(B, lo, hi);
                        B = trim(B, lo, hi);
                        if (B.n <= kCoopList) {
                            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8ull * (uint64_t)B.n;
                            add_count(acc, count_bits(B, bits, skip), carry);
                        } else {
                            longl = true;
                        }
                    }
                }
            }
        }
        uint64_t m = c.g.ballot(longl);
        while (m) {
            const int o = __builtin_ctzll(m);
            m &= m - 1;
            const int32_t ox = __shfl(x, o, G);
            const int32_t on = __shfl(B.n, o, G);
            const int32_t* op = (const int32_t*)__shfl((long long)B.p, o, G);
            int32_t w[K];
#pragma unroll
            for (int j = 0; j < K; ++j) w[j] = v[j];
            w[K - 2] = ox;
            uint32_t cnt = 0, all = 0;
            for (int32_t j = c.g.gl; j < on; j += G) {
                const int32_t y = op[j];
                if ((bits[y >> 5] >> (y & 31)) & 1u) {
                    ++all;
                    cnt += !inj_hit<K>(ll.inj, w, y);
                }
            }
            if constexpr (MODE == MODE_ACCOUNT)
                if (c.g.gl == 0) *c.bytes += 8ull * (uint64_t)on;
            add_count(acc, cnt, carry);
            if (c.memo && ox < c.n_hubs) {
                // the long list of a hub candidate: keep its whole count
                const uint32_t tot = (uint32_t)c.g.sum(all);
                if (c.g.gl == 0) {
                    c.memo[ox] = ((unsigned long long)c.tag << 32) | tot;
                    if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
                }
            }
        }
    }
    return true;
}

// Leaf mode 5 (table_kernel): the last level is N(x) & N(p) cut by root levels,
// p a root endpoint, so its size is a function of x alone while the root edge
// stays: the block's table holds it for every vertex below tab_n. A lane's
// element costs one coalesced list load and one LDS load; vertices past the
// table, the ones of lowest degree, have their lists walked. Of the images the
// last level must avoid, the other root endpoint is left out of the table;
// those that are parents of x lie in the set or not whatever x is, one
// number per call (corr); the rest (mask ex) are in the set only of the x
// adjacent to them, and only if they are in N(p) and the cut at all.
// Of levels [2, F), the images that the last level must avoid and that lie in
// N(p) and the cut: as a mask (the root endpoints are not among them).
template <int K, int G, int F>
__device__ __forceinline__ uint32_t table_images(const GpLevel& ll, const Ctx<G>& c, const int32_t (&v)[K], int32_t p,
                                                 int32_t lo, int32_t hi) {
    uint32_t m = 0;
#pragma unroll
    for (int j = 2; j < F; ++j)
        if ((ll.inj >> j) & 1u) {
            const int32_t y = v[j];
            if (y >= lo && y < hi && c.edge(y, p)) m |= 1u << j;
        }
    return (uint32_t)uni<G>((int32_t)m);
}

template <int K, int G, int MODE>
__device__ __forceinline__ void table_leaf(const GpPlanDesc& d, const Ctx<G>& c, const int32_t (&v)[K], Set S,
                                           int32_t slo, int32_t shi, uint32_t inj_l, uint32_t images, uint64_t& acc,
                                           uint64_t& carry) {
    const uint32_t corr = (uint32_t)__popc(images & d.lv[K - 2].parents);
    const uint32_t ex = images & ~(uint32_t)d.lv[K - 2].parents;
    const GpLevel& ll = d.lv[K - 1];
    const int32_t p = ll.pre_list == 0 ? v[0] : v[1];
    int32_t lo, hi;
    bounds<K>(ll.hi_src, ll.lo_src, v, lo, hi);
    // K = 4: level 2 itself, dealt to the block's waves in batches of G
    const int32_t first = K == 4 ? c.sj * G : 0, step = K == 4 ? c.sJ * G : G;
    if (S.n > 4 * G || K == 4) {
        if (slo > 0 || shi < 0x7fffffff) S = trim_u<G>(S, slo, shi);
        slo = 0;
        shi = 0x7fffffff;
    }
    uint32_t sum = 0, taken = 0;
    for (int32_t base = first; base < S.n; base += step) {
        const int32_t i = base + c.g.gl;
        const int32_t x = i < S.n ? S.p[i] : -1;
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += i < S.n ? 4 : 0;
        if (x >= slo && x < shi && !inj_hit<K>(inj_l, v, x)) {
            ++taken;
            if (x < c.tab_n) {
                sum += c.tab[x];
            } else {
                const Set N = c.nbr(x), P = c.nbr(p);
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += (uint64_t)N.n * (4 + test_bytes(P));
                auto none = [](int32_t) { return false; };
                if (P.bits) sum += count_bits_range(N, lo, hi, P.bits, none);
                else sum += intersect_count_serial(trim(N, lo, hi), trim(P, lo, hi));
                if (c.out >= lo && c.out < hi && c.edge(c.out, x)) --sum;
            }
            for (uint32_t m = ex; m; m &= m - 1) sum -= c.edge(pick<K>(v, __builtin_ctz(m)), x) ? 1u : 0u;
        }
    }
    // every unit of sum is an entry y of the list of a different x: fewer than the
    // graph's 2^31 entries (a load refuses more)
    add_count(acc, (uint64_t)sum - (uint64_t)corr * taken, carry);
}

// Level K-3 above a table_leaf over the list of its vertex: the lanes look up
// 64 candidates' list bounds (and whether the last level must avoid them) at
// once, so that a candidate costs its list's loads alone.
template <int K, int G, int MODE>
__device__ __forceinline__ void table_lists(const GpPlanDesc& d, const Ctx<G>& c, int32_t (&v)[K], Set S, int32_t st,
                                            uint32_t inj_l, uint64_t& acc, uint64_t& carry) {
    constexpr int L = K - 3;
    const GpLevel& l2 = d.lv[K - 2];
    const GpLevel& ll = d.lv[K - 1];
    const int32_t p = ll.pre_list == 0 ? v[0] : v[1];
    int32_t lo, hi;
    bounds<K>(ll.hi_src, ll.lo_src, v, lo, hi);
    const uint32_t images = table_images<K, G, L>(ll, c, v, p, lo, hi);
    const bool avoid = L >= 2 && ((ll.inj >> L) & 1u);
    for (int32_t base = 0; base < S.n; base += G) {
        if (c.expired()) break;
        const int32_t i = base + c.g.gl;
        int32_t x = 0, n = 0;
        long long q = 0;
        uint32_t own = 0;
        if (i < S.n) {
            x = S.p[(int64_t)i * st];
            if (!inj_hit<K>(inj_l, v, x)) {
                const int64_t b = c.row_ptr[x], e = c.row_ptr[x + 1];
                q = (long long)(c.col + b);
                n = (int32_t)(e - b);
                if (avoid && x >= lo && x < hi) own = c.edge(x, p) ? 1u : 0u;
            }
        }
        uint64_t m = c.g.ballot(n > 0);
        while (m) {
            const int src = __builtin_ctzll(m);
            m &= m - 1;
            v[L] = uni<G>(c.g.bcast(x, src));
            const Set N{(const int32_t*)uni64<G>(c.g.bcast(q, src)), uni<G>(c.g.bcast(n, src)), nullptr};
            int32_t slo, shi;
            bounds<K>(l2.hi_src, l2.lo_src, v, slo, shi);
            const uint32_t mine = (uint32_t)uni<G>((int32_t)c.g.bcast(own, src)) << L;
            table_leaf<K, G, MODE>(d, c, v, N, slo, shi, l2.inj, images | mine, acc, carry);
        }
    }
}

// The IEP leaf at the last outer level L (inner levels L+1 .. K-1): every
// candidate x of level L adds its inclusion-exclusion value, lanes taking
// different candidates. S: this task's candidates (every st-th), Sf: all of
// them. No build runs after level L is bound: an inner set whose last parent
// is level L is left unbuilt.
//
// Two inner levels, one of whose sets (term b) does not depend on x while the
// other's (term a) does (d.iep_sum): the sum over x of Pa(x) Pb(x) - P3(x) is
// taken apart. Pb is one number less [x in S_b]. P3(x) counts the y of
// Y = S_b & (S_a's other operands) adjacent to x, so its sum over x is the
// sum over y in Y of the candidates adjacent to y: |Y| pair sizes, kept in the
// memo where the candidates are a whole list, in place of a walk of Y or N(x)
// for each of the far more numerous x. A split task takes its slice of Y as it
// takes its slice of x: partial totals may be negative, and are exact mod
// 2^128.
//
// TAB: |N(p) & N(x)| of the x below tab_n comes from the block's table, p the
// root endpoint whose roots the block's wavefronts are working on; other x, of low
// degree, have their lists walked against the filter of N(p).

// Whether y (which passed the filter) is a neighbor of p, P = N(p).
template <int G>
__device__ __forceinline__ bool filt_hit(const Ctx<G>& c, const Set& P, int32_t y) {
    const uint32_t b = (uint32_t)y & (32u * kFiltWords - 1);
    return ((c.filt[b >> 5] >> (b & 31)) & 1u) && member(P, y);
}

// |N(p) & N(x)| of every active lane's x. Called by all lanes of the group.
template <int G, int MODE>
__device__ __forceinline__ uint32_t filt_count(const Ctx<G>& c, const Set& P, int32_t x, bool active) {
    uint32_t r = 0;
    bool longw = false;
    Set N{nullptr, 0, nullptr};
    if (active) {
        N = c.nbr(x);
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 4ull * (uint64_t)min(N.n, P.n);
        if (P.n * 8 < N.n) {
            // a search in N(x) for each of p's few neighbors
            if (P.n <= kIepLaneWork) {
                for (int32_t i = 0; i < P.n; ++i) r += contains(N.p, N.n, P.p[i]) ? 1u : 0u;
            } else {
                longw = true;
            }
        } else if (N.n > kIepLaneWork) {
            longw = true;
        } else {
            int32_t i = 0;
            for (; i + 4 <= N.n; i += 4) {
                const int32_t y0 = N.p[i], y1 = N.p[i + 1], y2 = N.p[i + 2], y3 = N.p[i + 3];
                r += (filt_hit<G>(c, P, y0) ? 1u : 0u) + (filt_hit<G>(c, P, y1) ? 1u : 0u) +
                     (filt_hit<G>(c, P, y2) ? 1u : 0u) + (filt_hit<G>(c, P, y3) ? 1u : 0u);
            }
            for (; i < N.n; ++i) r += filt_hit<G>(c, P, N.p[i]) ? 1u : 0u;
        }
    }
    uint64_t m = c.g.ballot(longw);
    while (m) {
        const int src = __builtin_ctzll(m);
        m &= m - 1;
        const int32_t* np = (const int32_t*)uni64<G>(c.g.bcast((long long)N.p, src));
        const int32_t nn = uni<G>(c.g.bcast(N.n, src));
        uint32_t mine = 0;
        for (int32_t i = c.g.gl; i < nn; i += G) mine += filt_hit<G>(c, P, np[i]) ? 1u : 0u;
        const uint32_t tot = c.g.sum(mine);
        if (c.g.gl == src) r = tot;
    }
    return r;
}

template <int K, int L, int G, int MODE, bool TAB>
__device__ __forceinline__ void iep_pair_sum(const GpPlanDesc& d, const Ctx<G>& c, const int32_t (&v)[K], Set S,
                                             int32_t st, Set Sf, uint32_t inj_l, uint64_t& acc, uint64_t& carry) {
    const GpIepTerm& ta = d.it[d.iep_sum - 1];
    const GpIepTerm& tb = d.it[2 - d.iep_sum];
    const GpIepTerm& t3 = d.it[2];
    int32_t lo, hi;
    // Pb but for x
    bounds<K>(tb.hi_src, tb.lo_src, v, lo, hi);
    Set Sb = tb.op[0] >= 0 ? c.nbr_u(pick<K>(v, tb.op[0])) : c.buf_u(-1 - tb.op[0]);
    if constexpr (MODE == MODE_ACCOUNT)
        if (c.g.gl == 0) *c.bytes += cut_bytes(Sb, lo, hi);
    Sb = trim_u<G>(Sb, lo, hi);
    const uint64_t pb = (uint64_t)Sb.n - iep_images<K, G, MODE, L>(d, c, tb, tb.inj, v, lo, hi);
    // Y: the first of term 3's other operands, tested in the second
    int32_t ylo, yhi;
    bounds<K>(t3.hi_src, t3.lo_src, v, ylo, yhi);
    Set Y = t3.op[0] >= 0 ? c.nbr_u(pick<K>(v, t3.op[0])) : c.buf_u(-1 - t3.op[0]);
    Set E{nullptr, 0, nullptr};
    if (t3.n_op > 2) {
        E = t3.op[1] >= 0 ? c.nbr_u(pick<K>(v, t3.op[1])) : c.buf_u(-1 - t3.op[1]);
        if (E.n < Y.n) {
            const Set t = Y;
            Y = E;
            E = t;
        }
    }
    if constexpr (MODE == MODE_ACCOUNT)
        if (c.g.gl == 0) *c.bytes += cut_bytes(Y, ylo, yhi);
    Y = trim_u<G>(Y, ylo, yhi);
    if constexpr (L == 2) {
        if (c.sJ > 1) {
            Y.n = Y.n > c.sj ? (Y.n - c.sj + c.sJ - 1) / c.sJ : 0;
            Y.p += c.sj;
        }
    }
    const GpLevel& lv = d.lv[L];
    const bool whole = lv.list >= 0 && (lv.hi_src | lv.lo_src) == 0;
    const int32_t a = whole ? pick<K>(v, lv.list) : 0;
    int32_t slo, shi;
    bounds<K>(lv.hi_src, lv.lo_src, v, slo, shi);
    if constexpr (TAB) {
        const Set N = c.nbr_u(pick<K>(v, ta.op[0]));
        for (int32_t base = 0; base < S.n; base += G) {
            if (c.expired()) break;
            const int32_t i = base + c.g.gl;
            int32_t x = 0;
            bool active = i < S.n;
            if (active) x = S.p[(int64_t)i * st];
            active = active && !inj_hit<K>(inj_l, v, x);
            const bool far = active && x >= c.tab_n;
            uint64_t q = far || !active ? 0 : c.tab[x];
            if (c.g.ballot(far)) q += filt_count<G, MODE>(c, N, x, far);
            if (!active) continue;
            int32_t w[K];
#pragma unroll
            for (int j = 0; j < K; ++j) w[j] = v[j];
            w[L] = x;
            if (ta.inj) q -= iep_images<K, G, MODE, L + 1>(d, c, ta, ta.inj, w, 0, 0x7fffffff);
            uint64_t b = pb;
            if ((tb.inj >> L) & 1u) b -= iep_images<K, G, MODE, L + 1>(d, c, tb, 1u << L, w, lo, hi);
            const unsigned __int128 val = (unsigned __int128)q * b;
            add_count128(acc, carry, (uint64_t)val, (uint64_t)(val >> 64));
        }
    }
    // the candidates x, then the y: one loop, so one copy of the walk
    const int32_t nx = TAB ? 0 : S.n, ny = Y.n;
    const int32_t xbatches = (nx + G - 1) / G, batches = xbatches + (ny + G - 1) / G;
#pragma unroll 1
    for (int32_t bt = 0; bt < batches; ++bt) {
        if (c.expired()) break;
        const bool is_x = bt < xbatches;
        const int32_t i = (is_x ? bt : bt - xbatches) * G + c.g.gl;
        int32_t z = 0;
        bool active = i < (is_x ? nx : ny);
        if (active) z = (is_x ? S.p : Y.p)[(int64_t)i * st];
        int32_t w[K];
#pragma unroll
        for (int j = 0; j < K; ++j) w[j] = v[j];
        w[L] = z;
        PairOps p;
        if (is_x) {
            active = active && !inj_hit<K>(inj_l, v, z);
            iep_operands<K, G>(c, ta, w, active, p);
        } else {
            if constexpr (MODE == MODE_ACCOUNT)
                if (active) *c.bytes += 4 + (t3.n_op > 2 ? test_bytes(E) : 0);
            active = active && !inj_hit<K>(t3.inj & ((1u << L) - 1), v, z) && (t3.n_op <= 2 || member(E, z));
            p.A = Sf;
            p.B = p.E1 = p.E2 = Set{nullptr, 0, nullptr};
            p.ne = 0;
            // Sf is cut, but its bitmap is the whole list's: N(z) must be cut too
            p.cut = (lv.hi_src | lv.lo_src) != 0;
            p.lo = slo;
            p.hi = shi;
            p.memo = nullptr;
            p.tag = 0x80000000u | (uint32_t)(a + 1);
            if (active) {
                p.B = c.nbr(z);
                if (whole) p.memo = iep_memo_word<G>(c, a, z);
            }
        }
        uint64_t q = pair_count<G, MODE>(c, p, active);
        if (!active) continue;
        if (is_x) {
            if (ta.inj) q -= iep_images<K, G, MODE, L + 1>(d, c, ta, ta.inj, w, p.lo, p.hi);
            uint64_t b = pb;
            if ((tb.inj >> L) & 1u) b -= iep_images<K, G, MODE, L + 1>(d, c, tb, 1u << L, w, lo, hi);
            const unsigned __int128 val = (unsigned __int128)q * b;
            add_count128(acc, carry, (uint64_t)val, (uint64_t)(val >> 64));
        } else {
            // earlier images are no candidates
            if (inj_l) {
#pragma unroll
                for (int o = 0; o < L; ++o) {
                    if (!((inj_l >> o) & 1u)) continue;
                    const int32_t u = v[o];
                    bool in = u >= slo && u < shi && u != z;
                    uint32_t need = lv.parents & ~(uint32_t)d.adj[o];
                    while (need) {
                        const int q2 = __builtin_ctz(need);
                        need &= need - 1;
                        if (in) in = adjacent<G, MODE>(c, u, pick<K>(v, q2));
                    }
                    if (in) q -= adjacent<G, MODE>(c, u, z) ? 1u : 0u;
                }
            }
            carry -= acc < q ? 1u : 0u;
            acc -= q;
        }
    }
}

template <int K, int L, int G, int MODE, bool TAB>
__device__ void iep_level(const GpPlanDesc& d, const Ctx<G>& c, int32_t (&v)[K], Set S, int32_t st, Set Sf,
                          uint32_t inj_l, uint64_t& acc, uint64_t& carry) {
    constexpr int N = K - 1 - L;
    if constexpr (N == 2) {
        if (d.iep_sum) {
            iep_pair_sum<K, L, G, MODE, TAB>(d, c, v, S, st, Sf, inj_l, acc, carry);
            return;
        }
    }
    if constexpr (TAB) return;  // the table kernel takes only such plans
    for (int32_t base = 0; base < S.n; base += G) {
        if (c.expired()) break;
        const int32_t i = base + c.g.gl;
        int32_t w[K];
#pragma unroll
        for (int j = 0; j < K; ++j) w[j] = v[j];
        bool active = false;
        if (i < S.n) {
            w[L] = S.p[(int64_t)i * st];
            active = !inj_hit<K>(inj_l, v, w[L]);
        }
        const unsigned __int128 val = iep_value<K, G, MODE, N>(d, c, w, active);
        if (active) add_count128(acc, carry, (uint64_t)val, (uint64_t)(val >> 64));
    }
}

// IEP: 0 (plain), else the number of inner levels counted with
// inclusion-exclusion (a kernel is built per depth, so each carries only the
// registers of its own depth).
template <int K, int L, int G, int LEAF, int MODE, int IEP>
__device__ void search(const GpPlanDesc& d, const Ctx<G>& c, int32_t (&v)[K], uint64_t& acc,
                       uint64_t& carry) {
    if constexpr (IEP > 0 && L > K - 1 - IEP) {
        return;  // an IEP search ends at its last outer level
    } else {
        const GpLevel& lv = d.lv[L];
        int32_t lo, hi;
        bounds<K>(lv.hi_src, lv.lo_src, v, lo, hi);
        Set S = lv.list >= 0 ? c.nbr_u(pick<K>(v, lv.list)) : c.buf_u(lv.buf);
        if constexpr (LEAF == 5 && IEP == 0 && L == K - 2) {
            const GpLevel& ll = d.lv[K - 1];
            int32_t llo, lhi;
            bounds<K>(ll.hi_src, ll.lo_src, v, llo, lhi);
            const uint32_t images = table_images<K, G, K - 2>(ll, c, v, ll.pre_list == 0 ? v[0] : v[1], llo, lhi);
            table_leaf<K, G, MODE>(d, c, v, S, lo, hi, lv.inj, images, acc, carry);
            return;
        }
        if (!lv.cut_done) {
            if constexpr (MODE == MODE_ACCOUNT)
                if (c.g.gl == 0) *c.bytes += cut_bytes(S, lo, hi);
            S = trim_u<G>(S, lo, hi);
        }
        // a split task binds only its slice of the level-2 candidates
        const Set Sf = S;
        int32_t st = 1;
        if constexpr (L == 2) {
            if (c.sJ > 1) {
                S.n = S.n > c.sj ? (S.n - c.sj + c.sJ - 1) / c.sJ : 0;
                S.p += c.sj;
                st = c.sJ;
            }
        }
        if constexpr (MODE == MODE_ACCOUNT)
            if (c.g.gl == 0) *c.bytes += 4ull * (uint64_t)S.n;
        if constexpr (IEP > 0 && L == K - 1 - IEP) {
            // the last outer level: the inner ones are counted, not enumerated
            iep_level<K, L, G, MODE, LEAF == 5>(d, c, v, S, st, Sf, lv.inj, acc, carry);
            return;
        }
        if constexpr (L == K - 2) {
            if constexpr (LEAF == 4)
                if (coop_bits_leaf<K, G, MODE>(d, c, v, S, st, lv.inj, acc, carry)) return;
            if constexpr (LEAF != 2) {
                for (int32_t base = 0; base < S.n; base += G) {
                    if (c.expired()) break;
                    int32_t i = base + c.g.gl;
                    if (i < S.n) {
                        int32_t x = S.p[(int64_t)i * st];
                        if (!inj_hit<K>(lv.inj, v, x)) {
                            int32_t w[K];
#pragma unroll
                            for (int j = 0; j < K; ++j) w[j] = v[j];
                            w[K - 2] = x;
                            // in a split task's slice the index steps by its ways
                            const int32_t at = L == 2 && c.sJ > 1 ? c.sj + i * st : i;
                            add_count(acc, leaf_serial<K, G, MODE>(d, c, w, at), carry);
                        }
                    }
                }
            } else {
                for (int32_t t = 0; t < S.n; ++t) {
                    if (c.expired()) break;
                    const int32_t x = uni<G>(S.p[(int64_t)t * st]);
                    if (inj_hit<K>(lv.inj, v, x)) continue;
                    v[K - 2] = x;
                    uint32_t cnt = leaf_group<K, G, MODE>(d, c, v);
                    if (c.g.gl == 0) add_count(acc, cnt, carry);
                }
            }
        } else {
            if constexpr (LEAF == 5 && IEP == 0 && L == K - 3) {
                if (d.build_begin[L] == d.build_end[L] && d.lv[K - 2].list == L) {
                    table_lists<K, G, MODE>(d, c, v, S, st, lv.inj, acc, carry);
                    return;
                }
            }
            if constexpr (LEAF == 3 && L == K - 3 && IEP == 0) {
                if (d.build_begin[L] == d.build_end[L]) {
                    flat_leaf<K, G, MODE>(d, c, v, S, st, lv.inj, acc, carry);
                    return;
                }
            }
            for (int32_t t = 0; t < S.n; ++t) {
                if (c.expired()) break;
                const int32_t x = uni<G>(S.p[(int64_t)t * st]);
                if (inj_hit<K>(lv.inj, v, x)) continue;
                v[L] = x;
                if (run_builds<K, G, MODE>(d, c, L, v)) search<K, L + 1, G, LEAF, MODE, IEP>(d, c, v, acc, carry);
            }
        }
    }
}

__device__ __forceinline__ int64_t entry_index(const int64_t* row_ptr, const int32_t* col,
                                               int32_t v0, int32_t v1) {
    int64_t b = row_ptr[v0];
    return b + lower_bound(col + b, (int32_t)(row_ptr[v0 + 1] - b), v1);
}

// One root edge's last level as roots_flat shares it out: element e of the
// wavefront's walk is walk[e] for the edge that holds it.
struct alignas(16) FlatRoot {
    const int32_t* walk;  // the walked list, moved back by where it starts in the walk
    const void* test;     // the other list, or its bitmap
    int32_t test_n;       // the other list's length; -1: a bitmap
    int32_t lo, hi;       // the level's cut
    int32_t pad;
};
constexpr int kFlatWindows = 4;  // windows of 64 elements in flight

// Last levels N(v0) & N(v1) of 64 root edges (k = 3), one per lane, walked
// as one list: the wavefront takes 64 elements of all the edges' shorter lists
// at a time, each lane finding its edge by a count of the lists that start up
// to its element. One lane per edge waits for the longest list of the 64,
// several times the mean on a power-law graph, and reads 64 lists at once; here
// the lanes read runs of a list. What bounds it is the chain from LDS to the
// element to the bitmap's word, and the first chunk, whose lists are the longest:
// four windows in flight. Triangles, a whole call, one lane per edge and 1, 2, 4
// windows: R-MAT 17 (971,517 edges) 159 and 139, 131, 129 us; R-MAT 20 (8.4M) 1,508
// and 993, 891, 860. Without bitmaps the test is a search per element, and lanes
// that merge two lists alone are as fast: there the old way stays.
template <int G, int MODE>
__device__ __forceinline__ uint32_t roots_flat(const GpPlanDesc& d, const Ctx<G>& c, int32_t v0, int32_t v1,
                                               bool active) {
    static_assert(G == 64, "one wavefront");
    const GpLevel& lv = d.lv[2];
    FlatRoot me{nullptr, nullptr, 0, 0, 0, 0};
    int32_t n = 0;
    if (active) {
        const int32_t v[3] = {v0, v1, 0};
        bounds<3>(lv.hi_src, lv.lo_src, v, me.lo, me.hi);
        Set W = c.nbr(v0), T = c.nbr(v1);
        if (T.n < W.n) {
            const Set t = W;
            W = T;
            T = t;
        }
        if (W.n > kShortList) {
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += cut_bytes(W, me.lo, me.hi);
            W = trim(W, me.lo, me.hi);
        }
        n = W.n;
        if constexpr (MODE == MODE_ACCOUNT) *c.bytes += (uint64_t)n * (4 + test_bytes(T));
        me.walk = W.p;
        me.test = T.bits ? (const void*)T.bits : (const void*)T.p;
        me.test_n = T.bits ? -1 : T.n;
    }
    int32_t end = n;  // inclusive scan
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t o = __shfl_up(end, off, 64);
        if (c.g.gl >= off) end += o;
    }
    const int32_t total = uni<64>(__shfl(end, 63, 64));
    const int32_t start = end - n;
    const uint64_t full = __ballot(n > 0);
    group_fence();  // the last call's reads
    if (n > 0) {
        me.walk = (const int32_t*)((uintptr_t)me.walk - 4 * (uintptr_t)start);
        c.flat[(int)__popcll(full & ((1ull << c.g.gl) - 1))] = me;
    }
#pragma unroll
    for (int u = 0; u < kFlatWindows; ++u) c.starts[u * 64 + c.g.gl] = 0;
    group_fence();
    uint32_t cnt = 0;
    int32_t before = -1;  // lists that start before the window, less one
    for (int32_t t = 0; t < total; t += 64 * kFlatWindows) {
        const bool in = n > 0 && start >= t && start < t + 64 * kFlatWindows;
        if (in) c.starts[start - t] = 1;
        group_fence();
        uint64_t m[kFlatWindows];
#pragma unroll
        for (int u = 0; u < kFlatWindows; ++u) m[u] = __ballot(c.starts[u * 64 + c.g.gl] != 0);
        group_fence();
        if (in) c.starts[start - t] = 0;
        FlatRoot r[kFlatWindows];
        int32_t x[kFlatWindows];
#pragma unroll
        for (int u = 0; u < kFlatWindows; ++u) {
            const int32_t e = t + u * 64 + c.g.gl;
            const int32_t own = before + (int)__popcll(m[u] & ((2ull << c.g.gl) - 1));
            before += (int)__popcll(m[u]);
            x[u] = -1;
            r[u] = FlatRoot{nullptr, nullptr, 0, 0, 0, 0};
            if (e < total) {
                r[u] = c.flat[own];
                x[u] = r[u].walk[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kFlatWindows; ++u) {
            if (x[u] >= r[u].lo && x[u] < r[u].hi) {
                if (r[u].test_n < 0) cnt += (((const uint32_t*)r[u].test)[x[u] >> 5] >> (x[u] & 31)) & 1u;
                else cnt += member(Set{(const int32_t*)r[u].test, r[u].test_n, nullptr}, x[u]) ? 1u : 0u;
            }
        }
    }
    return cnt;
}

// One group's root tasks [t0, t1) of task space ts: every task binds its root
// edge (levels 0 and 1) and searches the rest. Patterns whose search ends at
// the root (k <= 3, or IEP over all k-2 levels after it) take different roots
// in different lanes. per_root (MODE_PER_ROOT): each root's count at the CSR
// entry of the root edge.
template <int K, int G, int LEAF, int MODE, int IEP>
__device__ __forceinline__ void run_tasks(const GpPlanDesc& d, Ctx<G>& c, const TaskSpace& ts, int64_t t0,
                                          int64_t t1, uint64_t& acc, uint64_t& carry,
                                          unsigned long long* per_root) {
    constexpr bool PER_ROOT = MODE == MODE_PER_ROOT;
    if constexpr (IEP > 0 && IEP == K - 2) {
        // the root is the last outer level: lanes take different roots
        for (int64_t base = t0; base < t1; base += G) {
            const int64_t r = base + c.g.gl;
            int32_t w[K];
#pragma unroll
            for (int j = 0; j < K; ++j) w[j] = 0;
            const bool active = r < t1;
            if (active) {
                const int2 e = ts.roots[ts.offset + r * ts.stride];
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
                w[0] = e.x;
                w[1] = e.y;
            }
            const unsigned __int128 val = iep_value<K, G, MODE, K - 2>(d, c, w, active);
            if (active) {
                add_count128(acc, carry, (uint64_t)val, (uint64_t)(val >> 64));
                if constexpr (PER_ROOT) per_root[entry_index(c.row_ptr, c.col, w[0], w[1])] = (unsigned long long)val;
            }
        }
        return;
    }
    if constexpr (K == 3 && LEAF != 2 && G == 64 && !PER_ROOT) {
        // intersections of many edges shared out evenly, where bitmaps test the long lists
        // (and 64 shorter lists, of at most deg2 = cap elements, are counted in 32 bits)
        if (c.flat && d.lv[2].last_list >= 0 && d.lv[2].pre_buf < 0 && d.lv[2].inj == 0 && c.n_hubs > 0 &&
            c.cap < (1 << 25)) {
            for (int64_t base = t0; base < t1; base += G) {
                const int64_t r = base + c.g.gl;
                int2 e = make_int2(0, 0);
                if (r < t1) {
                    e = ts.roots[ts.offset + r * ts.stride];
                    if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
                }
                add_count(acc, roots_flat<G, MODE>(d, c, e.x, e.y, r < t1), carry);
            }
            return;
        }
    }
    if constexpr (K <= 3 && LEAF != 2) {
        // lanes take different roots
        for (int64_t base = t0; base < t1; base += G) {
            int64_t r = base + c.g.gl;
            if (r < t1) {
                int2 e = ts.roots[ts.offset + r * ts.stride];
                uint64_t cnt = 1;
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 8;
                if constexpr (K == 3) {
                    int32_t w[K] = {e.x, e.y, 0};
                    cnt = leaf_serial<K, G, MODE>(d, c, w);
                }
                add_count(acc, cnt, carry);
                if constexpr (PER_ROOT) per_root[entry_index(c.row_ptr, c.col, e.x, e.y)] = cnt;
            }
        }
    } else {
        for (int64_t t = t0; t < t1; ++t) {
            const int64_t r = task_root(t, ts.split_roots, ts.split_ways, c.sj, c.sJ);
            c.tag = ts.tag_base + (uint32_t)(r + 1);
            int2 e = ts.roots[ts.offset + r * ts.stride];
            e.x = uni<G>(e.x);
            e.y = uni<G>(e.y);
            const uint64_t before = acc;
            if constexpr (MODE == MODE_ACCOUNT)
                if (c.g.gl == 0) *c.bytes += 8;
            if constexpr (K <= 3) {
                uint64_t cnt = 1;
                if constexpr (K == 3) {
                    int32_t w[K] = {e.x, e.y, 0};
                    cnt = leaf_group<K, G, MODE>(d, c, w);
                }
                if (c.g.gl == 0) add_count(acc, cnt, carry);
            } else {
                int32_t v[K];
#pragma unroll
                for (int j = 0; j < K; ++j) v[j] = 0;
                v[0] = e.x;
                v[1] = e.y;
                if (run_builds<K, G, MODE>(d, c, 1, v)) search<K, 2, G, LEAF, MODE, IEP>(d, c, v, acc, carry);
            }
            if constexpr (PER_ROOT) {
                uint64_t mine = c.g.sum(acc - before);
                if (c.g.gl == 0) per_root[entry_index(c.row_ptr, c.col, e.x, e.y)] = mine;
            }
        }
    }
}

// Wavefronts per SIMD the compiler is asked to keep resident (it trims
// registers, spilling a few if it must). The searches are bound by the
// latency of scattered loads, so more resident wavefronts pay even against
// some spills. Measured on R-MAT 17 for k = 5 (64-lane groups with lanes on
// separate candidates: 8, others 6) and on Chung-Lu 7000 for k = 6 (64-lane
// groups 6, others 5); k >= 7 keeps the compiler's choice. IEP over 3 or 4
// inner levels keeps 7 or 15 set sizes and their 128-bit products live: 5
// and 4 wavefronts.
// XCDs of the device; workgroups are dealt to them round robin in launch
// order, so block b of a grid runs on XCD b mod kXcds.
constexpr int kXcds = 8;

// Tasks of XCD x when n tasks are dealt in blocks of B tasks, block b to
// XCD b mod kXcds.
__device__ __forceinline__ int64_t xcd_tasks(int64_t n, int64_t B, int x) {
    const int64_t round = (int64_t)kXcds * B;
    const int64_t full = n / round, rem = n - full * round;
    return full * B + min(max(rem - (int64_t)x * B, (int64_t)0), B);
}

// Global task of XCD x's j-th task.
__device__ __forceinline__ int64_t xcd_task(int64_t j, int64_t B, int x) {
    const int64_t b = j / B;
    return (b * kXcds + x) * B + (j - b * B);
}

// Next chunk of a group from the queue's cursors, or -1 once all are
// exhausted. *cur (in LDS: kept in a register through the search it cost
// spills): the cursor the group takes from (at first its home). When that one
// runs dry the group reads the others at once (plain loads, which do not queue
// up as atomics do) and moves on to the next one with chunks left, in cyclic
// order, so groups that run dry together spread out. Cursors only grow, so the
// search ends; the first group to see all of them dry says so in one word,
// which later ones read instead.
template <int G>
__device__ __forceinline__ int64_t next_chunk(const Group<G>& grp, unsigned long long* queue, int64_t n_chunks,
                                              int* cur) {
    // opaque, so that nothing computed from the lane for a grab is kept in
    // registers through the search between grabs
    int gl = grp.gl;
    asm volatile("" : "+v"(gl));
    for (;;) {
        const int c = uni<G>(*cur);
        unsigned long long v = 0;
        if (gl == 0) v = atomicAdd(&queue[c * (kCursorStep * kSlotWords) + SLOT_CURSOR], 1ull);
        const int64_t q = uni64<G>((int64_t)grp.bcast(v, 0)) * kCursors + c;
        if (q < n_chunks) return q;
        if (__hip_atomic_load(&queue[kDoneWord], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return -1;
        uint32_t left = 0;
#pragma unroll 1
        for (int base = 0; base < kCursors; base += G) {
            const int i = base + gl;
            bool some = false;
            if (i < kCursors) {
                const unsigned long long t = __hip_atomic_load(&queue[i * (kCursorStep * kSlotWords) + SLOT_CURSOR],
                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                some = (int64_t)t * kCursors + i < n_chunks;
            }
            left |= (uint32_t)grp.ballot(some) << base;
        }
        if (left == 0) {
            if (gl == 0)
                __hip_atomic_store(&queue[kDoneWord], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return -1;
        }
        const uint32_t from = (uint32_t)(c + 1) & (kCursors - 1);
        const uint32_t rot = (left >> from) | (left << (kCursors - from));
        group_fence();
        *cur = (int)((from + (uint32_t)__builtin_ctz(rot)) & (kCursors - 1));
        group_fence();
    }
}

// Next grab of a group: `chunk` tasks [*t0, *t1), or false once every cursor
// is exhausted. With XCD blocks the group starts at its own XCD's cursor
// (*q = 0) and moves on to the next XCD's when it runs dry; it never comes
// back to one that was dry.
template <int G>
__device__ __forceinline__ bool grab_tasks(const Group<G>& grp, unsigned long long* queue, int64_t n_tasks,
                                           int64_t n_chunks, int64_t chunk, int64_t xcd_block, int* q, int64_t* t0,
                                           int64_t* t1) {
    if (xcd_block <= 0) {
        const int64_t a = next_chunk<G>(grp, queue, n_chunks, q);
        if (a < 0) return false;
        *t0 = a * chunk;
        *t1 = min(*t0 + chunk, n_tasks);
        return true;
    }
    const int home = (int)(blockIdx.x % kXcds);
    for (int tries = *q; tries < kXcds; ++tries) {
        const int x = (home + tries) % kXcds;
        const int64_t nx = xcd_tasks(n_tasks, xcd_block, x);
        unsigned long long v = 0;
        if (grp.gl == 0) v = atomicAdd(&queue[x * (kCursorStep * kSlotWords) + SLOT_CURSOR], (unsigned long long)chunk);
        const int64_t j = uni64<G>((int64_t)grp.bcast(v, 0));
        if (j < nx) {
            *t0 = xcd_task(j, xcd_block, x);
            *t1 = *t0 + min(chunk, nx - j);
            *q = tries;
            return true;
        }
    }
    return false;
}

constexpr int occupancy_target(int K, int G, int LEAF, int IEP = 0) {
    return IEP > 0 ? (IEP == 2 ? 6 : 5)
           : K > 6  ? 1
           : K == 6 ? (G == 64 ? 6 : 5)
                    : (G == 64 && (LEAF == 1 || LEAF == 4) ? 8 : 6);
}

template <int K, int G, int LEAF, int MODE, int IEP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(occupancy_target(K, G, LEAF, IEP)))) void count_kernel(GpPlanDesc d, CountArgs a) {
    // a group's buffer lengths, then its task cursor's index
    __shared__ int32_t s_len[kBlock / G][GP_DESC_MAX_BUILDS + 1];
    Ctx<G> c;
    c.row_ptr = a.row_ptr;
    c.col = a.col;
    c.cap = a.buf_cap;
    c.hub_bits = a.hub_bits;
    c.hub_words = a.hub_words;
    c.n_hubs = a.n_hubs;
    const int grp = threadIdx.x / G;
    const int64_t group_id = (int64_t)blockIdx.x * (kBlock / G) + grp;
    c.bufs = a.scratch ? a.scratch + group_id * (int64_t)d.nbuf * a.buf_cap : nullptr;
    c.lens = s_len[grp];
    uint64_t bytes = 0;
    c.bytes = &bytes;
    c.sj = 0;
    c.sJ = 1;
    // leaf mode 4: a table per group; IEP: one table for the launch
    c.memo = a.memo ? (IEP > 0 ? a.memo : a.memo + group_id * (int64_t)a.n_hubs) : nullptr;
    c.tag = 0;
    c.memo_log2 = a.memo_ways_log2;
    c.tab = nullptr;
    c.tab_n = 0;
    c.filt = nullptr;
    constexpr bool kFlat = K == 3 && IEP == 0 && G == 64 && LEAF != 2 && MODE != MODE_PER_ROOT;
    __shared__ __attribute__((aligned(16))) FlatRoot s_flat[kFlat ? kBlock : 1];
    __shared__ int32_t s_starts[kFlat ? kBlock * kFlatWindows : 1];
    c.flat = kFlat ? s_flat + grp * G : nullptr;
    c.starts = s_starts + (kFlat ? grp * G * kFlatWindows : 0);
    __shared__ uint32_t s_cnt[IEP > 0 ? ((1 << IEP) - 1) * kBlock : 1];
    c.cnt = &s_cnt[IEP > 0 ? threadIdx.x : 0];
    const uint64_t t_begin = a.busy ? wall_clock64() : 0;
    c.deadline = a.busy && a.budget_ticks ? t_begin + a.budget_ticks : 0;
    uint64_t chunk_max = 0;
    bool stopped = false;
    TaskSpace ts;
    ts.roots = a.roots;
    ts.offset = a.root_offset;
    ts.stride = a.root_stride;
    ts.split_roots = a.split_roots;
    ts.split_ways = a.split_ways;
    ts.tag_base = 0;

    uint64_t acc = 0, carry = 0;
    const int64_t chunk = a.chunk;

    c.lens[GP_DESC_MAX_BUILDS] = a.xcd_block > 0 ? 0 : (int)(group_id & (kCursors - 1));
    group_fence();
    for (;;) {
        int64_t t0 = 0, t1 = 0;
        if (!grab_tasks<G>(c.g, a.queue, a.n_tasks, a.n_chunks, chunk, a.xcd_block, c.lens + GP_DESC_MAX_BUILDS, &t0, &t1)) break;
        const uint64_t t_chunk = a.busy ? wall_clock64() : 0;
        run_tasks<K, G, LEAF, MODE, IEP>(d, c, ts, t0, t1, acc, carry, a.per_root);
        if (a.busy) {
            const uint64_t now = wall_clock64();
            chunk_max = max(chunk_max, now - t_chunk);
            if (c.deadline && now > c.deadline) {
                stopped = true;
                break;
            }
        }
    }

    // exact 128-bit wavefront sum, one pair of atomics per wavefront
    uint64_t s = acc, s_hi = carry;
    wave_sum128(s, s_hi);
    if constexpr (MODE == MODE_ACCOUNT) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) bytes += __shfl_xor(bytes, off, 64);
    }
    uint64_t cm = chunk_max;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) cm = max(cm, (uint64_t)__shfl_xor(cm, off, 64));
    const bool any_stop = __ballot(stopped) != 0;
    if (__lane_id() == 0) {
        unsigned long long* slot = a.queue + (blockIdx.x & (kSlots - 1)) * kSlotWords;
        publish128(&slot[SLOT_LO], &slot[SLOT_HI], s, s_hi);
        if (any_stop) atomicOr(&a.result[1], 4ull);
        if constexpr (MODE == MODE_ACCOUNT) atomicAdd(&a.result[2], (unsigned long long)bytes);
        if (a.busy) {
            atomicAdd(&a.busy[0], (unsigned long long)(wall_clock64() - t_begin));
            atomicAdd(&a.busy[1], 1ull);
            atomicMax(&a.busy[2], (unsigned long long)cm);
        }
    }
}

}  // namespace gpcount
