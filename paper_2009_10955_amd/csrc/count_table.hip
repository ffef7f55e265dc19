// Counting kernel for plans whose last level depends on the root edge and one
// more vertex only: the last level is N(x) & N(p), x the vertex bound before
// it and p a root endpoint, cut by root levels (the cycles, and what ends in
// a cycle through a root endpoint). Its size for every x is then one table
// per root edge: T[x] = |{y in N(p), lo <= y < hi : x in N(y)}|, the number
// of two-paths from p to x, filled by walking the lists of N(p).
//
// How it maps to the machine:
//   * a block of 16 or 4 wavefronts works on one root edge with the table in
//     its LDS: 16-bit counts of the 32,768 or 8,192 vertices of highest degree
//     (64 or 16 KB, so 32 wavefronts per CU). In the degree-sorted layout the
//     first 32,768 hold nearly every list entry (95% on R-MAT 17);
//   * roots come in order of their hub endpoint, the other one ascending. While
//     p, the hub, stays and the cut only grows with the other endpoint, a root
//     adds the lists of the y that come in; else (p the other endpoint, or the
//     endpoint that the last level must avoid left out) the table is filled
//     anew, which walks N(p)'s lists once where the search walks N(x)'s for
//     every x;
//   * the wavefronts take different level-2 candidates (k = 4: different
//     batches of one list) and search on as 64-lane groups (leaf mode 5).
// The search reads lists in order and looks counts up in LDS: neither the
// lists of x nor a table of 8-byte words per group in HBM are touched. What bounds
// it now is reading the lists of the level-2 candidates, from L2: 5-cycle on
// R-MAT 17 (971,517 edges) 31 ms, against 481 ms in leaf mode 4.
#include "count_kernel.hpp"

namespace gpcount {

namespace {

// Adds 1 to T[x] for every x < tab_n other than p of the lists of N(p)[b, e),
// the block's wavefronts taking different lists.
template <int MODE>
__device__ __forceinline__ void add_lists(const Ctx<64>& c, int32_t p, const Set& P, int32_t b, int32_t e, int wave,
                                          int waves, uint32_t* tab) {
    for (int32_t t0 = b + wave; t0 < e; t0 += 64 * waves) {
        // the lanes look up 64 lists' bounds at once
        const int32_t t = t0 + c.g.gl * waves;
        long long q = 0;
        int32_t n = 0;
        int32_t y = c.out;
        if (t < e) y = P.p[t];
        if (y != c.out) {
            const int64_t rb = c.row_ptr[y], re = c.row_ptr[y + 1];
            q = (long long)(c.col + rb);
            n = (int32_t)(re - rb);
            if constexpr (MODE == MODE_ACCOUNT) *c.bytes += 4;
        }
        const int lists = (int)__popcll(c.g.ballot(t < e));
        for (int j = 0; j < lists; ++j) {
            const int32_t* np = (const int32_t*)uni64<64>(c.g.bcast(q, j));
            const int32_t nn = uni<64>(c.g.bcast(n, j));
            for (int32_t base = 0; base < nn; base += 64) {
                const int32_t i = base + c.g.gl;
                const int32_t x = i < nn ? np[i] : 0x7fffffff;
                if constexpr (MODE == MODE_ACCOUNT) *c.bytes += i < nn ? 4 : 0;
                // no carry into the neighbouring count: two different vertices
                // share at most deg2 < 2^16 neighbors
                if (x < c.tab_n && x != p) atomicAdd(&tab[x >> 1], 1u << ((x & 1) * 16));
                if (uni<64>(x) >= c.tab_n) break;  // the lane holding the smallest is past the table
            }
        }
    }
}

// Root edges of p in the root array that p, their hub, orders (L), and how many of them
// in a row a whole count's block takes with one fill of the table.
__device__ __forceinline__ int32_t whole_run(const Ctx<64>& c, int32_t p, const Set& P, int32_t whole_chunk, int32_t& L) {
    L = max(1, P.n - uni<64>(lower_bound_group<64>(c.g, P.p, P.n, p)));
    return min(whole_chunk, L);
}

// Time that a sample spent and a whole count, per root edge, does not: part of dt
// clock ticks, of which the whole count has the share num / den.
__device__ __forceinline__ uint64_t beyond_share(uint64_t dt, int32_t num, int32_t den) {
    return num >= den ? 0 : dt - (uint64_t)((float)dt * (float)num / (float)den);
}

template <int K, int MODE, int kWaves>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(8))) void table_kernel(GpPlanDesc d,
                                                                                                    CountArgs a) {
    constexpr int kTabBlock = kWaves * 64;
    __shared__ __attribute__((aligned(16))) uint32_t s_tab[table_max(kWaves) / 2];
    __shared__ int32_t s_len[kWaves][GP_DESC_MAX_BUILDS];
    __shared__ int64_t s_chunk;
    __shared__ int32_t s_cur;
    __shared__ uint64_t s_beyond[MODE == MODE_SAMPLE ? kWaves : 1];  // per wavefront: clock ticks that only a sample spends
    Ctx<64> c;
    const int wave = uni<64>((int)(threadIdx.x / 64));
    c.row_ptr = a.row_ptr;
    c.col = a.col;
    c.cap = a.buf_cap;
    c.hub_bits = a.hub_bits;
    c.hub_words = a.hub_words;
    c.n_hubs = a.n_hubs;
    c.bufs = a.scratch ? a.scratch + ((int64_t)blockIdx.x * kWaves + wave) * (int64_t)d.nbuf * a.buf_cap : nullptr;
    c.lens = s_len[wave];
    uint64_t bytes = 0;
    c.bytes = &bytes;
    c.sj = wave;
    c.sJ = kWaves;
    c.memo = nullptr;
    c.tag = 0;
    c.memo_log2 = 0;
    c.cnt = nullptr;
    c.tab = (const uint16_t*)s_tab;
    c.tab_n = a.tab_n;
    c.filt = nullptr;
    // with a.busy
    constexpr bool kTimed = MODE == MODE_SAMPLE;
    const uint64_t t_begin = kTimed ? wall_clock64() : 0;
    c.deadline = kTimed && a.budget_ticks ? t_begin + a.budget_ticks : 0;
    uint64_t chunk_max = 0;
    bool stopped = false;
    uint64_t acc = 0, carry = 0;

    const GpLevel& ll = d.lv[K - 1];
    // whether the roots of a hub p share a fill: p orders the array, and the other
    // endpoint only raises the cut
    const int hub = d.root_cut == 1 ? 1 : (d.root_cut == 2 ? 0 : -1), rest = 1 - ll.pre_list;
    const bool shared = hub == ll.pre_list && !(((ll.inj | ll.lo_src) >> rest) & 1u);
    if (kTimed && c.g.gl == 0) s_beyond[wave] = 0;
    int32_t cur_p = -1, cur_lo = 0, cur_hi = 0, cur_pos = 0;
    c.out = -1;
    if (threadIdx.x == 0) s_cur = (int)(blockIdx.x & (kCursors - 1));
    __syncthreads();
    for (;;) {
        if (wave == 0) {
            const int64_t q = next_chunk<64>(c.g, a.queue, a.n_chunks, &s_cur);
            if (c.g.gl == 0) s_chunk = q;
        }
        __syncthreads();
        const int64_t q = uni64<64>(s_chunk);
        __syncthreads();
        if (q < 0) break;
        const uint64_t t_chunk = kTimed ? wall_clock64() : 0;
        const int64_t r1 = min((q + 1) * a.chunk, a.n_roots);
        for (int64_t r = q * a.chunk; r < r1; ++r) {
            const int2 e = a.roots[a.root_offset + r * a.root_stride];
            if constexpr (MODE == MODE_ACCOUNT) bytes += threadIdx.x == 0 ? 8 : 0;
            int32_t v[K];
#pragma unroll
            for (int j = 0; j < K; ++j) v[j] = 0;
            v[0] = uni<64>(e.x);
            v[1] = uni<64>(e.y);
            const int32_t p = ll.pre_list == 0 ? v[0] : v[1];
            int32_t lo, hi;
            bounds<K>(ll.hi_src, ll.lo_src, v, lo, hi);
            const Set P = c.nbr_u(p);
            const int q = 1 - ll.pre_list;
            const int32_t out = (ll.inj >> q) & 1u ? v[q] : -1;
            const uint64_t t_fill = kTimed ? wall_clock64() : 0;
            const bool anew = p != cur_p || lo != cur_lo || hi < cur_hi || out != c.out;
            // every wavefront of the block takes the same way here
            if (anew) {
                for (int i = threadIdx.x; i < (a.tab_n + 7) / 8; i += kTabBlock)
                    reinterpret_cast<uint4*>(s_tab)[i] = make_uint4(0, 0, 0, 0);
                cur_pos = lo > 0 ? uni<64>(lower_bound_group<64>(c.g, P.p, P.n, lo)) : 0;
                __syncthreads();
            }
            const int32_t end = hi < 0x7fffffff
                                    ? cur_pos + uni<64>(lower_bound_group<64>(c.g, P.p + cur_pos, P.n - cur_pos, hi))
                                    : P.n;
            c.out = out;
            if (end > cur_pos) add_lists<MODE>(c, p, P, cur_pos, end, wave, kWaves, s_tab);
            cur_pos = max(cur_pos, end);
            cur_p = p;
            cur_lo = lo;
            cur_hi = hi;
            __syncthreads();
            if (kTimed && shared && a.root_stride > 1) {
                // a sampled root starts a table, or adds the lists of the roots left out;
                // a whole count does either once for a run of them
                const uint64_t dt = wall_clock64() - t_fill;
                const int32_t s = (int32_t)a.root_stride;
                int32_t L = 1;
                const int32_t run = whole_run(c, p, P, a.whole_chunk, L);
                if (c.g.gl == 0)
                    s_beyond[wave] +=
                        anew ? beyond_share(dt, min(a.chunk, max(1, L / s)), run) : beyond_share(dt, 1, s);
            }
            search<K, 2, 64, 5, MODE, 0>(d, c, v, acc, carry);
            __syncthreads();
        }
        if constexpr (kTimed) {
            const uint64_t now = wall_clock64();
            chunk_max = max(chunk_max, now - t_chunk);
            // the whole block stops together
            const bool late = c.deadline && now > c.deadline;
            if (__syncthreads_or(late)) {
                stopped = true;
                break;
            }
        }
    }
    uint64_t s = acc, s_hi = carry;
    wave_sum128(s, s_hi);
    if constexpr (MODE == MODE_ACCOUNT) bytes = c.g.sum(bytes);
    if (__lane_id() == 0) {
        if constexpr (MODE == MODE_ACCOUNT) atomicAdd(&a.result[2], (unsigned long long)bytes);
        unsigned long long* slot = a.queue + (blockIdx.x & (kSlots - 1)) * kSlotWords;
        publish128(&slot[SLOT_LO], &slot[SLOT_HI], s, s_hi);
        if (stopped) atomicOr(&a.result[1], 4ull);
        if constexpr (kTimed) {
            atomicAdd(&a.busy[0], (unsigned long long)(wall_clock64() - t_begin - s_beyond[wave]));
            atomicAdd(&a.busy[1], 1ull);
            atomicMax(&a.busy[2], (unsigned long long)chunk_max);
        }
    }
}

// The table with inclusion-exclusion: plans with two inner levels whose set of
// the last outer vertex x is N(p) & N(x), uncut, p the endpoint that the
// root array is ordered by. The table then holds for all roots of p: a block
// fills it once for a run of roots of one p (and hashes N(p) into the filter),
// and its wavefronts take the run's roots one by one, each searching on its
// own. What it replaces: a walk of N(p) or N(x) per (p, x), random words of
// hub bitmaps, which bounded the house count by memory lines (a 60th of
// R-MAT 22: 3.9 TB of lines fetched in 507 ms; now 1.06 TB in 223 ms, most of
// them for the pairs of term 3 that the memo does not hold yet. R-MAT 17 whole:
// 15.5 ms, 10.3 with the table).
constexpr int kIepWaves = kIepTableWaves;

template <int K, int MODE>
__global__ __launch_bounds__(kIepWaves * 64) __attribute__((amdgpu_waves_per_eu(6))) void table_iep_kernel(GpPlanDesc d,
                                                                                                           CountArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t s_tab[table_max(kIepWaves) / 2];
    __shared__ __attribute__((aligned(16))) uint32_t s_filt[kFiltWords];
    __shared__ int32_t s_len[kIepWaves][GP_DESC_MAX_BUILDS];
    __shared__ int64_t s_chunk;
    __shared__ int32_t s_cur, s_next;
    __shared__ uint64_t s_beyond[MODE == MODE_SAMPLE ? kIepWaves : 1];  // as above
    Ctx<64> c;
    const int wave = uni<64>((int)(threadIdx.x / 64));
    c.row_ptr = a.row_ptr;
    c.col = a.col;
    c.cap = a.buf_cap;
    c.hub_bits = a.hub_bits;
    c.hub_words = a.hub_words;
    c.n_hubs = a.n_hubs;
    c.bufs = a.scratch ? a.scratch + ((int64_t)blockIdx.x * kIepWaves + wave) * (int64_t)d.nbuf * a.buf_cap : nullptr;
    c.lens = s_len[wave];
    uint64_t bytes = 0;
    c.bytes = &bytes;
    c.sj = 0;
    c.sJ = 1;
    c.memo = a.memo;
    c.tag = 0;
    c.memo_log2 = a.memo_ways_log2;
    c.cnt = nullptr;
    c.tab = (const uint16_t*)s_tab;
    c.tab_n = a.tab_n;
    c.out = -1;
    c.filt = s_filt;
    // with a.busy
    constexpr bool kTimed = MODE == MODE_SAMPLE;
    const uint64_t t_begin = kTimed ? wall_clock64() : 0;
    c.deadline = kTimed && a.budget_ticks ? t_begin + a.budget_ticks : 0;
    uint64_t chunk_max = 0;
    bool stopped = false;
    uint64_t acc = 0, carry = 0;
    const bool second = d.it[d.iep_sum - 1].op[0] == 1;
    if (kTimed && c.g.gl == 0) s_beyond[wave] = 0;
    int32_t cur_p = -1;
    if (threadIdx.x == 0) s_cur = (int)(blockIdx.x & (kCursors - 1));
    __syncthreads();
    for (;;) {
        if (wave == 0) {
            const int64_t q = next_chunk<64>(c.g, a.queue, a.n_chunks, &s_cur);
            if (c.g.gl == 0) s_chunk = q;
        }
        __syncthreads();
        const int64_t q = uni64<64>(s_chunk);
        if (q < 0) break;
        const uint64_t t_chunk = kTimed ? wall_clock64() : 0;
        const int64_t r1 = min((q + 1) * a.chunk, a.n_roots);
        for (int64_t r = q * a.chunk; r < r1;) {
            // the chunk's next run of roots of one p (a chunk has at most 64)
            const int lanes = (int)(r1 - r);
            int32_t own = -1;
            if (c.g.gl < lanes) {
                const int2 e = a.roots[a.root_offset + (r + c.g.gl) * a.root_stride];
                own = second ? e.y : e.x;
            }
            const int32_t p = uni<64>(own);
            const uint64_t other = c.g.ballot(own != p);
            const int run = other ? __builtin_ctzll(other) : 64;
            __syncthreads();  // the last run's readers are done
            if (threadIdx.x == 0) s_next = 0;
            const uint64_t t_fill = kTimed ? wall_clock64() : 0;
            int32_t of_run = run;  // roots that a whole count takes with one fill
            if (kTimed && a.root_stride > 1) {
                int32_t L = 1;
                of_run = whole_run(c, p, c.nbr_u(p), a.whole_chunk, L);
            }
            const bool anew = p != cur_p;
            if (anew) {
                const Set P = c.nbr_u(p);
                for (int i = threadIdx.x; i < (a.tab_n + 7) / 8; i += kIepWaves * 64)
                    reinterpret_cast<uint4*>(s_tab)[i] = make_uint4(0, 0, 0, 0);
                reinterpret_cast<uint4*>(s_filt)[threadIdx.x] = make_uint4(0, 0, 0, 0);
                static_assert(kFiltWords == kIepWaves * 64 * 4, "one store per thread clears the filter");
                __syncthreads();
                for (int32_t i = threadIdx.x; i < P.n; i += kIepWaves * 64) {
                    const uint32_t b = (uint32_t)P.p[i] & (32u * kFiltWords - 1);
                    atomicOr(&s_filt[b >> 5], 1u << (b & 31));
                }
                add_lists<MODE>(c, p, P, 0, P.n, wave, kIepWaves, s_tab);
                cur_p = p;
            }
            __syncthreads();
            if (kTimed && anew && c.g.gl == 0) s_beyond[wave] += beyond_share(wall_clock64() - t_fill, run, of_run);
            for (;;) {
                int t = 0;
                if (c.g.gl == 0) t = atomicAdd(&s_next, 1);
                t = uni<64>(t);
                if (t >= run) break;
                const int2 e = a.roots[a.root_offset + (r + t) * a.root_stride];
                if constexpr (MODE == MODE_ACCOUNT) bytes += c.g.gl == 0 ? 8 : 0;
                int32_t v[K];
#pragma unroll
                for (int j = 0; j < K; ++j) v[j] = 0;
                v[0] = uni<64>(e.x);
                v[1] = uni<64>(e.y);
                if (run_builds<K, 64, MODE>(d, c, 1, v)) search<K, 2, 64, 5, MODE, 2>(d, c, v, acc, carry);
            }
            if constexpr (kTimed) {
                // a run of one sampled root leaves the other wavefronts waiting
                const uint64_t t_wait = wall_clock64();
                __syncthreads();
                if (c.g.gl == 0) s_beyond[wave] += beyond_share(wall_clock64() - t_wait, run, of_run);
            }
            r += run;
        }
        if constexpr (kTimed) {
            const uint64_t now = wall_clock64();
            chunk_max = max(chunk_max, now - t_chunk);
            if (__syncthreads_or(c.deadline && now > c.deadline)) {
                stopped = true;
                break;
            }
        } else {
            __syncthreads();  // s_chunk has been read
        }
    }
    uint64_t s = acc, s_hi = carry;
    wave_sum128(s, s_hi);
    if constexpr (MODE == MODE_ACCOUNT) bytes = c.g.sum(bytes);
    if (__lane_id() == 0) {
        if constexpr (MODE == MODE_ACCOUNT) atomicAdd(&a.result[2], (unsigned long long)bytes);
        unsigned long long* slot = a.queue + (blockIdx.x & (kSlots - 1)) * kSlotWords;
        publish128(&slot[SLOT_LO], &slot[SLOT_HI], s, s_hi);
        if (stopped) atomicOr(&a.result[1], 4ull);
        if constexpr (kTimed) {
            atomicAdd(&a.busy[0], (unsigned long long)(wall_clock64() - t_begin - s_beyond[wave]));
            atomicAdd(&a.busy[1], 1ull);
            atomicMax(&a.busy[2], (unsigned long long)chunk_max);
        }
    }
}

}  // namespace

// The kernel for IEP plans: k from 5 on (two inner levels below one more outer
// level than the root edge).
KernelFn pick_table_iep_kernel(int k, int mode) {
#define GP_TABLE_CASE(KK)                                                 \
    case KK:                                                              \
        if (mode == MODE_PLAIN) return table_iep_kernel<KK, MODE_PLAIN>;  \
        if (mode == MODE_SAMPLE) return table_iep_kernel<KK, MODE_SAMPLE>; \
        return mode == MODE_ACCOUNT ? table_iep_kernel<KK, MODE_ACCOUNT> : nullptr;
    switch (k) {
        GP_TABLE_CASE(5)
        GP_TABLE_CASE(6)
        GP_TABLE_CASE(7)
        GP_TABLE_CASE(8)
        default: return nullptr;
    }
#undef GP_TABLE_CASE
}

template <int K, int W>
static KernelFn table_kernel_of(int mode) {
    if (mode == MODE_PLAIN) return table_kernel<K, MODE_PLAIN, W>;
    if (mode == MODE_SAMPLE) return table_kernel<K, MODE_SAMPLE, W>;
    return mode == MODE_ACCOUNT ? table_kernel<K, MODE_ACCOUNT, W> : nullptr;
}

KernelFn pick_table_kernel(int k, int mode, int waves) {
    if (waves != 4 && waves != 16) return nullptr;
#define GP_TABLE_CASE(KK) \
    case KK: return waves == 4 ? table_kernel_of<KK, 4>(mode) : table_kernel_of<KK, 16>(mode);
    switch (k) {
        GP_TABLE_CASE(4)
        GP_TABLE_CASE(5)
        GP_TABLE_CASE(6)
        GP_TABLE_CASE(7)
        GP_TABLE_CASE(8)
        default: return nullptr;
    }
#undef GP_TABLE_CASE
}

}  // namespace gpcount
