// Graph layout in HBM (device side of gp_load_graph).
//
// Input: an undirected simple graph as CSR with sorted, contiguous neighbor
// lists (Section IV-E). Steps, all on the device:
//   1. validate: rows non-decreasing, columns in range, each list strictly
//      ascending (no duplicates), no self-loops, every (u,v) has (v,u);
//   2. relabel by descending degree, ties by ascending id (radix sort of
//      (degree, id) keys), rebuild the CSR by a radix sort of relabelled
//      (src, dst) keys, so every list is again ascending;
//   3. root-edge arrays: all entries, entries with v1 < v0, entries with
//      v1 > v0, each in CSR order (hubs first);
//   4. content hash of the input (order-independent sum of mixed entries).
// The triangle count for the cost model is taken afterwards by the counting
// kernel itself (see the API layer).
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <vector>

#include "internal.hpp"
#include "sets.hpp"

using namespace gpdev;

namespace {

enum : unsigned {
    F_RANGE = 1,
    F_UNSORTED = 2,
    F_SELFLOOP = 4,
    F_DUP = 8,
    F_ASYM = 16,
};

__device__ __forceinline__ int64_t row_of(const int64_t* row_ptr, int64_t n, int64_t e) {
    // last v with row_ptr[v] <= e
    int64_t lo = 0, hi = n;  // answer in [0, n)
    while (hi - lo > 1) {
        int64_t mid = (lo + hi) >> 1;
        if (row_ptr[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
}

__global__ void check_rows(const int64_t* row_ptr, int64_t n, int64_t nnz, unsigned* flags) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        int64_t b = row_ptr[v], e = row_ptr[v + 1];
        if (b > e || b < 0 || e > nnz || e - b > 0x7fffffff) atomicOr(flags, (unsigned)F_UNSORTED);
    }
}

__global__ void check_entries(const int64_t* row_ptr, const int32_t* col, int64_t n, int64_t nnz,
                              unsigned* flags) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x) {
        int64_t v = row_of(row_ptr, n, e);
        int32_t w = col[e];
        unsigned f = 0;
        if (w < 0 || w >= n) {
            f |= F_RANGE;
        } else {
            if (w == v) f |= F_SELFLOOP;
            if (e + 1 < row_ptr[v + 1]) {
                int32_t nx = col[e + 1];
                if (nx == w) f |= F_DUP;
                else if (nx < w) f |= F_UNSORTED;
            }
            int64_t b = row_ptr[w];
            int64_t len = row_ptr[w + 1] - b;
            if (len < 0 || b < 0 || b + len > nnz) {
                f |= F_UNSORTED;
            } else if (!contains(col + b, (int32_t)len, (int32_t)v)) {
                f |= F_ASYM;
            }
        }
        if (f) atomicOr(flags, f);
    }
}

__device__ __forceinline__ uint64_t mix64(uint64_t x) {
    // splitmix64 finaliser
    x += 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

__global__ void hash_input(const int64_t* row_ptr, const int32_t* col, int64_t n, int64_t nnz,
                           unsigned long long* out) {
    uint64_t h = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nnz + n + 1;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i < nnz) h += mix64(((uint64_t)i << 32) ^ (uint32_t)col[i]);
        else h += mix64(0xabcdef0000000000ull ^ ((uint64_t)(i - nnz) << 40) ^ (uint64_t)row_ptr[i - nnz]);
    }
    // one atomic per block of a grid that fills the device once: atomics on one
    // address take 12 ns each (a wavefront's each: 3.1 of a load's 11 ms at 16M entries)
    __shared__ uint64_t s_h[4];
    for (int off = 32; off >= 1; off >>= 1) h += __shfl_xor(h, off, 64);
    if (__lane_id() == 0) s_h[threadIdx.x / 64] = h;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(out, (unsigned long long)(s_h[0] + s_h[1] + s_h[2] + s_h[3]));
}

__global__ void degree_keys(const int64_t* row_ptr, int64_t n, uint64_t* keys) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        uint64_t deg = (uint64_t)(row_ptr[v + 1] - row_ptr[v]);
        keys[v] = ((uint64_t)(0xffffffffu - (uint32_t)deg) << 32) | (uint64_t)v;
    }
}

__global__ void assign_ids(const uint64_t* sorted, const int64_t* row_ptr, int64_t n,
                           int32_t* new_id, int64_t* new_deg) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        int64_t old = (int64_t)(sorted[p] & 0xffffffffu);
        new_id[old] = (int32_t)p;
        new_deg[p] = row_ptr[old + 1] - row_ptr[old];
    }
}

__global__ void edge_keys(const int64_t* row_ptr, const int32_t* col, const int32_t* new_id,
                          int64_t n, int64_t nnz, int shift, uint64_t* keys) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x) {
        int64_t v = row_of(row_ptr, n, e);
        keys[e] = ((uint64_t)(uint32_t)new_id[v] << shift) | (uint64_t)(uint32_t)new_id[col[e]];
    }
}

__global__ void unpack_edges(const uint64_t* keys, int64_t nnz, int shift, int32_t* col,
                             int2* roots_all) {
    const uint64_t mask = (uint64_t(1) << shift) - 1;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x) {
        uint64_t k = keys[e];
        int32_t w = (int32_t)(k & mask);
        int32_t v = (int32_t)(k >> shift);
        col[e] = w;
        roots_all[e] = make_int2(v, w);
    }
}

// Number of neighbors below v (the lower part of each sorted list).
__global__ void count_lower(const int64_t* row_ptr, const int32_t* col, int64_t n, int64_t* lower,
                            int64_t* upper) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        int64_t b = row_ptr[v];
        int32_t len = (int32_t)(row_ptr[v + 1] - b);
        int32_t lo = lower_bound(col + b, len, (int32_t)v);
        lower[v] = lo;
        upper[v] = len - lo;
    }
}

// out[0..2] += the sums over the vertices of degree^2, lower * degree and lower^2,
// lower: a vertex's neighbors of smaller id.
__global__ void degree_sums(const int64_t* row_ptr, const int64_t* lower, int64_t n, unsigned long long* out) {
    uint64_t s[3] = {0, 0, 0};
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t d = (uint64_t)(row_ptr[v + 1] - row_ptr[v]), l = (uint64_t)lower[v];
        s[0] += d * d;
        s[1] += l * d;
        s[2] += l * l;
    }
    __shared__ uint64_t s_sum[4];
    for (int i = 0; i < 3; ++i) {
        for (int off = 32; off >= 1; off >>= 1) s[i] += __shfl_xor(s[i], off, 64);
        __syncthreads();
        if (__lane_id() == 0) s_sum[threadIdx.x / 64] = s[i];
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(&out[i], (unsigned long long)(s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]));
    }
}

// The numbers the host keeps of a layout, gathered for one copy (a copy each was
// 37 round trips).
struct LayoutWords {
    unsigned long long sums[3];  // degree_sums
    unsigned long long hash;
    int64_t n_lower, n_upper, deg[2];
    int64_t first_entries[3];
    int64_t upper_pref[32];
};

// w->sums and w->hash are there already; one block.
__global__ void layout_words(const int64_t* row_ptr, const int64_t* lower_off, const int64_t* upper_off, int64_t n,
                             int64_t t0, int64_t t1, int64_t t2, LayoutWords* w) {
    const int i = threadIdx.x;
    if (i < 32) w->upper_pref[i] = upper_off[min(int64_t(1) << i, n)];
    if (i < 2) w->deg[i] = i < n ? row_ptr[i + 1] - row_ptr[i] : 0;
    if (i < 3) w->first_entries[i] = row_ptr[min(i == 0 ? t0 : (i == 1 ? t1 : t2), n)];
    if (i == 0) {
        w->n_lower = lower_off[n];
        w->n_upper = upper_off[n];
    }
}

__global__ void scatter_roots(const int64_t* row_ptr, const int2* roots_all, int64_t n, int64_t nnz,
                              const int64_t* lower_cnt, const int64_t* lower_off,
                              const int64_t* upper_off, int2* roots_lower, int2* roots_upper) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x) {
        int2 r = roots_all[e];
        int64_t v = r.x;
        int64_t k = e - row_ptr[v];
        if (k < lower_cnt[v]) roots_lower[lower_off[v] + k] = r;
        else roots_upper[upper_off[v] + (k - lower_cnt[v])] = r;
    }
}

// Root arrays ordered by their smaller endpoint, which in the degree-sorted
// layout is the higher-degree one: the heaviest roots come first (they start
// first, and the kernel can split a prefix of them). roots_upper stays in CSR
// order (v0 < v1, v0 ascending); roots_lower holds the same edges reversed in
// the same order; roots_all interleaves the two.
__global__ void order_roots(const int2* roots_upper, int64_t n_upper, int2* roots_lower, int2* roots_all) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_upper;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int2 u = roots_upper[k];
        const int2 r = make_int2(u.y, u.x);
        roots_lower[k] = r;
        roots_all[2 * k] = u;
        roots_all[2 * k + 1] = r;
    }
}

__global__ void fill_hub_bits(const int64_t* row_ptr, const int32_t* col, int64_t n_hubs,
                              int64_t n_entries, int64_t words, uint32_t* bits) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n_entries;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = row_of(row_ptr, n_hubs, e);
        const int32_t w = col[e];
        atomicOr(&bits[v * words + (w >> 5)], 1u << (w & 31));
    }
}

// Of the degree-descending layout: out[0] = vertices of degree >= min_degree
// among the first cap, out[1] = vertices of degree > 0, out[2] = CSR entries of
// the first out[0] vertices.
__global__ void degree_bounds(const int64_t* row_ptr, int64_t n, int64_t cap, int64_t min_degree, int64_t* out) {
    const int64_t at_least[2] = {min_degree, 1};
    const int64_t end[2] = {cap, n};
    if (threadIdx.x < 2) {
        int64_t lo = 0, hi = end[threadIdx.x];  // first vertex of a smaller degree
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (row_ptr[mid + 1] - row_ptr[mid] >= at_least[threadIdx.x]) lo = mid + 1;
            else hi = mid;
        }
        out[threadIdx.x] = lo;
        if (threadIdx.x == 0) out[2] = row_ptr[lo];
    }
}

unsigned grid_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > 65536) b = 65536;
    return (unsigned)b;
}

struct TempPool {
    hipStream_t s;
    void* ptrs[32];
    int n = 0;
    explicit TempPool(hipStream_t st) : s(st) {}
    hipError_t get(void** p, size_t bytes) {
        hipError_t e = gpint::stream_malloc(p, bytes ? bytes : 8, s);
        if (e == hipSuccess && n < 32) ptrs[n++] = *p;
        return e;
    }
    ~TempPool() {
        for (int i = 0; i < n; ++i) (void)hipFreeAsync(ptrs[i], s);
    }
};

}  // namespace

namespace gpint {

// Fills g (device buffers owned by g). row_ptr/col are device pointers.
gp_status build_layout(const int64_t* row_ptr, const int32_t* col, int64_t n, int64_t nnz,
                       hipStream_t s, DeviceGraph* g) {
    TempPool tmp(s);
    unsigned* flags = nullptr;
    LayoutWords* words = nullptr;
    GP_HIP_TRY(tmp.get((void**)&flags, sizeof(unsigned)));
    GP_HIP_TRY(tmp.get((void**)&words, sizeof(LayoutWords)));
    GP_HIP_TRY(hipMemsetAsync(flags, 0, sizeof(unsigned), s));
    GP_HIP_TRY(hipMemsetAsync(words, 0, sizeof(LayoutWords), s));
    if (n > 0) hipLaunchKernelGGL(check_rows, dim3(grid_for(n)), dim3(256), 0, s, row_ptr, n, nnz, flags);
    unsigned hflags = 0;
    GP_HIP_TRY(hipMemcpyAsync(&hflags, flags, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    GP_HIP_TRY(hipStreamSynchronize(s));
    if (hflags) return GP_ERR_CSR_UNSORTED;
    if (nnz > 0) {
        hipLaunchKernelGGL(check_entries, dim3(grid_for(nnz)), dim3(256), 0, s, row_ptr, col, n, nnz,
                           flags);
        GP_HIP_TRY(hipGetLastError());
        GP_HIP_TRY(hipMemcpyAsync(&hflags, flags, sizeof(unsigned), hipMemcpyDeviceToHost, s));
        GP_HIP_TRY(hipStreamSynchronize(s));
        if (hflags & F_RANGE) return GP_ERR_CSR_RANGE;
        if (hflags & F_UNSORTED) return GP_ERR_CSR_UNSORTED;
        if (hflags & F_SELFLOOP) return GP_ERR_CSR_SELFLOOP;
        if (hflags & F_DUP) return GP_ERR_CSR_DUPLICATE;
        if (hflags & F_ASYM) return GP_ERR_CSR_ASYMMETRIC;
    }
    hipLaunchKernelGGL(hash_input, dim3(std::min(2048u, grid_for(nnz + n + 1))), dim3(256), 0, s, row_ptr, col, n, nnz,
                       &words->hash);

    // device buffers owned by the graph
    const int64_t nn = n > 0 ? n : 1;
    const int64_t ne = nnz > 0 ? nnz : 1;
    GP_HIP_TRY(device_malloc((void**)&g->row_ptr, sizeof(int64_t) * (n + 1)));
    GP_HIP_TRY(device_malloc((void**)&g->col, sizeof(int32_t) * ne));
    GP_HIP_TRY(device_malloc((void**)&g->roots_all, sizeof(int2) * ne));
    GP_HIP_TRY(device_malloc((void**)&g->new_id, sizeof(int32_t) * nn));

    // 2. relabel by descending degree, ties by ascending id
    uint64_t *vkeys = nullptr, *vkeys_sorted = nullptr;
    int64_t* new_deg = nullptr;
    GP_HIP_TRY(tmp.get((void**)&vkeys, sizeof(uint64_t) * nn));
    GP_HIP_TRY(tmp.get((void**)&vkeys_sorted, sizeof(uint64_t) * nn));
    GP_HIP_TRY(tmp.get((void**)&new_deg, sizeof(int64_t) * (n + 1)));
    if (n > 0) hipLaunchKernelGGL(degree_keys, dim3(grid_for(n)), dim3(256), 0, s, row_ptr, n, vkeys);
    size_t tb = 0;
    GP_HIP_TRY(hipcub::DeviceRadixSort::SortKeys(nullptr, tb, vkeys, vkeys_sorted, (int)n, 0, 64, s));
    void* tstore = nullptr;
    GP_HIP_TRY(tmp.get(&tstore, tb));
    GP_HIP_TRY(hipcub::DeviceRadixSort::SortKeys(tstore, tb, vkeys, vkeys_sorted, (int)n, 0, 64, s));
    if (n > 0)
        hipLaunchKernelGGL(assign_ids, dim3(grid_for(n)), dim3(256), 0, s, vkeys_sorted, row_ptr, n,
                           g->new_id, new_deg);
    GP_HIP_TRY(hipMemsetAsync(new_deg + n, 0, sizeof(int64_t), s));
    // row_ptr of the layout = exclusive scan of new degrees (n+1 entries)
    tb = 0;
    GP_HIP_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, tb, new_deg, g->row_ptr, (int)(n + 1), s));
    void* tscan = nullptr;
    GP_HIP_TRY(tmp.get(&tscan, tb));
    GP_HIP_TRY(hipcub::DeviceScan::ExclusiveSum(tscan, tb, new_deg, g->row_ptr, (int)(n + 1), s));

    int bits = 1;
    while ((int64_t(1) << bits) < nn) ++bits;
    const int shift = bits;
    uint64_t *ekeys = nullptr, *ekeys_sorted = nullptr;
    GP_HIP_TRY(tmp.get((void**)&ekeys, sizeof(uint64_t) * ne));
    GP_HIP_TRY(tmp.get((void**)&ekeys_sorted, sizeof(uint64_t) * ne));
    if (nnz > 0)
        hipLaunchKernelGGL(edge_keys, dim3(grid_for(nnz)), dim3(256), 0, s, row_ptr, col, g->new_id, n,
                           nnz, shift, ekeys);
    tb = 0;
    GP_HIP_TRY(hipcub::DeviceRadixSort::SortKeys(nullptr, tb, ekeys, ekeys_sorted, (int)nnz, 0,
                                                 2 * bits, s));
    void* tsort = nullptr;
    GP_HIP_TRY(tmp.get(&tsort, tb));
    GP_HIP_TRY(hipcub::DeviceRadixSort::SortKeys(tsort, tb, ekeys, ekeys_sorted, (int)nnz, 0,
                                                 2 * bits, s));
    if (nnz > 0)
        hipLaunchKernelGGL(unpack_edges, dim3(grid_for(nnz)), dim3(256), 0, s, ekeys_sorted, nnz, shift,
                           g->col, g->roots_all);

    // 3. oriented root arrays
    int64_t *lower_cnt = nullptr, *upper_cnt = nullptr, *lower_off = nullptr, *upper_off = nullptr;
    GP_HIP_TRY(tmp.get((void**)&lower_cnt, sizeof(int64_t) * (n + 1)));
    GP_HIP_TRY(tmp.get((void**)&upper_cnt, sizeof(int64_t) * (n + 1)));
    GP_HIP_TRY(tmp.get((void**)&lower_off, sizeof(int64_t) * (n + 1)));
    GP_HIP_TRY(tmp.get((void**)&upper_off, sizeof(int64_t) * (n + 1)));
    GP_HIP_TRY(hipMemsetAsync(lower_cnt + n, 0, sizeof(int64_t), s));
    GP_HIP_TRY(hipMemsetAsync(upper_cnt + n, 0, sizeof(int64_t), s));
    if (n > 0)
        hipLaunchKernelGGL(count_lower, dim3(grid_for(n)), dim3(256), 0, s, g->row_ptr, g->col, n,
                           lower_cnt, upper_cnt);
    tb = 0;
    GP_HIP_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, tb, lower_cnt, lower_off, (int)(n + 1), s));
    void* tscan2 = nullptr;
    GP_HIP_TRY(tmp.get(&tscan2, tb));
    GP_HIP_TRY(hipcub::DeviceScan::ExclusiveSum(tscan2, tb, lower_cnt, lower_off, (int)(n + 1), s));
    GP_HIP_TRY(hipcub::DeviceScan::ExclusiveSum(tscan2, tb, upper_cnt, upper_off, (int)(n + 1), s));
    if (n > 0)
        hipLaunchKernelGGL(degree_sums, dim3(std::min(1024u, grid_for(n))), dim3(256), 0, s, g->row_ptr, lower_cnt, n,
                           words->sums);
    hipLaunchKernelGGL(layout_words, dim3(1), dim3(64), 0, s, g->row_ptr, lower_off, upper_off, n,
                       (int64_t)kTableSizes[0], (int64_t)kTableSizes[1], (int64_t)kTableSizes[2], words);
    LayoutWords lw;
    GP_HIP_TRY(hipMemcpyAsync(&lw, words, sizeof lw, hipMemcpyDeviceToHost, s));
    GP_HIP_TRY(hipStreamSynchronize(s));
    const int64_t hv[2] = {lw.n_lower, lw.n_upper};
    g->n_lower = hv[0];
    g->n_upper = hv[1];
    GP_HIP_TRY(device_malloc((void**)&g->roots_lower, sizeof(int2) * (hv[0] > 0 ? hv[0] : 1)));
    GP_HIP_TRY(device_malloc((void**)&g->roots_upper, sizeof(int2) * (hv[1] > 0 ? hv[1] : 1)));
    if (nnz > 0)
        hipLaunchKernelGGL(scatter_roots, dim3(grid_for(nnz)), dim3(256), 0, s, g->row_ptr, g->roots_all,
                           n, nnz, lower_cnt, lower_off, upper_off, g->roots_lower, g->roots_upper);
    GP_HIP_TRY(hipGetLastError());
    if (hv[0] != hv[1] || hv[0] + hv[1] != nnz) return GP_ERR_INTERNAL;  // validated symmetric, loop-free
    if (hv[1] > 0)
        hipLaunchKernelGGL(order_roots, dim3(grid_for(hv[1])), dim3(256), 0, s, g->roots_upper, hv[1],
                           g->roots_lower, g->roots_all);
    GP_HIP_TRY(hipGetLastError());
    GP_HIP_TRY(hipStreamSynchronize(s));
    for (int i = 0; i < 32; ++i) g->upper_pref[i] = lw.upper_pref[i];
    for (int i = 0; i < 3; ++i) g->first_entries[i] = lw.first_entries[i];
    g->n = n;
    g->nnz = nnz;
    g->max_deg = lw.deg[0];
    g->deg2 = lw.deg[1];
    if (nnz > 0) {
        // a vertex is the other endpoint of as many root edges as it has
        // neighbors of smaller id, and the hub of the rest
        const double m = (double)nnz / 2, dd = (double)lw.sums[0], ld = (double)lw.sums[1], ll = (double)lw.sums[2];
        g->mean_deg = dd / (double)nnz;
        g->other_deg = ld / m;
        g->hub_deg = (dd - ld) / m;
        g->other_below = (ll - m) / 2 / m;
        g->hub_below = (ld - ll) / m;
    }
    g->stats.n = n;
    g->stats.m = nnz / 2;
    g->stats.max_degree = lw.deg[0];
    g->stats.hash = lw.hash;
    return GP_OK;
}

// Dense neighbor bitmaps for the highest-degree vertices. In the
// degree-descending layout they are ids [0, n_hubs), whose lists are the first
// row_ptr[n_hubs] CSR entries. A vertex qualifies with degree >= min_degree;
// the count is capped so that all bitmaps fit in budget_bytes.
// The budget counts n bits per vertex, but a bitmap ends at the last vertex with
// a neighbor: isolated vertices are in no list. On R-MAT 20 that is half the
// memory, and a freed graph's memory costs its size: the driver clears it at
// 24 GB/s, 190 of a load and free's 206 ms before.
gp_status build_hub_bitmaps(DeviceGraph* g, int64_t min_degree, int64_t budget_bytes, hipStream_t s) {
    g->n_hubs = 0;
    g->hub_words = (g->n + 31) / 32;
    if (g->n == 0 || g->nnz == 0) return GP_OK;
    const int64_t cap = std::min<int64_t>(g->n, budget_bytes / (g->hub_words * 4));
    if (cap <= 0) return GP_OK;
    int64_t found[3] = {0, 0, 0};
    {
        TempPool tmp(s);
        int64_t* bounds = nullptr;
        GP_HIP_TRY(tmp.get((void**)&bounds, sizeof found));
        hipLaunchKernelGGL(degree_bounds, dim3(1), dim3(64), 0, s, g->row_ptr, g->n, cap, min_degree, bounds);
        GP_HIP_TRY(hipMemcpyAsync(found, bounds, sizeof found, hipMemcpyDeviceToHost, s));
        GP_HIP_TRY(hipStreamSynchronize(s));
    }
    const int64_t h = found[0], entries = found[2];
    if (h == 0) return GP_OK;
    g->hub_words = (found[1] + 31) / 32;
    const int64_t per = g->hub_words * 4;
    // The runtime keeps freed blocks of up to 64 MB, 64 MB in total, and gives all of them
    // back once it holds more, 0.25 ms each: bitmaps that do not fit beside the
    // graph's other arrays would push these out with them. A block just too large to be kept
    // is freed alone (R-MAT, 205,598 vertices, 847,715 edges, 52 MB of bitmaps:
    // load and free 3.9 ms, 2.1 so).
    constexpr int64_t kKept = int64_t(64) << 20;
    int64_t kept = h * per;
    for (const int64_t bytes : {8 * (g->n + 1), 4 * g->n, 4 * g->nnz, 8 * g->nnz, 4 * g->nnz, 4 * g->nnz})
        if (bytes <= kKept) kept += bytes;
    const int64_t block = h * per <= kKept && kept > kKept ? kKept + (int64_t(2) << 20) : h * per;
    // (row_ptr, new_id, col and the three arrays of root edges)
    GP_HIP_TRY(device_malloc((void**)&g->hub_bits, (size_t)block));
    GP_HIP_TRY(hipMemsetAsync(g->hub_bits, 0, (size_t)(h * per), s));
    hipLaunchKernelGGL(fill_hub_bits, dim3(grid_for(entries)), dim3(256), 0, s, g->row_ptr, g->col, h,
                       entries, g->hub_words, g->hub_bits);
    GP_HIP_TRY(hipGetLastError());
    GP_HIP_TRY(hipStreamSynchronize(s));
    g->n_hubs = (int32_t)h;
    g->stats.hub_vertices = h;
    g->stats.hub_bitmap_bytes = h * per;
    return GP_OK;
}

}  // namespace gpint
