// Host side of the counting kernel: launch geometry, scratch, dispatch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "count_kernel.hpp"

namespace gpcount {
KernelFn pick_kernel_k2(int group, int leaf, int mode, int iep);
KernelFn pick_kernel_k3(int group, int leaf, int mode, int iep);
KernelFn pick_kernel_k4(int group, int leaf, int mode, int iep);
KernelFn pick_kernel_k5(int group, int leaf, int mode, int iep);
KernelFn pick_kernel_k6(int group, int leaf, int mode, int iep);
KernelFn pick_kernel_k7(int group, int leaf, int mode, int iep);
KernelFn pick_kernel_k8(int group, int leaf, int mode, int iep);
KernelFn pick_table_kernel(int k, int mode, int waves);
KernelFn pick_table_iep_kernel(int k, int mode);
BatchFn batch_kernel_k2_2(int group, int leaf, int iep);
BatchFn batch_kernel_k3_3(int group, int leaf, int iep);
BatchFn batch_kernel_k4_4(int group, int leaf, int iep);
BatchFn batch_kernel_k5_5(int group, int leaf, int iep);
BatchFn batch_kernel_k6_6(int group, int leaf, int iep);
BatchFn batch_kernel_k7_8(int group, int leaf, int iep);

// The batched kernel of a run whose plans have k in [kmin, kmax]: one pattern
// size up to 6, or sizes 7 and 8.
BatchFn pick_batch_kernel(int kmin, int kmax, int group, int leaf, int iep) {
    if (kmin == kmax) {
        switch (kmin) {
            case 2: return batch_kernel_k2_2(group, leaf, iep);
            case 3: return batch_kernel_k3_3(group, leaf, iep);
            case 4: return batch_kernel_k4_4(group, leaf, iep);
            case 5: return batch_kernel_k5_5(group, leaf, iep);
            case 6: return batch_kernel_k6_6(group, leaf, iep);
            default: break;
        }
    }
    if (kmin >= 7 && kmax <= 8) return batch_kernel_k7_8(group, leaf, iep);
    return nullptr;
}

namespace {
// A launch's counters cleared: n words at p, nr at r, nb at b (one block; r
// and b may be null with nr, nb 0).
__global__ void init_counters(unsigned long long* p, int n, unsigned long long* r, int nr, unsigned long long* b,
                              int nb) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
    if ((int)threadIdx.x < nr) r[threadIdx.x] = 0;
    if ((int)threadIdx.x < nb) b[threadIdx.x] = 0;
}

// Batch plan blockIdx.x's slots summed into its result words {count low word,
// flags, busy clock ticks, count high word}.
__global__ void collect_batch(const unsigned long long* queues, unsigned long long* result) {
    const unsigned long long* q = queues + (int64_t)blockIdx.x * kQueueWords;
    uint64_t lo, hi, busy = q[(int64_t)__lane_id() * kSlotWords + SLOT_BUSY];
    slot_sum128(q, lo, hi);
    busy = Group<64>().sum(busy);
    if (threadIdx.x == 0) {
        unsigned long long* r = result + 4 * (int64_t)blockIdx.x;
        r[0] = lo;
        r[1] = 0;
        r[2] = busy;
        r[3] = hi;
    }
}

KernelFn pick_kernel(int k, int group, int leaf, int mode, int iep) {
    switch (k) {
        case 2: return pick_kernel_k2(group, leaf, mode, iep);
        case 3: return pick_kernel_k3(group, leaf, mode, iep);
        case 4: return pick_kernel_k4(group, leaf, mode, iep);
        case 5: return pick_kernel_k5(group, leaf, mode, iep);
        case 6: return pick_kernel_k6(group, leaf, mode, iep);
        case 7: return pick_kernel_k7(group, leaf, mode, iep);
        case 8: return pick_kernel_k8(group, leaf, mode, iep);
        default: return nullptr;
    }
}

__global__ void zero_u64(unsigned long long* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// IEP plans: some inner set is left unbuilt as N(a) & N(x) with a an outer
// vertex's list and no cut, so its size depends on (a, x) alone and the
// kernel keeps it in a table shared by the launch's groups
// (count_kernel.hpp, pair_count); likewise the sizes that iep_pair_sum adds.
bool iep_memo_eligible(const GpPlanDesc& d) {
    if (!d.iep) return false;
    for (int m = 0; m < (1 << d.iep) - 1; ++m)
        if (d.it[m].memo && d.it[m].alias < 0) return true;
    const GpLevel& lv = d.lv[d.k - d.iep - 1];
    return d.iep_sum && lv.list >= 0 && (lv.hi_src | lv.lo_src) == 0;
}

// log2 of the IEP memo's rows of n_hubs words: the most ways, up to
// kIepMemoWaysMax, whose table of n_hubs x ways words fits words_cap
// words; -1 if not even one way fits.
int iep_memo_log2(int64_t n_hubs, int64_t words_cap) {
    if (n_hubs <= 0 || words_cap < n_hubs) return -1;
    int l = 0;
    while ((int64_t(2) << l) <= kIepMemoWaysMax && (n_hubs << (l + 1)) <= words_cap) ++l;
    return l;
}

// Whether leaf mode 4 may keep its last-level counts per root: the last
// level is pre & N(v[k-2]) with pre the list of a root level, its cut comes
// from the root levels only, and every earlier image it must avoid is a
// parent of level k-2.
bool memo_eligible(const GpPlanDesc& d) {
    if (d.k < 4 || d.iep) return false;
    const GpLevel& ll = d.lv[d.k - 1];
    if (ll.last_list != d.k - 2 || ll.pre_buf >= 0 || ll.pre_list < 0 || ll.pre_list > 1) return false;
    if ((ll.hi_src | ll.lo_src) & ~3u) return false;
    return (ll.inj & ~(uint32_t)d.lv[d.k - 2].parents) == 0;
}

// Whether the table kernel (count_table.hip) can count d over g: every
// plan whose last level is N(x) & N(root endpoint) cut by root levels, whole
// counts and samples alike, while its sizes fit 16 bits. Not with builds at the
// root level, which each of the block's 16 wavefronts would repeat, and not
// per root. With inclusion-exclusion: plans whose set of the last outer vertex x is
// N(root endpoint) & N(x). Without and with the table: R-MAT 17 5-cycle (64 lanes, split 4
// ways, leaf mode 4 with a memo) 481 and 31 ms; 5-cycle of the cost model's plan on
// R-MAT (20,000 vertices, 160K edges) 100 and 11.5 ms; 6-cycle on Chung-Lu (3,000
// vertices, 30K edges) 199 and 24 ms.
bool table_form(const gpint::DeviceGraph& g, const GpPlanDesc& d) {
    if (d.k < 4 || g.deg2 >= 65536) return false;
    if (d.iep) {
        // the set of the last outer vertex: N(p) & N(x), uncut, p the endpoint
        // that the root array is ordered by
        if (d.iep != 2 || !d.iep_sum || d.root_cut == 0) return false;
        const GpIepTerm& t = d.it[d.iep_sum - 1];
        return t.n_op == 2 && t.memo && t.op[0] == (d.root_cut == 2 ? 0 : 1) && t.op[1] == d.k - 3;
    }
    if (d.build_begin[1] != d.build_end[1]) return false;
    const GpLevel& ll = d.lv[d.k - 1];
    return ll.last_list == d.k - 2 && ll.pre_buf < 0 && (ll.pre_list == 0 || ll.pre_list == 1) &&
           ((ll.hi_src | ll.lo_src) & ~3u) == 0;
}

// Bindings that a search of d is expected to make below one root edge, through
// level to: the product of the levels' candidate sets, from the graph's means. Cuts
// count only where they are by the root's hub, which leaves few candidates; sets
// built from several lists count as an edge's common neighbors.
double expected_bindings(const gpint::DeviceGraph& g, const GpPlanDesc& d, int to) {
    const int hub = d.root_cut == 1 ? 1 : (d.root_cut == 2 ? 0 : -1);  // its level
    double w = 1;
    for (int l = 2; l <= to; ++l) {
        const GpLevel& L = d.lv[l];
        if (L.list < 0) w *= g.mean_common();
        else if (L.list >= 2 || hub < 0) w *= g.mean_deg;
        else if ((L.hi_src >> hub) & 1) w *= L.list == hub ? g.hub_below : g.other_below;
        else w *= L.list == hub ? g.hub_deg : g.other_deg;
    }
    return w;
}

int table_waves(const gpint::DeviceGraph& g, const GpPlanDesc& d);

// Whether the table pays for its fills. A fill costs a block a fixed time (clearing
// 16 to 64 KB of LDS, barriers), 6 to 8 us per root edge where every root has one. What
// it saves is a walk per binding of the level above the last, where the table covers
// it; the eighth is what a lookup costs itself. The lines lie where the table
// began to win on uniform, Chung-Lu and R-MAT graphs of 200 to 1M vertices (below, V, E:
// vertices, edges of uniform graphs; saved as a multiple of the line; table and general kernel).
// Four levels: 4-cycle 1M V, 8M E below 0: 37 and 6.3 ms; 20K, 160K 0.5: 0.37 and
// 0.16; 20K, 400K 1.1: 1.23 and 1.34; 20K, 1M 2.8: 4.5 and 10.6. More levels, a walk counted
// with mean_deg elements: 5-cycle on a 4-regular torus of 1M V 0: 26 and 1.2; 1M, 8M 0:
// 219 and 86; 20K, 160K 0.8: 2.03 and 1.32; 100K, 1.6M 1.8: 57 and 72; 20K, 400K 11:
// 6.5 and 26. 6-cycle 100K, 400K 0.2: 18 and 9; 40K, 200K 1.1: 6.4 and 7.5; 20K, 160K 6.8:
// 7.6 and 19.6. House with inclusion-exclusion 20K, 400K 0.94: 0.81 and 0.73; 20K, 1M 5.8:
// 4.5 and 11.
// A small graph's roots do not fill the device, and a block finishes one sooner than a
// group: 4-cycle on R-MAT (451 V, 2,541 E) 48 and 110 us, G(606, 5,861 E) 61 and 66.
bool table_pays(const gpint::DeviceGraph& g, const GpPlanDesc& d) {
    const int waves = table_waves(g, d);
    const int t = waves == 4 ? 0 : (waves == 8 ? 1 : 2);
    static_assert(gpint::kTableSizes[0] == table_max(4) && gpint::kTableSizes[1] == table_max(8) &&
                      gpint::kTableSizes[2] == table_max(16),
                  "entries counted for the tables' sizes");
    const double covered = (double)g.first_entries[t] / (double)std::max<int64_t>(1, g.nnz);
    if (g.nnz <= 2 * 8192 && covered > 0.99) return true;
    double saved = expected_bindings(g, d, d.iep ? d.k - 3 : d.k - 2) * (covered - 0.125);
    if (d.k == 4) {
        const int hub = d.root_cut == 1 ? 1 : 0;
        const bool below = d.root_cut != 0 && ((d.lv[2].hi_src >> hub) & 1);  // candidates of higher degree than the hub
        return saved >= (below ? 3.5 : 10);
    }
    saved *= g.mean_deg;
    return saved >= (d.iep ? 1200 : (waves == 4 ? 600 : (d.k == 5 ? 6000 : 12000)));
}

bool table_rule(const gpint::DeviceGraph& g, const GpPlanDesc& d) {
    return table_form(g, d) && table_pays(g, d);
}

// With inclusion-exclusion a table is filled once for all of p's roots, so a sparse
// sample pays for the fills: taken while the heaviest endpoint keeps 1,024 sampled
// roots. House with and without the table, every 1st and 7th root of R-MAT 17: 10.3 and
// 15.5, 4.4 and 3.8 ms; every 60th, 237th and 1,001st of R-MAT 22 (largest degree
// 95,042): 221 and 504, 144 and 200, 116 and 68 ms.
bool table_sample(const gpint::DeviceGraph& g, const GpPlanDesc& d, int64_t stride) {
    return !d.iep || stride <= 1 || stride * 1024 <= g.max_deg;
}

// Its blocks: 4 wavefronts where a root edge has little work (one level of lanes,
// k = 4) or the small table covers the graph, else 16: 5-cycle on G(5000, 0.004) 0.74
// ms with 16 and 0.31 with 4.
int table_waves(const gpint::DeviceGraph& g, const GpPlanDesc& d) {
    if (d.iep) return kIepTableWaves;
    return d.k == 4 || g.n <= table_max(4) ? 4 : 16;
}

// Its launch: blocks that keep waves_per_cu wavefronts (a multiple of the
// block's, at least one block) per CU, and up to 16 roots (IEP: 64) per grab,
// which share a hub endpoint and so a table.
int64_t table_blocks(const gpint::DeviceGraph& g, const GpPlanDesc& d, int waves_per_cu, int64_t n_roots) {
    const int w = table_waves(g, d);
    const int64_t most = (int64_t)g.num_cus * std::max(1, std::min(waves_per_cu, d.iep ? 3 * w : 32) / w);
    return std::max<int64_t>(1, std::min(most, n_roots));
}
int32_t table_chunk(const GpPlanDesc& d, int64_t blocks, int64_t n_roots) {
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(d.iep ? 64 : 16, n_roots / (blocks * 8)));
}
KernelFn pick_table(const GpPlanDesc& d, int mode, int waves) {
    return d.iep ? pick_table_iep_kernel(d.k, mode) : pick_table_kernel(d.k, mode, waves);
}

// The count's last step (one wavefront): the sum of the queue's 128-bit totals
// divided by the IEP over-count (1 for plain counts), with the overflow flag
// set only if the quotient does not fit in 64 bits; check: flag a remainder (a
// whole count must divide exactly).
__global__ void finish_count(unsigned long long* result, const unsigned long long* queue, unsigned long long div,
                             int check, unsigned long long* host) {
    uint64_t lo, hi;
    slot_sum128(queue, lo, hi);
    if (threadIdx.x == 0) {
        const unsigned long long flags = result[1];
        result[0] = lo;
        finish128(&result[0], &result[1], hi, div);
        if (!check) result[1] = (result[1] & ~2ull) | (flags & 2ull);
        if (host) {
            host[0] = result[0];
            host[1] = result[1];
        }
    }
}

// The counting kernels' accumulation on given values: each lane adds its
// share with add_count (carries counted), the wavefronts sum exactly in 128
// bits and publish into the queue's slots, as a count's wavefronts do.
__global__ void sum_check_kernel(const unsigned long long* vals, int64_t n, unsigned long long* queue) {
    uint64_t acc = 0, carry = 0;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step)
        add_count(acc, vals[i], carry);
    wave_sum128(acc, carry);
    if (__lane_id() == 0) {
        const int wave = (int)((blockIdx.x * blockDim.x + threadIdx.x) / 64);
        unsigned long long* slot = queue + (int64_t)(wave & (kSlots - 1)) * kSlotWords;
        publish128(&slot[SLOT_LO], &slot[SLOT_HI], acc, carry);
    }
}
}  // namespace
}  // namespace gpcount

using namespace gpcount;

namespace gpint {

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_pool_mu;
hipMemPool_t g_pool[kMaxDevices] = {};
bool g_pool_failed[kMaxDevices] = {};
int g_pool_graphs[kMaxDevices] = {};

// The device's pool, made on first use; null if it cannot be made or no graph is
// there (nothing would give its memory back).
hipMemPool_t device_pool(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (g_pool_graphs[device] <= 0) return nullptr;
    if (!g_pool[device] && !g_pool_failed[device]) {
        hipMemPoolProps props;
        std::memset(&props, 0, sizeof props);
        props.allocType = hipMemAllocationTypePinned;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = device;
        hipMemPool_t p = nullptr;
        uint64_t keep = kPoolKeepBytes;
        if (hipMemPoolCreate(&p, &props) != hipSuccess) p = nullptr;
        else if (hipMemPoolSetAttribute(p, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) {
            (void)hipMemPoolDestroy(p);
            p = nullptr;
        }
        g_pool[device] = p;
        g_pool_failed[device] = p == nullptr;
        if (!p) (void)hipGetLastError();
    }
    return g_pool[device];
}
}  // namespace

// Gives the device memory that its pool holds and no call uses back to the driver.
static void pool_trim() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (g_pool[dev]) (void)hipMemPoolTrimTo(g_pool[dev], 0);
}

hipError_t device_malloc(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    pool_trim();
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

hipError_t stream_malloc(void** p, size_t bytes, hipStream_t stream) {
    hipError_t e = hipMallocAsync(p, bytes, stream);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    pool_trim();
    e = hipMallocAsync(p, bytes, stream);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

hipError_t pool_malloc(void** p, size_t bytes, hipStream_t stream) {
    size_t size = size_t(64) << 10;
    while (size < bytes && size < kPoolMostBytes) size *= 2;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    int dev = -1;
    hipMemPool_t pool = nullptr;
    if (bytes <= size && hipStreamIsCapturing(stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone &&
        hipGetDevice(&dev) == hipSuccess)
        pool = device_pool(dev);
    if (pool && hipMallocFromPoolAsync(p, size, pool, stream) == hipSuccess) return hipSuccess;
    (void)hipGetLastError();  // the default pool decides
    return stream_malloc(p, bytes, stream);
}

void pool_add_graph(int device) {
    if (device < 0 || device >= kMaxDevices) return;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    ++g_pool_graphs[device];
}

void pool_drop_graph(int device) {
    if (device < 0 || device >= kMaxDevices) return;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (--g_pool_graphs[device] == 0 && g_pool[device]) (void)hipMemPoolTrimTo(g_pool[device], 0);
}

// Plans whose search ends at the root edge: lanes take different root edges.
static bool lanes_take_roots(const GpPlanDesc& d) { return d.k <= 3 || d.iep == d.k - 2; }

// Tasks per grab of a launch: at least one per lane where lanes take root edges.
static int32_t grab_tasks_of(const GpPlanDesc& d, const LaunchCfg& cfg, int group) {
    return lanes_take_roots(d) ? std::max(cfg.chunk, group) : cfg.chunk;
}

LaunchCfg default_launch(const GpPlanDesc& d) {
    LaunchCfg cfg;
    // Plain searches run widest on 16 lanes: their sets are short, and four paths
    // per wavefront hide each other's loads. 64 and 16 lanes: R-MAT 19 4-clique 3.0
    // and 2.2 ms, R-MAT 17 diamond 4.8 and 2.8, 5-clique (model plan) 10.2 and 6.3,
    // Chung-Lu 7000 prism 268 and 121, 5-wheel 74 and 36, house 13.3 and 7.1.
    // Where lanes take root edges, and with inclusion-exclusion (lanes take the
    // last outer level), the width of a wavefront.
    cfg.group = d.k >= 4 && !d.iep ? 16 : 64;
    cfg.own_group = cfg.own_chunk = true;
    cfg.waves_per_cu = 32;
    // where lanes take different root edges (k <= 3, or IEP over every level
    // after the root) a grab fills the lanes of a group: the 4-star with IEP on
    // R-MAT (91K vertices, 907K edges) takes 116 ms at 4 per grab, 0.13 at 64
    cfg.chunk = lanes_take_roots(d) ? 64 : 4;
    cfg.leaf = 1;
    cfg.split_ways = 16;
    cfg.split_vertices = 256;
    return cfg;
}

bool uses_table(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& cfg) {
    return cfg.table >= 0 && table_rule(g, d) && (cfg.table > 0 || table_sample(g, d, cfg.root_stride));
}

int resident_waves_per_cu(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& cfg) {
    if (uses_table(g, d, cfg)) {
        const int w = table_waves(g, d);
        return std::max(1, std::min(cfg.waves_per_cu, d.iep ? 3 * w : 32) / w) * w;
    }
    const bool iep = d.iep != 0;
    const int group = iep ? (cfg.group >= 64 ? 64 : 32) : cfg.group;
    KernelFn fn = pick_kernel(d.k, group, cfg.leaf, MODE_PLAIN, d.iep);
    (void)g;
    int nb = 0;
    if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)fn, kBlock, 0) != hipSuccess || nb <= 0)
        return cfg.waves_per_cu;
    return std::min(cfg.waves_per_cu, nb * (kBlock / 64));
}

int64_t xcd_block_tasks(const DeviceGraph& g, const LaunchCfg& cfg, int group) {
    (void)g;
    (void)group;
    if (cfg.xcd <= 0) return 0;  // the default: one task order for the device (measured faster)
    const int64_t chunk = std::max(1, cfg.chunk);
    return (cfg.xcd + chunk - 1) / chunk * chunk;
}

LaunchCfg apply_launch(LaunchCfg cfg, const gp_launch* l) {
    if (l) {
        if (l->group) {
            cfg.group = l->group;
            cfg.own_group = false;
        }
        if (l->waves_per_cu) cfg.waves_per_cu = l->waves_per_cu;
        if (l->chunk) {
            cfg.chunk = l->chunk;
            cfg.own_chunk = false;
        }
        if (l->leaf_mode) cfg.leaf = l->leaf_mode;
        if (l->root_stride) cfg.root_stride = l->root_stride;
        cfg.root_offset = l->root_offset;
        if (l->split_ways) cfg.split_ways = l->split_ways;
        if (l->split_vertices) cfg.split_vertices = l->split_vertices;
        if (l->xcd_tasks) cfg.xcd = l->xcd_tasks;
        if (l->batch_runs) cfg.batch_runs = l->batch_runs;
    }
    return cfg;
}

// Five and more levels, on graphs whose heaviest roots decide (a root edge's endpoints
// have 64 neighbors or more in the mean): where the level-2 candidates are a list that is
// not cut below the hub, a grab of four such roots by a group a quarter as wide
// ends last, so grabs are single tasks: R-MAT (131,072 vertices, 200K edges)
// 5-cycle of schedule 0,1,2,4,3 301 and 100 ms (64 lanes, four a grab: 152), house of
// 1,4,2,3,0 120 and 43 (81). Below 64 neighbors, tasks are short and even, and the
// queue counts: 5-cycle on G(100,000, 400K edges) 1.07 and 1.35 ms.
// Where they are a built set, but the lanes then take whole lists (the level above the
// last), 32 lanes, two a grab, while the heaviest root has more work than a group's
// share: R-MAT (131,072, 200K) house of 4,1,0,2,3 131 ms on 16 lanes, 54 on 32 (64: 67).
static void settle_tail(const DeviceGraph& g, const GpPlanDesc& d, LaunchCfg* cfg, int64_t roots) {
    if (d.k < 5 || d.iep || g.mean_deg < 64) return;
    const int hub = d.root_cut == 1 ? 1 : (d.root_cut == 2 ? 0 : -1);
    const GpLevel &l2 = d.lv[2], &lanes = d.lv[d.k - 2];
    if (l2.list >= 0) {
        if (cfg->own_chunk && (hub < 0 || !((l2.hi_src >> hub) & 1))) cfg->chunk = 1;
    } else if (lanes.list >= 0 && lanes.hi_src == 0) {
        const int64_t most = (int64_t)g.num_cus * cfg->waves_per_cu * (64 / cfg->group);
        // of six levels and more it has to be well above: K4 + path of 2,1,0,3,4,5 on R-MAT
        // (200,000 vertices, 600K edges; 1.2 shares) 970 ms on 16 lanes, 1,151 on 32
        const double share = (double)roots / (double)most * g.mean_deg;
        if ((double)g.max_deg < (d.k > 5 ? 1.5 : 1.0) * share) return;
        cfg->group = 32;
        if (cfg->own_chunk) cfg->chunk = 2;
    }
}

void settle_group(const DeviceGraph& g, const GpPlanDesc& d, LaunchCfg* cfg, int64_t room) {
    if (!cfg->own_group || cfg->group >= 64) return;
    const int64_t most = (int64_t)g.num_cus * cfg->waves_per_cu * (64 / cfg->group);
    const int64_t roots = root_task_count(g, d);
    const int64_t groups = std::min(most, roots / std::max(1, cfg->chunk) + 1);
    // fewer roots than groups: the heaviest decide, and finish sooner on more lanes
    // (5-cycle per root on Chung-Lu, 4,709 edges: 7.3 ms on 16 lanes, 5.6 on 64)
    if (roots < most || groups * d.nbuf * std::max<int64_t>(1, g.deg2) * 4 > room) {
        cfg->group = 64;
        return;
    }
    settle_tail(g, d, cfg, roots);
}

static const int2* pick_roots(const DeviceGraph& g, int root_cut, int64_t* n) {
    if (root_cut == 1) {
        *n = g.n_lower;
        return g.roots_lower;
    }
    if (root_cut == 2) {
        *n = g.n_upper;
        return g.roots_upper;
    }
    *n = g.nnz;
    return g.roots_all;
}

// Roots split into several tasks: the first `roots` of the (sampled) root
// array, whose smaller endpoint is below 2^floor(log2(split_vertices)).
// Per-root counts stay one task per root, and so do patterns with no level-2
// loop (k <= 3, or IEP over every level after the root).
// So do 4-vertex plans whose level-2 candidates are cut below the root's hub
// endpoint (as the 4-clique's are): fewer candidates than the hub's id, and each
// of the ways would build the root's sets again. R-MAT 19 4-clique (3.2M edges),
// default launch: 14.6 ms split 16 ways, 3.6 not. With one more level the
// tail of the heaviest roots decides: R-MAT 17 5-clique 5.3 ms split, 7.6 not.
struct SplitPlan {
    int64_t roots = 0;
    int ways = 1;
};

static SplitPlan split_plan(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& cfg, int mode,
                            int64_t n_roots, int64_t stride, int64_t offset) {
    SplitPlan sp;
    if (mode == MODE_PER_ROOT || d.k < 4 || (d.iep && d.iep == d.k - 2) || cfg.split_ways <= 1 ||
        cfg.split_vertices <= 0)
        return sp;
    const unsigned hub = d.root_cut == 1 ? 2u : (d.root_cut == 2 ? 1u : 0u);  // the level of the smaller id
    if (d.k == 4 && (d.lv[2].hi_src & hub)) return sp;
    int i = 0;
    while (i < 31 && (int64_t(1) << (i + 1)) <= cfg.split_vertices) ++i;
    const int64_t pref = g.upper_pref[i] * (d.root_cut == 0 ? 2 : 1);
    const int64_t sampled = pref > offset ? (pref - offset + stride - 1) / stride : 0;
    sp.roots = std::min(n_roots, sampled);
    sp.ways = cfg.split_ways;
    // where lanes take the level-2 candidates, a way of fewer than a group's
    // width leaves lanes idle: the 5-vertex patterns with IEP on Chung-Lu (3,000
    // vertices, 30K edges, largest degree 281) take 1.5-2.2 ms each split 16
    // ways, 0.3-0.6 split 4 ways
    if (d.k - (d.iep ? d.iep + 1 : 2) == 2)
        sp.ways = (int)std::min<int64_t>(sp.ways, std::max<int64_t>(1, g.max_deg / std::max(cfg.group, 1)));
    if (sp.ways <= 1) sp = SplitPlan{};
    return sp;
}

int64_t task_count(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& cfg, TaskSplit* split) {
    int64_t n = 0;
    (void)pick_roots(g, d.root_cut, &n);
    const SplitPlan sp = split_plan(g, d, cfg, MODE_PLAIN, n, 1, 0);
    split->tasks = sp.roots * sp.ways;
    split->ways = sp.ways;
    return n + sp.roots * (sp.ways - 1);
}

namespace {
constexpr size_t kAlign = 256;
constexpr size_t kQueueBytes = sizeof(unsigned long long) * kQueueWords;  // a multiple of kAlign
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
}  // namespace

namespace {
// What one launch of the counting kernels is made of.
struct CountShape {
    LaunchCfg cfg;
    KernelFn fn = nullptr;
    bool table = false;  // the table kernel
    int mode = MODE_PLAIN, group = 64, tab_waves = 16;
    int64_t cap = 1;
    const int2* roots = nullptr;
    int64_t n_roots = 0, split_roots = 0, n_tasks = 0, need = 0;
    int split_ways = 1;
    int32_t chunk = 1, whole_chunk = 1;
    int64_t blocks = 1, groups_per_block = 4;
    size_t scratch_bytes = 0;
    int iep_log2 = -1;
    int64_t memo_words = 0;
    bool use_memo = false;
    int threads() const { return table ? tab_waves * 64 : kBlock; }
};
}  // namespace

static gp_status count_shape(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& launch, int mode,
                             const Workspace* ws, CountShape* out) {
    CountShape& z = *out;
    // keep scratch within a fixed budget (or the caller's workspace): fewer
    // resident groups if needed
    const int64_t budget = ws ? (int64_t)ws->bytes - (int64_t)kQueueBytes : int64_t(16) << 30;
    if (ws && budget < 0) return GP_ERR_ARG;
    z.cfg = launch;
    LaunchCfg& cfg = z.cfg;
    if (ws) settle_group(g, d, &cfg, budget);
    if (cfg.group != 64 && cfg.group != 32 && cfg.group != 16 && cfg.group != 8) return GP_ERR_ARG;
    if (cfg.leaf < 1 || cfg.leaf > 4) return GP_ERR_ARG;
    if (cfg.waves_per_cu < 1 || cfg.waves_per_cu > 32 || cfg.chunk < 1) return GP_ERR_ARG;
    z.mode = mode;
    const bool iep = d.iep != 0;
    z.group = iep ? (cfg.group >= 64 ? 64 : 32) : cfg.group;  // IEP kernels: 64 or 32 lanes
    z.tab_waves = table_waves(g, d);
    z.cap = std::max<int64_t>(1, g.deg2);
    // the table kernel, unless a workspace has no room for its larger blocks
    z.table = mode != MODE_PER_ROOT && uses_table(g, d, cfg) && z.tab_waves * d.nbuf * z.cap * 4 <= budget;
    z.fn = z.table ? pick_table(d, mode, z.tab_waves) : pick_kernel(d.k, z.group, cfg.leaf, mode, d.iep);
    if (!z.fn) return GP_ERR_UNSUPPORTED;

    int64_t all_roots = 0;
    z.roots = pick_roots(g, d.root_cut, &all_roots);
    if (cfg.root_stride < 1 || cfg.root_offset < 0) return GP_ERR_ARG;
    if (cfg.split_ways < 1 || cfg.split_ways > 4096 || cfg.split_vertices < 0 || cfg.budget_ms < 0)
        return GP_ERR_ARG;
    // sampled roots: roots[offset + r * stride]
    z.n_roots =
        all_roots > cfg.root_offset ? (all_roots - cfg.root_offset + cfg.root_stride - 1) / cfg.root_stride : 0;
    const SplitPlan sp = split_plan(g, d, cfg, mode, z.n_roots, cfg.root_stride, cfg.root_offset);
    z.split_roots = sp.roots;
    z.split_ways = sp.ways;
    z.n_tasks = z.n_roots + sp.roots * (sp.ways - 1);

    const int waves_per_block = kBlock / 64;
    z.blocks = std::max<int64_t>(1, (int64_t)g.num_cus * cfg.waves_per_cu / waves_per_block);
    z.groups_per_block = kBlock / z.group;
    z.chunk = grab_tasks_of(d, cfg, z.group);
    if (z.table) {
        z.groups_per_block = z.tab_waves;
        z.blocks = table_blocks(g, d, cfg.waves_per_cu, z.n_roots);
        z.chunk = table_chunk(d, z.blocks, z.n_roots);
        z.whole_chunk = table_chunk(d, table_blocks(g, d, cfg.waves_per_cu, all_roots), all_roots);
    }
    const int64_t per_block = d.nbuf > 0 ? z.groups_per_block * d.nbuf * z.cap * 4 : 0;
    // the memo that the launch may use (below): one for all of it, or a word per
    // hub in every group
    const bool leaf4_memo = cfg.leaf == 4 && !z.table && mode != MODE_PER_ROOT && !iep && memo_eligible(d) &&
                            z.n_tasks < (int64_t(1) << 31);
    const bool iep_memo = iep && iep_memo_eligible(d);
    if (per_block > 0) {
        if (ws && per_block > budget) return GP_ERR_NOMEM;  // not even one block's buffers fit
        z.blocks = std::min(z.blocks, std::max<int64_t>(1, budget / per_block));
        // within what the pool hands out, if that leaves half the grid: larger
        // regions are freed after the call, and the driver clears them at 24 GB/s
        const int64_t l = iep_memo ? iep_memo_log2(g.n_hubs, kIepMemoBytes / 8) : -1;
        const int64_t room = (int64_t)kPoolMostBytes - (int64_t(1) << 20) - (l >= 0 ? ((int64_t)g.n_hubs * 8) << l : 0);
        const int64_t kept = room / (per_block + (leaf4_memo ? z.groups_per_block * (int64_t)g.n_hubs * 8 : 0));
        if (!ws && 2 * kept >= z.blocks) z.blocks = std::min(z.blocks, kept);
    }
    // a grid larger than the number of root tasks only adds idle groups
    z.need = (z.n_tasks + z.chunk - 1) / z.chunk;
    if (!z.table)
        z.blocks =
            std::min(z.blocks, std::max<int64_t>(1, (z.need + z.groups_per_block - 1) / z.groups_per_block));

    z.scratch_bytes = (size_t)(z.blocks * per_block);
    // leaf mode 4's per-task memo: one word per hub per group, within 4 GiB
    // (within what the workspace has left); the IEP memo: one table for the
    // launch, 2^l words per hub, within 2 GiB (or the room left)
    const int64_t memo_cap = ws ? budget - (int64_t)align_up(z.scratch_bytes) : (int64_t(4) << 30);
    z.iep_log2 = iep_memo ? iep_memo_log2(g.n_hubs, std::min(memo_cap, kIepMemoBytes) / 8) : -1;
    z.memo_words = iep ? (z.iep_log2 >= 0 ? (int64_t)g.n_hubs << z.iep_log2 : 0)
                       : z.blocks * z.groups_per_block * (int64_t)g.n_hubs;
    z.use_memo = (leaf4_memo || z.iep_log2 >= 0) && g.n_hubs > 0 && z.memo_words * 8 <= memo_cap;
    return GP_OK;
}

gp_status describe_count(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& cfg, gp_shape* out) {
    CountShape z;
    const gp_status st = count_shape(g, d, cfg, MODE_PLAIN, nullptr, &z);
    if (st != GP_OK) return st;
    out->table = z.table ? 1 : 0;
    out->memo = z.use_memo ? 1 : 0;
    out->group = z.table ? 64 : z.group;
    out->chunk = z.chunk;
    out->blocks = (int32_t)z.blocks;
    out->threads = z.threads();
    return GP_OK;
}

gp_status launch_count(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& launch,
                       hipStream_t stream, unsigned long long* result_dev,
                       unsigned long long* per_root, bool account, unsigned long long* busy,
                       const Workspace* ws, unsigned long long* result_host) {
    CountShape z;
    const gp_status shaped =
        count_shape(g, d, launch, account ? MODE_ACCOUNT : (per_root ? MODE_PER_ROOT : MODE_PLAIN), ws, &z);
    if (shaped != GP_OK) return shaped;
    if (z.table && busy) z.fn = pick_table(d, MODE_SAMPLE, z.tab_waves);
    const LaunchCfg& cfg = z.cfg;
    const size_t scratch_bytes = z.scratch_bytes;
    const bool use_memo = z.use_memo;
    const int64_t memo_words = z.memo_words;

    int32_t* scratch = nullptr;
    unsigned long long* queue = nullptr;
    unsigned long long* memo = nullptr;
    // one region: the queue, (without result_dev) the result words, the
    // candidate buffers, the memo
    if (!result_dev && (ws || !result_host)) return GP_ERR_ARG;
    const size_t head = kQueueBytes + (result_dev ? 0 : kAlign);
    char* base = ws ? (char*)ws->base : nullptr;
    if (!ws && pool_malloc((void**)&base, head + align_up(scratch_bytes) + (use_memo ? (size_t)memo_words * 8 : 0),
                           stream) != hipSuccess)
        return GP_ERR_NOMEM;
    queue = (unsigned long long*)base;
    if (!result_dev) result_dev = (unsigned long long*)(base + kQueueBytes);
    if (scratch_bytes) scratch = (int32_t*)(base + head);
    if (use_memo) memo = (unsigned long long*)(base + head + align_up(scratch_bytes));
    if (use_memo)
        hipLaunchKernelGGL(zero_u64, dim3((unsigned)std::min<int64_t>(4096, (memo_words + 255) / 256)), dim3(256), 0,
                           stream, memo, memo_words);
    hipLaunchKernelGGL(init_counters, dim3(1), dim3(1024), 0, stream, queue, kQueueWords, result_dev, account ? 3 : 2,
                       busy, busy ? 3 : 0);

    CountArgs a;
    a.row_ptr = g.row_ptr;
    a.col = g.col;
    a.roots = z.roots;
    a.n_roots = z.n_roots;
    a.n_tasks = z.n_tasks;
    a.n_chunks = z.table ? (z.n_roots + z.chunk - 1) / z.chunk : z.need;
    a.tab_n = (int32_t)std::min<int64_t>(g.n, table_max(z.tab_waves));
    a.whole_chunk = z.whole_chunk;
    a.split_roots = z.split_roots;
    a.split_ways = z.split_ways;
    a.budget_ticks = busy && cfg.budget_ms > 0 ? (uint64_t)(cfg.budget_ms * g.wall_khz) : 0;
    a.root_offset = cfg.root_offset;
    a.hub_bits = g.hub_bits;
    a.hub_words = g.hub_words;
    a.n_hubs = g.n_hubs;
    a.root_stride = cfg.root_stride;
    a.scratch = scratch;
    a.buf_cap = z.cap;
    a.queue = queue;
    a.result = result_dev;
    a.per_root = per_root;
    a.busy = busy;
    a.memo = memo;
    a.chunk = z.chunk;
    a.memo_ways_log2 = std::max(z.iep_log2, 0);
    LaunchCfg grab = cfg;
    grab.chunk = z.chunk;
    a.xcd_block = xcd_block_tasks(g, grab, z.group);
    if (z.n_tasks > 0)
        hipLaunchKernelGGL(z.fn, dim3((unsigned)z.blocks), dim3((unsigned)z.threads()), 0, stream, d, a);
    // a sample's total need not be a multiple of the over-count: its quotient
    // is an estimate, not checked
    const bool whole = cfg.root_stride == 1 && cfg.root_offset == 0 && !(busy && cfg.budget_ms > 0);
    hipLaunchKernelGGL(finish_count, dim3(1), dim3(64), 0, stream, result_dev, queue,
                       (unsigned long long)(d.iep ? d.iep_div : 1), whole ? 1 : 0, result_host);
    hipError_t le = hipGetLastError();
    if (!ws) (void)hipFreeAsync(base, stream);
    if (le != hipSuccess) return GP_ERR_HIP;
    return GP_OK;
}

gp_status check_sum(const uint64_t* values, int64_t n, uint64_t div, hipStream_t stream, uint64_t* out,
                    uint32_t* flags) {
    if (n < 0 || (n > 0 && !values) || div < 1) return GP_ERR_ARG;
    unsigned long long* w = nullptr;  // the queue's slots, {low word, flags}, then the values
    GP_HIP_TRY(pool_malloc((void**)&w, kQueueBytes + sizeof(unsigned long long) * (2 + (size_t)n), stream));
    unsigned long long* res = w + kQueueWords;
    unsigned long long h[2] = {0, 0};
    hipError_t e = hipSuccess;
    hipLaunchKernelGGL(init_counters, dim3(1), dim3(1024), 0, stream, w, kQueueWords, res, 2,
                       (unsigned long long*)nullptr, 0);
    if (n > 0)
        e = hipMemcpyAsync(res + 2, values, sizeof(unsigned long long) * (size_t)n, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(sum_check_kernel, dim3(4), dim3(kBlock), 0, stream, res + 2, n, w);
        hipLaunchKernelGGL(finish_count, dim3(1), dim3(64), 0, stream, res, w, (unsigned long long)div, 1,
                           (unsigned long long*)nullptr);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(h, res, sizeof h, hipMemcpyDeviceToHost, stream);
    (void)hipFreeAsync(w, stream);
    if (hipStreamSynchronize(stream) != hipSuccess || e != hipSuccess) return GP_ERR_HIP;
    *out = h[0];
    *flags = (uint32_t)h[1];
    return GP_OK;
}

// Workspace of launch_count_noalloc: every GPU the library runs on holds one
// copy of this array until the process ends. In host code its name is only a
// stand-in; the device address of each GPU's copy comes from
// hipGetSymbolAddress, taken once per device.
static __device__ __align__(256) unsigned char scratch[kNoallocWorkspaceBytes + kNoallocQueueBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};
}  // namespace

// The device address of this GPU's copy of `scratch` (the device must be
// current), looked up on the first call per device.
static gp_status scratch_address(int device, void** ptr) {
    if (device < 0 || device >= 64) return GP_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GP_ERR_HIP;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return GP_OK;
}

gp_status launch_count_noalloc(const DeviceGraph& g, const GpPlanDesc& d, const LaunchCfg& cfg,
                               hipStream_t stream, unsigned long long* result_dev) {
    void* base = nullptr;
    const gp_status st = scratch_address(g.device, &base);
    if (st != GP_OK) return st;
    Workspace ws;
    ws.base = base;
    static_assert(kQueueBytes <= kNoallocQueueBytes, "room for the queue");
    ws.bytes = kNoallocWorkspaceBytes + kQueueBytes;
    return launch_count(g, d, cfg, stream, result_dev, nullptr, false, nullptr, &ws);
}

int64_t root_task_count(const DeviceGraph& g, const GpPlanDesc& d) {
    int64_t n = 0;
    (void)pick_roots(g, d.root_cut, &n);
    return n;
}

void batch_release(BatchState* st) {
    (void)hipFree(st->scratch);
    (void)hipFree(st->memo);
    (void)hipFree(st->queues);
    (void)hipFree(st->result);
    *st = BatchState{};
}

// A plan's shape inside a batch: IEP plans run in 64- or 32-lane groups,
// others in 64, 32, 16 or 8 (floored at min_group); leaf modes 1, 3 or 4 (2
// runs as 1).
static void batch_shape(const GpPlanDesc& d, const LaunchCfg& c, int min_group, BatchPlan* bp) {
    const int want = std::max(c.group, min_group);
    if (d.iep) bp->group = want >= 64 ? 64 : 32;
    else bp->group = want >= 64 ? 64 : (want >= 32 ? 32 : (want >= 16 ? 16 : 8));
    bp->leaf = d.iep ? 1 : (c.leaf == 3 || c.leaf == 4 ? c.leaf : 1);
    bp->chunk = std::max(1, grab_tasks_of(d, c, bp->group));
}

int batch_shape_key(const GpPlanDesc& d, const LaunchCfg& c, int min_group) {
    BatchPlan bp;
    batch_shape(d, c, min_group, &bp);
    return (std::min(d.k, 7) << 16) | (bp.group << 8) | (bp.leaf << 4) | d.iep;
}

// The host copy of a batch's plan table (launches pass it by value).
static void store_plans(BatchState* b, const std::vector<BatchPlan>& plans) {
    b->h_plans.assign((const char*)plans.data(), (const char*)(plans.data() + plans.size()));
}

// Per-plan task ranges, shapes and the launch geometry for np plans.
static gp_status batch_layout(const DeviceGraph& g, const GpPlanDesc* descs, const LaunchCfg* cfgs,
                              const int64_t* offsets, const int64_t* counts, int np, int min_group_floor,
                              BatchState* b, std::vector<BatchPlan>* plans) {
    plans->resize(np);
    b->runs.clear();
    std::vector<int64_t> nroots(np, 0);
    std::vector<bool> whole(np, false);
    int32_t nbuf = 0;
    b->kmax = 2;
    int64_t tag_next = 1;  // memo tags of the eligible plans: disjoint ranges
    bool any_memo = false;
    for (int i = 0; i < np; ++i) {
        int64_t n_all = 0;
        const int2* roots = pick_roots(g, descs[i].root_cut, &n_all);
        // a strided root sample per plan, as in launch_count
        const int64_t stride = std::max<int64_t>(1, cfgs[i].root_stride);
        const int64_t roff = std::max<int64_t>(0, cfgs[i].root_offset);
        const int64_t n_sampled = n_all > roff ? (n_all - roff + stride - 1) / stride : 0;
        // offsets and counts are in the plan's task space (split roots count once per task)
        const SplitPlan sp = split_plan(g, descs[i], cfgs[i], MODE_PLAIN, n_sampled, stride, roff);
        const int64_t n_tasks = n_sampled + sp.roots * (sp.ways - 1);
        int64_t off = offsets ? offsets[i] : 0;
        int64_t cnt = counts ? counts[i] : n_tasks;
        if (off < 0 || cnt < 0) return GP_ERR_ARG;
        off = std::min(off, n_tasks);
        cnt = std::min(cnt, n_tasks - off);
        whole[i] = off == 0 && cnt == n_tasks;
        nroots[i] = n_sampled;
        BatchPlan& bp = (*plans)[i];
        std::memset(&bp, 0, sizeof bp);
        bp.roots = roots;
        bp.root_offset = roff;
        bp.root_stride = stride;
        bp.n_tasks = cnt;
        bp.task_offset = off;
        bp.split_roots = sp.roots;
        bp.split_ways = sp.ways;
        batch_shape(descs[i], cfgs[i], min_group_floor, &bp);
        const int64_t grab = (int64_t)(64 / bp.group) * bp.chunk;
        bp.n_chunks = (cnt + grab - 1) / grab;
        // consecutive plans of one shape share a launch (up to kRunMaxPlans:
        // their descriptors are its kernel arguments)
        const int iep_depth = descs[i].iep;
        const int ksize = std::min((int)descs[i].k, 7);  // sizes 7 and 8 share a kernel
        // runs are laid out for every sample that the batch may be set to: a plan that may
        // run on path tables is alone, whether its present sample does or not
        const bool may_table = whole[i] && cfgs[i].table >= 0 && table_rule(g, descs[i]);
        if (b->runs.empty() || may_table || b->runs.back().may_table || b->runs.back().group != bp.group || b->runs.back().leaf != bp.leaf ||
            b->runs.back().iep != iep_depth || std::min(b->runs.back().kmin, 7) != ksize ||
            b->runs.back().p1 - b->runs.back().p0 >= kRunMaxPlans || cfgs[i].batch_runs == 2) {
            BatchRun r;
            r.p0 = i;
            r.group = bp.group;
            r.leaf = bp.leaf;
            r.iep = iep_depth;
            r.kmin = r.kmax = descs[i].k;
            r.may_table = may_table;
            r.table = may_table && uses_table(g, descs[i], cfgs[i]);
            r.tab_waves = table_waves(g, descs[i]);
            b->runs.push_back(r);
        }
        b->runs.back().p1 = i + 1;
        b->runs.back().kmin = std::min(b->runs.back().kmin, (int)descs[i].k);
        b->runs.back().kmax = std::max(b->runs.back().kmax, (int)descs[i].k);
        b->runs.back().waves_per_cu = std::max(b->runs.back().waves_per_cu, cfgs[i].waves_per_cu);
        bp.tag_base = 0;
        if (bp.leaf == 4 && !may_table && !descs[i].iep && g.n_hubs > 0 && memo_eligible(descs[i]) &&
            tag_next + n_all < (int64_t(1) << 31) - 1) {  // below the IEP memo's tags
            bp.tag_base = (uint32_t)tag_next - 1;  // tags tag_base + root + 1 >= tag_next
            tag_next += n_all;
            any_memo = true;
        }
        // an IEP plan run alone keeps its inner set sizes in the same region
        if (descs[i].iep && g.n_hubs > 0 && iep_memo_eligible(descs[i])) any_memo = true;
        nbuf = std::max(nbuf, descs[i].nbuf);
        b->kmax = std::max(b->kmax, (int)descs[i].k);
    }
    b->np = np;
    b->nbuf = nbuf;
    b->use_memo = any_memo;
    for (BatchRun& r : b->runs) {
        const BatchPlan& bp = (*plans)[r.p0];
        r.solo = r.p1 - r.p0 == 1 && whole[r.p0] && bp.tag_base == 0 && r.kmin == r.kmax;
        r.roots = bp.roots;
        r.n_roots = nroots[r.p0];
        r.root_offset = bp.root_offset;
        r.root_stride = bp.root_stride;
        r.n_tasks = bp.n_tasks;
        r.split_roots = bp.split_roots;
        r.split_ways = bp.split_ways;
        r.chunk = bp.chunk;
    }
    b->h_descs.assign(descs, descs + np);
    store_plans(b, *plans);
    return GP_OK;
}

// Wavefront-resident blocks: the device's share, within the scratch and memo
// budgets. Scratch per wavefront: slots_per_wave groups x nbuf x cap int32.
static int64_t batch_blocks(const DeviceGraph& g, int waves_per_cu, int slots_per_wave, int32_t nbuf, int64_t cap,
                            bool memo) {
    const int waves_per_block = kBlock / 64;
    int64_t blocks = std::max<int64_t>(1, (int64_t)g.num_cus * waves_per_cu / waves_per_block);
    if (nbuf > 0) {
        const int64_t budget = int64_t(16) << 30;
        blocks = std::min(blocks, std::max<int64_t>(1, budget / ((int64_t)waves_per_block * slots_per_wave * nbuf *
                                                                  cap * 4)));
    }
    if (memo && g.n_hubs > 0) {
        const int64_t budget = int64_t(4) << 30;
        blocks = std::min(blocks, std::max<int64_t>(1, budget / ((int64_t)waves_per_block * slots_per_wave *
                                                                  g.n_hubs * 8)));
    }
    return blocks;
}

// Group slots (scratch and memo tables) a run's launch addresses, on path tables or not.
static int64_t run_group_slots(const BatchRun& r, bool table) {
    return table ? r.table_blocks * r.tab_waves : r.plain_blocks * (kBlock / 64) * (64 / r.group);
}

gp_status batch_prepare(const DeviceGraph& g, const GpPlanDesc* descs, const LaunchCfg* cfgs,
                        const int64_t* offsets, const int64_t* counts, int np, int waves_per_cu,
                        hipStream_t stream, BatchState* st) {
    if (np < 1 || np > kBatchMaxPlans) return GP_ERR_ARG;
    BatchState b;
    b.cap = std::max<int64_t>(1, g.deg2);
    std::vector<BatchPlan> plans;
    gp_status rc = batch_layout(g, descs, cfgs, offsets, counts, np, 8, &b, &plans);
    if (rc != GP_OK) return rc;
    // every run at its own width and residency; the regions fit the largest
    int64_t slots = 0;
    for (BatchRun& r : b.runs) {
        r.plain_blocks =
            batch_blocks(g, std::min(waves_per_cu, r.waves_per_cu), 64 / r.group, b.nbuf, b.cap, b.use_memo);
        slots = std::max(slots, run_group_slots(r, false));
        if (r.may_table) {
            // within the scratch budget, as batch_blocks keeps the others
            r.table_blocks = table_blocks(g, descs[r.p0], std::min(waves_per_cu, r.waves_per_cu),
                                          std::max<int64_t>(1, r.n_roots));
            if (b.nbuf > 0)
                r.table_blocks = std::max<int64_t>(
                    1, std::min(r.table_blocks, (int64_t(16) << 30) / (r.tab_waves * b.nbuf * b.cap * 4)));
            slots = std::max(slots, run_group_slots(r, true));
        }
        r.blocks = r.table ? r.table_blocks : r.plain_blocks;
    }
    b.memo_words = b.use_memo ? slots * (int64_t)g.n_hubs : 0;
    // room for the IEP memo's most ways when an eligible IEP plan runs alone
    for (const BatchRun& r : b.runs)
        for (int p = r.p0; p < r.p1 && b.use_memo; ++p)
            if (r.solo && descs[p].iep && iep_memo_eligible(descs[p])) {
                const int l = iep_memo_log2(g.n_hubs, kIepMemoBytes / 8);
                if (l >= 0) b.memo_words = std::max(b.memo_words, (int64_t)g.n_hubs << l);
            }
    if (device_malloc((void**)&b.queues, kQueueBytes * np) != hipSuccess ||
        device_malloc((void**)&b.result, 4 * sizeof(unsigned long long) * np) != hipSuccess ||
        (b.nbuf > 0 && device_malloc((void**)&b.scratch, (size_t)(slots * b.nbuf * b.cap * 4)) != hipSuccess) ||
        (b.memo_words > 0 && device_malloc((void**)&b.memo, (size_t)b.memo_words * 8) != hipSuccess))
        rc = GP_ERR_NOMEM;
    if (rc == GP_OK && hipStreamSynchronize(stream) != hipSuccess) rc = GP_ERR_HIP;
    if (rc != GP_OK) {
        batch_release(&b);
        return rc;
    }
    *st = b;
    return GP_OK;
}

gp_status batch_update(const DeviceGraph& g, BatchState* st, const GpPlanDesc* descs, const LaunchCfg* cfgs,
                       hipStream_t stream) {
    BatchState b = *st;
    std::vector<BatchPlan> plans;
    gp_status rc = batch_layout(g, descs, cfgs, nullptr, nullptr, st->np, 8, &b, &plans);
    if (rc != GP_OK) return rc;
    bool same = b.nbuf == st->nbuf && b.use_memo == st->use_memo && b.runs.size() == st->runs.size();
    for (size_t i = 0; same && i < b.runs.size(); ++i)
        same = b.runs[i].p0 == st->runs[i].p0 && b.runs[i].p1 == st->runs[i].p1 &&
               b.runs[i].group == st->runs[i].group && b.runs[i].leaf == st->runs[i].leaf &&
               b.runs[i].iep == st->runs[i].iep && b.runs[i].may_table == st->runs[i].may_table;
    if (!same) return GP_ERR_ARG;  // the shapes the buffers were carved for must not change
    (void)stream;
    // launches take their task ranges as kernel arguments: the caller
    // enqueues (or captures) the batch again
    for (size_t i = 0; i < b.runs.size(); ++i) {
        BatchRun& r = b.runs[i];
        r.table_blocks = st->runs[i].table_blocks;  // the carved grids
        r.plain_blocks = st->runs[i].plain_blocks;
        r.blocks = r.table ? r.table_blocks : r.plain_blocks;
    }
    st->runs = b.runs;
    st->h_plans = b.h_plans;
    return GP_OK;
}

gp_status describe_batch(const BatchState& st, int plan, gp_shape* out) {
    for (const BatchRun& r : st.runs) {
        if (plan < r.p0 || plan >= r.p1) continue;
        const BatchPlan& bp = reinterpret_cast<const BatchPlan*>(st.h_plans.data())[plan];
        const bool iep = st.h_descs[plan].iep != 0;
        out->table = r.table ? 1 : 0;
        out->memo = st.memo_words > 0 && (iep ? iep_memo_eligible(st.h_descs[plan]) : bp.tag_base != 0) ? 1 : 0;
        out->group = r.table ? 64 : r.group;
        out->chunk = r.table ? table_chunk(st.h_descs[plan], r.blocks, r.n_roots) : bp.chunk;
        out->blocks = (int32_t)r.blocks;
        out->threads = r.table ? r.tab_waves * 64 : kBlock;
        return GP_OK;
    }
    return GP_ERR_ARG;
}

gp_status batch_enqueue(const DeviceGraph& g, const BatchState& st, hipStream_t stream) {
    if (st.runs.empty()) return GP_ERR_ARG;
    for (const BatchRun& r : st.runs)
        if (!pick_batch_kernel(r.kmin, r.kmax, r.group, r.leaf, r.iep) || r.blocks < 1) return GP_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(zero_u64, dim3((unsigned)(st.np * (kQueueWords / 256))), dim3(256), 0, stream, st.queues,
                       (int64_t)st.np * kQueueWords);
    if (st.memo_words > 0)
        hipLaunchKernelGGL(zero_u64, dim3((unsigned)std::min<int64_t>(4096, (st.memo_words + 255) / 256)), dim3(256),
                           0, stream, st.memo, st.memo_words);
    // one persistent launch per run of same-shape plans, in batch order. The
    // runs share the scratch and memo regions: launches on one stream never
    // overlap, and memo tags are disjoint per plan.
    for (size_t ri = 0; ri < st.runs.size(); ++ri) {
        const BatchRun& r = st.runs[ri];
        if (r.solo) {
            // the plain counting kernel over the plan's whole task space
            const int p = r.p0;
            const GpPlanDesc& d = st.h_descs[p];
            KernelFn fn = r.table ? pick_table(d, MODE_PLAIN, r.tab_waves) : pick_kernel(d.k, r.group, r.leaf, MODE_PLAIN, d.iep);
            if (!fn) return GP_ERR_UNSUPPORTED;
            const int32_t chunk = r.table ? table_chunk(d, r.blocks, r.n_roots) : r.chunk;
            CountArgs a;
            a.row_ptr = g.row_ptr;
            a.col = g.col;
            a.roots = r.roots;
            a.n_roots = r.n_roots;
            a.n_tasks = r.n_tasks;
            a.n_chunks = ((r.table ? r.n_roots : r.n_tasks) + chunk - 1) / chunk;
            a.tab_n = (int32_t)std::min<int64_t>(g.n, table_max(r.tab_waves));
            a.whole_chunk = chunk;
            a.split_roots = r.split_roots;
            a.split_ways = r.split_ways;
            a.budget_ticks = 0;
            a.root_offset = r.root_offset;
            a.hub_bits = g.hub_bits;
            a.hub_words = g.hub_words;
            a.n_hubs = g.n_hubs;
            a.root_stride = r.root_stride;
            a.scratch = st.scratch;
            a.buf_cap = st.cap;
            a.queue = st.queues + (int64_t)p * kQueueWords;
            a.result = st.result + 4 * p;
            a.per_root = nullptr;
            a.busy = nullptr;
            // the IEP memo holds sizes fixed by the graph, valid in every
            // launch: the region needs no clearing between runs
            const int iep_log2 = d.iep && iep_memo_eligible(d) && st.memo_words > 0
                                     ? iep_memo_log2(g.n_hubs, std::min(st.memo_words, kIepMemoBytes / 8))
                                     : -1;
            a.memo = iep_log2 >= 0 ? st.memo : nullptr;
            a.memo_ways_log2 = std::max(iep_log2, 0);
            a.chunk = chunk;
            a.xcd_block = 0;
            if (r.n_tasks > 0)
                hipLaunchKernelGGL(fn, dim3((unsigned)r.blocks), dim3(r.table ? r.tab_waves * 64 : kBlock), 0, stream, d, a);
            continue;
        }
        BatchArgs a;
        a.row_ptr = g.row_ptr;
        a.col = g.col;
        a.np = r.p1 - r.p0;
        a.hub_bits = g.hub_bits;
        a.hub_words = g.hub_words;
        a.n_hubs = g.n_hubs;
        a.scratch = st.scratch;
        a.buf_cap = st.cap;
        a.nbuf = st.nbuf;
        a.slots_per_wave = 64 / r.group;
        a.memo = st.memo_words > 0 ? st.memo : nullptr;
        a.iep_memo_log2 = r.iep && st.memo_words > 0
                              ? iep_memo_log2(g.n_hubs, std::min(st.memo_words, kIepMemoBytes / 8))
                              : -1;
        a.queues = st.queues + (int64_t)r.p0 * kQueueWords;
        RunDescs rd;
        std::memset(&rd, 0, sizeof rd);
        for (int p = r.p0; p < r.p1; ++p) {
            rd.d[p - r.p0] = st.h_descs[p];
            rd.bp[p - r.p0] = reinterpret_cast<const BatchPlan*>(st.h_plans.data())[p];
        }
        hipLaunchKernelGGL(pick_batch_kernel(r.kmin, r.kmax, r.group, r.leaf, r.iep), dim3((unsigned)r.blocks), dim3(kBlock),
                           0, stream, a, rd);
    }
    hipLaunchKernelGGL(collect_batch, dim3((unsigned)st.np), dim3(64), 0, stream, st.queues, st.result);
    return hipGetLastError() == hipSuccess ? GP_OK : GP_ERR_HIP;
}

gp_status arena_create(const DeviceGraph& g, int nbuf_cap, int waves_per_cu, int min_group, BatchArena* ar) {
    BatchArena a;
    a.waves_per_cu = waves_per_cu;
    BatchState& b = a.st;
    b.cap = std::max<int64_t>(1, g.deg2);
    a.min_group = min_group >= 64 ? 64 : (min_group >= 32 ? 32 : (min_group >= 16 ? 16 : 8));
    a.nbuf_cap = std::max(0, std::min(nbuf_cap, GP_DESC_MAX_BUILDS));
    // room for the smallest group width and for the memo of leaf-4 plans
    a.blocks_cap = batch_blocks(g, waves_per_cu, 64 / a.min_group, a.nbuf_cap, b.cap, true);
    a.slots_cap = a.blocks_cap * (kBlock / 64) * (64 / a.min_group);
    a.memo_words_cap = g.n_hubs > 0 ? a.slots_cap * (int64_t)g.n_hubs : 0;
    bool ok = device_malloc((void**)&b.queues, kQueueBytes * kBatchMaxPlans) == hipSuccess &&
              device_malloc((void**)&b.result, 4 * sizeof(unsigned long long) * kBatchMaxPlans) == hipSuccess &&
              (a.nbuf_cap == 0 ||
               device_malloc((void**)&b.scratch, (size_t)(a.slots_cap * a.nbuf_cap * b.cap * 4)) == hipSuccess) &&
              (a.memo_words_cap == 0 || device_malloc((void**)&b.memo, (size_t)a.memo_words_cap * 8) == hipSuccess) &&
              hipHostMalloc((void**)&a.h_result, 4 * sizeof(unsigned long long) * kBatchMaxPlans,
                            hipHostMallocDefault) == hipSuccess;
    if (!ok) {
        arena_release(&a);
        return GP_ERR_NOMEM;
    }
    *ar = a;
    return GP_OK;
}

gp_status arena_launch(const DeviceGraph& g, BatchArena* ar, const GpPlanDesc* descs, const LaunchCfg* cfgs,
                       const int64_t* offsets, const int64_t* counts, int np, hipStream_t stream) {
    if (np < 1 || np > kBatchMaxPlans) return GP_ERR_ARG;
    BatchState& b = ar->st;
    std::vector<BatchPlan> plans;
    gp_status rc = batch_layout(g, descs, cfgs, offsets, counts, np, ar->min_group, &b, &plans);
    if (rc != GP_OK) return rc;
    if (b.nbuf > ar->nbuf_cap) return GP_ERR_NOMEM;
    // each run within the regions carved at creation: group slots x nbuf
    // buffers of scratch, group slots x n_hubs memo words
    int64_t room = b.nbuf > 0 ? ar->slots_cap * ar->nbuf_cap / b.nbuf : ar->slots_cap;
    if (b.use_memo) room = std::min(room, ar->slots_cap);
    int64_t slots = 0;
    for (BatchRun& r : b.runs) {
        r.table = r.table && room >= r.tab_waves;  // else no block's buffers fit
        const int64_t per_block = r.table ? r.tab_waves : (kBlock / 64) * (64 / r.group);
        r.blocks = r.table ? table_blocks(g, descs[r.p0], std::min(ar->waves_per_cu, r.waves_per_cu),
                                          std::max<int64_t>(1, r.n_roots))
                           : batch_blocks(g, std::min(ar->waves_per_cu, r.waves_per_cu), 64 / r.group, b.nbuf, b.cap,
                                          b.use_memo);
        r.blocks = std::max<int64_t>(1, std::min(r.blocks, room / per_block));
        slots = std::max(slots, r.blocks * per_block);
    }
    b.memo_words = b.use_memo ? slots * (int64_t)g.n_hubs : 0;
    if (b.memo_words > ar->memo_words_cap) {
        // no room for every wave's table: run the leaf-4 plans without the memo
        for (auto& bp : plans) bp.tag_base = 0;
        b.memo_words = 0;
    }
    store_plans(&b, plans);
    rc = batch_enqueue(g, b, stream);
    if (rc != GP_OK) return rc;
    GP_HIP_TRY(hipMemcpyAsync(ar->h_result, b.result, 4 * sizeof(unsigned long long) * np, hipMemcpyDeviceToHost,
                              stream));
    return GP_OK;
}

gp_status batch_result(const GpPlanDesc& d, const unsigned long long* r, uint64_t* out, bool whole) {
    unsigned __int128 t = ((unsigned __int128)r[3] << 64) | (unsigned __int128)r[0];
    const uint64_t div = d.iep ? (uint64_t)d.iep_div : 1;
    if (div > 1) {
        // a whole count is a multiple of the over-count; a sample's need not be
        if (whole && t % div) return GP_ERR_INTERNAL;
        t /= div;
    }
    if (t >> 64) return GP_ERR_OVERFLOW;
    *out = (uint64_t)t;
    return GP_OK;
}

void arena_release(BatchArena* ar) {
    batch_release(&ar->st);
    if (ar->h_result) (void)hipHostFree(ar->h_result);
    *ar = BatchArena{};
}

}  // namespace gpint
