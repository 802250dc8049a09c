// vm_fused.hip -- RANSAC planes and boundary polygons of a whole cluster set
// with its inlier counting in one persistent launch (Sec. III-C "Multi-plane
// estimation" (a)-(c) and "Boundary polygon generation", run cluster-parallel
// as in the paper's pipeline, with thousands of clusters of very uneven size).
//
// A one-workgroup preparation sorts the clusters by cost (point count,
// largest first) and lays out a device work queue of items: one per
// (4096-point tile, chunk of hypotheses), or, for a cluster of at most
// small_max points, one for all its hypotheses.  A grid-wide pass draws and
// fits every hypothesis plane.  The persistent workgroups then take items
// from the queue with one atomic each (no workgroup ever waits for another),
// then those of the smallest clusters in turn;
// each wave keeps up to 128 of the item's planes in registers, sweeps the
// tile's points on the matrix cores (PlaneGroups) and stores its integer
// counts in the tile's own row, so the sums do not depend on the order.
// Selection sums a cluster's rows; the inlier lists and the polygons are made
// by the tiled passes of vm_ransac_planes and vm_hulls, which spread a
// 200k-point cluster over the chip.  (Built by the workgroup that completed
// the cluster, inside the persistent kernel, they took it a few milliseconds
// for such a cluster, serial chains of dependent gathers, and the device-scope
// release and acquire that hand over a cluster's counts write back and
// invalidate an XCD's L2 for every other workgroup: counting 48M points x 1024
// hypotheses took 6.6-8.2 ms that way and takes 4.2 ms as a kernel of its
// own.)  Results are bit-identical to vm_ransac_planes followed by vm_hulls.
#include "vm_common.h"
#include "vm_dev.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

namespace vm {
namespace {

using namespace dev;

constexpr int kFBlock = 256;                         // threads of the counting kernel
constexpr uint32_t kFTile = kPointTile;              // points per tile item
constexpr int kFGroups = 2;                          // groups of 64 planes per wave at most
constexpr uint32_t kFMaxChunk = kFGroups * kFBlock;  // hypotheses per item (512)
constexpr uint32_t kFSmallMax = 256;                 // most points of a cluster with one item
constexpr int kBuckets = 33;                         // cost classes: floor(log2(points)) + 1

// Clusters of fewer points are not queued: their items, the last in cost order,
// go to the workgroups in turn.  The queue's head takes an atomic every 12 ns,
// which is all that 60000 clusters of at most 11 points waited for (700 us for
// their counting, 162 so); items this small need no balance.
constexpr uint32_t kFQueueMin = 256;
constexpr int kFQueueClass = kBuckets - 1 - 8;   // the last class of queued clusters
static_assert(kFQueueMin == 1u << 8, "a class boundary");

// device scalars of the queue, beside those of the shared passes
constexpr int kQueueItems = 16, kQueueHead = 17, kAllItems = 18;

struct FusedWork {
    WorkLayout w;          // the shared passes'; its counts hold the tiles' rows, [tiles][H]
    uint32_t* order;       // [k_cap] clusters by cost, largest first
    uint32_t* item_off;    // [k_cap + 1] first queue item of order[i]
    size_t bytes;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The passes' arrays without those that only more than kOneBlockMax clusters or
// the tiled counting kernel use; a tile's cluster is not needed any more when
// the survivors' positions come to lie there (a tile has at least one point).
// (The size is what callers may have a buffer of: no more than it was with the
// results of the persistent pass in these places.)
FusedWork fused_layout(void* base, uint32_t k_cap, uint32_t n_cap, uint32_t H)
{
    FusedWork f{};
    WorkLayout& w = f.w;
    w.k_cap = k_cap;
    char* p = (char*)base;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char* r = p ? p + o : nullptr;
        o += align256(bytes);
        return r;
    };
    const size_t rows = (size_t)n_cap / kFTile + (size_t)k_cap + 1;
    const size_t kb = ((size_t)k_cap + 1) * 4, nb = ((size_t)n_cap + 1) * 4;
    w.counts = (int32_t*)take(rows * H * sizeof(int32_t));
    w.hyp = (float4*)take((size_t)k_cap * H * sizeof(float4));
    f.order = (uint32_t*)take(kb);
    f.item_off = (uint32_t*)take(kb);
    w.tile_off = (uint32_t*)take(kb);
    w.hull_tile_off = (uint32_t*)take(kb);
    w.hull_cnt = (uint32_t*)take(kb);
    w.surv_cnt = (uint32_t*)take(kb);
    w.margin = (double*)take(kb);   // and the next kb bytes
    (void)take(kb);
    w.flags = (uint32_t*)take(nb);
    w.hull_tmp = (uint32_t*)take(nb + kb);
    w.hull_u = (double*)take(2 * nb);
    w.hull_v = (double*)take(2 * nb);
    w.hull_i = (uint32_t*)take(nb);
    w.tile_k = w.hull_i;
    w.small = (uint32_t*)take(64 * 4);
    f.bytes = o;
    return f;
}

// the work split of the counting kernel (vm_fused_config)
struct Split {
    uint32_t H, chunk, nch, small_max;
};

__device__ __forceinline__ bool is_small(uint32_t n, const Split& s) { return n <= s.small_max; }

// queue items of a cluster of n points
__device__ __forceinline__ uint32_t items_of(uint32_t n, const Split& s)
{
    if (n == 0) return 0;
    return is_small(n, s) ? 1u : (n + kFTile - 1) / kFTile * s.nch;
}

// ---- preparation: validate, cost order, queue and tile layout (one workgroup) ----
__global__ void __launch_bounds__(kOneBlockThreads) k_fused_prepare(const uint32_t* __restrict__ meta, uint32_t k_cap,
                                                                    uint32_t out_k_cap, uint32_t n_cap,
                                                                    const uint32_t* __restrict__ off, Split sp,
                                                                    FusedWork f, uint32_t* __restrict__ status)
{
    __shared__ int bad;
    __shared__ uint32_t bucket[kBuckets + 1];
    const uint32_t K = validate_clusters(meta, off, k_cap, n_cap, status, &bad);
    for (int b = threadIdx.x; b <= kBuckets; b += blockDim.x) bucket[b] = 0;
    __syncthreads();
    // cost class of each cluster (largest first), counted per class
    auto cls = [&](uint32_t n) -> uint32_t { return n ? (uint32_t)(kBuckets - 1 - (31 - __clz(n))) : (uint32_t)kBuckets - 1; };
    for (uint32_t k = threadIdx.x; k < K; k += blockDim.x) atomicAdd(&bucket[cls(off[k + 1] - off[k]) + 1], 1u);
    __syncthreads();
    if (threadIdx.x == 0)
        for (int b = 1; b <= kBuckets; ++b) bucket[b] += bucket[b - 1];   // class starts
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < K; k += blockDim.x) f.order[atomicAdd(&bucket[cls(off[k + 1] - off[k])], 1u)] = k;
    __syncthreads();
    // queue offsets in cost order, tiles in cluster order
    uint32_t tot[1];
    one_block_scan<kOneBlockThreads, 4, 1>(
        K, [&](uint32_t i, uint32_t(&v)[1]) { v[0] = items_of(off[f.order[i] + 1] - off[f.order[i]], sp); },
        [&](uint32_t i, const uint32_t(&e)[1]) { f.item_off[i] = e[0]; }, tot);
    __syncthreads();
    uint32_t tiles[1];
    one_block_scan<kOneBlockThreads, 4, 1>(
        K, [&](uint32_t k, uint32_t(&v)[1]) { v[0] = (off[k + 1] - off[k] + kFTile - 1) / kFTile; },
        [&](uint32_t k, const uint32_t(&e)[1]) { f.w.tile_off[k] = e[0]; }, tiles);
    if (threadIdx.x == 0) {
        f.w.small[0] = K;
        f.w.small[1] = tiles[0];
        f.w.small[3] = 0;
        // (a class' start has moved to its end: the queued clusters' number)
        const uint32_t queued = bucket[kFQueueClass];
        f.w.small[kQueueItems] = queued < K ? f.item_off[queued] : tot[0];
        f.w.small[kAllItems] = tot[0];
        f.w.small[kQueueHead] = 0;
        f.item_off[K] = tot[0];
        if (meta[0] > out_k_cap) atomicOr(status, (uint32_t)VM_FLAG_CLUSTERS_CAP);
    }
}

// ---- the persistent counting kernel ------------------------------------------------
struct FusedArgs {
    const uint32_t* off;
    const float* X;
    const float* Y;
    const float* Z;
    EpsTest eps;
    Split sp;
    FusedWork f;
};

// (the bound of four workgroups per compute unit also keeps the matrix results
// out of the accumulation registers, each of which would cost a move to read)
template <int G, bool kFloat>
__global__ void __launch_bounds__(kFBlock, 4) k_fused(FusedArgs a)
{
    __shared__ uint32_t s_item;
    const FusedWork& f = a.f;
    const Split& sp = a.sp;
    const uint32_t H = sp.H;
    const uint32_t K = f.w.small[0], queued = f.w.small[kQueueItems], total = f.w.small[kAllItems];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t own = queued + blockIdx.x;   // the next item in turn
    for (bool queue = queued != 0;;) {
        uint32_t item = own;
        if (queue) {
            if (threadIdx.x == 0) s_item = atomicAdd(&f.w.small[kQueueHead], 1u);
            __syncthreads();
            item = __builtin_amdgcn_readfirstlane(s_item);
            __syncthreads();   // s_item is rewritten for the next item
            queue = item < queued;   // (workgroup-uniform)
            if (!queue) item = own;
        }
        if (!queue) {
            if (item >= total) break;   // workgroup-uniform: every wave leaves
            own += gridDim.x;
        }
        // the queue position holding the item
        const uint32_t i = __builtin_amdgcn_readfirstlane(last_at_or_below(f.item_off, K, item));
        const uint32_t k = f.order[i], j = item - f.item_off[i];
        const uint32_t base = a.off[k], n = a.off[k + 1] - base;
        const bool small = is_small(n, sp);
        const uint32_t c0 = small ? 0u : j % sp.nch, c1 = small ? sp.nch : c0 + 1, t = small ? 0u : j / sp.nch;
        int32_t* part = f.w.counts + (size_t)(f.w.tile_off[k] + t) * H;
        const float4* hk = f.w.hyp + (size_t)k * H;
        const uint32_t p0 = base + t * kFTile, np = min(kFTile, n - t * kFTile);
        for (uint32_t c = c0; c < c1; ++c) {
            // wave w takes planes [64 G w, 64 G (w + 1)) of the chunk against
            // all points of the tile (the four waves' reads of a row share its
            // cache lines); a wave past the chunk's end has none
            const uint32_t h1 = min(H, (c + 1) * sp.chunk), hw = c * sp.chunk + wave * (uint32_t)(G * kWave);
            if (hw >= h1) continue;
            PlaneGroups<G> pg;
            pg.load(hk, hw, h1, lane);
            pg.template sweep<kFloat>(a.X + p0, a.Y + p0, a.Z + p0, np, a.eps, lane);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const uint32_t h = hw + (uint32_t)(g * kWave + lane);
                const uint32_t v = pg.count(g, lane);
                if (h < h1) part[h] = (int32_t)v;
            }
        }
    }
}

// ---- the work split: process-wide setting and per-shape autotuned choices ------
std::mutex g_fused_mu;
vm_fused_config g_fused_cfg = {512, 0, 5, 0};   // fused_config_default()
std::map<std::tuple<uint32_t, uint32_t, uint32_t>, vm_fused_config> g_fused_cache;

std::tuple<uint32_t, uint32_t, uint32_t> shape_bucket(uint32_t k_cap, uint32_t n_cap, uint32_t H)
{
    auto lg = [](uint32_t x) { uint32_t r = 0; while (x > 1) { x >>= 1; ++r; } return r; };
    return {lg(k_cap), lg(n_cap), lg(H)};
}

}  // namespace

bool fused_config_valid(const vm_fused_config& c)
{
    return c.hyp_chunk >= 64 && c.hyp_chunk <= kFMaxChunk && c.hyp_chunk % 64 == 0 && c.small_max <= kFSmallMax &&
           c.groups_per_cu >= 1 && c.groups_per_cu <= 8 && c.reserved == 0;
}

vm_fused_config fused_config_default() { return vm_fused_config{512, 0, 5, 0}; }

vm_fused_config fused_config_get()
{
    std::lock_guard<std::mutex> g(g_fused_mu);
    return g_fused_cfg;
}

void fused_config_set(const vm_fused_config& c)
{
    std::lock_guard<std::mutex> g(g_fused_mu);
    g_fused_cfg = c;
}

void fused_cache_put(uint32_t k_cap, uint32_t n_cap, uint32_t H, const vm_fused_config& c)
{
    std::lock_guard<std::mutex> g(g_fused_mu);
    g_fused_cache[shape_bucket(k_cap, n_cap, H)] = c;
}

bool fused_cache_get(uint32_t k_cap, uint32_t n_cap, uint32_t H, vm_fused_config* c)
{
    std::lock_guard<std::mutex> g(g_fused_mu);
    auto it = g_fused_cache.find(shape_bucket(k_cap, n_cap, H));
    if (it == g_fused_cache.end()) return false;
    *c = it->second;
    return true;
}

void fused_cache_clear()
{
    std::lock_guard<std::mutex> g(g_fused_mu);
    g_fused_cache.clear();
}

size_t fused_workspace_bytes(uint32_t k_cap, uint32_t n_cap, uint32_t H)
{
    return fused_layout(nullptr, k_cap, n_cap, H).bytes;
}

namespace {

Split make_split(uint32_t H, const vm_fused_config& cfg)
{
    Split sp;
    sp.H = H;
    sp.chunk = std::min<uint32_t>(cfg.hyp_chunk, ((H + kWave - 1) / kWave) * kWave);
    sp.nch = (H + sp.chunk - 1) / sp.chunk;
    sp.small_max = cfg.small_max;
    return sp;
}

int device_cus()
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
    }
    return cus;
}

}  // namespace

vm_status planes_and_hulls(const vm_clusters& cl, const vm_ransac_params& p, const uint32_t* d_cframe,
                           const vm_planes& planes_in, const vm_hulls_out& hulls_in, void* d_work, size_t work_bytes,
                           const vm_fused_config& cfg, hipStream_t s)
{
    // both outputs take the clusters that the smaller of them holds
    vm_planes planes = planes_in;
    vm_hulls_out hull_out = hulls_in;
    planes.k_cap = hull_out.k_cap = std::min(planes_in.k_cap, hulls_in.k_cap);
    const uint32_t kc = std::min(cl.k_cap, planes.k_cap);
    if (kc > kOneBlockMax) return VM_E_CAPACITY;
    const uint32_t H = p.n_hyp;
    const FusedWork f = fused_layout(d_work, kc, cl.n_cap, H);
    if (f.bytes > work_bytes) return VM_E_CAPACITY;
    const Split sp = make_split(H, cfg);
    {
        StageScope t(VM_STAGE_HYPOTHESES, s);
        k_fused_prepare<<<1, kOneBlockThreads, 0, s>>>(cl.d_meta, kc, planes.k_cap, cl.n_cap, cl.d_off, sp, f,
                                                       planes.d_status);
        VM_HIP(hipGetLastError());
        // no cluster is left to the tiled counting kernel of the two-pass form
        VM_HIP(launch_hypotheses(cl, p, f.w, kc, 0xFFFFFFFFu, d_cframe, s));
    }
    {
        StageScope t(VM_STAGE_COUNT, s);
        FusedArgs a;
        a.off = cl.d_off;
        a.X = cl.d_x;
        a.Y = cl.d_y;
        a.Z = cl.d_z;
        a.eps = eps_test(p.eps);
        a.sp = sp;
        a.f = f;
        const int grid = device_cus() * (int)cfg.groups_per_cu;
        // one plane group per wave fills the four waves with chunks up to 256
        if (p.eps < kMinFloatEps) k_fused<kFGroups, false><<<grid, kFBlock, 0, s>>>(a);
        else if (sp.chunk > (uint32_t)kFBlock) k_fused<kFGroups, true><<<grid, kFBlock, 0, s>>>(a);
        else k_fused<1, true><<<grid, kFBlock, 0, s>>>(a);
        VM_HIP(hipGetLastError());
    }
    vm_status st = select_and_list(cl, p, planes, f.w, kc, true, s);
    if (st != VM_OK) return st;
    return hulls(cl, planes, hull_out, f.w, s);
}

}  // namespace vm
