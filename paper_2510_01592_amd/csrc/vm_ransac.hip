// vm_ransac.hip -- cluster-parallel RANSAC (Sec. III-C, "Multi-plane
// estimation"): (a) hypotheses from three sampled points, (b) inlier
// counting, (c) selection of the best hypothesis and extraction of its inliers.
//
// All clusters are processed together.  Work is cut into tiles of a fixed
// number of points inside one cluster (the tile list is built on the device
// from the cluster offsets), so thousands of clusters of very different sizes
// load-balance across the 256 CUs without the host knowing any size.
//
// Inlier counting is the arithmetic hot spot (sum over clusters of n_k x H
// point-plane tests).  It runs on the matrix cores: a wave keeps 64 or 128
// planes in registers and sweeps points (PlaneGroups in vm_dev.h); three K = 1
// fp32 matrix steps give the specified fma chain bit for bit.  Counts are
// integers added with atomics, hence independent of the order of tiles.
// (6.7M clustered points x 1024 hypotheses: 0.65 ms, 10.6 T tests/s, from 0.95
// ms with ballots over points in registers and planes in scalar registers;
// clusters of at most 256 points, 11k of them x 512: 14 us, from 24.)
#include "vm_common.h"
#include "vm_dev.h"

#include <mutex>

#include <math.h>

namespace vm {
namespace {

using namespace dev;

constexpr int kCountBlock = 256;
constexpr int kInlierBlock = 512;   // of k_inlier_count
constexpr int kPtsPerLane = 16;
constexpr int kTile = (int)kPointTile;             // points per tile
constexpr uint32_t kXcds = 8;                      // accelerator complex dies (separate L2s)

// (a) hypothesis (k, h): three distinct points -> unit normal (+z first) and
// offset in fp64, rounded to float32.  Degenerate triples get a NaN plane.
__global__ void __launch_bounds__(kBlock) k_hypotheses(const uint32_t* __restrict__ small,
                                                       const uint32_t* __restrict__ off,
                                                       const uint32_t* __restrict__ tag, const float* __restrict__ X,
                                                       const float* __restrict__ Y, const float* __restrict__ Z,
                                                       uint32_t H, uint64_t seed, uint32_t frame_arg,
                                                       const uint32_t* __restrict__ d_frame,
                                                       const uint32_t* __restrict__ cframe,
                                                       const uint32_t* __restrict__ tile_off,
                                                       uint32_t* __restrict__ tile_k,
                                                       const uint32_t* __restrict__ tile_off_big,
                                                       uint32_t* __restrict__ tile_k_big, uint32_t wave_max,
                                                       int32_t* __restrict__ counts, float4* __restrict__ hyp)
{
    const uint32_t frame_all = d_frame ? *d_frame : frame_arg;
    const uint32_t K = small[0];
    const uint64_t total = (uint64_t)K * H;
    for (uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (uint64_t)gridDim.x * blockDim.x) {
        // (32-bit division where the index fits: the 64-bit one is a long
        // instruction sequence per hypothesis)
        uint32_t k, h;
        if (total <= 0xFFFFFFFFull) {
            k = (uint32_t)idx / H;
            h = (uint32_t)idx - k * H;
        } else {
            k = (uint32_t)(idx / H);
            h = (uint32_t)(idx % H);
        }
        const uint32_t base = off[k];
        const uint64_t n = (uint64_t)(off[k + 1] - base);
        // the cluster of each of its point tiles, for the inlier kernels and
        // (clusters beyond one wave's points) for the tiled counting kernel
        const uint32_t nt = (uint32_t)((n + kTile - 1) / kTile);
        for (uint32_t q = h; q < nt; q += H) tile_k[tile_off[k] + q] = k;
        if (n > wave_max)
            for (uint32_t q = h; q < nt; q += H) tile_k_big[tile_off_big[k] + q] = k;
        const uint32_t frame = cframe ? cframe[k] : frame_all;   // a merged set's clusters carry their own
        const float4 pl = hyp_plane(X + base, Y + base, Z + base, n, h, tag[k], frame, seed);
        // the tiled kernel adds into the counts; the wave kernel stores every
        // count of its clusters, and clusters of fewer than 3 points have no
        // valid hypothesis (their counts are never read)
        if (n > wave_max) counts[idx] = 0;
        hyp[idx] = pl;
    }
}

// the clusters this pass processes (small[0] = K, 0 if the CSR is invalid)
__global__ void __launch_bounds__(kBlock) k_validate(const uint32_t* __restrict__ meta, uint32_t k_cap,
                                                     uint32_t out_k_cap, uint32_t n_cap,
                                                     const uint32_t* __restrict__ off, uint32_t* __restrict__ small,
                                                     uint32_t* __restrict__ status)
{
    __shared__ int bad;
    const uint32_t K = validate_clusters(meta, off, k_cap, n_cap, status, &bad);
    if (threadIdx.x == 0) {
        small[0] = K;
        if (meta[0] > out_k_cap) atomicOr(status, (uint32_t)VM_FLAG_CLUSTERS_CAP);
    }
}

// validate, tiles per cluster and both tile-offset scans in one workgroup
// (the capacity is at most kOneBlockMax clusters)
__global__ void __launch_bounds__(kOneBlockThreads) k_prepare(const uint32_t* __restrict__ meta, uint32_t k_cap,
                                                              uint32_t out_k_cap, uint32_t n_cap,
                                                              const uint32_t* __restrict__ off,
                                                              uint32_t* __restrict__ small,
                                                              uint32_t* __restrict__ tile_off,
                                                              uint32_t* __restrict__ tile_off_big, uint32_t wave_max,
                                                              uint32_t* __restrict__ status)
{
    __shared__ int bad;
    const uint32_t K = validate_clusters(meta, off, k_cap, n_cap, status, &bad);
    uint32_t total[2];
    one_block_scan<kOneBlockThreads, 4, 2>(
        K,
        [&](uint32_t k, uint32_t(&v)[2]) {
            const uint32_t n = off[k + 1] - off[k];
            v[0] = (n + kTile - 1) / kTile;
            v[1] = n > wave_max ? v[0] : 0u;   // counted by the tiled kernel
        },
        [&](uint32_t k, const uint32_t(&e)[2]) {
            tile_off[k] = e[0];
            tile_off_big[k] = e[1];
        },
        total);
    if (threadIdx.x == 0) {
        small[0] = K;
        small[1] = total[0];
        small[3] = total[1];
        if (meta[0] > out_k_cap) atomicOr(status, (uint32_t)VM_FLAG_CLUSTERS_CAP);
    }
}

// tiles per cluster (for the device-built tile list)
__global__ void __launch_bounds__(kBlock) k_tiles(const uint32_t* __restrict__ small,
                                                  const uint32_t* __restrict__ off, uint32_t* __restrict__ ntiles,
                                                  uint32_t* __restrict__ ntiles_big, uint32_t wave_max)
{
    const uint32_t K = small[0];
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x) {
        const uint32_t n = off[k + 1] - off[k];
        ntiles[k] = (n + kTile - 1) / kTile;
        ntiles_big[k] = n > wave_max ? (n + kTile - 1) / kTile : 0u;   // counted by the tiled kernel
    }
}

// (b) inlier counting.  The rows form, for clusters that vm_count_config gives
// to one wave with its lanes over points: a wave evaluates only the rows of 64
// points that hold points of its cluster.
template <int R>
__device__ __forceinline__ uint32_t count_rows(const float4 pl, const float* px, const float* py, const float* pz,
                                               float eps)
{
    uint32_t acc = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const float dd = fmaf(pl.z, pz[j], fmaf(pl.y, py[j], fmaf(pl.x, px[j], pl.w)));
        acc += (uint32_t)__popcll(__ballot(fabsf(dd) < eps));
    }
    return acc;
}

// All planes of a cluster that one wave holds: the counts are final, stored.
// With few points per lane the work per plane is short, so the planes of a
// 64-plane batch are fetched with one vector load (lane q loads plane
// hb + q) and broadcast lane by lane, instead of one scalar load per few
// planes whose latency the short work cannot hide.
template <int R>
__device__ __forceinline__ void count_all(const float4* __restrict__ hk, uint32_t h0, uint32_t h1, const float* px,
                                          const float* py, const float* pz, float eps, int32_t* __restrict__ ck,
                                          int lane)
{
    for (uint32_t hb = h0; hb < h1; hb += kWave) {
        const uint32_t nb = min(h1 - hb, (uint32_t)kWave);
        const float4 mine = (uint32_t)lane < nb ? hk[hb + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
        int cv = 0;
        for (uint32_t b = 0; b < nb; ++b) {
            float4 pl;
            pl.x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine.x), (int)b));
            pl.y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine.y), (int)b));
            pl.z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine.z), (int)b));
            pl.w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine.w), (int)b));
            if (pl.x != pl.x) continue;   // degenerate hypothesis
            const uint32_t acc = count_rows<R>(pl, px, py, pz, eps);
            cv = (lane == (int)b) ? (int)acc : cv;
        }
        if ((uint32_t)lane < nb) ck[hb + (uint32_t)lane] = cv;
    }
}

// Clusters of at most a few rows of points: the wave's lanes hold 64 G planes
// at a time against all the points (PlaneGroups).
template <int G, bool kFloat>
__device__ __forceinline__ void count_by_planes(const float4* __restrict__ hk, uint32_t h0, uint32_t h1, uint32_t n,
                                                const float* __restrict__ X, const float* __restrict__ Y,
                                                const float* __restrict__ Z, const EpsTest& eps,
                                                int32_t* __restrict__ ck, int lane)
{
    for (uint32_t hb = h0; hb < h1; hb += G * kWave) {
        PlaneGroups<G> pg;
        pg.load(hk, hb, h1, lane);
        pg.template sweep<kFloat>(X, Y, Z, n, eps, lane);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t h = hb + (uint32_t)(g * kWave + lane);
            const uint32_t c = pg.count(g, lane);
            if (h < h1) ck[h] = (int32_t)c;
        }
    }
}

// Clusters of at most wave_max points (at most 1024: one wave's registers)
// are counted by waves without LDS or workgroup barriers, a wave per
// (cluster, chunk of hypotheses) item: the counts of a chunk are final.  The
// hypotheses are split into chunks (multiples of 64) only as far as needed
// for about chunk_mult items per wave, so few clusters still fill the chip.
// Larger clusters go through the tiled kernel below.  Clusters of at most
// plane_max points (at most 256) put the lanes over planes.
constexpr uint32_t kWaveMaxPts = kWave * kPtsPerLane;   // 1024
constexpr uint32_t kPlaneMaxPts = 4 * kWave;            // 256

template <bool kFloat>
__global__ void __launch_bounds__(kCountBlock, 4) k_count_small(const uint32_t* __restrict__ small,
                                                             const uint32_t* __restrict__ off,
                                                             const float* __restrict__ X, const float* __restrict__ Y,
                                                             const float* __restrict__ Z, uint32_t H, EpsTest eps,
                                                             const float4* __restrict__ hyp,
                                                             int32_t* __restrict__ counts, uint32_t wave_max,
                                                             uint32_t plane_max, uint32_t chunk_mult)
{
    const uint32_t K = small[0];
    if (K == 0) return;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t waves = gridDim.x * (kCountBlock / kWave);
    const float qnan = __builtin_nanf("");
    // chunks of cb 64-plane batches, HC chunks per cluster
    const uint32_t nb64 = (H + kWave - 1) / kWave;
    uint32_t HC = (uint32_t)min((uint64_t)nb64, ((uint64_t)chunk_mult * waves + K - 1) / K);
    if (HC < 1) HC = 1;
    const uint32_t cb = (nb64 + HC - 1) / HC;
    HC = (nb64 + cb - 1) / cb;
    const uint64_t items = (uint64_t)K * HC;
    // the wave's item index, made explicitly wave-uniform so that its loads
    // (offsets, points, planes' addresses) are scalar
    const uint32_t w0 = __builtin_amdgcn_readfirstlane(blockIdx.x * (kCountBlock / kWave) + threadIdx.x / kWave);
    for (uint64_t item = w0; item < items; item += waves) {
        const uint32_t k = (uint32_t)(item / HC), hc = (uint32_t)(item % HC);
        const uint32_t h0 = hc * cb * kWave, h1 = min(H, h0 + cb * kWave);
        const uint32_t base = off[k], n = off[k + 1] - base;
        if (n < 3 || n > wave_max) continue;   // fewer than 3: no planes; more: the tiled kernel
        const float4* hk = hyp + (size_t)k * H;
        int32_t* ck = counts + (size_t)k * H;
        if (n <= plane_max) {
            count_by_planes<2, kFloat>(hk, h0, h1, n, X + base, Y + base, Z + base, eps, ck, lane);
            continue;
        }
        const int rows = (int)((n + kWave - 1) / kWave);
        float px[kPtsPerLane], py[kPtsPerLane], pz[kPtsPerLane];
#pragma unroll
        for (int j = 0; j < kPtsPerLane; ++j) {
            const uint32_t i = (uint32_t)(j * kWave + lane);
            const bool v = i < n;
            px[j] = v ? X[base + i] : qnan;   // NaN never passes |d| < eps
            py[j] = v ? Y[base + i] : qnan;
            pz[j] = v ? Z[base + i] : qnan;
        }
        if (rows > 8) count_all<16>(hk, h0, h1, px, py, pz, eps.eps, ck, lane);
        else if (rows > 4) count_all<8>(hk, h0, h1, px, py, pz, eps.eps, ck, lane);
        else if (rows > 2) count_all<4>(hk, h0, h1, px, py, pz, eps.eps, ck, lane);
        else if (rows > 1) count_all<2>(hk, h0, h1, px, py, pz, eps.eps, ck, lane);
        else count_all<1>(hk, h0, h1, px, py, pz, eps.eps, ck, lane);
    }
}

// Larger clusters: an item is a slice of a 4096-point tile against a chunk of
// hypotheses, 64 G per wave, so each wave holds its planes in registers and
// sweeps the slice's points (PlaneGroups).  A tile is cut into slices (down to
// 256 points) until there are about chunk_mult items per resident workgroup:
// the frame's few hundred tiles alone would leave most of the chip idle.
constexpr uint32_t kMaxSlices = 16;          // slices of a tile (256 points each)
constexpr uint32_t kCountResident = 1280;    // workgroups of this kernel on the chip at once

// (the bound of four workgroups per compute unit also keeps the matrix results
// out of the accumulation registers, each of which would cost a move to read)
template <int G, bool kFloat>
__global__ void __launch_bounds__(kCountBlock, 4) k_count(const uint32_t* __restrict__ small,
                                                       const uint32_t* __restrict__ tile_off, const uint32_t* __restrict__ tile_k,
                                                       const uint32_t* __restrict__ off, const float* __restrict__ X,
                                                       const float* __restrict__ Y, const float* __restrict__ Z,
                                                       uint32_t H, EpsTest eps, const float4* __restrict__ hyp,
                                                       int32_t* __restrict__ counts, uint32_t chunk_mult)
{
    const uint32_t T = small[3];   // tiles of the clusters beyond one wave
    if (T == 0) return;
    constexpr uint32_t kChunk = (uint32_t)(G * kCountBlock);
    const uint32_t HC = (H + kChunk - 1) / kChunk;
    uint32_t S = 1;
    while (S < kMaxSlices && (uint64_t)T * HC * S < (uint64_t)chunk_mult * kCountResident) S <<= 1;
    const uint32_t slice = kTile / S;
    // Workgroups are dispatched round-robin over the XCDs, each with its own
    // L2: tile t is handled on XCD t mod kXcds only, so the items of a tile
    // (run at about the same time) fetch its points from memory once.
    const uint32_t xcd = blockIdx.x % kXcds, sub = blockIdx.x / kXcds, nsub = gridDim.x / kXcds;
    const uint32_t tiles_x = T > xcd ? (T - xcd + kXcds - 1) / kXcds : 0u;
    const uint64_t items = (uint64_t)tiles_x * HC * S;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (uint64_t item = sub; item < items; item += nsub) {
        const uint32_t t = (uint32_t)(item / (HC * S)) * kXcds + xcd, q = (uint32_t)(item % (HC * S));
        const uint32_t hc = q / S, sl = q % S;
        const uint32_t k = tile_k[t];
        const uint32_t p0 = off[k] + (t - tile_off[k]) * kTile + sl * slice;
        const uint32_t pend = off[k + 1];
        const uint32_t h0 = hc * kChunk + wave * (uint32_t)(G * kWave);
        if (p0 >= pend || h0 >= H) continue;   // wave-uniform; no barriers below
        PlaneGroups<G> pg;
        pg.load(hyp + (size_t)k * H, h0, H, lane);
        pg.template sweep<kFloat>(X + p0, Y + p0, Z + p0, min(slice, pend - p0), eps, lane);
        int32_t* ck = counts + (size_t)k * H;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t h = h0 + (uint32_t)(g * kWave + lane);
            const uint32_t c = pg.count(g, lane);
            if (h < H && c) atomicAdd(&ck[h], (int32_t)c);
        }
    }
}

// (c) best hypothesis per cluster: largest count, first index on ties
__global__ void __launch_bounds__(kBlock) k_select(const uint32_t* __restrict__ small, uint32_t H,
                                                   const int32_t* __restrict__ counts, const float4* __restrict__ hyp,
                                                   float4* __restrict__ plane_out, int32_t* __restrict__ best_out,
                                                   int32_t* __restrict__ nin_out, int32_t* __restrict__ counts_out,
                                                   float4* __restrict__ hyp_out)
{
    constexpr uint32_t kAhead = 4;
    const uint32_t K = small[0];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t waves = gridDim.x * (blockDim.x / kWave);
    for (uint32_t k = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; k < K; k += waves) {
        const float4* hk = hyp + (size_t)k * H;
        const int32_t* ck = counts + (size_t)k * H;
        int32_t bc = -1;
        uint32_t bh = 0xFFFFFFFFu;
        float4 bp = make_float4(0.f, 0.f, 0.f, 0.f);
        // kAhead rounds' reads are in flight together, and the best plane is
        // kept, not read again (one round after another, 512 hypotheses took
        // a frame's clusters 7.7 us, 4.7 so; 1024 took 13 us and 6.6)
        for (uint32_t h0 = lane; h0 < H; h0 += kAhead * kWave) {
            float4 pl[kAhead];
            int32_t c[kAhead];
#pragma unroll
            for (uint32_t j = 0; j < kAhead; ++j) {
                const uint32_t h = min(h0 + j * kWave, H - 1u);
                pl[j] = hk[h];
                c[j] = ck[h];
            }
#pragma unroll
            for (uint32_t j = 0; j < kAhead; ++j) {
                const uint32_t h = h0 + j * kWave;
                if (h >= H) break;
                const bool degen = pl[j].x != pl[j].x;
                if (degen) {
                    c[j] = -1;
                    pl[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
                if (c[j] > bc) {
                    bc = c[j];
                    bh = h;
                    bp = pl[j];
                }
                if (counts_out) counts_out[(size_t)k * H + h] = c[j];
                if (hyp_out) hyp_out[(size_t)k * H + h] = pl[j];
            }
        }
        const uint32_t own = bh;
#pragma unroll
        for (int d = kWave / 2; d >= 1; d >>= 1) {
            const int32_t oc = __shfl_xor(bc, d, kWave);
            const uint32_t oh = __shfl_xor(bh, d, kWave);
            if (oc > bc || (oc == bc && oh < bh)) { bc = oc; bh = oh; }
        }
        // the lane that found it, or without one any (its plane is zero then)
        if (bc < 0 ? lane == 0 : own == bh) {
            best_out[k] = bc < 0 ? -1 : (int32_t)bh;
            nin_out[k] = bc < 0 ? 0 : bc;
            plane_out[k] = bp;
        }
    }
}

// the same from a row of counts per point tile, a workgroup per cluster: a
// cluster's count is the sum of its tiles' rows
__global__ void __launch_bounds__(kBlock) k_select_rows(const uint32_t* __restrict__ small,
                                                        const uint32_t* __restrict__ off,
                                                        const uint32_t* __restrict__ tile_off, uint32_t H,
                                                        const int32_t* __restrict__ rows, const float4* __restrict__ hyp,
                                                        float4* __restrict__ plane_out, int32_t* __restrict__ best_out,
                                                        int32_t* __restrict__ nin_out, int32_t* __restrict__ counts_out,
                                                        float4* __restrict__ hyp_out)
{
    __shared__ int32_t sc[kBlock / kWave];
    __shared__ uint32_t sh[kBlock / kWave];
    const uint32_t K = small[0];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (uint32_t k = blockIdx.x; k < K; k += gridDim.x) {
        const uint32_t nt = (off[k + 1] - off[k] + kTile - 1) / kTile;
        const int32_t* row = rows + (size_t)tile_off[k] * H;
        int32_t bc = -1;
        uint32_t bh = 0xFFFFFFFFu;
        for (uint32_t h = threadIdx.x; h < H; h += kBlock) {
            const float4 pl = hyp[(size_t)k * H + h];
            const bool degen = pl.x != pl.x;
            int32_t c = 0;
#pragma unroll 8
            for (uint32_t t = 0; t < nt; ++t) c += row[(size_t)t * H + h];
            if (degen) c = -1;
            if (c > bc) { bc = c; bh = h; }
            if (counts_out) counts_out[(size_t)k * H + h] = c;
            if (hyp_out) hyp_out[(size_t)k * H + h] = degen ? make_float4(0.f, 0.f, 0.f, 0.f) : pl;
        }
#pragma unroll
        for (int d = kWave / 2; d >= 1; d >>= 1) {
            const int32_t oc = __shfl_xor(bc, d, kWave);
            const uint32_t oh = __shfl_xor(bh, d, kWave);
            if (oc > bc || (oc == bc && oh < bh)) { bc = oc; bh = oh; }
        }
        if (lane == 0) {
            sc[wave] = bc;
            sh[wave] = bh;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kBlock / kWave; ++w)
                if (sc[w] > bc || (sc[w] == bc && sh[w] < bh)) { bc = sc[w]; bh = sh[w]; }
            best_out[k] = bc < 0 ? -1 : (int32_t)bh;
            nin_out[k] = bc < 0 ? 0 : bc;
            plane_out[k] = bc < 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : hyp[(size_t)k * H + bh];
        }
        __syncthreads();   // sc and sh are reused by the next cluster
    }
}

// (c) the inlier lists of the winning planes, over the same point tiles, in
// three launches: the inliers of each tile, as a bit mask and their number;
// one workgroup's scan of the tile counts (which also gives each cluster's
// list offset); the lists, written from the masks.  The first reads every
// point (bound by that: 118 us for the 48M points of 2000 clusters, 4.9 TB/s),
// the last reads a bit per point and consecutive lanes write consecutive
// places (testing the points again, with a thread writing out 32 points in
// turn, took 364 us there, this 46 us).  512 threads leave a thread eight
// points in the first (81 tiles: 4.9 us, 6.5 us with 256; clusters of a few
// points: 5.2 us, 8.6 us with 1024); the last has little to wait for (2000
// clusters: 46 us with 256, 55 with 512).
// the mask words of tile t, whose first point is p0: tiles start at distinct
// words that do not overlap, whatever their sizes (a tile of n points needs
// n / 32 rounded up, at most one more than the quotient)
__device__ __forceinline__ uint32_t* tile_mask(uint32_t* mask, uint32_t p0, uint32_t t)
{
    return mask + (p0 / 32 + t);
}

__global__ void __launch_bounds__(kInlierBlock) k_inlier_count(const uint32_t* __restrict__ small,
                                                              const uint32_t* __restrict__ tile_off,
                                                              const uint32_t* __restrict__ tile_k,
                                                              const uint32_t* __restrict__ off,
                                                              const float* __restrict__ X, const float* __restrict__ Y,
                                                              const float* __restrict__ Z, float eps,
                                                              const int32_t* __restrict__ best,
                                                              const float4* __restrict__ plane,
                                                              uint32_t* __restrict__ mask,
                                                              uint32_t* __restrict__ tile_cnt)
{
    __shared__ uint32_t wsum[kInlierBlock / kWave];
    const uint32_t T = small[1];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (uint32_t t = blockIdx.x; t < T; t += gridDim.x) {
        const uint32_t k = tile_k[t];
        const uint32_t p0 = off[k] + (t - tile_off[k]) * kTile;
        const uint32_t n = min(kTile, off[k + 1] - p0);
        uint32_t c = 0;
        if (best[k] >= 0) {
            const float4 pl = plane[k];
            uint32_t* m = tile_mask(mask, p0, t);
#pragma unroll 4
            for (uint32_t j0 = wave * kWave; j0 < n; j0 += kInlierBlock) {
                const uint32_t j = j0 + (uint32_t)lane, i = p0 + min(j, n - 1u);
                const bool in = j < n && inlier_test(pl, X[i], Y[i], Z[i], eps);
                const uint64_t b = __ballot(in);
                c += (uint32_t)__popcll(b);
                if (lane < 2 && j0 + 32 * lane < n) m[j0 / 32 + lane] = lane ? (uint32_t)(b >> 32) : (uint32_t)b;
            }
        }
        if (lane == 0) wsum[wave] = c;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
#pragma unroll
            for (int w = 0; w < kInlierBlock / kWave; ++w) tot += wsum[w];
            tile_cnt[t] = tot;
        }
        __syncthreads();   // wsum is reused by the next tile
    }
}

__global__ void __launch_bounds__(kOneBlockThreads) k_inlier_scan(uint32_t* __restrict__ small,
                                                                  const uint32_t* __restrict__ tile_off,
                                                                  uint32_t* __restrict__ tile_cnt,
                                                                  uint32_t* __restrict__ in_off)
{
    const uint32_t K = small[0], T = small[1];
    uint32_t total[1];
    one_block_scan<kOneBlockThreads, 4, 1>(
        T, [&](uint32_t t, uint32_t(&v)[1]) { v[0] = tile_cnt[t]; },
        [&](uint32_t t, const uint32_t(&e)[1]) { tile_cnt[t] = e[0]; }, total);
    __syncthreads();   // the prefixes other threads wrote
    // a cluster's list starts at the prefix of its first tile (a cluster
    // without points has no tile: the next cluster's start, or the total)
    for (uint32_t k = threadIdx.x; k <= K; k += blockDim.x)
        in_off[k] = (k < K && tile_off[k] < T) ? tile_cnt[tile_off[k]] : total[0];
    if (threadIdx.x == 0) small[2] = total[0];
}

__global__ void __launch_bounds__(kCountBlock) k_inlier_write(const uint32_t* __restrict__ small,
                                                              const uint32_t* __restrict__ tile_off,
                                                              const uint32_t* __restrict__ tile_k,
                                                              const uint32_t* __restrict__ off,
                                                              const int32_t* __restrict__ best,
                                                              uint32_t* __restrict__ mask,
                                                              const uint32_t* __restrict__ tile_pre, uint32_t in_cap,
                                                              uint32_t* __restrict__ in_idx, uint32_t* __restrict__ status)
{
    // a point's place: the tile's prefix, the inliers in the mask words before
    // its own, and those below it in the word
    constexpr uint32_t kWords = kTile / 32;   // 128
    static_assert(kWords == 2 * kWave && kWords <= kCountBlock, "two waves scan the words");
    __shared__ uint32_t sm[kWords], pre[kWords];
    __shared__ uint32_t half;
    const uint32_t T = small[1];
    const int lane = threadIdx.x & (kWave - 1);
    bool over = false;
    for (uint32_t t = blockIdx.x; t < T; t += gridDim.x) {
        const uint32_t k = tile_k[t];
        if (best[k] < 0) continue;   // workgroup-uniform
        const uint32_t base = off[k];
        const uint32_t p0 = base + (t - tile_off[k]) * kTile;
        const uint32_t n = min(kTile, off[k + 1] - p0);
        if (threadIdx.x < kWords) {
            const uint32_t m = threadIdx.x * 32 < n ? tile_mask(mask, p0, t)[threadIdx.x] : 0u;
            const uint32_t c = (uint32_t)__popc(m);
            uint32_t inc = c;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t o = __shfl_up(inc, d, kWave);
                if (lane >= d) inc += o;
            }
            sm[threadIdx.x] = m;
            pre[threadIdx.x] = inc - c;
            if (threadIdx.x == kWave - 1) half = inc;
        }
        __syncthreads();
        const uint32_t first = tile_pre[t];
#pragma unroll 4
        for (uint32_t j = threadIdx.x; j < n; j += kCountBlock) {
            const uint32_t w = j / 32, m = sm[w], bit = 1u << (j & 31);
            if (!(m & bit)) continue;
            const uint32_t p = first + pre[w] + (w >= (uint32_t)kWave ? half : 0u) + (uint32_t)__popc(m & (bit - 1u));
            if (p < in_cap) in_idx[p] = p0 - base + j;
            else over = true;
        }
        __syncthreads();   // the words are reused by the next tile
    }
    if (over) atomicOr(status, (uint32_t)VM_FLAG_INLIERS_CAP);
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

WorkLayout work_layout(void* base, uint32_t k_cap, uint32_t n_cap, uint32_t n_hyp)
{
    WorkLayout w{};
    w.k_cap = k_cap;
    char* p = (char*)base;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char* r = p ? p + o : nullptr;
        o += align256(bytes);
        return r;
    };
    const size_t kh = (size_t)k_cap * (size_t)n_hyp;
    w.counts = (int32_t*)take(kh * sizeof(int32_t));
    w.hyp = (float4*)take(kh * sizeof(float4));
    w.tile_off = (uint32_t*)take(((size_t)k_cap + 2) * sizeof(uint32_t));
    w.tile_k = (uint32_t*)take(((size_t)n_cap / kTile + k_cap + 2) * sizeof(uint32_t));
    w.tile_off_big = (uint32_t*)take(((size_t)k_cap + 2) * sizeof(uint32_t));
    w.tile_k_big = (uint32_t*)take(((size_t)n_cap / kTile + k_cap + 2) * sizeof(uint32_t));
    w.flags = (uint32_t*)take(((size_t)n_cap + 1) * sizeof(uint32_t));
    const size_t blk_words = scan_blk_words((uint64_t)n_cap + k_cap + 2) + 64;
    w.blk = (uint32_t*)take(blk_words * sizeof(uint32_t));
    w.hull_cnt = (uint32_t*)take(((size_t)k_cap + 2) * sizeof(uint32_t));
    w.hull_off = (uint32_t*)take(((size_t)k_cap + 2) * sizeof(uint32_t));
    w.hull_tmp = (uint32_t*)take(((size_t)n_cap + k_cap + 2) * sizeof(uint32_t));
    w.hull_u = (double*)take(((size_t)n_cap + 1) * sizeof(double));
    w.hull_v = (double*)take(((size_t)n_cap + 1) * sizeof(double));
    w.hull_i = (uint32_t*)take(((size_t)n_cap + 1) * sizeof(uint32_t));
    w.hull_tile_off = (uint32_t*)take(((size_t)k_cap + 2) * sizeof(uint32_t));
    // The size decides which buffers and which calls of the allocation-free form
    // are accepted, so it stays what it was while the tiles' extremes (96 bytes
    // per hull tile; they share hull_u and hull_v now), 18 doubles of a filter
    // polygon (now its margin) and a list of clusters lay here.
    const size_t ht = hull_tiles_bound(k_cap, n_cap);
    (void)take(ht * 64);
    (void)take(ht * 32);
    w.margin = (double*)take((size_t)k_cap * 18 * sizeof(double) + 8);
    w.surv_cnt = (uint32_t*)take(((size_t)k_cap + 1) * sizeof(uint32_t));
    (void)take(((size_t)k_cap + 1) * sizeof(uint32_t));
    w.small = (uint32_t*)take(64 * sizeof(uint32_t));
    w.bytes = o;
    return w;
}

namespace {
std::mutex g_count_mu;
vm_count_config g_count_cfg = count_config_default();
}   // namespace

vm_count_config count_config_default()
{
    vm_count_config c;
    c.count_grid = 16384;
    c.chunk_mult = 2;
    c.wave_max_points = kPlaneMaxPts;   // larger clusters: the tiled kernel splits their hypotheses
    c.plane_max_points = kPlaneMaxPts;
    return c;
}

bool count_config_valid(const vm_count_config& c)
{
    if (c.count_grid < kXcds || c.count_grid > 65536 || c.count_grid % kXcds != 0) return false;
    if (c.chunk_mult < 1 || c.chunk_mult > 16) return false;
    if (c.wave_max_points > kWaveMaxPts) return false;
    return c.plane_max_points <= kPlaneMaxPts && c.plane_max_points <= c.wave_max_points;
}

vm_count_config count_config_get()
{
    std::lock_guard<std::mutex> g(g_count_mu);
    return g_count_cfg;
}

void count_config_set(const vm_count_config& c)
{
    std::lock_guard<std::mutex> g(g_count_mu);
    g_count_cfg = c;
}

hipError_t launch_hypotheses(const vm_clusters& cl, const vm_ransac_params& p, const WorkLayout& w, uint32_t kc,
                             uint32_t wave_max, const uint32_t* d_cframe, hipStream_t s)
{
    const uint64_t kh = (uint64_t)kc * p.n_hyp;
    k_hypotheses<<<grid_for(kh, kBlock, 16384), kBlock, 0, s>>>(w.small, cl.d_off, cl.d_tag, cl.d_x, cl.d_y, cl.d_z,
                                                                p.n_hyp, p.seed, p.frame, p.d_frame, d_cframe,
                                                                w.tile_off, w.tile_k, w.tile_off_big, w.tile_k_big,
                                                                wave_max, w.counts, w.hyp);
    return hipGetLastError();
}

vm_status select_and_list(const vm_clusters& cl, const vm_ransac_params& p, const vm_planes& out, const WorkLayout& w,
                          uint32_t kc, bool tile_rows, hipStream_t s)
{
    const uint32_t H = p.n_hyp;
    StageScope t(VM_STAGE_SELECT, s);
    if (tile_rows)
        k_select_rows<<<grid_for(kc, 1, 8192), kBlock, 0, s>>>(w.small, cl.d_off, w.tile_off, H, w.counts, w.hyp,
                                                               (float4*)out.d_plane, out.d_best_h, out.d_n_inliers,
                                                               out.d_counts, (float4*)out.d_hyp);
    else
        k_select<<<grid_for((uint64_t)kc * kWave), kBlock, 0, s>>>(w.small, H, w.counts, w.hyp, (float4*)out.d_plane,
                                                                   out.d_best_h, out.d_n_inliers, out.d_counts,
                                                                   (float4*)out.d_hyp);
    const int tgrid = grid_for((uint64_t)cl.n_cap / kTile + kc + 1, 1, 8192);   // most tiles are small: many workgroups
    // w.flags holds the per-tile counts, then their prefixes (tiles <= points);
    // the mask takes at most n_cap / 32 + tiles + 1 words of what the polygons
    // use later (2 n_cap + 2 words, tiles <= points)
    uint32_t* mask = (uint32_t*)w.hull_u;
    k_inlier_count<<<tgrid, kInlierBlock, 0, s>>>(w.small, w.tile_off, w.tile_k, cl.d_off, cl.d_x, cl.d_y, cl.d_z,
                                                p.eps, out.d_best_h, (const float4*)out.d_plane, mask, w.flags);
    k_inlier_scan<<<1, kOneBlockThreads, 0, s>>>(w.small, w.tile_off, w.flags, out.d_in_off);
    k_inlier_write<<<tgrid, kCountBlock, 0, s>>>(w.small, w.tile_off, w.tile_k, cl.d_off, out.d_best_h, mask, w.flags,
                                                out.in_cap, out.d_in_idx, out.d_status);
    VM_HIP(hipGetLastError());
    return VM_OK;
}

vm_status ransac_planes(const vm_clusters& cl, const vm_ransac_params& p, const vm_planes& out,
                        const WorkLayout& w, hipStream_t s, const uint32_t* d_cframe)
{
    // the workspace is laid out for kc = min(cl.k_cap, out.k_cap) clusters
    const uint32_t kc = cl.k_cap < out.k_cap ? cl.k_cap : out.k_cap;
    if (kc > w.k_cap) return VM_E_STATE;
    const uint32_t H = p.n_hyp;
    const vm_count_config cc = count_config_get();
    // small[0] = K (clamped), small[1] = tiles, small[2] = inliers, small[3] = tiles of clusters beyond one wave
    {
        StageScope t(VM_STAGE_HYPOTHESES, s);
        if (kc <= kOneBlockMax) {
            k_prepare<<<1, kOneBlockThreads, 0, s>>>(cl.d_meta, kc, out.k_cap, cl.n_cap, cl.d_off, w.small, w.tile_off,
                                                     w.tile_off_big, cc.wave_max_points, out.d_status);
        } else {
            k_validate<<<1, kBlock, 0, s>>>(cl.d_meta, kc, out.k_cap, cl.n_cap, cl.d_off, w.small, out.d_status);
            k_tiles<<<grid_for(kc), kBlock, 0, s>>>(w.small, cl.d_off, w.tile_off, w.tile_off_big,
                                                    cc.wave_max_points);
            VM_HIP(scan_exclusive_dev(w.tile_off, w.tile_off, w.small, kc, w.small + 1, w.blk, s));
            VM_HIP(scan_exclusive_dev(w.tile_off_big, w.tile_off_big, w.small, kc, w.small + 3, w.blk, s));
        }
        VM_HIP(launch_hypotheses(cl, p, w, kc, cc.wave_max_points, d_cframe, s));
    }
    {
        StageScope t(VM_STAGE_COUNT, s);
        const EpsTest et = eps_test(p.eps);
        const bool flt = p.eps >= kMinFloatEps;
        if (cc.wave_max_points >= 3) {
            const int grid = grid_for((uint64_t)kc * ((H + kWave - 1) / kWave) * kWave, kCountBlock, 1024);
            auto count_small = [&](auto kernel) {
                kernel<<<grid, kCountBlock, 0, s>>>(w.small, cl.d_off, cl.d_x, cl.d_y, cl.d_z, H, et, w.hyp, w.counts,
                                                    cc.wave_max_points, cc.plane_max_points, cc.chunk_mult);
            };
            if (flt) count_small(k_count_small<true>);
            else count_small(k_count_small<false>);
        }
        auto count = [&](auto kernel) {
            kernel<<<cc.count_grid, kCountBlock, 0, s>>>(w.small, w.tile_off_big, w.tile_k_big, cl.d_off, cl.d_x,
                                                         cl.d_y, cl.d_z, H, et, w.hyp, w.counts, cc.chunk_mult);
        };
        // two plane groups per wave need fewer point reads per test, one
        // fills four waves with up to 256 hypotheses
        if (!flt) count(k_count<1, false>);
        else if (H > (uint32_t)kCountBlock) count(k_count<2, true>);
        else count(k_count<1, true>);
        VM_HIP(hipGetLastError());
    }
    return select_and_list(cl, p, out, w, kc, false, s);
}

}  // namespace vm
