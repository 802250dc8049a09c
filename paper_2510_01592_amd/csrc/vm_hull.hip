// vm_hull.hip -- boundary polygons (Sec. III-C, "Boundary polygon
// generation"): the convex hull of each plane's inliers, in the plane.
//
// The paper filters most points on the GPU and finishes each hull on the CPU
// from the few candidates left.  Here the whole hull stays on the device and
// every pass over the inliers is tile-parallel, so one huge cluster (a floor)
// spreads over the whole chip instead of one workgroup:
//   B. per tile of inliers: project onto the in-plane basis (fp64) and find an
//      extreme inlier in each of 64 directions, a lane per direction;
//   C. per cluster: combine the tiles' extremes; the convex polygon through
//      them lies inside the hull, so a point strictly inside it (by a margin
//      far above the fp64 rounding of the test) cannot be a hull vertex;
//   D. per tile: keep only the points not strictly inside that polygon
//      (block-aggregated compaction into the cluster's own region);
//   E. per cluster: sort the survivors by (u, v, inlier index) -- in a
//      wave's registers for at most 64, by a workgroup in LDS up to kLdsCap, in
//      global memory beyond -- and find both chains of the hull (strictly
//      convex, counter-clockwise from the smallest point);
//   F. scan the vertex counts and pack the polygons, each vertex projected
//      onto the plane.
// The stage is bound by latency, not by bytes: nine launches with serial
// chains in between took 130-280 us on the frames measured (an octagon filter
// that left hundreds to thousands of survivors on a ray-cast floor, thinned by
// one workgroup; one lane pruning each polygon; one lane per chain popping
// point after point); with the 64-gon found by all tiles and the polygon and
// the chains found by whole waves, six launches take 36-75 us.
#include "vm_common.h"
#include "vm_dev.h"

#include <math.h>

namespace vm {
namespace {

using namespace dev;

constexpr int kTileThreads = 256;
constexpr int kTileItems = 4;
constexpr int kHullTile = kTileThreads * kTileItems;   // inliers per tile
constexpr int kDirs = 64;          // support directions of the filter polygon, a lane each
constexpr double kMargin = 4e-9;   // of the extent's square: the margin of the polygon's corners and of the filter
constexpr int kTileGrid = 16384;   // workgroups of the tile kernels, at most
constexpr int kPolyGrid = 2048;    // workgroups of the polygon kernel
constexpr int kFinishGrid = 512;   // workgroups of the hull kernel: two per compute unit (76 KB of LDS)
constexpr int kLdsCap = 2048;      // survivors sorted in LDS
static_assert(kDirs == kWave, "a lane per direction");

// Whether cluster k gets a polygon: it has a plane, its inlier list fits the
// output and indexes its own points.
__device__ __forceinline__ bool cluster_ok(uint32_t k, const uint32_t* off, const int32_t* best,
                                           const uint32_t* in_off, const uint32_t* in_idx, uint32_t in_cap)
{
    const uint32_t ib = in_off[k], ie = in_off[k + 1];
    if (best[k] < 0 || ie <= ib || ie > in_cap) return false;
    return in_idx[ib] < off[k + 1] - off[k];
}

__device__ __forceinline__ ClusterFrame cluster_frame(uint32_t k, const uint32_t* off, const float* X, const float* Y,
                                                      const float* Z, const float4* plane, const uint32_t* in_off,
                                                      const uint32_t* in_idx)
{
    ClusterFrame f;
    f.ib = in_off[k];
    f.m = in_off[k + 1] - f.ib;
    f.pb = off[k];
    f.nk = off[k + 1] - f.pb;
    f.B = plane_basis(plane[k]);
    const uint32_t i0 = f.pb + in_idx[f.ib];
    f.ox = X[i0];
    f.oy = Y[i0];
    f.oz = Z[i0];
    return f;
}

// tiles of cluster k: [tile_off[k], end)
__device__ __forceinline__ uint32_t tiles_end(const uint32_t* tile_off, uint32_t k, uint32_t K, uint32_t total)
{
    return k + 1 < K ? tile_off[k + 1] : total;
}

// ---- A: validate, tiles per cluster ------------------------------------------
__global__ void __launch_bounds__(kBlock) k_hull_validate(const uint32_t* __restrict__ meta, uint32_t kc,
                                                          uint32_t n_cap, const uint32_t* __restrict__ off,
                                                          uint32_t* small, uint32_t* status)
{
    __shared__ int bad;
    const uint32_t K = validate_clusters(meta, off, kc, n_cap, status, &bad);
    if (threadIdx.x == 0) {
        small[4] = K;
    }
}

__global__ void __launch_bounds__(kBlock) k_hull_tiles(const uint32_t* __restrict__ small,
                                                       const uint32_t* __restrict__ off,
                                                       const int32_t* __restrict__ best,
                                                       const uint32_t* __restrict__ in_off,
                                                       const uint32_t* __restrict__ in_idx, uint32_t in_cap,
                                                       uint32_t* __restrict__ ntiles, uint32_t* __restrict__ status)
{
    const uint32_t K = small[4];
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x) {
        const bool ok = cluster_ok(k, off, best, in_off, in_idx, in_cap);
        const uint32_t m = ok ? in_off[k + 1] - in_off[k] : 0u;
        // clusters with at most one wave of inliers skip the tiled filter
        ntiles[k] = m > (uint32_t)kWave ? (m + kHullTile - 1) / kHullTile : 0u;
        if (best[k] >= 0 && in_off[k + 1] > in_cap) atomicOr(status, (uint32_t)VM_FLAG_INLIERS_CAP);
    }
}

// validate, tiles per cluster and their offsets in one workgroup (the
// capacity is at most kOneBlockMax clusters)
__global__ void __launch_bounds__(kOneBlockThreads) k_hull_prepare(
    const uint32_t* __restrict__ meta, uint32_t kc, uint32_t n_cap, const uint32_t* __restrict__ off,
    const int32_t* __restrict__ best, const uint32_t* __restrict__ in_off, const uint32_t* __restrict__ in_idx,
    uint32_t in_cap, uint32_t* __restrict__ small, uint32_t* __restrict__ tile_off, uint32_t* __restrict__ status)
{
    __shared__ int bad;
    const uint32_t K = validate_clusters(meta, off, kc, n_cap, status, &bad);
    uint32_t total[1];
    one_block_scan<kOneBlockThreads, 4, 1>(
        K,
        [&](uint32_t k, uint32_t(&v)[1]) {
            const bool ok = cluster_ok(k, off, best, in_off, in_idx, in_cap);
            const uint32_t m = ok ? in_off[k + 1] - in_off[k] : 0u;
            v[0] = m > (uint32_t)kWave ? (m + kHullTile - 1) / kHullTile : 0u;
            if (best[k] >= 0 && in_off[k + 1] > in_cap) atomicOr(status, (uint32_t)VM_FLAG_INLIERS_CAP);
        },
        [&](uint32_t k, const uint32_t(&e)[1]) { tile_off[k] = e[0]; }, total);
    if (threadIdx.x == 0) {
        small[4] = K;
        small[6] = total[0];
    }
}

// ---- B: projection + directional extremes per tile --------------------------------
// The polygon that the extremes give may be through any inliers (it only has to
// lie inside the hull), so the extremes are compared in fp32, with a point's
// number in the value's lowest bits: one instruction makes the key,
// half of one keeps the largest.  The points are projected in fp64 and rounded
// then: an fp32 projection errs by the whole distance from the first inlier,
// which along the normal may be any multiple of the cluster's width.  (An
// eighth of the coordinates is compared, so that none of them overflows: an
// extreme lost would let the polygon say nothing about the cluster's extent.)  Opposite directions share the product, and
// a lane has four directions (q, q + 16 and their opposites) for a quarter of
// its wave's points: a point per lane and direction took 64 LDS reads per
// wave and 5 instructions each and was bound by both (526 us for the 34M
// inliers of 2000 clusters, 249 us so, 220 with the projection in fp32; the
// bytes take about 130).  A tile's 64
// extremes (value, position in the inlier list) go to ext_v / ext_i.
__device__ __forceinline__ float key_of(float v, uint32_t pos, uint32_t mask)
{
    return __uint_as_float((__float_as_uint(v) & ~mask) | pos);
}

// largest / smallest of three, a NaN loses (the compiler's own form quiets
// every operand first)
__device__ __forceinline__ float max3f(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__device__ __forceinline__ float min3f(float a, float b, float c)
{
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__global__ void __launch_bounds__(kTileThreads) k_hull_extremes(
    const uint32_t* __restrict__ small, const uint32_t* __restrict__ tile_off, const uint32_t* __restrict__ off,
    const float* __restrict__ X, const float* __restrict__ Y, const float* __restrict__ Z,
    const float4* __restrict__ plane, const uint32_t* __restrict__ in_off, const uint32_t* __restrict__ in_idx,
    float* __restrict__ ext_v, uint32_t* __restrict__ ext_i)
{
    constexpr int kWaves = kTileThreads / kWave;
    constexpr int kQuarter = kHullTile / kWaves;       // points of a wave
    constexpr int kGroups = 4;                         // lane groups that share them, two points at a time
    constexpr int kStep = 2 * kGroups;
    constexpr uint32_t kPosMask = kQuarter / kGroups - 1;
    static_assert(kDirs == 4 * (kWave / kGroups) && (kPosMask & (kPosMask + 1)) == 0, "four directions per lane");
    __shared__ __align__(16) float2 uv[kHullTile];
    __shared__ float rv[kWaves * kGroups][kDirs];
    __shared__ uint32_t ri[kWaves * kGroups][kDirs];
    const uint32_t K = small[4];
    const uint32_t T = small[6];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int dir = lane & (kDirs / 4 - 1), grp = lane / (kDirs / 4);
    float sn, cs;
    sincospif((float)dir / (kDirs / 2), &sn, &cs);
    for (uint32_t t = blockIdx.x; t < T; t += gridDim.x) {
        const uint32_t k = last_at_or_below(tile_off, K, t);
        const ClusterFrame f = cluster_frame(k, off, X, Y, Z, plane, in_off, in_idx);
        const uint32_t j0 = (t - tile_off[k]) * kHullTile, m = min((uint32_t)kHullTile, f.m - j0);
        // a wave projects and then searches its own quarter of the tile; what
        // is not a point of the cluster is NaN and never an extreme
        const int q0 = wave * kQuarter;
        uint32_t li[kQuarter / kWave];
#pragma unroll
        for (int it = 0; it < kQuarter / kWave; ++it) {
            const uint32_t j = (uint32_t)(q0 + it * kWave + lane);
            li[it] = in_idx[f.ib + j0 + min(j, m - 1u)];
            if (j >= m) li[it] = f.nk;
        }
#pragma unroll
        for (int it = 0; it < kQuarter / kWave; ++it) {
            const uint32_t i = f.pb + min(li[it], f.nk - 1u);
            double u, v;
            project(f, X[i], Y[i], Z[i], &u, &v);
            uv[q0 + it * kWave + lane] =
                li[it] < f.nk ? make_float2((float)(0.125 * u), (float)(0.125 * v)) : make_float2(__builtin_nanf(""), 0.0f);
        }
        wave_sync();
        float hi0 = -INFINITY, hi1 = -INFINITY, lo0 = INFINITY, lo1 = INFINITY;
        const int n = min(kQuarter, (int)m - q0);
#pragma unroll 4
        for (int j = 0; j < n; j += kStep) {
            const float4 p = *(const float4*)&uv[q0 + j + 2 * grp];
            const uint32_t pos = (uint32_t)(j / kGroups);
            const float a0 = key_of(fmaf(p.x, cs, p.y * sn), pos, kPosMask);
            const float b0 = key_of(fmaf(p.z, cs, p.w * sn), pos + 1u, kPosMask);
            const float a1 = key_of(fmaf(p.y, cs, -(p.x * sn)), pos, kPosMask);
            const float b1 = key_of(fmaf(p.w, cs, -(p.z * sn)), pos + 1u, kPosMask);
            hi0 = max3f(hi0, a0, b0);
            lo0 = min3f(lo0, a0, b0);
            hi1 = max3f(hi1, a1, b1);
            lo1 = min3f(lo1, a1, b1);
        }
        const auto put = [&](int d, float key, bool none) {
            const uint32_t pos = __float_as_uint(key) & kPosMask;
            rv[wave * kGroups + grp][d] = none ? -INFINITY : d < kDirs / 2 ? key : -key;
            ri[wave * kGroups + grp][d] = j0 + (uint32_t)q0 + (pos >> 1) * kStep + 2u * (uint32_t)grp + (pos & 1u);
        };
        put(dir, hi0, hi0 == -INFINITY);
        put(dir + kDirs / 4, hi1, hi1 == -INFINITY);
        put(dir + kDirs / 2, lo0, lo0 == INFINITY);
        put(dir + 3 * kDirs / 4, lo1, lo1 == INFINITY);
        __syncthreads();
        if (wave == 0) {
            float bv = -INFINITY;
            uint32_t bi = 0xFFFFFFFFu;
#pragma unroll
            for (int w = 0; w < kWaves * kGroups; ++w)
                if (rv[w][lane] > bv) {
                    bv = rv[w][lane];
                    bi = ri[w][lane];
                }
            ext_v[kDirs * (size_t)t + lane] = bv;
            ext_i[kDirs * (size_t)t + lane] = bi;
        }
        __syncthreads();
    }
}

// ---- C: per-cluster extreme polygon -----------------------------------------------
// The corners among `alive` (a lane each, in the order of their directions, at
// (su, sv); this lane's is (u, v)) that a convex polygon can have: those that do
// not turn left by more than mg are dropped, all lanes at once, until every one
// left does.  Of a run of such corners every other one goes in a round, from its
// first: the rounds end, and no two neighbours go together, which two
// coincident points at a true corner may both look like (with such a corner
// lost, a lattice of 150 x 150 cells left 60k survivors: 8.8 ms, 0.1 so).
__device__ __forceinline__ uint64_t convex_corners(uint64_t alive, double u, double v, const double* su, const double* sv,
                                                   double mg, int lane)
{
    const uint64_t below = (1ull << lane) - 1ull, above = ~below & ~(1ull << lane);
    while (__popcll(alive) >= 3) {
        bool bad = false;
        if ((alive >> lane) & 1ull) {
            // neighbours on the circle of corners
            const int p = (alive & below) ? 63 - __clzll((long long)(alive & below)) : 63 - __clzll((long long)alive);
            const int n = __ffsll((long long)((alive & above) ? (alive & above) : alive)) - 1;
            bad = cross3(su[p], sv[p], u, v, su[n], sv[n]) <= mg;
        }
        const uint64_t b = __ballot(bad), good = alive & ~b;
        if (b == 0) break;
        // this corner's place in its run of bad ones
        const uint64_t start = (good & below) ? good & below : good;
        const uint64_t past = start ? ~((2ull << (63 - __clzll((long long)start))) - 1ull) : 0ull;
        uint32_t place = (uint32_t)__popcll(alive & below & ((good & below) ? past : ~0ull));
        if (!(good & below)) place += (uint32_t)__popcll(alive & past);
        // (all bad: the run closes on itself)
        const bool joins = good == 0 && place + 1u == (uint32_t)__popcll(alive);
        alive &= ~__ballot(bad && (place & 1u) == 0 && !joins);
    }
    return alive;
}

// A workgroup per cluster: its waves share the tiles, lane d its extreme in
// direction d; then one wave merges repeated extremes and drops the corners that
// are not strictly convex.  The rest bound a convex polygon inside the
// hull.  Its corners, as positions in the inlier list, counter-clockwise, go
// to the first 64 words of the cluster's own region of hull_tmp, their number
// (below 3: no filtering) to the next one; the filtered clusters have more
// than 64 inliers, so the region holds them.  margin[k] is far above the fp64
// rounding of a cross product at the polygon's scale.
__global__ void __launch_bounds__(kBlock) k_hull_poly(const uint32_t* __restrict__ small,
                                                     const uint32_t* __restrict__ tile_off,
                                                     const uint32_t* __restrict__ off, const float* __restrict__ X,
                                                     const float* __restrict__ Y, const float* __restrict__ Z,
                                                     const float4* __restrict__ plane,
                                                     const uint32_t* __restrict__ in_off,
                                                     const uint32_t* __restrict__ in_idx,
                                                     const float* __restrict__ ext_v,
                                                     const uint32_t* __restrict__ ext_i, double* __restrict__ margin,
                                                     uint32_t* __restrict__ hull_tmp, uint32_t* __restrict__ surv_cnt)
{
    constexpr int kWaves = kBlock / kWave;
    constexpr uint32_t kAhead = 8;   // tiles whose reads a wave has in flight
    __shared__ double su[kWave], sv[kWave];
    __shared__ float rv[kWaves][kDirs];
    __shared__ uint32_t ri[kWaves][kDirs];
    const uint32_t K = small[4];
    const uint32_t T = small[6];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (uint32_t k = blockIdx.x; k < K; k += gridDim.x) {
        const uint32_t t0 = tile_off[k], t1 = tiles_end(tile_off, k, K, T);
        if (threadIdx.x == 0) surv_cnt[k] = 0;
        if (t0 == t1) continue;   // workgroup-uniform
        float bv = -INFINITY;
        uint32_t e = 0xFFFFFFFFu;
        for (uint32_t t = t0 + wave * kAhead; t < t1; t += kWaves * kAhead) {
            float v[kAhead];
            uint32_t i[kAhead];
#pragma unroll
            for (uint32_t q = 0; q < kAhead; ++q) {
                const size_t x = kDirs * (size_t)min(t + q, t1 - 1u) + lane;
                v[q] = ext_v[x];
                i[q] = ext_i[x];
            }
#pragma unroll
            for (uint32_t q = 0; q < kAhead; ++q)
                if (v[q] > bv) {
                    bv = v[q];
                    e = i[q];
                }
        }
        rv[wave][lane] = bv;
        ri[wave][lane] = e;
        __syncthreads();
        if (wave != 0) {
            __syncthreads();   // (the end of the round below)
            continue;
        }
#pragma unroll
        for (int w = 1; w < kWaves; ++w)
            if (rv[w][lane] > bv) {
                bv = rv[w][lane];
                e = ri[w][lane];
            }
        const ClusterFrame f = cluster_frame(k, off, X, Y, Z, plane, in_off, in_idx);
        double u = 0.0, v = 0.0;
        const bool found = e < f.m;
        if (found) {
            const uint32_t i = f.pb + min(in_idx[f.ib + e], f.nk - 1u);
            project(f, X[i], Y[i], Z[i], &u, &v);
        }
        su[lane] = u;
        sv[lane] = v;
        wave_sync();
        // the corners: extremes that differ from the one before
        const uint32_t prev = __shfl(e, (lane + kWave - 1) & (kWave - 1), kWave);
        uint64_t alive = __ballot(found) == ~0ull ? __ballot(e != prev) : 0ull;
        const double span = wave_max_d(fmax(fabs(u - su[0]), fabs(v - sv[0])));
        // (the largest distance from one corner is at least half the extent)
        const double mg = kMargin * span * span + 1e-300;
        alive = convex_corners(alive, u, v, su, sv, mg, lane);
        const uint64_t below = (1ull << lane) - 1ull;
        const uint32_t np = (uint32_t)__popcll(alive);
        uint32_t* out = hull_tmp + f.ib + k;
        if ((alive >> lane) & 1ull) out[__popcll(alive & below)] = e;
        if (lane == 0) {
            out[kDirs] = np;
            margin[k] = mg;
        }
        __syncthreads();   // the scratch is reused by the next cluster
    }
}

// ---- D: survivors of the polygon test, compacted per cluster ---------------------
// Whether (u, v) lies strictly inside the convex polygon P[0..np): the wedge
// at corner 0 that holds it is found by bisection, then the wedge's outer
// edge and both edges at corner 0 (a point that nearly coincides with that
// corner may be put in any wedge) are tested by the margin.
template <typename F2, typename F>
__device__ __forceinline__ bool inside_polygon(const F2* P, int np, F mg, F u, F v)
{
    const F2 c0 = P[0];
    const F wu = u - c0.x, wv = v - c0.y;
    const auto side = [&](int i) { return (P[i].x - c0.x) * wv - (P[i].y - c0.y) * wu; };
    int lo = 1, hi = np - 1;   // the wedge (lo, hi)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (side(mid) >= F(0)) lo = mid;
        else hi = mid;
    }
    const F2 a = P[lo], b = P[hi];
    return (b.x - a.x) * (v - a.y) - (b.y - a.y) * (u - a.x) > mg && side(1) > mg && side(np - 1) < -mg;
}

// A point is first tested in fp32, by a margin above the rounding there; the
// few near the border or outside are collected and tested in fp64 by margin[k],
// so that one wave does for a tile what else nearly every wave would run for a
// lane or two (34M inliers in no order, 2048 workgroups: 277 us with fp64 alone,
// 355 with both in place, 312 so; with 16384 workgroups and the points projected
// once 227).  The fp32 coordinates are the fp64 ones relative
// to corner 0, rounded: each errs by 2^-24 of itself and none exceeds the
// extent E of the inliers in the plane, wherever they lie along the normal.
// Differences then err by 3 * 2^-24 E, a product of two of them by 7 * 2^-24
// E^2, and a side's value by 16 * 2^-24 E^2.  E is at most 2.0001 spans (the
// extremes hold the largest and the smallest of both coordinates to 2^-16), so
// that is 4e-6 of the span's square.
constexpr double kMarginF = 3e-5;   // of the span's square

// (extents whose square leaves fp32's range are left to fp64)
__device__ __forceinline__ float margin_f(double mg)
{
    const double m = mg * (kMarginF / kMargin);
    return m < 1e30 ? (float)m + 1e-37f : INFINITY;
}

__global__ void __launch_bounds__(kTileThreads) k_hull_filter(
    const uint32_t* __restrict__ small, const uint32_t* __restrict__ tile_off, const uint32_t* __restrict__ off,
    const float* __restrict__ X, const float* __restrict__ Y, const float* __restrict__ Z,
    const float4* __restrict__ plane, const uint32_t* __restrict__ in_off, const uint32_t* __restrict__ in_idx,
    const double* __restrict__ margin, const uint32_t* __restrict__ hull_tmp, uint32_t* __restrict__ surv_cnt,
    double* __restrict__ gu, double* __restrict__ gv, uint32_t* __restrict__ gi)
{
    __shared__ double2 poly[kDirs];
    __shared__ float2 polyf[kDirs];
    __shared__ double2 rest[kHullTile];   // the points left for the fp64 test, and their numbers in the tile
    __shared__ uint16_t rest_no[kHullTile];
    __shared__ uint32_t nrest;
    const uint32_t K = small[4];
    const uint32_t T = small[6];
    const int lane = threadIdx.x & (kWave - 1);
    for (uint32_t t = blockIdx.x; t < T; t += gridDim.x) {
        const uint32_t k = last_at_or_below(tile_off, K, t);
        const ClusterFrame f = cluster_frame(k, off, X, Y, Z, plane, in_off, in_idx);
        const uint32_t* corner = hull_tmp + f.ib + k;
        const int np = (int)corner[kDirs];
        const double mg = margin[k];
        const float mgf = margin_f(mg);
        const uint32_t j0 = (t - tile_off[k]) * kHullTile;
        // the tile's points, while the polygon's come in
        uint32_t pt[kTileItems];
        float x[kTileItems], y[kTileItems], z[kTileItems];
        bool in[kTileItems];
#pragma unroll
        for (int it = 0; it < kTileItems; ++it) {
            const uint32_t j = j0 + it * kTileThreads + threadIdx.x;
            const uint32_t li = in_idx[f.ib + min(j, f.m - 1u)];
            in[it] = j < f.m && li < f.nk;
            pt[it] = f.pb + min(li, f.nk - 1u);
        }
#pragma unroll
        for (int it = 0; it < kTileItems; ++it) {
            x[it] = X[pt[it]];
            y[it] = Y[pt[it]];
            z[it] = Z[pt[it]];
        }
        if ((int)threadIdx.x < np) {
            const uint32_t i = f.pb + in_idx[f.ib + corner[threadIdx.x]], i0 = f.pb + in_idx[f.ib + corner[0]];
            double2 c, c0;
            project(f, X[i], Y[i], Z[i], &c.x, &c.y);
            project(f, X[i0], Y[i0], Z[i0], &c0.x, &c0.y);
            poly[threadIdx.x] = c;
            polyf[threadIdx.x] = make_float2((float)(c.x - c0.x), (float)(c.y - c0.y));
        }
        if (threadIdx.x == 0) nrest = 0;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kTileItems; ++it) {
            double2 p;
            project(f, x[it], y[it], z[it], &p.x, &p.y);
            if (in[it] && !(np >= 3 && inside_polygon(polyf, np, mgf, (float)(p.x - poly[0].x), (float)(p.y - poly[0].y)))) {
                const uint32_t r = atomicAdd(&nrest, 1u);
                rest[r] = p;
                rest_no[r] = (uint16_t)(it * kTileThreads + threadIdx.x);
            }
        }
        __syncthreads();
        const uint32_t n = nrest;
        for (uint32_t r0 = 0; r0 < n; r0 += kTileThreads) {
            const uint32_t r = r0 + threadIdx.x;
            double2 p;
            bool out = false;
            if (r < n) {
                p = rest[r];
                out = !(np >= 3 && inside_polygon(poly, np, mg, p.x, p.y));
            }
            const uint64_t b = __ballot(out);
            if (b == 0) continue;
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&surv_cnt[k], (uint32_t)__popcll(b));
            base = __shfl(base, 0, kWave);
            if (out) {
                const uint32_t dst = f.ib + base + (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
                gu[dst] = p.x;
                gv[dst] = p.y;
                gi[dst] = j0 + rest_no[r];
            }
        }
        __syncthreads();
    }
}

// ---- E: the hulls of the survivors -------------------------------------------------
// Survivor sets beyond LDS are thinned once more before they are sorted, by the
// polygon of their own extremes, found in fp64: the first polygon's extremes are
// compared to 2^-18 of their distance, and where a straight edge's points differ
// by less (a lattice's edge under a plane that tilts by 1e-3), most of them lie
// outside it and few outside this one (600k points on 400 x 400 cells: 2.9 ms
// without, the sort in memory and one thread's chain; 0.2 so).
struct RefineLds {
    double rv[kChainBlock / kWave][kDirs];
    uint32_t ri[kChainBlock / kWave][kDirs];
    double su[kDirs], sv[kDirs];
    double2 poly[kDirs];
    double margin;
    uint32_t np;
    uint32_t wcnt[kChainBlock / kWave];
};

// compacts U/V/I[0, ns) in place to the points not strictly inside the polygon
// of their extremes; returns their number (every thread of the workgroup calls it)
__device__ __forceinline__ uint32_t refine_survivors(RefineLds& R, double* U, double* V, uint32_t* I, uint32_t ns)
{
    constexpr uint32_t kWaves = kChainBlock / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // a lane per direction, the waves share the points
    double sn, cs, bv = -INFINITY;
    uint32_t bi = 0xFFFFFFFFu;
    sincospi((double)lane / (kDirs / 2), &sn, &cs);
#pragma unroll 8
    for (uint32_t t = wave; t < ns; t += kWaves) {
        const double val = U[t] * cs + V[t] * sn;
        if (val > bv) {
            bv = val;
            bi = t;
        }
    }
    R.rv[wave][lane] = bv;
    R.ri[wave][lane] = bi;
    __syncthreads();
    if (wave == 0) {
        for (uint32_t w = 1; w < kWaves; ++w)
            if (R.rv[w][lane] > bv) {
                bv = R.rv[w][lane];
                bi = R.ri[w][lane];
            }
        const bool found = bi < ns;
        const double u = found ? U[bi] : 0.0, v = found ? V[bi] : 0.0;
        R.su[lane] = u;
        R.sv[lane] = v;
        wave_sync();
        const uint32_t prev = __shfl(bi, (lane + kWave - 1) & (kWave - 1), kWave);
        uint64_t alive = __ballot(found) == ~0ull ? __ballot(bi != prev) : 0ull;
        const double span = wave_max_d(fmax(fabs(u - R.su[0]), fabs(v - R.sv[0])));
        const double mg = kMargin * span * span + 1e-300;
        alive = convex_corners(alive, u, v, R.su, R.sv, mg, lane);
        if ((alive >> lane) & 1ull) R.poly[__popcll(alive & ((1ull << lane) - 1ull))] = make_double2(u, v);
        if (lane == 0) {
            R.np = (uint32_t)__popcll(alive);
            R.margin = mg;
        }
    }
    __syncthreads();
    const int np = (int)R.np;
    const double mg = R.margin;
    if (np < 3) return ns;
    // a workgroup's row at a time: its points are read before any is written,
    // and writes land at or below them
    uint32_t nout = 0;
    for (uint32_t t0 = 0; t0 < ns; t0 += kChainBlock) {
        const uint32_t t = t0 + threadIdx.x;
        double u = 0.0, v = 0.0;
        uint32_t id = 0;
        bool keep = false;
        if (t < ns) {
            u = U[t];
            v = V[t];
            id = I[t];
            keep = !inside_polygon(R.poly, np, mg, u, v);
        }
        const uint64_t bal = __ballot(keep);
        if (lane == 0) R.wcnt[wave] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t o = nout + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        for (uint32_t w = 0; w < kWaves; ++w) {
            o += w < wave ? R.wcnt[w] : 0u;
            nout += R.wcnt[w];
        }
        if (keep) {
            U[o] = u;
            V[o] = v;
            I[o] = id;
        }
        __syncthreads();   // wcnt is reused, the next row may be written to
    }
    return nout;
}

// A survivor set beyond LDS: sorted in global memory (bitonic, partners beyond
// ns are +infinity) by the workgroup, chained by one thread.
__device__ void global_chain(uint32_t k, uint32_t ns, uint32_t ib, double* U, double* Vv, uint32_t* I,
                             const uint32_t* __restrict__ in_idx, uint32_t* hull_cnt, uint32_t* hull_tmp,
                             double* area_out)
{
    uint32_t N = 1;
    while (N < ns) N <<= 1;
    for (uint32_t size = 2; size <= N; size <<= 1) {
        for (uint32_t t = threadIdx.x; t < N / 2; t += kChainBlock) {
            const uint32_t blk = t / (size >> 1), r = t % (size >> 1);
            const uint32_t a = blk * size + r, b = blk * size + size - 1 - r;
            if (b < ns && p2_less(U[b], Vv[b], I[b], U[a], Vv[a], I[a])) swap3(U, Vv, I, a, b);
        }
        __syncthreads();
        for (uint32_t stride = size >> 2; stride > 0; stride >>= 1) {
            for (uint32_t t = threadIdx.x; t < N / 2; t += kChainBlock) {
                const uint32_t a = 2 * t - (t & (stride - 1)), b = a + stride;
                if (b < ns && p2_less(U[b], Vv[b], I[b], U[a], Vv[a], I[a])) swap3(U, Vv, I, a, b);
            }
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) {
        // single-stack chain; cluster k's stack is hull_tmp[ib + k, ib + k + m + 1)
        // and never holds more than ns + 1 <= m + 1 entries
        uint32_t* st = hull_tmp + ib + k;
        uint32_t h = 0;
        for (uint32_t i = 0; i < ns; ++i) {
            while (h >= 2) {
                const uint32_t a = st[h - 2], b = st[h - 1];
                if (cross3(U[a], Vv[a], U[b], Vv[b], U[i], Vv[i]) <= 0.0) --h;
                else break;
            }
            st[h++] = i;
        }
        const uint32_t lower = h + 1;
        for (int32_t i = (int32_t)ns - 2; i >= 0; --i) {
            while (h >= lower) {
                const uint32_t a = st[h - 2], b = st[h - 1];
                if (cross3(U[a], Vv[a], U[b], Vv[b], U[i], Vv[i]) <= 0.0) --h;
                else break;
            }
            st[h++] = (uint32_t)i;
        }
        --h;   // the last point repeats the first
        double s = 0.0;
        if (h >= 3) {
            for (uint32_t q = 0; q < h; ++q) {
                const uint32_t p0 = st[q], p1 = st[q + 1 == h ? 0 : q + 1];
                s = s + (U[p0] * Vv[p1] - U[p1] * Vv[p0]);
            }
        }
        area_out[k] = h >= 3 ? 0.5 * s : 0.0;
        // entry q of the stack is read before slot q is overwritten
        for (uint32_t q = 0; q < h; ++q) hull_tmp[ib + k + q] = in_idx[ib + I[st[q]]];
        hull_cnt[k] = h;
    }
    __syncthreads();
}

// Workgroup b takes clusters b, b + G, ..., b + 7 G of each round of 8 G (G
// workgroups): while there are fewer clusters than workgroups each gets one,
// so the large ones, neighbours in label order, run side by side.  First the
// workgroup chains together those of them with more than 64 survivors of the
// filter, then each wave its own of the others: at most 64 survivors, or (a
// cluster that the filter skips) all inliers, projected here exactly as the
// filter projects them.
__global__ void __launch_bounds__(kChainBlock) k_hull_finish(
    const uint32_t* __restrict__ small, const uint32_t* __restrict__ tile_off, const uint32_t* __restrict__ off,
    const float* __restrict__ X, const float* __restrict__ Y, const float* __restrict__ Z,
    const float4* __restrict__ plane, const int32_t* __restrict__ best, uint32_t in_cap,
    const uint32_t* __restrict__ in_off, const uint32_t* __restrict__ in_idx, const uint32_t* __restrict__ surv_cnt,
    double* __restrict__ gu, double* __restrict__ gv, uint32_t* __restrict__ gi, uint32_t* __restrict__ hull_cnt,
    uint32_t* __restrict__ hull_tmp, double* __restrict__ area_out)
{
    constexpr uint32_t kWaves = kChainBlock / kWave;
    __shared__ double su[kWaves][kWave];
    __shared__ double sv[kWaves][kWave];
    __shared__ uint32_t si[kWaves][kWave];
    __shared__ uint8_t st[kWaves][2 * kWave + 2];
    __shared__ ChainLds<kLdsCap> L;
    __shared__ RefineLds R;
    const uint32_t K = small[4];
    const uint32_t T = small[6];
    const uint32_t G = gridDim.x;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (uint32_t c0 = blockIdx.x; c0 < K; c0 += kWaves * G) {
        for (uint32_t w = 0; w < kWaves && c0 + w * G < K; ++w) {   // workgroup-uniform
            const uint32_t k = c0 + w * G;
            if (tile_off[k] == tiles_end(tile_off, k, K, T)) continue;
            uint32_t ns = surv_cnt[k];
            if (ns <= (uint32_t)kWave) continue;
            const uint32_t ib = in_off[k];
            if (ns > (uint32_t)kLdsCap) ns = refine_survivors(R, gu + ib, gv + ib, gi + ib, ns);
            if (ns > (uint32_t)kLdsCap) {
                global_chain(k, ns, ib, gu + ib, gv + ib, gi + ib, in_idx, hull_cnt, hull_tmp, area_out);
                continue;
            }
            double area = 0.0;
            const uint32_t hh = block_chain(L, ns,
                                            [&](uint32_t t, double* u, double* v, uint32_t* id) {
                                                *u = gu[ib + t];
                                                *v = gv[ib + t];
                                                *id = gi[ib + t];
                                            },
                                            [&](uint32_t q, uint32_t p) { hull_tmp[ib + k + q] = in_idx[ib + L.si[p]]; },
                                            &area);
            if (threadIdx.x == 0) {
                area_out[k] = area;
                hull_cnt[k] = hh;
            }
            __syncthreads();   // L is reused by the next cluster
        }
        const uint32_t k = c0 + wv * G;
        if (k >= K) continue;   // wave-uniform, no barriers below
        uint32_t ns;
        double u = INFINITY, v = INFINITY;
        uint32_t i = 0xFFFFFFFFu;
        const uint32_t ib = in_off[k];
        if (tile_off[k] != tiles_end(tile_off, k, K, T)) {
            ns = surv_cnt[k];
            if (ns > (uint32_t)kWave) continue;   // done by the workgroup
            if ((uint32_t)lane < ns) {
                u = gu[ib + lane];
                v = gv[ib + lane];
                i = gi[ib + lane];
            }
        } else {
            if (!cluster_ok(k, off, best, in_off, in_idx, in_cap)) {   // no polygon
                if (lane == 0) {
                    hull_cnt[k] = 0;
                    area_out[k] = 0.0;
                }
                continue;
            }
            ns = in_off[k + 1] - ib;
            const ClusterFrame f = cluster_frame(k, off, X, Y, Z, plane, in_off, in_idx);
            if ((uint32_t)lane < ns) {
                const uint32_t p = f.pb + in_idx[ib + lane];
                project(f, X[p], Y[p], Z[p], &u, &v);
                i = (uint32_t)lane;
            }
        }
        const WaveHull r = wave_hull(u, v, i, ns, lane, su[wv], sv[wv], si[wv], st[wv]);
        if (lane == 0) {
            area_out[k] = r.area;
            hull_cnt[k] = r.h;
        }
        if ((uint32_t)lane < r.h) hull_tmp[ib + k + lane] = in_idx[ib + si[wv][r.vi]];
        wave_sync();
    }
}

// ---- F: pack --------------------------------------------------------------------------
// Groups of kPackClusters clusters, a workgroup each.  scan is the exclusive
// scan of the vertex counts and small[5] their total, or, when scan is null
// (at most kOneBlockMax clusters), a group sums the counts of the clusters
// before it itself, which saves a launch that took longer than this one.
constexpr uint32_t kPackClusters = 64;

__global__ void __launch_bounds__(kBlock) k_hull_pack(const uint32_t* __restrict__ small,
                                                      const uint32_t* __restrict__ off, const float* __restrict__ X,
                                                      const float* __restrict__ Y, const float* __restrict__ Z,
                                                      const float4* __restrict__ plane,
                                                      const uint32_t* __restrict__ in_off,
                                                      const uint32_t* __restrict__ hull_cnt,
                                                      const uint32_t* __restrict__ hull_tmp,
                                                      const uint32_t* __restrict__ scan, uint32_t v_cap,
                                                      uint32_t* __restrict__ v_off, uint32_t* __restrict__ v_idx,
                                                      float* __restrict__ v_xyz, uint32_t* __restrict__ status)
{
    __shared__ uint32_t part[kBlock / kWave];
    __shared__ uint32_t s_off[kPackClusters + 1];   // first vertex of each cluster of the group, and the end
    const uint32_t K = small[4];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    bool over = false;
    if (K == 0 && blockIdx.x == 0 && threadIdx.x == 0) v_off[0] = 0;
    for (uint32_t k0 = blockIdx.x * kPackClusters; k0 < K; k0 += gridDim.x * kPackClusters) {
        uint32_t pre = 0;
        if (!scan) {
#pragma unroll 4
            for (uint32_t k = threadIdx.x; k < k0; k += kBlock) pre += hull_cnt[k];
        }
#pragma unroll
        for (int d = kWave / 2; d >= 1; d >>= 1) pre += __shfl_xor(pre, d, kWave);
        if (lane == 0) part[wave] = pre;
        __syncthreads();
        if (wave == 0) {
            const uint32_t k = k0 + (uint32_t)lane, c = k < K ? hull_cnt[k] : 0u;
            uint32_t base = scan ? scan[k0] : 0u;
#pragma unroll
            for (int w = 0; w < kBlock / kWave; ++w) base += part[w];
            uint32_t inc = c;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t o = __shfl_up(inc, d, kWave);
                if (lane >= d) inc += o;
            }
            s_off[lane] = base + inc - c;
            if (lane == kWave - 1) s_off[kPackClusters] = base + inc;
            if (k < K) v_off[k] = base + inc - c;
            if (k + 1 == K) v_off[K] = base + inc;
        }
        __syncthreads();
        for (uint32_t pos = s_off[0] + threadIdx.x; pos < s_off[kPackClusters]; pos += kBlock) {
            if (pos >= v_cap) {
                over = true;
                continue;
            }
            uint32_t lo = 0;   // the cluster: the last one starting at or before pos (empty ones precede it)
#pragma unroll
            for (uint32_t h = kPackClusters / 2; h; h >>= 1)
                if (s_off[lo + h] <= pos) lo += h;
            const uint32_t k = k0 + lo;
            const float4 pl = plane[k];
            const double nx = pl.x, ny = pl.y, nz = pl.z, d = pl.w;
            const uint32_t j = hull_tmp[in_off[k] + k + (pos - s_off[lo])], i = off[k] + j;
            const double px = X[i], py = Y[i], pz = Z[i];
            const double dist = nx * px + ny * py + nz * pz + d;
            v_idx[pos] = j;
            v_xyz[3 * (size_t)pos + 0] = (float)(px - dist * nx);
            v_xyz[3 * (size_t)pos + 1] = (float)(py - dist * ny);
            v_xyz[3 * (size_t)pos + 2] = (float)(pz - dist * nz);
        }
        __syncthreads();   // part and s_off are reused by the next group
    }
    if (over) atomicOr(status, (uint32_t)VM_FLAG_HULL_CAP);
}

static_assert(kPackClusters == (uint32_t)kWave, "a lane per cluster of a group");

}  // namespace

uint64_t hull_tiles_bound(uint32_t k_cap, uint32_t n_cap)
{
    return (uint64_t)n_cap / kHullTile + (uint64_t)k_cap + 2;
}

vm_status hulls(const vm_clusters& cl, const vm_planes& planes, const vm_hulls_out& out, const WorkLayout& w,
                hipStream_t s)
{
    uint32_t kc = cl.k_cap;
    if (planes.k_cap < kc) kc = planes.k_cap;
    if (out.k_cap < kc) kc = out.k_cap;
    if (kc > w.k_cap) return VM_E_STATE;
    StageScope t(VM_STAGE_HULL, s);
    const float4* pl = (const float4*)planes.d_plane;
    if (kc <= kOneBlockMax) {
        k_hull_prepare<<<1, kOneBlockThreads, 0, s>>>(cl.d_meta, kc, cl.n_cap, cl.d_off, planes.d_best_h,
                                                      planes.d_in_off, planes.d_in_idx, planes.in_cap, w.small,
                                                      w.hull_tile_off, out.d_status);
    } else {
        k_hull_validate<<<1, kBlock, 0, s>>>(cl.d_meta, kc, cl.n_cap, cl.d_off, w.small, out.d_status);
        k_hull_tiles<<<grid_for(kc), kBlock, 0, s>>>(w.small, cl.d_off, planes.d_best_h, planes.d_in_off,
                                                     planes.d_in_idx, planes.in_cap, w.hull_tile_off, out.d_status);
        VM_HIP(scan_exclusive_dev(w.hull_tile_off, w.hull_tile_off, w.small + 4, kc, w.small + 6, w.blk, s));
    }
    // the tile kernels stride over the device-side counts; many more workgroups
    // than fit at once even out what they find (34k tiles of 2000 clusters:
    // extremes 259 us and filter 316 with 2048, of which 1792 fit, 249 and 227
    // with 16384; a frame's few hundred tiles: 19 us either way)
    const int tgrid = grid_for(hull_tiles_bound(kc, cl.n_cap), 1, kTileGrid);
    // the tiles' extremes lie where the survivors go afterwards: a filtered
    // cluster of m > 64 inliers has at most m / 1024 + 1 tiles of 256 bytes in
    // each table, less than the 8 m bytes of its part of hull_u or hull_v
    float* ext_v = (float*)w.hull_u;
    uint32_t* ext_i = (uint32_t*)w.hull_v;
    k_hull_extremes<<<tgrid, kTileThreads, 0, s>>>(w.small, w.hull_tile_off, cl.d_off, cl.d_x, cl.d_y, cl.d_z, pl,
                                                   planes.d_in_off, planes.d_in_idx, ext_v, ext_i);
    k_hull_poly<<<grid_for(kc, 1, kPolyGrid), kBlock, 0, s>>>(
        w.small, w.hull_tile_off, cl.d_off, cl.d_x, cl.d_y, cl.d_z, pl, planes.d_in_off, planes.d_in_idx, ext_v, ext_i,
        w.margin, w.hull_tmp, w.surv_cnt);
    k_hull_filter<<<tgrid, kTileThreads, 0, s>>>(w.small, w.hull_tile_off, cl.d_off, cl.d_x, cl.d_y, cl.d_z, pl,
                                                 planes.d_in_off, planes.d_in_idx, w.margin, w.hull_tmp, w.surv_cnt,
                                                 w.hull_u, w.hull_v, w.hull_i);
    k_hull_finish<<<grid_for(kc, 1, kFinishGrid), kChainBlock, 0, s>>>(
        w.small, w.hull_tile_off, cl.d_off, cl.d_x, cl.d_y, cl.d_z, pl, planes.d_best_h, planes.in_cap, planes.d_in_off,
        planes.d_in_idx, w.surv_cnt, w.hull_u, w.hull_v, w.hull_i, w.hull_cnt, w.hull_tmp, out.d_area);
    VM_HIP(hipGetLastError());
    const uint32_t* scan = nullptr;
    if (kc > kOneBlockMax) {
        VM_HIP(scan_exclusive_dev(w.hull_cnt, w.hull_off, w.small + 4, kc, w.small + 5, w.blk, s));
        scan = w.hull_off;
    }
    k_hull_pack<<<grid_for(kc, (int)kPackClusters, 1024), kBlock, 0, s>>>(
        w.small, cl.d_off, cl.d_x, cl.d_y, cl.d_z, pl, planes.d_in_off, w.hull_cnt, w.hull_tmp, scan, out.v_cap,
        out.d_v_off, out.d_v_idx, out.d_v_xyz, out.d_status);
    VM_HIP(hipGetLastError());
    return VM_OK;
}

}  // namespace vm
