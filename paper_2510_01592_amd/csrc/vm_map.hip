// vm_map.hip -- the sparse voxel map (Sec. III-B): insertion of a point frame
// (Eq. (1)), the occupancy index, and map export/import.
//
// Storage.  Occupied voxels live in an open-addressing hash keyed by the
// voxel's linear index; the payload per slot is a point count and three
// 64-bit sums of fixed-point in-voxel offsets (quantum s*2^-20).  Integer
// atomics make the accumulated mean exact and independent of the order in
// which points (and lanes, and XCDs) arrive.  Beside the hash, one bit per
// grid cell marks occupancy; its popcount prefix gives every occupied voxel a
// dense rank in ascending key order, which the clustering stages use as their
// index space (4 MB of bits for a 400x400x200 grid).
#include "vm_common.h"
#include "vm_tilescan.h"

#include <stddef.h>

#include <algorithm>

namespace vm {
namespace {

// Counters are reduced per block before one atomic each (same-address device
// atomics from every wave would serialise).  Grids stay at most kMapGrid
// blocks; threads stride over the points.
constexpr int kMapGrid = 1024;

// A point's voxel and its offsets in it (20 bits per axis): map_from_sensor in
// fp64, one fused chain per output coordinate, then whole steps of s * 2^-20
// from the origin, split exactly (a step's number has at most 52 bits, so the
// products with 2^-20 and 2^20 and the difference are exact).  False outside
// the grid; the negated range tests also reject NaN.
struct Cell {
    uint32_t key, off[3];
};

__device__ __forceinline__ bool cell_of(const Pose& pose, const Geom& g, float x, float y, float z, Cell* c)
{
    const double px = (double)x, py = (double)y, pz = (double)z;
    const double wx = fma(pose.R[2], pz, fma(pose.R[1], py, fma(pose.R[0], px, pose.t[0])));
    const double wy = fma(pose.R[5], pz, fma(pose.R[4], py, fma(pose.R[3], px, pose.t[1])));
    const double wz = fma(pose.R[8], pz, fma(pose.R[7], py, fma(pose.R[6], px, pose.t[2])));
    const double fx = floor((wx - g.origin[0]) * g.inv_q);
    const double fy = floor((wy - g.origin[1]) * g.inv_q);
    const double fz = floor((wz - g.origin[2]) * g.inv_q);
    if (!(fx >= 0.0 && fx < (double)g.dims[0] * 0x1p20 && fy >= 0.0 && fy < (double)g.dims[1] * 0x1p20 && fz >= 0.0 &&
          fz < (double)g.dims[2] * 0x1p20))
        return false;
    const double cx = floor(fx * 0x1p-20), cy = floor(fy * 0x1p-20), cz = floor(fz * 0x1p-20);
    c->key = (uint32_t)cx + (uint32_t)g.dims[0] * ((uint32_t)cy + (uint32_t)g.dims[1] * (uint32_t)cz);
    c->off[0] = (uint32_t)(fx - cx * 0x1p20);
    c->off[1] = (uint32_t)(fy - cy * 0x1p20);
    c->off[2] = (uint32_t)(fz - cz * 0x1p20);
    return true;
}

// key and count of a slot as one word, as they lie in memory
__device__ __forceinline__ unsigned long long slot_head(uint32_t key, uint32_t cnt)
{
    static_assert(offsetof(Slot, key) == 0 && offsetof(Slot, cnt) == 4, "one aligned 8-byte word");
    return (unsigned long long)cnt << 32 | key;
}

// Bound by the atomics of points that share voxels, and for few points by the
// chain of waits.  A slot's key and count are read first: a voxel that holds
// points already needs no claim, and its count, which only grows here, no
// answer.  An empty slot is claimed with its first point counted, one atomic
// for both.  (Claiming by a compare-and-swap without a read was an atomic more
// for every point: the call of 100k points into 2000 voxels that are there took
// 49 us, 44 so, 20k points into one voxel 1186 us, 965 so, and 100k points into
// an empty map 39 us, 37 so.)
__global__ void __launch_bounds__(kBlock) k_insert(const float* __restrict__ xyz, int64_t n, Pose pose, Geom g,
                                                   Hash h, uint32_t* __restrict__ bits,
                                                   DevCounters* __restrict__ ctr)
{
    uint32_t n_in = 0, n_drop = 0, n_lost = 0, n_new = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        Cell c;
        if (!cell_of(pose, g, xyz[3 * i + 0], xyz[3 * i + 1], xyz[3 * i + 2], &c)) {
            ++n_drop;
            continue;
        }
        const uint32_t key = c.key;
        uint32_t s = hash_slot(key, h.log2cap), cnt = 0;
        bool ok = false, claimed = false;
        for (uint32_t p = 0; p < kMaxProbe && p <= h.mask; ++p) {
            unsigned long long* head = reinterpret_cast<unsigned long long*>(&h.slot[s]);
            unsigned long long old = *head;
            if ((uint32_t)old == kEmpty) {   // (an empty slot's count is 0)
                const unsigned long long none = slot_head(kEmpty, 0u);
                old = atomicCAS(head, none, slot_head(key, 1u));
                claimed = old == none;
            }
            ok = claimed || (uint32_t)old == key;
            cnt = (uint32_t)(old >> 32);
            if (ok) break;
            s = (s + 1) & h.mask;
        }
        if (!ok) {
            ++n_lost;
            continue;
        }
        Slot* sl = &h.slot[s];
        // the point that takes a slot's count from 0 marks the voxel occupied:
        // a newly claimed slot, or one whose voxel was cleared (cleared voxels
        // keep their key, so probe chains stay intact)
        bool first = claimed;
        if (!claimed) {
            // (one into the word's upper half: as an add to the count itself the
            // compiler makes this and the next one a single add with an answer)
            if (cnt) atomicAdd(reinterpret_cast<unsigned long long*>(sl), slot_head(0u, 1u));
            else first = atomicAdd(&sl->cnt, 1u) == 0u;
        }
        if (first) {
            atomicOr(&bits[key >> 5], 1u << (key & 31));
            ++n_new;
        }
        atomicAdd(&sl->sum[0], (unsigned long long)c.off[0]);
        atomicAdd(&sl->sum[1], (unsigned long long)c.off[1]);
        atomicAdd(&sl->sum[2], (unsigned long long)c.off[2]);
        ++n_in;
    }
    {
        unsigned long long* const dst[4] = {&ctr->points_in, &ctr->points_dropped, &ctr->points_lost, &ctr->occupied};
        const uint32_t v[4] = {n_in, n_drop, n_lost, n_new};
        block_add_counters<4>(dst, v);
    }
    if (n_lost) atomicOr(&ctr->flags, (uint32_t)VM_FLAG_HASH_FULL);
}

// ---- grouped insert (large calls) ---------------------------------------------
// The points of a batch are partitioned into hash buckets of about kBucketAvg
// points (a bucket is a range of home slots of the map's hash, so every point
// of a voxel lands in the same bucket), and each bucket is then aggregated by
// one workgroup in an LDS table: one slot update per distinct voxel, a plain
// read-modify-write since no other workgroup touches those voxels.
//   count:   a workgroup counts the buckets of its points, a row of the
//            histogram;
//   cols:    each bucket's column becomes prefixes and a total;
//   scatter: the points are voxelised a second time (their 12 bytes are read
//            again, from the cache for a frame, instead of 12 written and read)
//            and go to their buckets as 16-byte records;
//   insert.
// Rows are written and read whole: with a row per bucket the workgroups'
// words lay scattered, and two scan kernels passed over them (4M points: count
// 57 us, scan 34, scatter 81; now
// 24, 5, 69; 1M points: 14, 14, 16; now 11, 4, 16).
constexpr int kPartBlock = 1024;          // partition workgroup: 16 waves
constexpr uint32_t kPartAhead = 4;        // points a thread has in flight
constexpr uint32_t kBucketBlocks = 256;   // partition workgroups per batch, at most: one per compute unit
                                          // (512: 3 to 5 us longer for 0.3M and 1M points, the same for 4M)
// workgroups of the aggregation, what fits at once (five per compute unit, by
// registers): their counters meet on one line, a workgroup per bucket made
// 2048 or 4096 of them do so (1M points: 38 us, 30 so; 4M new: 120, 111)
constexpr uint32_t kInsertBlocks = 1280;
constexpr uint32_t kBucketAvg = 512;      // target points per bucket
constexpr uint32_t kBucketMaxLog2 = 12;   // at most 4096 buckets (LDS counters)
constexpr uint32_t kBucketChunk = 1024;   // points aggregated per LDS table fill
constexpr uint32_t kBucketTableLog2 = 10;
constexpr uint32_t kBucketTable = 1u << kBucketTableLog2;   // LDS table slots: 20 KB (eight workgroups' on
                                                             // a CU, where registers let five); a bucket
                                                             // averages kBucketAvg points, so the table is
                                                             // about half full
static_assert(kBucketTable >= kBucketChunk, "a chunk's distinct keys always fit: every probe ends");
constexpr uint32_t kRecPerThread = kBucketChunk / kBlock;   // records per thread per fill
constexpr uint32_t kSlotPerThread = kBucketTable / kBlock;  // table entries per thread
static_assert(kRecPerThread * kBlock == kBucketChunk && kSlotPerThread * kBlock == kBucketTable, "whole rows per thread");

__device__ __forceinline__ uint32_t bucket_of(uint32_t key, uint32_t lb)
{
    // the top lb bits of the map's own slot hash
    return lb ? (key * 2654435769u) >> (32 - lb) : 0u;
}

// The next bits of the same hash, so that the table's order is the order of the
// home slots and the lanes of a wave update neighbouring lines (4M points: 111
// -> 107 us when every voxel is new, 190 -> 181 when few are; bound by the
// random 32-byte accesses themselves: probing a thread's four entries together
// instead of one after another changed nothing).
__device__ __forceinline__ uint32_t table_slot(uint32_t key, uint32_t lb)
{
    return ((key * 2654435769u) << lb) >> (32 - kBucketTableLog2);
}

// f(in the grid, cell) for the points of workgroup blockIdx.x's tile
template <class F>
__device__ __forceinline__ void each_point(const float* __restrict__ xyz, uint32_t n, const Pose& pose, const Geom& g,
                                           uint32_t tile, F f)
{
    const uint32_t i0 = blockIdx.x * tile, end = min(n - i0, tile) + i0;   // (the grid covers n: i0 < n)
    for (uint32_t b = i0 + threadIdx.x; b < end; b += kPartAhead * kPartBlock) {
        float x[kPartAhead], y[kPartAhead], z[kPartAhead];
#pragma unroll
        for (uint32_t u = 0; u < kPartAhead; ++u) {
            const size_t i = min(b + u * kPartBlock, end - 1u);
            x[u] = xyz[3 * i + 0];
            y[u] = xyz[3 * i + 1];
            z[u] = xyz[3 * i + 2];
        }
#pragma unroll
        for (uint32_t u = 0; u < kPartAhead; ++u) {
            Cell c;
            if (b + u * kPartBlock < end) f(cell_of(pose, g, x[u], y[u], z[u], &c), c);
        }
    }
}

__global__ void __launch_bounds__(kPartBlock) k_bucket_count(const float* __restrict__ xyz, uint32_t n, Pose pose,
                                                             Geom g, uint32_t lb, uint32_t tile, bool first_batch,
                                                             uint32_t* __restrict__ hist, DevCounters* __restrict__ ctr)
{
    __shared__ uint32_t cnt[1u << kBucketMaxLog2];
    const uint32_t B = 1u << lb;
    for (uint32_t b = threadIdx.x; b < B; b += kPartBlock) cnt[b] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && first_batch) ctr->touched = 0;
    __syncthreads();
    uint32_t n_in = 0, n_drop = 0;
    each_point(xyz, n, pose, g, tile, [&](bool in, const Cell& c) {
        if (in) {
            atomicAdd(&cnt[bucket_of(c.key, lb)], 1u);
            ++n_in;
        } else {
            ++n_drop;
        }
    });
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < B; b += kPartBlock) hist[(size_t)blockIdx.x * B + b] = cnt[b];
    unsigned long long* const dst[2] = {&ctr->points_in, &ctr->points_dropped};
    const uint32_t v[2] = {n_in, n_drop};
    block_add_counters<2, kPartBlock>(dst, v);
}

// Columns of the histogram (B buckets, a row per partition workgroup): each
// workgroup takes 32 of them, its 32 groups of lanes an equal share of the rows.
constexpr uint32_t kCols = 32;
constexpr uint32_t kColRows = kBucketBlocks / (kPartBlock / kCols);   // rows of a thread, at most

__global__ void __launch_bounds__(kPartBlock) k_bucket_cols(uint32_t* __restrict__ hist, uint32_t B, uint32_t nblk,
                                                            uint32_t* __restrict__ total)
{
    constexpr uint32_t kGroups = kPartBlock / kCols;
    __shared__ uint32_t sum[kGroups][kCols];
    const uint32_t col = threadIdx.x % kCols, grp = threadIdx.x / kCols;
    const uint32_t b = blockIdx.x * kCols + col, rows = (nblk + kGroups - 1) / kGroups, r0 = grp * rows;
    uint32_t v[kColRows], s = 0;
#pragma unroll
    for (uint32_t j = 0; j < kColRows; ++j) {
        v[j] = j < rows && r0 + j < nblk && b < B ? hist[(size_t)(r0 + j) * B + b] : 0u;
        s += v[j];
    }
    sum[grp][col] = s;
    __syncthreads();
    uint32_t run = 0;
    for (uint32_t q = 0; q < grp; ++q) run += sum[q][col];
    if (b >= B) return;
    if (grp == kGroups - 1) total[b] = run + s;
#pragma unroll
    for (uint32_t j = 0; j < kColRows; ++j) {
        if (j < rows && r0 + j < nblk) hist[(size_t)(r0 + j) * B + b] = run;
        run += v[j];
    }
}

// Points to their buckets; workgroup 0 also writes where the buckets start
// (start[B]: the points in the grid).
__global__ void __launch_bounds__(kPartBlock) k_bucket_scatter(const float* __restrict__ xyz, uint32_t n, Pose pose,
                                                               Geom g, uint32_t lb, uint32_t tile,
                                                               const uint32_t* __restrict__ hist,
                                                               const uint32_t* __restrict__ total,
                                                               uint32_t* __restrict__ start,
                                                               uint4* __restrict__ rec_out)
{
    __shared__ uint32_t pos[1u << kBucketMaxLog2];
    const uint32_t B = 1u << lb;
    const uint32_t* row = hist + (size_t)blockIdx.x * B;
    uint32_t all[1];
    one_block_scan<kPartBlock, 4, 1>(
        B, [&](uint32_t b, uint32_t(&v)[1]) { v[0] = total[b]; },
        [&](uint32_t b, const uint32_t(&e)[1]) {
            pos[b] = e[0] + row[b];
            if (blockIdx.x == 0) start[b] = e[0];
        },
        all);
    if (blockIdx.x == 0 && threadIdx.x == 0) start[B] = all[0];
    __syncthreads();
    each_point(xyz, n, pose, g, tile, [&](bool in, const Cell& c) {
        if (!in) return;
        const uint32_t p = atomicAdd(&pos[bucket_of(c.key, lb)], 1u);
        rec_out[p] = make_uint4(c.key, c.off[0], c.off[1], c.off[2]);   // one 16-byte store
    });
}

// One workgroup per bucket: sum its points per voxel in LDS (at most
// kBucketChunk points per fill, so the 32-bit sums of 20-bit offsets cannot
// overflow), then update each voxel's slot once per fill.
__global__ void __launch_bounds__(kBlock) k_bucket_insert(const uint4* __restrict__ rec, uint32_t lb,
                                                          const uint32_t* __restrict__ first, Hash h,
                                                          uint32_t* __restrict__ bits, DevCounters* __restrict__ ctr)
{
    __shared__ uint32_t tkey[kBucketTable];
    __shared__ uint32_t tcnt[kBucketTable];
    __shared__ uint32_t tsum[3][kBucketTable];
    const uint32_t B = 1u << lb;
    uint32_t n_lost = 0, n_new = 0, n_upd = 0;
    for (uint32_t b = blockIdx.x; b < B; b += gridDim.x) {
        const uint32_t start = first[b], end = first[b + 1];
        for (uint32_t c0 = start; c0 < end; c0 += kBucketChunk) {
            const uint32_t c1 = min(end, c0 + kBucketChunk);
            for (uint32_t q = threadIdx.x; q < kBucketTable; q += kBlock) {
                tkey[q] = kEmpty;
                tcnt[q] = 0;
                tsum[0][q] = tsum[1][q] = tsum[2][q] = 0;
            }
            __syncthreads();
            // a chunk is kRecPerThread records per thread: all loaded before the
            // table inserts
            uint4 rr[kRecPerThread];
#pragma unroll
            for (uint32_t u = 0; u < kRecPerThread; ++u) {
                const uint32_t i = c0 + threadIdx.x + u * kBlock;
                if (i < c1) rr[u] = rec[i];
            }
#pragma unroll
            for (uint32_t u = 0; u < kRecPerThread; ++u) {
                if (c0 + threadIdx.x + u * kBlock >= c1) continue;
                const uint32_t k = rr[u].x;
                uint32_t q = table_slot(k, lb);
                for (;;) {   // at most kBucketChunk keys in a table of kBucketTable slots: ends
                    const uint32_t old = atomicCAS(&tkey[q], kEmpty, k);
                    if (old == kEmpty || old == k) break;
                    q = (q + 1) & (kBucketTable - 1);
                }
                atomicAdd(&tcnt[q], 1u);
                atomicAdd(&tsum[0][q], rr[u].y);
                atomicAdd(&tsum[1][q], rr[u].z);
                atomicAdd(&tsum[2][q], rr[u].w);
            }
            __syncthreads();
            // the thread's kSlotPerThread table entries: first probes (whole
            // 32-byte slots) issued together
            uint32_t tk[kSlotPerThread], sl[kSlotPerThread];
            uint4 sa[kSlotPerThread], sb[kSlotPerThread];
#pragma unroll
            for (uint32_t u = 0; u < kSlotPerThread; ++u) {
                tk[u] = tkey[threadIdx.x + u * kBlock];
                sl[u] = hash_slot(tk[u], h.log2cap);
                if (tk[u] != kEmpty) {
                    const uint4* sp = reinterpret_cast<const uint4*>(&h.slot[sl[u]]);
                    sa[u] = sp[0];
                    sb[u] = sp[1];
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < kSlotPerThread; ++u) {
                const uint32_t q = threadIdx.x + u * kBlock;
                const uint32_t k = tk[u];
                if (k == kEmpty) continue;
                ++n_upd;
                uint32_t s = sl[u];
                uint4 a = sa[u], b2 = sb[u];
                bool ok = a.x == k;
                if (!ok) {
                    for (uint32_t p = 0; p < kMaxProbe && p <= h.mask; ++p) {
                        if (p) a.x = h.slot[s].key;
                        if (a.x == k) { ok = true; break; }
                        if (a.x == kEmpty) {
                            const uint32_t old = atomicCAS(&h.slot[s].key, kEmpty, k);
                            if (old == kEmpty || old == k) { ok = true; break; }
                        }
                        s = (s + 1) & h.mask;
                    }
                    if (ok) {
                        // claimed or found past the first probe: the slot's
                        // counts as they stand now
                        const uint4* sp = reinterpret_cast<const uint4*>(&h.slot[s]);
                        a = sp[0];
                        b2 = sp[1];
                    }
                }
                if (!ok) {
                    n_lost += tcnt[q];
                    continue;
                }
                uint4* sp = reinterpret_cast<uint4*>(&h.slot[s]);
                const unsigned long long s0 = ((unsigned long long)a.w << 32 | a.z) + tsum[0][q];
                const unsigned long long s1 = ((unsigned long long)b2.y << 32 | b2.x) + tsum[1][q];
                const unsigned long long s2 = ((unsigned long long)b2.w << 32 | b2.z) + tsum[2][q];
                // the key is stored as claimed, not as loaded: a load served
                // from a line fetched before the claim would read it empty
                a.x = k;
                if (a.y == 0u) {   // new, or cleared since: occupied again
                    atomicOr(&bits[k >> 5], 1u << (k & 31));
                    ++n_new;
                }
                a.y += tcnt[q];
                a.z = (uint32_t)s0;
                a.w = (uint32_t)(s0 >> 32);
                b2 = make_uint4((uint32_t)s1, (uint32_t)(s1 >> 32), (uint32_t)s2, (uint32_t)(s2 >> 32));
                sp[0] = a;
                sp[1] = b2;
            }
            __syncthreads();
        }
    }
    {
        unsigned long long* const dst[3] = {&ctr->points_lost, &ctr->occupied, &ctr->touched};
        const uint32_t v[3] = {n_lost, n_new, n_upd};
        block_add_counters<3>(dst, v);
    }
    if (n_lost) {
        // points lost here were counted as inserted by the voxelise pass
        atomicAdd(&ctr->points_in, 0ull - (unsigned long long)n_lost);
        atomicOr(&ctr->flags, (uint32_t)VM_FLAG_HASH_FULL);
    }
}

// ---- occupancy index ------------------------------------------------------------
// Word ranks (exclusive popcount prefixes) and the occupied keys in rank order,
// in two kernels over tiles of 256 grid words: the tiles' popcounts, a tile
// per wave; then, per tile, the sum of the tiles before it (scanned by one
// workgroup in between if there are many), the ranks of its words, and their
// keys, laid out in LDS at their ranks (at most 32 per word) and stored as
// contiguous rows with the component-size counters of the ranks, cleared on
// the way (the labelling accumulates into them).  With the ranks and the keys
// in a kernel each, the second read bits and ranks again: a 400x400x200 grid
// took 18 us and takes 14.5, one of 800x800x400 85 and 67.  (With the keys of
// 1024 words per workgroup 28: the dense rows of a floor hold few of them up.)
constexpr uint32_t kRankTile = kBlock;          // words per tile
constexpr uint32_t kRankDirectTiles = 4096;     // up to this many a tile sums those before it itself

__global__ void __launch_bounds__(kBlock) k_rank_tiles(const uint32_t* __restrict__ bits, uint32_t nwords, uint32_t nt,
                                                       Vec<1>* __restrict__ blk)
{
    constexpr int kPerLane = kRankTile / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t waves = gridDim.x * (kBlock / kWave);
    for (uint32_t t = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; t < nt; t += waves) {
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const uint32_t w = t * kRankTile + j * kWave + lane;
            c += w < nwords ? (uint32_t)__popc(bits[w]) : 0u;
        }
#pragma unroll
        for (int d = kWave / 2; d >= 1; d >>= 1) c += __shfl_xor(c, d, kWave);
        if (lane == 0) blk[t].v[0] = c;
    }
}

__global__ void __launch_bounds__(kBlock) k_rank_keys(const uint32_t* __restrict__ bits, uint32_t nwords, uint32_t nt,
                                                      const Vec<1>* __restrict__ blk, bool scanned,
                                                      uint32_t* __restrict__ wrank, uint32_t* __restrict__ occ_key,
                                                      uint32_t* __restrict__ csize, DevCounters* __restrict__ ctr)
{
    __shared__ uint16_t keys[kRankTile * 32];   // from the tile's first cell
    __shared__ Vec<1> lds[kBlock / kWave];
    for (uint32_t t = blockIdx.x; t < nt; t += gridDim.x) {
        const uint32_t w = t * kRankTile + threadIdx.x;
        uint32_t b = w < nwords ? bits[w] : 0u;
        Vec<1> pre{{0u}}, n, c{{(uint32_t)__popc(b)}};
        if (scanned) {
            pre = blk[t];
        } else {
            Vec<1> p{{0u}};
#pragma unroll 4
            for (uint32_t q = threadIdx.x; q < t; q += kBlock) p.v[0] += blk[q].v[0];
            ts_block_excl(p, lds, &pre);
        }
        uint32_t q = ts_block_excl(c, lds, &n).v[0];
        if (w < nwords) wrank[w] = pre.v[0] + q;
        for (; b; b &= b - 1, ++q) keys[q] = (uint16_t)((threadIdx.x << 5) | (uint32_t)(__ffs(b) - 1));
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n.v[0]; i += kBlock) {
            occ_key[pre.v[0] + i] = t * kRankTile * 32u + keys[i];
            csize[pre.v[0] + i] = 0u;
        }
        if (t + 1 == nt && threadIdx.x == 0) ctr->n_occ = pre.v[0] + n.v[0];
        __syncthreads();   // keys is reused by the next tile
    }
}

__global__ void __launch_bounds__(kBlock) k_export(Geom g, Hash h, const uint32_t* __restrict__ occ_key,
                                                   const DevCounters* __restrict__ ctr, uint32_t* key_out,
                                                   uint32_t* cnt_out, unsigned long long* sum_out, float* mean_out,
                                                   uint64_t cap, uint32_t* __restrict__ n_host)
{
    const uint64_t n = ctr->n_occ < cap ? ctr->n_occ : cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_host = ctr->n_occ;
    for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t k = occ_key[r];
        // linear probing as in hash_find, with the whole slot in one read
        uint32_t s = hash_slot(k, h.log2cap);
        Slot sl = h.slot[s];
        for (uint32_t p = 1; sl.key != k && sl.key != kEmpty && p < kMaxProbe && p <= h.mask; ++p) {
            s = (s + 1) & h.mask;
            sl = h.slot[s];
        }
        const bool found = sl.key == k;
        const uint32_t c = found ? sl.cnt : 0u;
        const unsigned long long sx = found ? sl.sum[0] : 0, sy = found ? sl.sum[1] : 0, sz = found ? sl.sum[2] : 0;
        if (key_out) key_out[r] = k;
        if (cnt_out) cnt_out[r] = c;
        if (sum_out) {
            sum_out[3 * r + 0] = sx;
            sum_out[3 * r + 1] = sy;
            sum_out[3 * r + 2] = sz;
        }
        if (mean_out && c) {
            const uint32_t ix = k % (uint32_t)g.dims[0];
            const uint32_t iy = (k / (uint32_t)g.dims[0]) % (uint32_t)g.dims[1];
            const uint32_t iz = k / ((uint32_t)g.dims[0] * (uint32_t)g.dims[1]);
            mean_out[3 * r + 0] = voxel_mean_axis(ix, sx, c, g.voxel_size, g.origin[0]);
            mean_out[3 * r + 1] = voxel_mean_axis(iy, sy, c, g.voxel_size, g.origin[1]);
            mean_out[3 * r + 2] = voxel_mean_axis(iz, sz, c, g.voxel_size, g.origin[2]);
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_import(Geom g, Hash h, uint32_t* __restrict__ bits, DevCounters* ctr,
                                                   const uint32_t* __restrict__ key, const uint32_t* __restrict__ cnt,
                                                   const unsigned long long* __restrict__ sum, uint64_t n)
{
    uint32_t n_new = 0, n_lost = 0;
    const uint64_t ncell = (uint64_t)g.dims[0] * (uint64_t)g.dims[1] * (uint64_t)g.dims[2];
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t k = key[i];
        if ((uint64_t)k >= ncell || cnt[i] == 0) { ++n_lost; continue; }   // not a voxel of this grid
        uint32_t s = hash_slot(k, h.log2cap);
        bool ok = false;
        for (uint32_t p = 0; p < kMaxProbe && p <= h.mask; ++p) {
            const uint32_t old = atomicCAS(&h.slot[s].key, kEmpty, k);
            if (old == kEmpty || old == k) { ok = true; break; }
            s = (s + 1) & h.mask;
        }
        if (!ok) { ++n_lost; continue; }
        h.slot[s].cnt = cnt[i];
        h.slot[s].sum[0] = sum[3 * i + 0];
        h.slot[s].sum[1] = sum[3 * i + 1];
        h.slot[s].sum[2] = sum[3 * i + 2];
        atomicOr(&bits[k >> 5], 1u << (k & 31));
        ++n_new;
    }
    {
        unsigned long long* const dst[1] = {&ctr->occupied};
        const uint32_t v[1] = {n_new};
        block_add_counters<1>(dst, v);
    }
    if (n_lost) atomicOr(&ctr->flags, (uint32_t)VM_FLAG_HASH_FULL);
}

// ---- scrolling (the robot-centric map): a whole-voxel shift of the grid ------------
// 1. k_scroll_gather: every ranked voxel's slot content, with its key in the
//    shifted grid (kEmpty when it leaves), into staging arrays (32 bytes per
//    voxel: new key, count, the three sums as 32-bit halves);
// 2. the hash and the occupancy bits are emptied (fill kernels);
// 3. k_scroll_scatter: the staged voxels that stay are inserted under their
//    new keys.  Rebuilding the hash also drops the slots of cleared voxels.
struct ScrollStage {
    uint32_t* key;
    uint32_t* cnt;
    uint32_t* s[6];   // sum0 lo, hi, sum1 lo, hi, sum2 lo, hi
};

__global__ void __launch_bounds__(kBlock) k_scroll_gather(Geom g, Hash h, const DevCounters* __restrict__ ctr,
                                                          const uint32_t* __restrict__ occ_key, int32_t dx, int32_t dy,
                                                          int32_t dz, ScrollStage st)
{
    const uint32_t V = ctr->n_occ;
    const int64_t NX = g.dims[0], NY = g.dims[1], NZ = g.dims[2];
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += gridDim.x * blockDim.x) {
        const uint32_t k = occ_key[r];
        const int64_t x = (int64_t)(k % (uint32_t)NX) - dx, y = (int64_t)((k / (uint32_t)NX) % (uint32_t)NY) - dy,
                      z = (int64_t)(k / ((uint32_t)NX * (uint32_t)NY)) - dz;
        const bool in = x >= 0 && y >= 0 && z >= 0 && x < NX && y < NY && z < NZ;
        const uint32_t s = hash_find(h, k);
        Slot sl{};
        if (s != kEmpty) sl = h.slot[s];
        st.key[r] = in && s != kEmpty ? (uint32_t)(x + NX * (y + NY * z)) : kEmpty;
        st.cnt[r] = sl.cnt;
        for (int a = 0; a < 3; ++a) {
            st.s[2 * a][r] = (uint32_t)sl.sum[a];
            st.s[2 * a + 1][r] = (uint32_t)(sl.sum[a] >> 32);
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_fill_zero(uint32_t* __restrict__ p, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

// occupied restarts from zero (the scatter counts the voxels that stay); the
// voxels that leave are added to the scrolled-out counter
__global__ void k_scroll_counters(DevCounters* ctr)
{
    if (threadIdx.x == 0) ctr->occupied = 0ull;
}

__global__ void __launch_bounds__(kBlock) k_scroll_scatter(Hash h, uint32_t* __restrict__ bits, ScrollStage st,
                                                           DevCounters* ctr)
{
    uint32_t n_new = 0, n_out = 0, n_lost = 0;
    const uint32_t V = ctr->n_occ;
    const int lane = threadIdx.x & (kWave - 1);
    for (uint32_t b0 = blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); b0 < V; b0 += gridDim.x * blockDim.x) {
        const uint32_t r = b0 + (uint32_t)lane, k = r < V ? st.key[r] : kEmpty;
        bool ok = false;
        if (k != kEmpty) {
            uint32_t sum[6];
            const uint32_t cnt = st.cnt[r];   // (read while the slot is claimed)
#pragma unroll
            for (int a = 0; a < 6; ++a) sum[a] = st.s[a][r];
            uint32_t s = hash_slot(k, h.log2cap);
            for (uint32_t p = 0; p < kMaxProbe && p <= h.mask; ++p) {
                const uint32_t old = atomicCAS(&h.slot[s].key, kEmpty, k);
                if (old == kEmpty) { ok = true; break; }   // keys are distinct: never old == k
                s = (s + 1) & h.mask;
            }
            if (ok) {
                Slot* sl = &h.slot[s];
                sl->cnt = cnt;
                for (int a = 0; a < 3; ++a)
                    sl->sum[a] = (unsigned long long)sum[2 * a] | ((unsigned long long)sum[2 * a + 1] << 32);
                ++n_new;
            } else {
                ++n_lost;
            }
        } else if (r < V) {
            ++n_out;
        }
        // the occupancy bits, one atomic per word: a word's voxels are
        // neighbours in key order
        const uint32_t w = ok ? k >> 5 : kEmpty;
        uint32_t m = ok ? 1u << (k & 31) : 0u;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {   // (a word has at most 32 of them)
            const uint32_t om = __shfl_up(m, d, kWave), ow = __shfl_up(w, d, kWave);
            if (lane >= d && ow == w) m |= om;
        }
        const uint32_t next = __shfl_down(w, 1, kWave);
        if (ok && (lane == kWave - 1 || next != w)) atomicOr(&bits[w], m);
    }
    {
        unsigned long long* const dst[2] = {&ctr->occupied, &ctr->shifted_out};
        const uint32_t v[2] = {n_new, n_out};
        block_add_counters<2>(dst, v);
    }
    if (n_lost) atomicOr(&ctr->flags, (uint32_t)VM_FLAG_HASH_FULL);
}

// Empty slots, half a slot per thread so that a wave's stores are one row of
// 1 KB (with a slot per thread each store left gaps: 64 us for 268 MB, 41 so).
__device__ __forceinline__ void clear_slots(Slot* __restrict__ slot, uint32_t cap)
{
    static_assert(sizeof(Slot) == 2 * sizeof(uint4) && offsetof(Slot, key) == 0, "halves of a slot");
    uint4* p = reinterpret_cast<uint4*>(slot);
    const uint64_t n = 2 * (uint64_t)cap, stride = (uint64_t)gridDim.x * blockDim.x;
    const uint4 v = make_uint4(threadIdx.x & 1u ? 0u : kEmpty, 0u, 0u, 0u);   // (the stride is even)
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ void __launch_bounds__(kBlock) k_clear_slots(Slot* __restrict__ slot, uint32_t cap)
{
    clear_slots(slot, cap);
}

// slots, occupancy and counters of an empty map, in one launch
__global__ void __launch_bounds__(kBlock) k_clear_map(Slot* __restrict__ slot, uint32_t cap, uint32_t* __restrict__ bits,
                                                      uint32_t nwords, DevCounters* __restrict__ ctr)
{
    clear_slots(slot, cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += gridDim.x * blockDim.x) bits[i] = 0u;
    static_assert(sizeof(DevCounters) % 4 == 0 && sizeof(DevCounters) / 4 <= kBlock, "a word per thread");
    if (blockIdx.x == 0 && threadIdx.x < sizeof(DevCounters) / 4) reinterpret_cast<uint32_t*>(ctr)[threadIdx.x] = 0u;
}

__global__ void k_stats(const DevCounters* __restrict__ c, uint32_t log2cap, vm_map_stats_t* out)
{
    if (threadIdx.x == 0) {
        out->last_touched = c->touched;
        out->occupied = c->occupied;
        out->points_in = c->points_in;
        out->points_dropped = c->points_dropped;
        out->points_lost = c->points_lost;
        out->status_flags = c->flags;
        out->hash_capacity_log2 = log2cap;
        out->voxels_cleared = c->cleared;
        out->voxels_shifted_out = c->shifted_out;
    }
}

}  // namespace

hipError_t launch_stats(const DevCounters* ctr, uint32_t log2cap, vm_map_stats_t* out, hipStream_t s)
{
    k_stats<<<1, 64, 0, s>>>(ctr, log2cap, out);
    return hipGetLastError();
}

uint32_t bucket_log2(uint32_t m)
{
    uint32_t lb = 0;
    while (lb < kBucketMaxLog2 && ((uint64_t)kBucketAvg << lb) < m) ++lb;
    return lb;
}

// points per partition workgroup: as few rows of them as leave at most
// kBucketBlocks workgroups (bounds the histogram)
static uint32_t bucket_tile(uint32_t m)
{
    uint32_t t = kPartBlock;
    while ((uint64_t)t * kBucketBlocks < m) t <<= 1;
    return t;
}

size_t bucket_hist_words(uint32_t batch)
{
    const uint32_t tile = bucket_tile(batch);
    const uint32_t nblk = (batch + tile - 1) / tile;
    return ((size_t)(nblk + 2) << bucket_log2(batch)) + 1;   // rows, totals and starts
}

hipError_t launch_insert(const float* xyz, int64_t n, const Pose& pose, const Geom& g, const Hash& h,
                         uint32_t* bits, DevCounters* ctr, const InsertScratch& sc, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n < kSortedInsertMin || sc.cap == 0) {
        k_insert<<<grid_for((uint64_t)n, kBlock, kMapGrid), kBlock, 0, s>>>(xyz, n, pose, g, h, bits, ctr);
        return hipGetLastError();
    }
    for (int64_t done = 0; done < n; done += sc.cap) {
        const uint32_t m = (uint32_t)((n - done) < (int64_t)sc.cap ? (n - done) : (int64_t)sc.cap);
        // the batch size is known here, so grids and the bucket count follow it
        const uint32_t lb = bucket_log2(m);
        const uint32_t tile = bucket_tile(m);
        const uint32_t nblk = (m + tile - 1) / tile;
        uint32_t* total = sc.hist + ((size_t)nblk << lb);
        uint32_t* start = total + (1u << lb);
        k_bucket_count<<<nblk, kPartBlock, 0, s>>>(xyz + 3 * done, m, pose, g, lb, tile, done == 0, sc.hist, ctr);
        k_bucket_cols<<<((1u << lb) + kCols - 1) / kCols, kPartBlock, 0, s>>>(sc.hist, 1u << lb, nblk, total);
        k_bucket_scatter<<<nblk, kPartBlock, 0, s>>>(xyz + 3 * done, m, pose, g, lb, tile, sc.hist, total, start, sc.rec);
        k_bucket_insert<<<std::min(1u << lb, kInsertBlocks), kBlock, 0, s>>>(sc.rec, lb, start, h, bits, ctr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// words of launch_rank's tile totals
size_t rank_blk_words(uint32_t nwords) { return (size_t)(nwords + kRankTile - 1) / kRankTile; }

hipError_t launch_rank(const Geom& g, const uint32_t* bits, SegBuffers& b, DevCounters* ctr, hipStream_t s)
{
    Vec<1>* blk = reinterpret_cast<Vec<1>*>(b.blk);
    const uint32_t nt = (uint32_t)rank_blk_words(g.nwords);
    const bool scanned = nt > kRankDirectTiles;
    k_rank_tiles<<<grid_for((uint64_t)nt * kWave), kBlock, 0, s>>>(bits, g.nwords, nt, blk);
    if (scanned) k_tile_totals<1><<<1, kOneBlockThreads, 0, s>>>(blk, nt);
    k_rank_keys<<<grid_for(nt, 1, 16384), kBlock, 0, s>>>(bits, g.nwords, nt, blk, scanned, b.wrank, b.occ_key, b.csize,
                                                          ctr);
    return hipGetLastError();
}

hipError_t launch_clear(const Geom& g, const Hash& h, uint32_t* bits, DevCounters* ctr, hipStream_t s)
{
    const uint32_t cap = h.mask + 1;
    k_clear_map<<<grid_for(std::max<uint64_t>(cap, g.nwords / 4), kBlock, 16384), kBlock, 0, s>>>(h.slot, cap, bits,
                                                                                                  g.nwords, ctr);
    return hipGetLastError();
}

hipError_t launch_scroll(const Geom& g, const Hash& h, uint32_t* bits, SegBuffers& b, uint32_t cap, int32_t dx,
                         int32_t dy, int32_t dz, DevCounters* ctr, hipStream_t s)
{
    // staging in segmentation buffers that are free between frames
    ScrollStage st;
    st.key = b.parent;
    st.cnt = b.csize;
    st.s[0] = b.scan_a;
    st.s[1] = b.scan_b;
    st.s[2] = b.sort_k[0];
    st.s[3] = b.sort_k[1];
    st.s[4] = b.sort_v[0];
    st.s[5] = b.sort_v[1];
    k_scroll_gather<<<grid_for(cap), kBlock, 0, s>>>(g, h, ctr, b.occ_key, dx, dy, dz, st);
    const uint32_t hcap = h.mask + 1;
    k_clear_slots<<<grid_for(hcap, kBlock, 16384), kBlock, 0, s>>>(h.slot, hcap);
    k_fill_zero<<<grid_for(g.nwords), kBlock, 0, s>>>(bits, g.nwords);
    k_scroll_counters<<<1, kWave, 0, s>>>(ctr);
    k_scroll_scatter<<<grid_for(cap, kBlock, kMapGrid), kBlock, 0, s>>>(h, bits, st, ctr);
    return hipGetLastError();
}

hipError_t launch_export(const Geom& g, const Hash& h, const SegBuffers& b, const DevCounters* ctr, uint32_t* key,
                         uint32_t* cnt, unsigned long long* sum, float* mean, uint64_t cap,
                         uint32_t* n_host, hipStream_t s)
{
    k_export<<<grid_for(cap), kBlock, 0, s>>>(g, h, b.occ_key, ctr, key, cnt, sum, mean, cap, n_host);
    return hipGetLastError();
}

hipError_t launch_import(const Geom& g, const Hash& h, uint32_t* bits, DevCounters* ctr, const uint32_t* key,
                         const uint32_t* cnt, const unsigned long long* sum, uint64_t n, hipStream_t s)
{
    hipError_t e = launch_clear(g, h, bits, ctr, s);
    if (e != hipSuccess || n == 0) return e;
    k_import<<<grid_for(n, kBlock, kMapGrid), kBlock, 0, s>>>(g, h, bits, ctr, key, cnt, sum, n);
    return hipGetLastError();
}

}  // namespace vm
