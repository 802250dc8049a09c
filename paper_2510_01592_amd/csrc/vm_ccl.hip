// vm_ccl.hip -- connected-component labelling of the occupied voxels and the
// grouping of voxels into clusters (Sec. III-C, "Clustering", Alg. 1).
//
// Alg. 1 propagates the smaller label over every adjacency until nothing
// changes; from L_i = i its fixed point is the smallest index of each
// connected component.  That fixed point is reached here with a lock-free
// union-find over the occupied ranks (rank order == key order, so the
// smallest rank of a component is its smallest key):
//   * init:    every voxel points at the start of its run along x (runs of
//              consecutive occupied cells share a component trivially);
//   * merge:   runs in the four neighbouring rows with smaller keys
//              (dz = -1, any dy; dz = 0, dy = -1) are united, each pair of
//              touching runs once: inside tiles in LDS, then across their
//              faces;
//   * flatten: every voxel takes its root.
// Hooks always put the larger root under the smaller one with a CAS on the
// root, so every root ends as the minimum of its tree and the labels are
// exact whatever the interleaving.  Path halving keeps trees shallow.  The
// 26-neighbourhood never needs the hash: occupancy and ranks come from the
// 1-bit-per-cell index.
#include "vm_common.h"
#include "vm_dev.h"
#include "vm_tilescan.h"

#include <algorithm>

namespace vm {
namespace {

// Parent pointers are read through the ordinary caches.  A stale value is
// still an ancestor (parents only ever move to smaller ranks of the same
// component), so finds stay correct; the hook itself is a device-coherent
// CAS.  The path-halving and flattening stores are device-scope stores
// (written through to memory): with stores left in an XCD's L2, repeated
// labelling of one large map (5.3M voxels, 99k components) now and then left
// a voxel pointing at an intermediate ancestor after the flatten (3 calls in
// 400); with device-scope stores none did in 800.  Relaxed atomics keep the
// compiler from caching or tearing the accesses.
__device__ __forceinline__ uint32_t ld_parent(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

__device__ __forceinline__ void st_parent(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a moves to the root of its set and b to the root of its own, with path
// halving (each visited node is re-pointed at its grandparent; concurrent
// writes only ever store an ancestor); a step of one and a step of the other
// wait for memory together
__device__ __forceinline__ void uf_roots(uint32_t* parent, uint32_t& a, uint32_t& b)
{
    while (a != b) {
        const uint32_t pa = ld_parent(&parent[a]), pb = ld_parent(&parent[b]);
        const uint32_t ga = ld_parent(&parent[pa]), gb = ld_parent(&parent[pb]);
        const bool ra = ga == pa, rb = gb == pb;   // pa (pb) is a root
        if (!ra) st_parent(&parent[a], ga);
        if (!rb) st_parent(&parent[b], gb);
        a = ga;
        b = gb;
        if (ra && rb) return;
    }
}

__device__ __forceinline__ void uf_unite(uint32_t* parent, uint32_t a, uint32_t b)
{
    uf_roots(parent, a, b);
    while (a != b) {
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        const uint32_t old = atomicCAS(&parent[a], a, b);   // hook root a under b
        if (old == a) return;
        a = old;
        uf_roots(parent, a, b);
    }
}

struct Dims {
    uint32_t nx, ny, nz;
};


// ---- tiled labelling ------------------------------------------------------------
// The grid is cut into 32 x 16 x 16-cell tiles, one workgroup each.  Thread
// j of the workgroup owns local row j (y = j % 16, z = j / 16), 32 cells along
// x as one 32-bit occupancy word.  Inside a tile the components are found with
// a union-find in LDS over the runs of the rows (a row holds at most 16
// runs; run q of row j has index 16 j + q, hooked with LDS CAS); run index
// order is the order of the runs' first keys, so every local root is the
// smallest key of its local component.  Each occupied voxel then stores, as
// its global parent, the rank of its local root.  Adjacencies that cross a
// tile face are hooked afterwards by k_ccl_boundary with the global
// union-find; only those need device-wide atomics.
constexpr int kTX = 32, kTY = 16, kTZ = 16;
constexpr int kTileRows = kTY * kTZ;          // 256 = threads per workgroup
constexpr int kRowRuns = kTX / 2;             // runs per row at most
constexpr int kTileRuns = kTileRows * kRowRuns;   // 4096
static_assert(kTileRows == kBlock, "one thread per tile row");
constexpr int kJumps = 16;   // steps towards the root before the unions, a walk's first ones

struct TileGrid {
    uint32_t ntx, nty, ntz;
};

// Workgroups are dealt to the eight XCDs in turn, each with its own L2.  The
// loop index v (v % 8 names its XCD while the grid is a multiple of 8) is
// mapped so that every row of tiles along x (which share bitmap, rank and
// parent lines) is visited on one XCD, and rows go to the XCDs in turn (the
// map's dense regions stay spread over all of them).  Indices past the last
// row map to no tile.
constexpr uint32_t kXcds = 8;

__host__ __device__ inline uint32_t xcd_virtual_tiles(const TileGrid& tg)
{
    const uint32_t rows = tg.nty * tg.ntz;
    return kXcds * tg.ntx * ((rows + kXcds - 1) / kXcds);
}

__device__ __forceinline__ bool xcd_tile(uint32_t v, const TileGrid& tg, uint32_t* t)
{
    const uint32_t x = v % kXcds, i = v / kXcds;
    const uint32_t row = x + kXcds * (i / tg.ntx);
    *t = row * tg.ntx + i % tg.ntx;
    return row < tg.nty * tg.ntz;
}

// 32 occupancy bits of grid row (y, z) starting at x0 (bits beyond NX cleared)
__device__ __forceinline__ uint32_t row_bits(const uint32_t* __restrict__ bits, uint32_t nwords, const Dims& d,
                                             uint32_t x0, uint32_t y, uint32_t z, uint32_t* key0_out)
{
    if (y >= d.ny || z >= d.nz) {
        *key0_out = 0;
        return 0u;
    }
    const uint32_t key0 = x0 + d.nx * (y + d.ny * z);
    *key0_out = key0;
    const uint32_t w = key0 >> 5, sh = key0 & 31;
    uint32_t v = bits[w] >> sh;
    if (sh && w + 1 < nwords) v |= bits[w + 1] << (32 - sh);
    const uint32_t xcount = d.nx - x0 < 32u ? d.nx - x0 : 32u;
    if (xcount < 32u) v &= (1u << xcount) - 1u;
    return v;
}

// first cells of the runs of w, and last cells
__device__ __forceinline__ uint32_t run_starts(uint32_t w) { return w & ~(w << 1); }
__device__ __forceinline__ uint32_t run_ends(uint32_t w) { return w & ~(w >> 1); }

// rank of the first cell of a row segment (occupied cells with smaller keys)
__device__ __forceinline__ uint32_t seg_rank0(const uint32_t* __restrict__ bits, const uint32_t* __restrict__ wrank,
                                              uint32_t key0)
{
    return wrank[key0 >> 5] + __popc(bits[key0 >> 5] & ((1u << (key0 & 31)) - 1u));
}

// Hooks between the runs of row segment v and those of an adjacent row
// segment w (same x range), as masks of the cells xl of v: with cell xl of w
// for the bits of a, with xl - 1 for those of b and with xl + 1 for those of
// c.  Two runs touch iff their x ranges, one widened by a cell on each side,
// overlap: an overlap begins where the run of v or the run of w starts (a);
// a purely diagonal touch is the start of one run against the end of the
// other (b and c).
struct HookMasks {
    uint32_t a, b, c;
};

__device__ __forceinline__ HookMasks hook_masks(uint32_t v, uint32_t w)
{
    const uint32_t sv = run_starts(v), ev = run_ends(v);
    const uint32_t m = v & (sv | ev | run_starts(w));
    HookMasks h;
    h.a = m & w & (sv | ~(w << 1));
    h.b = m & sv & (w << 1);
    h.c = m & ev & (w >> 1);
    return h;
}

// LDS union-find.  Finds halve the path (a node is re-pointed at its
// grandparent: a store of an ancestor, harmless to concurrent finds), hooks
// put the larger root under the smaller one with a CAS on the root.
__device__ __forceinline__ uint32_t lds_ld(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void lds_st(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// a moves to the root of its set and b to the root of its own, a step of each
// at a time, so that the two walks wait for LDS together
__device__ __forceinline__ void lds_roots(uint32_t* par, uint32_t& a, uint32_t& b)
{
    while (a != b) {
        const uint32_t pa = lds_ld(&par[a]), pb = lds_ld(&par[b]);
        const uint32_t ga = lds_ld(&par[pa]), gb = lds_ld(&par[pb]);
        const bool ra = ga == pa, rb = gb == pb;   // pa (pb) is a root
        if (!ra) lds_st(&par[a], ga);
        if (!rb) lds_st(&par[b], gb);
        a = ga;
        b = gb;
        if (ra && rb) return;
    }
}

// Root of x without writing anything on the way, for when the unions are
// done and other threads are storing roots: a path-halving store could
// replace the root another thread has just stored for a node by an
// intermediate ancestor.
__device__ __forceinline__ uint32_t lds_root(const uint32_t* par, uint32_t x)
{
    uint32_t p = lds_ld(&par[x]);
    while (p != x) {
        x = p;
        p = lds_ld(&par[x]);
    }
    return x;
}

// unites the sets of a and b; returns a node above both
__device__ __forceinline__ uint32_t lds_unite(uint32_t* par, uint32_t a, uint32_t b)
{
    lds_roots(par, a, b);
    while (a != b) {
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        const uint32_t old = atomicCAS(&par[a], a, b);
        if (old == a) return b;
        a = old;
        lds_roots(par, a, b);
    }
    return a;
}

// ordinal of that run in its row (runs counted from x = 0)
__device__ __forceinline__ uint32_t run_ordinal(uint32_t starts, int x)
{
    return (uint32_t)__popc(starts & ((2u << x) - 1u)) - 1u;
}

// The workgroup's runs are numbered through (a row's first number is its
// prefix), so that each step below gives every thread as many runs as any
// other, however the runs lie.  A run first takes one run it touches as its
// parent, with a plain store (only its own entry, a smaller number); pointers
// are then jumped, after which most of the other touching pairs already have
// one root and take two reads and no CAS.  (With rows as the unit, their pairs
// listed and each united from scratch, the longest row and the longest chain
// of a wave set the pace: a map of 916k voxels took 38 us and takes 26,
// one of 29k, with a tile per compute unit, 30 and 13.)
__global__ void __launch_bounds__(kBlock) k_ccl_tile(const uint32_t* __restrict__ bits, uint32_t nwords,
                                                     const uint32_t* __restrict__ wrank, Dims d, TileGrid tg,
                                                     uint32_t* __restrict__ parent, uint32_t* __restrict__ csize)
{
    __shared__ uint32_t rowv[kTileRows];
    __shared__ uint32_t rowrank[kTileRows];
    __shared__ uint16_t rowbase[kTileRows];
    __shared__ uint16_t info[kTileRuns];   // a run's row and first cell: 32 row + x
    __shared__ uint32_t par[kTileRuns];
    __shared__ uint32_t wtot[kBlock / kWave];
    const uint32_t j = threadIdx.x;
    const int lane = (int)(j & (kWave - 1)), wave = (int)(j / kWave);
    const int yl = (int)(j % kTY), zl = (int)(j / kTY);
    // tiles in the XCD-ordered walk of the face kernel: a row of tiles along
    // x shares its bitmap and rank lines in one L2 (7 % faster than the
    // launch order once the per-run count atomics were gone; with them, the
    // launch order had been faster)
    const uint32_t nv = xcd_virtual_tiles(tg);
    for (uint32_t v0 = blockIdx.x; v0 < nv; v0 += gridDim.x) {
        uint32_t t;
        if (!xcd_tile(v0, tg, &t)) continue;
        const uint32_t tx = t % tg.ntx, ty = (t / tg.ntx) % tg.nty, tz = t / (tg.ntx * tg.nty);
        const uint32_t x0 = tx * kTX, y = ty * kTY + yl, z = tz * kTZ + zl;
        uint32_t key0;
        const uint32_t v = row_bits(bits, nwords, d, x0, y, z, &key0);
        // (unconditional, so that its loads overlap those of the row; rows
        // outside the grid read key 0, and empty rows' ranks are never used)
        const uint32_t rank0 = seg_rank0(bits, wrank, key0);
        const uint32_t sv = run_starts(v), cnt = (uint32_t)__popc(sv);
        uint32_t inc = cnt;
#pragma unroll
        for (int dd = 1; dd < kWave; dd <<= 1) {
            const uint32_t o = __shfl_up(inc, dd, kWave);
            if (lane >= dd) inc += o;
        }
        if (lane == kWave - 1) wtot[wave] = inc;
        rowv[j] = v;
        rowrank[j] = rank0;
        __syncthreads();
        uint32_t c0 = inc - cnt, nruns = 0;
#pragma unroll
        for (int w2 = 0; w2 < kBlock / kWave; ++w2) {
            const uint32_t t2 = wtot[w2];
            c0 += (w2 < wave) ? t2 : 0u;
            nruns += t2;
        }
        rowbase[j] = (uint16_t)c0;
        for (uint32_t m = sv; m; m &= m - 1, ++c0) info[c0] = (uint16_t)(32u * j + (uint32_t)__ffs(m) - 1u);
        __syncthreads();
        if (nruns == 0) continue;   // (block-uniform; the next write to LDS follows no read here)

        // f(number) for the runs that run c touches in the neighbouring rows
        // with smaller keys, until it returns false
        const auto touching = [&](uint32_t c, auto f) {
            const uint32_t in = info[c], row = in / 32u, s0 = in & 31u;
            const uint32_t e0 = (uint32_t)__ffs(run_ends(rowv[row]) >> s0) - 1u + s0;
            const uint32_t win = (~0u >> (31u - min(e0 + 1u, 31u))) & (~0u << (s0 ? s0 - 1u : 0u));
            const int ry = (int)(row % kTY), rz = (int)(row / kTY);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int dy = (q < 2) ? q - 1 : (q == 2 ? -1 : 1), dz = (q == 0) ? 0 : -1;
                if (ry + dy < 0 || ry + dy >= kTY || rz + dz < 0) continue;
                const uint32_t nr = (uint32_t)(ry + dy + kTY * (rz + dz)), w = rowv[nr], sw = run_starts(w);
                const uint32_t m0 = w & win;
                for (uint32_t m = run_starts(m0); m; m &= m - 1)
                    if (!f(rowbase[nr] + run_ordinal(sw, __ffs(m) - 1))) return;
            }
        };
        for (uint32_t c = j; c < nruns; c += kBlock) {
            uint32_t p = c;
            touching(c, [&](uint32_t o) {
                p = o;
                return false;
            });
            par[c] = p;
        }
        __syncthreads();
        // (a parent's entry may be jumped meanwhile: any value read is an ancestor)
        for (uint32_t c = j; c < nruns; c += kBlock) {
            uint32_t p = lds_ld(&par[c]);
#pragma unroll 1
            for (int i = 0; i < kJumps; ++i) {
                const uint32_t g = lds_ld(&par[p]);
                if (g == p) break;
                p = g;
                lds_st(&par[c], p);
            }
        }
        __syncthreads();
        for (uint32_t c = j; c < nruns; c += kBlock) {
            uint32_t a = c;
            bool first = true;
            touching(c, [&](uint32_t o) {
                if (!first) a = lds_unite(par, a, o);   // (the first is its parent)
                first = false;
                return true;
            });
        }
        __syncthreads();
        // roots of the runs (a run's entry then holds its root; every value
        // a walk reads is an ancestor or the root) ...
        for (uint32_t c = j; c < nruns; c += kBlock) lds_st(&par[c], lds_root(par, c));
        __syncthreads();
        // ... then each run adds its length to its root's count, kept in the
        // upper 16 bits of the root's entry (run numbers take 12 bits, a tile
        // holds at most 8192 cells)
        const auto run_len = [&](uint32_t row, uint32_t s0) { return (uint32_t)__ffs(run_ends(rowv[row]) >> s0); };
        for (uint32_t c = j; c < nruns; c += kBlock) {
            const uint32_t in = info[c];
            atomicAdd(&par[par[c] & 0xFFFFu], run_len(in / 32u, in & 31u) << 16);
        }
        __syncthreads();
        // global parents: the rank of the local root, for a whole run at once
        // (consecutive cells of a run have consecutive ranks); the local
        // root's entry of csize receives its component's voxel count in the
        // tile
        const auto rank_at = [&](uint32_t row, uint32_t x) { return rowrank[row] + __popc(rowv[row] & ((1u << x) - 1u)); };
        for (uint32_t c = j; c < nruns; c += kBlock) {
            const uint32_t in = info[c], pc = par[c], rt = pc & 0xFFFFu, ri = info[rt];
            const uint32_t rr = rank_at(ri / 32u, ri & 31u), r = rank_at(in / 32u, in & 31u);
            // the run's entries: single stores up to a 16-byte boundary, then
            // 16-byte stores, then the rest
            uint32_t p0 = r;
            const uint32_t pe = r + run_len(in / 32u, in & 31u);
            for (; p0 < pe && (p0 & 3u); ++p0) parent[p0] = rr;
            for (; p0 + 4 <= pe; p0 += 4) *reinterpret_cast<uint4*>(parent + p0) = make_uint4(rr, rr, rr, rr);
            for (; p0 < pe; ++p0) parent[p0] = rr;
            // the local root's count, stored once by the tile that owns it (no
            // device atomic: other tiles never write this entry here)
            if (rt == c) csize[r] = pc >> 16;
        }
        // LDS is reused by the next tile (a block with no next tile skips the
        // barrier, which would wait for the stores above to complete)
        if (v0 + gridDim.x < nv) __syncthreads();
    }
}

// A row segment of 32 cells from x0 with the cells beside it, and the rank of
// its first cell (occupied cells with smaller keys): `prev` and `next` have
// the ranks rank0 - 1 and rank0 + popc(v).  Four reads without a branch, so
// that those of several rows are in flight together.
struct Segment {
    uint32_t v, rank0;
    bool prev, next;
};

__device__ __forceinline__ Segment segment_at(const uint32_t* __restrict__ bits, uint32_t nwords,
                                              const uint32_t* __restrict__ wrank, const Dims& d, uint32_t x0,
                                              uint32_t y, uint32_t z)
{
    const bool ok = y < d.ny && z < d.nz;
    const uint32_t key0 = ok ? x0 + d.nx * (y + d.ny * z) : 0u, w = key0 >> 5, sh = key0 & 31u;
    const uint32_t a = bits[w ? w - 1u : 0u], b = bits[w], c = bits[min(w + 1u, nwords - 1u)], wr = wrank[w];
    Segment s;
    s.v = b >> sh;
    if (sh && w + 1u < nwords) s.v |= c << (32u - sh);
    const uint32_t n = min(d.nx - x0, 32u);
    if (n < 32u) s.v &= (1u << n) - 1u;
    if (!ok) s.v = 0u;
    s.prev = ok && x0 > 0u && ((sh ? b >> (sh - 1u) : a >> 31) & 1u);
    s.next = ok && x0 + 32u < d.nx && ((c >> sh) & 1u);
    s.rank0 = wr + (uint32_t)__popc(b & ((1u << sh) - 1u));
    return s;
}

// Cross-tile adjacencies, from the cell with the larger key.
//  * y/z faces: a row segment whose neighbouring row (dz = -1 any dy, or
//    dz = 0 and dy = -1) lies in another tile with the same x range hooks the
//    runs of the two segments with the run rule above (runs cut at the tile's
//    x edges are joined inside their tiles).
//  * x faces: the first cell of a segment links each occupied neighbour with
//    a smaller key at x - 1 (five of them), the last cell each one at x + 1
//    (four); these pairs lie in tiles of another x range.
// Each pair is replaced by the parents of its two voxels (the labelling pass
// left every voxel pointing at its tile-local root, and another tile's unions
// may have moved that on to another ancestor), and a tile keeps one copy of
// each distinct pair (an LDS hash set): along a dense surface many cells link
// the same two local components.  The distinct pairs are listed in LDS and
// united a thread each; pairs beyond the list are united where they are found.
// A row's reads (its own words, then those of its four neighbours with
// smaller keys, which also hold the cells beyond the x faces) are in flight
// together; cell by cell they were up to 18 waits in turn.  Each face pair of
// rows has a thread of its own: with up to four in a row's thread, the longest
// row of a wave set the pace of twelve loops in turn.  Unions by another
// kernel cost a launch and the list's way through memory: boundary and pairs
// took 28 + 12 us for 916k voxels, 18 + 9 for 29k (a tile per compute unit);
// now 28 and 14.
// Every pair has a cell of the tile, so an empty tile can end with the two words
// of its own rows, read before all else.  That pays where most tiles are empty
// (2000x2000x500 cells with 2000 points: 1059 us without, 387 so; with the empty
// tile left after a row's four reads 777) and is one more wait elsewhere (916k
// voxels in 400x400x200 cells, 217 a tile, 28 -> 32 us, 7.9M in 800x800x400, 254 a
// tile, 174 -> 198).  A tile that holds a surface has some 512 voxels, so with
// fewer than 64 a tile most are empty.
constexpr uint64_t kSkipVoxels = 64;

constexpr uint32_t kPairHash = 1024;   // LDS hash set of root pairs per tile
constexpr uint32_t kTilePairs = 256;   // distinct pairs listed per tile
constexpr uint32_t kRawPairs = 1024;   // voxel pairs gathered per tile before the root lookups

// The tile's pairs of a row and a neighbouring row (dy, dz) of smaller key in
// another tile, a thread each: 16 with dy = -1, dz = 0; 31 with dy = -1, 16
// with dy = 0 and 31 with dy = 1 at dz = -1 (the rows of the tile's lowest
// layer, and those at the y face).
constexpr uint32_t kFacePairs = 4 * kTY + 2 * (kTZ - 1);   // 94
static_assert(kTY == 16 && kTZ == 16 && kFacePairs <= kBlock, "a thread per face pair");

struct FacePair {
    int y, z, dy, dz;
};

__device__ __forceinline__ FacePair face_pair(uint32_t t)
{
    if (t < 64u) {   // the four neighbours of 16 rows: at the y face for dz = 0, else of the lowest layer
        const int i = (int)(t % 16u), q = (int)(t / 16u);
        return q == 0 ? FacePair{0, i, -1, 0} : FacePair{i, 0, q - 2, -1};
    }
    const int i = (int)(t - 64u);   // the higher layers' rows at the y faces, one layer down
    return i < kTZ - 1 ? FacePair{0, 1 + i, -1, -1} : FacePair{kTY - 1, i - (kTZ - 2), 1, -1};
}

__global__ void __launch_bounds__(kBlock) k_ccl_boundary(const DevCounters* __restrict__ ctr,
                                                         const uint32_t* __restrict__ bits, uint32_t nwords,
                                                         const uint32_t* __restrict__ wrank, Dims d, TileGrid tg,
                                                         uint32_t* parent)
{
    __shared__ uint64_t raw[kRawPairs];
    __shared__ uint64_t buf[kTilePairs];
    __shared__ unsigned long long hset[kPairHash];
    __shared__ uint32_t nbuf;
    const uint32_t j = threadIdx.x;
    const int yl = (int)(j % kTY), zl = (int)(j / kTY);
    // a distinct root pair goes to the tile's list (united in place if full)
    auto add_roots = [&](uint32_t ra, uint32_t rb) {
        const unsigned long long key = ((unsigned long long)ra << 32) | rb;
        uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 54);   // kPairHash = 2^10 slots
        for (uint32_t probe = 0; probe < kPairHash; ++probe) {
            const unsigned long long old = atomicCAS(&hset[h], ~0ull, key);
            if (old == key) return;          // this root pair is already listed
            if (old == ~0ull) break;         // first time
            h = (h + 1) & (kPairHash - 1);
        }
        const uint32_t i = atomicAdd(&nbuf, 1u);
        if (i < kTilePairs) buf[i] = key;
        else uf_unite(parent, ra, rb);
    };
    __shared__ uint32_t wtot[kBlock / kWave];
    const int lane = (int)(j & (kWave - 1)), wave = (int)(j / kWave);
    const uint32_t nv = xcd_virtual_tiles(tg);
    const bool skip = ctr->n_occ < kSkipVoxels * nv;
    for (uint32_t v0 = blockIdx.x; v0 < nv; v0 += gridDim.x) {
        uint32_t t;
        if (!xcd_tile(v0, tg, &t)) continue;   // uniform over the workgroup
        const uint32_t tx = t % tg.ntx, ty = (t / tg.ntx) % tg.nty, tz = t / (tg.ntx * tg.nty);
        const uint32_t x0 = tx * kTX;
        const int y = (int)(ty * kTY) + yl, z = (int)(tz * kTZ) + zl;
        if (skip) {
            uint32_t key0;
            if (!__syncthreads_or(row_bits(bits, nwords, d, x0, (uint32_t)y, (uint32_t)z, &key0) != 0u)) continue;
        }
        const Segment own = segment_at(bits, nwords, wrank, d, x0, (uint32_t)y, (uint32_t)z);
        if (j == 0) nbuf = 0;
        for (uint32_t i = j; i < kPairHash; i += kBlock) hset[i] = ~0ull;
        // first the voxel pairs (no loads of parents yet): each thread finds
        // and counts those of its row's ends and of one of the tile's face
        // pairs, a block scan places them in the raw list
        Segment fa, fb;
        HookMasks hm = {0, 0, 0};
        if (j < kFacePairs) {
            const FacePair fp = face_pair(j);
            const int fy = (int)(ty * kTY) + fp.y, fz = (int)(tz * kTZ) + fp.z;
            fa = segment_at(bits, nwords, wrank, d, x0, (uint32_t)fy, (uint32_t)fz);
            fb = segment_at(bits, nwords, wrank, d, x0, (uint32_t)(fy + fp.dy), (uint32_t)(fz + fp.dz));
            hm = hook_masks(fa.v, fb.v);
        }
        const uint32_t v = own.v, r0 = own.rank0;
        const bool first = (v & 1u) && x0 > 0, last = (v >> 31) & 1u;
        uint32_t cnt = (uint32_t)(__popc(hm.a) + __popc(hm.b) + __popc(hm.c));
        uint32_t fr[5], lr[4], fmask = 0, lmask = 0;
        if (first || last) {
            Segment nb[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                nb[q] = segment_at(bits, nwords, wrank, d, x0, (uint32_t)(y + (q == 0 ? -1 : q - 2)),
                                   (uint32_t)(z + (q == 0 ? 0 : -1)));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                fr[q] = nb[q].rank0 - 1u;
                lr[q] = nb[q].rank0 + (uint32_t)__popc(nb[q].v);
                fmask |= first && nb[q].prev ? 1u << q : 0u;
                lmask |= last && nb[q].next ? 1u << q : 0u;
            }
            fr[4] = r0 - 1u;
            fmask |= first && own.prev ? 1u << 4 : 0u;
            cnt += (uint32_t)(__popc(fmask) + __popc(lmask));
        }
        uint32_t inc = cnt;
#pragma unroll
        for (int dd = 1; dd < kWave; dd <<= 1) {
            const uint32_t o = __shfl_up(inc, dd, kWave);
            if (lane >= dd) inc += o;
        }
        if (lane == kWave - 1) wtot[wave] = inc;
        __syncthreads();
        uint32_t slot = inc - cnt, nraw = 0;
#pragma unroll
        for (int w2 = 0; w2 < kBlock / kWave; ++w2) {
            const uint32_t t2 = wtot[w2];
            slot += (w2 < wave) ? t2 : 0u;
            nraw += t2;
        }
        // ... then, a list's worth at a time, the local roots of the pairs,
        // deduplicated (nraw is block-uniform)
        for (uint32_t q0 = 0; q0 < nraw; q0 += kRawPairs) {
            if (cnt && slot < q0 + kRawPairs && slot + cnt > q0) {
                uint32_t sl = slot;
                auto emit = [&](uint32_t a, uint32_t b) {
                    if (sl >= q0 && sl < q0 + kRawPairs) raw[sl - q0] = ((uint64_t)a << 32) | b;
                    ++sl;
                };
                for (uint32_t m = hm.a | hm.b | hm.c; m; m &= m - 1) {
                    const int xa = __ffs(m) - 1;
                    const uint32_t bit = m & (0u - m), ra = fa.rank0 + (uint32_t)__popc(fa.v & (bit - 1u));
                    const uint32_t rb = fb.rank0 + (uint32_t)__popc(fb.v & (bit - 1u));   // of cell xa of the other row
                    if (hm.b & bit) emit(ra, rb - 1u);
                    if (hm.a & bit) emit(ra, rb);
                    if (hm.c & bit) emit(ra, rb + ((fb.v >> xa) & 1u));
                }
#pragma unroll
                for (int q = 0; q < 5; ++q)
                    if ((fmask >> q) & 1u) emit(r0, fr[q]);
                const uint32_t rl = r0 + (uint32_t)__popc(v) - 1u;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((lmask >> q) & 1u) emit(rl, lr[q]);
            }
            __syncthreads();
            const uint32_t nr = min(nraw - q0, kRawPairs);
            for (uint32_t i = j; i < nr; i += kBlock) {
                const uint64_t pr = raw[i];
                add_roots(ld_parent(&parent[(uint32_t)(pr >> 32)]), ld_parent(&parent[(uint32_t)pr]));
            }
            __syncthreads();
        }
        const uint32_t np = min(nbuf, kTilePairs);
        for (uint32_t i = j; i < np; i += kBlock) uf_unite(parent, (uint32_t)(buf[i] >> 32), (uint32_t)buf[i]);
        // LDS is reused by the next tile (a block with no next tile skips the
        // barrier, which would wait for the stores above to complete)
        if (v0 + gridDim.x < nv) __syncthreads();
    }
}

// After the merge every tree is final.  Each voxel walks to its root without
// writing anything on the way (a path-halving store here could overwrite the
// root another thread has just stored for that node) and stores only its own
// entry; every value a walk can read is an ancestor, so walks stay correct.
// A tile-local root joined to another tile's component hands its count to the
// component's root; a large component has many local roots, so a workgroup
// gathers the counts of its roots in LDS first (an atomic per wave and root,
// most of them on a floor's word, took most of the kernel's time: 2.4M voxels 33 us, so 21).
constexpr int kFlatBlock = 1024;
constexpr uint32_t kFlatSlots = 64;

__global__ void __launch_bounds__(kFlatBlock) k_ccl_flatten(const DevCounters* __restrict__ ctr, uint32_t* parent,
                                                            uint32_t* csize)
{
    __shared__ uint32_t root_of[kFlatSlots], count[kFlatSlots];
    const uint32_t V = ctr->n_occ;
    if (threadIdx.x < kFlatSlots) {
        root_of[threadIdx.x] = kEmpty;
        count[threadIdx.x] = 0;
    }
    __syncthreads();
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += stride) {
        // only roots receive counts below, and the count is used only when r
        // is not a root: it is final, and can be read before the walk
        const uint32_t own = csize[r];
        const uint32_t p0 = ld_parent(&parent[r]);
        uint32_t p = p0, x = r;
        while (p != x) {
            x = p;
            p = ld_parent(&parent[x]);
        }
        if (x != p0) st_parent(&parent[r], x);   // most voxels already point at their root
        if (x == r || own == 0) continue;
        const uint32_t at = (x * 0x9E3779B1u) >> 26;
        const uint32_t old = atomicCAS(&root_of[at], kEmpty, x);
        if (old == kEmpty || old == x) atomicAdd(&count[at], own);
        else atomicAdd(&csize[x], own);   // another root has the slot
    }
    __syncthreads();
    if (threadIdx.x < kFlatSlots && count[threadIdx.x]) atomicAdd(&csize[root_of[threadIdx.x]], count[threadIdx.x]);
}
static_assert(kFlatSlots == 1u << (32 - 26), "the slot is a hash's top bits");

// ---- grouping -------------------------------------------------------------------
// One fused scan over the ranks gives, in rank order: the cluster id of each
// root (kEmpty for components below min_cluster voxels) and the cluster
// offsets (running sum of the kept roots' sizes, i.e. clusters in label
// order).
struct GroupF {
    const uint32_t* parent;
    const uint32_t* csize;
    uint32_t* cid;
    uint32_t min_cluster;
    __device__ Vec<2> operator()(uint32_t r) const
    {
        const bool root = parent[r] == r;
        const uint32_t sz = root ? csize[r] : 0u;
        const bool kept = sz >= min_cluster;   // (min_cluster is at least 1)
        if (root && !kept) cid[r] = kEmpty;
        Vec<2> x;
        x.v[0] = kept ? 1u : 0u;
        x.v[1] = kept ? sz : 0u;
        return x;
    }
};

struct GroupG {
    uint32_t* cid;        // cluster id, at roots
    uint32_t* cl_off;
    uint32_t* cl_tag;
    const uint32_t* occ_key;
    DevCounters* ctr;
    __device__ void operator()(uint32_t r, const Vec<2>&, const Vec<2>& pre) const
    {
        cid[r] = pre.v[0];
        cl_off[pre.v[0]] = pre.v[1];
        cl_tag[pre.v[0]] = occ_key[r];
    }
    __device__ void total(const Vec<2>& t) const
    {
        ctr->meta[0] = t.v[0];
        ctr->meta[1] = t.v[1];
        cl_off[t.v[0]] = t.v[1];
        ctr->kmax = t.v[0] ? t.v[0] - 1 : 0;
    }
};

// The kept voxels in cluster-major order: a stable radix sort by cluster id
// (ascending keys inside each cluster).  11-bit digits: ids up to 2048, the
// usual case, take one pass, up to 4M two; the passes that the largest id of
// the frame does not need do nothing.  A pass is three launches:
//   hist:    digits per tile, digit-major; a tile is as many steps of 1024
//            items as leave about 1024 tiles (for 916k voxels one, and the
//            scatter takes 23 us, 30 with 2048 items a step; for 2.4M voxels
//            three, and the first two kernels take 28 us, 49 with one);
//   rows:    a workgroup per digit turns its row into prefixes and a total;
//   scatter: the digits' totals are scanned by every workgroup (2048 words
//            from L2), then the tile's voxels go to their places.
// The first pass takes the voxels by rank, straight from their roots, and
// leaves out those of no cluster; the last one that runs also looks up each
// voxel and writes the cluster points themselves.  (As pairs made by a kernel
// of their own, a sort with two scan kernels per pass and a gather after it,
// 916k voxels took 74 us from the scan on, and take 60; 29k took 47 and take 36.)
constexpr int kSortBits = 11;
constexpr uint32_t kSortBins = 1u << kSortBits;
constexpr int kSortIters = 4;
constexpr uint32_t kSortStep = kBlock * kSortIters;   // 1024 items, a workgroup's step
constexpr uint32_t kSortTiles = 1024;                 // tiles aimed at: a row of a histogram stays short
constexpr int kWaveSpan = kWave * kSortIters;         // a wave's voxels, consecutive

struct GroupSort {
    const DevCounters* ctr;
    const uint32_t* parent;
    const uint32_t* cid;
    const uint32_t* occ_key;
    uint32_t* k[2];       // cluster id and key of each kept voxel, between passes; k[1]: first every voxel's id
    uint32_t* v[2];
    uint32_t* hist;       // [digits * tiles]
    uint32_t* tot;        // [kSortBins]
    Geom g;
    Hash h;
    uint32_t* cl_key;
    float* cl_x;
    float* cl_y;
    float* cl_z;
};

// What pass p (shift = p * kSortBits) covers.
struct SortPass {
    uint32_t n, bins;     // items, digits in use
    uint32_t tile, nt;    // items per tile, tiles
    bool last, runs;
};

__device__ __forceinline__ SortPass sort_pass(const GroupSort& a, int shift)
{
    const uint32_t top = a.ctr->kmax >> shift;
    SortPass p;
    p.n = shift == 0 ? a.ctr->n_occ : a.ctr->meta[1];
    p.last = top < kSortBins;
    p.bins = p.last ? top + 1u : kSortBins;
    p.runs = shift == 0 || top != 0u;
    const uint32_t steps = (p.n + kSortStep - 1) / kSortStep;
    p.tile = max((steps + kSortTiles - 1) / kSortTiles, 1u) * kSortStep;
    p.nt = (p.n + p.tile - 1) / p.tile;
    return p;
}

template <bool kFirst>
__global__ void __launch_bounds__(kBlock) k_group_hist(GroupSort a, int shift)
{
    __shared__ uint32_t cnt[kSortBins];
    const SortPass sp = sort_pass(a, shift);
    if (!sp.runs) return;
    const int src = (shift / kSortBits + 1) & 1, lane = threadIdx.x & (kWave - 1);
    for (uint32_t t = blockIdx.x; t < sp.nt; t += gridDim.x) {
        for (uint32_t d = threadIdx.x; d < sp.bins; d += kBlock) cnt[d] = 0;
        __syncthreads();
        const uint32_t end = min((t + 1) * sp.tile, sp.n);
        for (uint32_t i0 = t * sp.tile + threadIdx.x; i0 - threadIdx.x < end; i0 += kSortStep) {
            uint32_t k[kSortIters];
#pragma unroll
            for (int j = 0; j < kSortIters; ++j) {
                const uint32_t i = i0 + j * kBlock;
                k[j] = i < end ? (kFirst ? a.cid[a.parent[i]] : a.k[src][i]) : kEmpty;
            }
            if (kFirst) {
#pragma unroll
                for (int j = 0; j < kSortIters; ++j)
                    if (i0 + j * kBlock < end) a.k[src][i0 + j * kBlock] = k[j];
            }
#pragma unroll
            for (int j = 0; j < kSortIters; ++j) {
                // neighbours are mostly of one cluster: the first one's lanes add together
                const bool in = k[j] != kEmpty;
                const uint32_t d = (k[j] >> shift) & (kSortBins - 1);
                const uint64_t m = __ballot(in);
                if (m == 0) continue;
                const int lead = __ffsll((long long)m) - 1;
                const uint32_t dl = __shfl(d, lead, kWave);
                const bool same = in && d == dl;
                const uint32_t c = (uint32_t)__popcll(__ballot(same));
                if (lane == lead) atomicAdd(&cnt[d], c);
                else if (in && !same) atomicAdd(&cnt[d], 1u);
            }
        }
        __syncthreads();
        for (uint32_t d = threadIdx.x; d < sp.bins; d += kBlock) a.hist[(size_t)d * sp.nt + t] = cnt[d];
        __syncthreads();   // cnt is reused by the next tile
    }
}

__global__ void __launch_bounds__(kBlock) k_group_rows(GroupSort a, int shift)
{
    __shared__ Vec<1> lds[kBlock / kWave];
    const SortPass sp = sort_pass(a, shift);
    if (!sp.runs) return;
    const uint32_t nt = sp.nt;
    for (uint32_t d = blockIdx.x; d < sp.bins; d += gridDim.x) {
        uint32_t* row = a.hist + (size_t)d * nt;
        uint32_t carry = 0;
        for (uint32_t t0 = 0; t0 < nt; t0 += 4 * kBlock) {
            const uint32_t t = t0 + 4 * threadIdx.x;
            uint32_t x[4];
            Vec<1> s{{0u}}, all;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[j] = t + j < nt ? row[t + j] : 0u;
                s.v[0] += x[j];
            }
            uint32_t run = carry + ts_block_excl(s, lds, &all).v[0];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (t + j < nt) row[t + j] = run;
                run += x[j];
            }
            carry += all.v[0];
        }
        if (threadIdx.x == 0) a.tot[d] = carry;
    }
}

template <bool kFirst>
__global__ void __launch_bounds__(kBlock) k_group_scatter(GroupSort a, int shift)
{
    constexpr int kWaves = kBlock / kWave;
    constexpr uint32_t kOwn = kSortBins / kBlock;   // digits of a thread, consecutive
    __shared__ uint32_t place[kWaves][kSortBins];   // counts, then places, of each wave's digits
    __shared__ Vec<1> lds[kWaves];
    const SortPass sp = sort_pass(a, shift);
    if (!sp.runs) return;
    const uint32_t bins = sp.bins;
    const bool last = sp.last;
    const int src = (shift / kSortBits + 1) & 1;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = threadIdx.x / kWave;
    if (blockIdx.x >= sp.nt) return;
    uint32_t tot[kOwn];
    Vec<1> s{{0u}}, all;
#pragma unroll
    for (uint32_t q = 0; q < kOwn; ++q) {
        const uint32_t d = threadIdx.x * kOwn + q;
        tot[q] = d < bins ? a.tot[d] : 0u;
        s.v[0] += tot[q];
    }
    const uint32_t first = ts_block_excl(s, lds, &all).v[0];   // items of the digits before this thread's
    const uint64_t lt = (1ull << lane) - 1ull;
    for (uint32_t t = blockIdx.x; t < sp.nt; t += gridDim.x) {
        // the places of the tile's next item of each of this thread's digits
        uint32_t at[kOwn], run = first;
#pragma unroll
        for (uint32_t q = 0; q < kOwn; ++q) {
            const uint32_t d = threadIdx.x * kOwn + q;
            at[q] = run + (d < bins ? a.hist[(size_t)d * sp.nt + t] : 0u);
            run += tot[q];
        }
        const uint32_t end = min((t + 1) * sp.tile, sp.n);
        for (uint32_t s0 = t * sp.tile; s0 < end; s0 += kSortStep) {
            const uint32_t i0 = s0 + wave * kWaveSpan + (uint32_t)lane;
            uint32_t k[kSortIters], v[kSortIters], p[kSortIters];
#pragma unroll
            for (int j = 0; j < kSortIters; ++j) {
                const uint32_t i = i0 + j * kWave;
                k[j] = i < end ? a.k[src][i] : kEmpty;
                v[j] = i < end ? (kFirst ? a.occ_key[i] : a.v[src][i]) : 0u;
            }
            // the last pass writes the points: the first probes of all its slots
            // are in flight while the places are found, and a probe loads the
            // whole 32-byte slot, so a hit needs no second load for the sums
            Slot sl[kSortIters];
            if (last) {
#pragma unroll
                for (int j = 0; j < kSortIters; ++j)
                    sl[j] = a.h.slot[k[j] != kEmpty ? hash_slot(v[j], a.h.log2cap) : 0u];
            }
            for (uint32_t d = threadIdx.x; d < bins; d += kBlock) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) place[w][d] = 0;
            }
            __syncthreads();
            // a wave counts its digits in item order and notes each item's number
            // among the wave's items of its digit
#pragma unroll
            for (int j = 0; j < kSortIters; ++j) {
                const bool in = k[j] != kEmpty;
                const uint32_t d = (k[j] >> shift) & (kSortBins - 1);
                uint64_t m = __ballot(in);   // the lanes with this lane's digit
#pragma unroll
                for (int b = 0; b < kSortBits; ++b) {
                    const bool bit = (d >> b) & 1u;
                    const uint64_t bb = __ballot(in && bit);
                    m &= bit ? bb : ~bb;
                }
                p[j] = 0;
                if (in) p[j] = place[wave][d] + (uint32_t)__popcll(m & lt);
                dev::wave_sync();
                if (in && (m & lt) == 0) place[wave][d] += (uint32_t)__popcll(m);
                dev::wave_sync();
            }
            __syncthreads();
#pragma unroll
            for (uint32_t q = 0; q < kOwn; ++q) {
                const uint32_t d = threadIdx.x * kOwn + q;
                if (d >= bins) continue;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const uint32_t c = place[w][d];
                    place[w][d] = at[q];
                    at[q] += c;
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kSortIters; ++j)
                if (k[j] != kEmpty) p[j] += place[wave][(k[j] >> shift) & (kSortBins - 1)];
            if (!last) {
#pragma unroll
                for (int j = 0; j < kSortIters; ++j)
                    if (k[j] != kEmpty) {
                        a.k[src ^ 1][p[j]] = k[j];
                        a.v[src ^ 1][p[j]] = v[j];
                    }
            } else {
                // the points: key and Eq. (1) mean of each voxel
                const uint32_t nx = (uint32_t)a.g.dims[0], ny = (uint32_t)a.g.dims[1];
                const uint32_t nprobe = a.h.mask < kMaxProbe ? a.h.mask + 1u : kMaxProbe;
#pragma unroll
                for (int j = 0; j < kSortIters; ++j) {
                    const uint32_t key = v[j], to = p[j];
                    if (k[j] == kEmpty) continue;
                    // linear probing as in hash_find
                    uint32_t sx = hash_slot(key, a.h.log2cap);
                    for (uint32_t q = 1; sl[j].key != key && sl[j].key != kEmpty && q < nprobe; ++q) {
                        sx = (sx + 1) & a.h.mask;
                        sl[j] = a.h.slot[sx];
                    }
                    float mx = 0.0f, my = 0.0f, mz = 0.0f;
                    if (sl[j].key == key) {
                        mx = voxel_mean_axis(key % nx, sl[j].sum[0], sl[j].cnt, a.g.voxel_size, a.g.origin[0]);
                        my = voxel_mean_axis((key / nx) % ny, sl[j].sum[1], sl[j].cnt, a.g.voxel_size, a.g.origin[1]);
                        mz = voxel_mean_axis(key / (nx * ny), sl[j].sum[2], sl[j].cnt, a.g.voxel_size, a.g.origin[2]);
                    }
                    a.cl_key[to] = key;
                    a.cl_x[to] = mx;
                    a.cl_y[to] = my;
                    a.cl_z[to] = mz;
                }
            }
            __syncthreads();   // place is reused by the next step
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_labels(const DevCounters* __restrict__ ctr,
                                                   const uint32_t* __restrict__ parent,
                                                   const uint32_t* __restrict__ occ_key, uint32_t* __restrict__ labels)
{
    const uint32_t V = ctr->n_occ;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += gridDim.x * blockDim.x)
        labels[r] = occ_key[parent[r]];
}

Dims dims_of(const Geom& g)
{
    Dims d;
    d.nx = (uint32_t)g.dims[0];
    d.ny = (uint32_t)g.dims[1];
    d.nz = (uint32_t)g.dims[2];
    return d;
}

}  // namespace

hipError_t launch_ccl(const Geom& g, const uint32_t* bits, SegBuffers& b, uint32_t cap, DevCounters* ctr,
                      hipStream_t s)
{
    const Dims d = dims_of(g);
    TileGrid tg;
    tg.ntx = (d.nx + kTX - 1) / kTX;
    tg.nty = (d.ny + kTY - 1) / kTY;
    tg.ntz = (d.nz + kTZ - 1) / kTZ;
    // the labelling and face kernels walk the XCD-ordered tile indices (a
    // multiple of 8, and so is 16384)
    const uint32_t nv = xcd_virtual_tiles(tg);
    const int vgrid = (int)(nv < 16384u ? nv : 16384u);
    {
        StageScope t(VM_STAGE_CCL, s);
        k_ccl_tile<<<vgrid, kBlock, 0, s>>>(bits, g.nwords, b.wrank, d, tg, b.parent, b.csize);
    }
    {
        StageScope t(VM_STAGE_CCL_LINK, s);
        k_ccl_boundary<<<vgrid, kBlock, 0, s>>>(ctr, bits, g.nwords, b.wrank, d, tg, b.parent);
        k_ccl_flatten<<<grid_for(cap, kFlatBlock, 1024), kFlatBlock, 0, s>>>(ctr, b.parent, b.csize);
    }
    return hipGetLastError();
}

// words of the sort's histograms and digit totals
size_t group_hist_words(uint64_t cap)
{
    return (size_t)kSortBins * (std::min<uint64_t>((cap + kSortStep - 1) / kSortStep, kSortTiles) + 1);
}

hipError_t launch_group(const Geom& g, const Hash& h, SegBuffers& b, uint32_t cap, uint32_t min_cluster,
                        uint32_t* d_labels, DevCounters* ctr, hipStream_t s)
{
    StageScope t(VM_STAGE_GROUP, s);
    if (min_cluster < 1) min_cluster = 1;
    const GroupF f{b.parent, b.csize, b.scan_a, min_cluster};
    const GroupG gg{b.scan_a, b.cl_off, b.cl_tag, b.occ_key, ctr};
    tile_scan<2>(f, gg, &ctr->n_occ, cap, reinterpret_cast<Vec<2>*>(b.blk), s);
    GroupSort a;
    a.ctr = ctr;
    a.parent = b.parent;
    a.cid = b.scan_a;
    a.occ_key = b.occ_key;
    for (int i = 0; i < 2; ++i) {
        a.k[i] = b.sort_k[i];
        a.v[i] = b.sort_v[i];
    }
    a.hist = b.hist;
    a.tot = b.hist + (group_hist_words(cap) - kSortBins);
    a.g = g;
    a.h = h;
    a.cl_key = b.cl_key;
    a.cl_x = b.cl_x;
    a.cl_y = b.cl_y;
    a.cl_z = b.cl_z;
    int tgrid = grid_for(cap, (int)kSortStep, (int)kSortTiles), dgrid = (int)kSortBins;
    k_group_hist<true><<<tgrid, kBlock, 0, s>>>(a, 0);
    k_group_rows<<<dgrid, kBlock, 0, s>>>(a, 0);
    k_group_scatter<true><<<tgrid, kBlock, 0, s>>>(a, 0);
    // the further passes mostly have nothing to do: small grids end sooner
    tgrid = std::min(tgrid, 512);
    dgrid = 512;
    const uint32_t kmax = cap / min_cluster;   // no more clusters than this
    for (int shift = kSortBits; shift < 32 && kmax >> shift; shift += kSortBits) {
        k_group_hist<false><<<tgrid, kBlock, 0, s>>>(a, shift);
        k_group_rows<<<dgrid, kBlock, 0, s>>>(a, shift);
        k_group_scatter<false><<<tgrid, kBlock, 0, s>>>(a, shift);
    }
    if (d_labels) k_labels<<<grid_for(cap), kBlock, 0, s>>>(ctr, b.parent, b.occ_key, d_labels);
    return hipGetLastError();
}

}  // namespace vm
