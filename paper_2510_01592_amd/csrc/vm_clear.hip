// vm_clear.hip -- free space along the sensor rays (Sec. III-B, Eq. (2)).
//
//   k_clear_prepare: a lane per point transformed as the insert does it, the
//                  cells holding a point of the frame, with a list of the
//                  first point found in each: points of one cell cast the
//                  same line (it runs from voxel to voxel), so one of them
//                  casts it.  Points outside the grid are all listed.
//   k_clear_cast:  a lane per listed point works out the 3D Bresenham line
//                  from the sensor's voxel towards it (its own voxel excluded,
//                  cut at the grid's faces); then the wave walks its lines
//                  four at a time, 16 lanes over the steps of each, marking
//                  every occupied voxel passed.  A mark is an atomic OR only
//                  when a plain read shows the bit still clear.
//   k_clear_apply: a thread per 32-cell word frees the cells marked on a ray
//                  and holding no point (count and sums zeroed in the hash
//                  slot, the occupancy bit cleared), and leaves the bitmaps
//                  zero for the next call.
// The cells' order.  For many rays the preparation also copies the occupancy
// into bricks of up to 8x8x8 cells beside the marks, 128 bytes a brick, so that
// neighbouring steps of a ray in any direction share a line.  That costs three
// passes over the grid, whatever the number of rays; few of them walk the
// occupancy index as it lies, with a bitmap of marks beside it (bricks_pay).
// The marks deduplicate the removal set: whatever the number of rays through a
// voxel, its slot is written once, by the one thread that owns its word, after
// every ray has been cast.
//
// What bounds the cast: VALU work per step (some 30 instructions) and the
// 16-cycle address rate of a gather.  A wave per line spent its time on the
// line's 64-bit divisions, made by all 64 lanes alike, and on one cache-line
// lookup per step, 200M steps for 1M points in the 4x4x2 m map: 794 us.  A lane
// per line's setup and a 4x4x4-cell occupancy in LDS took 538 us (spurious
// returns near the sensor, where every ray passes, fill the cubes), the bricks
// with four steps' reads in flight 400 us, and one line per end cell 170 us
// beside 76 us for the pass that lists them.
#include "vm_common.h"

#include <algorithm>

namespace vm {
namespace {

// A 32-cell word: which cells are occupied, and which of those lie on a ray.
// One read (in bricks, two in the grid's order) per step serves the test and the
// check whether the cell is marked already (the marks in it may be of a stale
// line: the atomic OR is then made once more).
struct CellWord {
    uint32_t occ, ray;
};

__device__ __forceinline__ bool unmarked(const CellWord w, uint32_t bit) { return (w.occ & ~w.ray & bit) != 0u; }

// The words by address: cells in bricks, or the occupancy index and the marks.
template <bool kBricked>
struct Cells {
    CellWord* brick;
    const uint32_t* bits;
    uint32_t* ray;

    template <typename A>
    __device__ __forceinline__ CellWord at(A a) const
    {
        if (!kBricked) return {bits[a >> 5], ray[a >> 5]};
        const uint2 v = *reinterpret_cast<const uint2*>(&brick[a >> 5]);
        return {v.x, v.y};
    }

    template <typename A>
    __device__ __forceinline__ void mark(A a) const
    {
        const uint32_t bit = 1u << ((uint32_t)a & 31u);
        if (unmarked(at(a), bit)) atomicOr(kBricked ? &brick[a >> 5].ray : &ray[a >> 5], bit);
    }
};

// Cells found by a wave, waiting in LDS for their marks: a device-scope atomic
// takes some two microseconds to return, and the reads issued after it wait
// behind it, so the marks are made in bursts.
constexpr uint32_t kMarkCap = 512;   // per wave

template <typename A>
struct MarkList {
    A* at;        // [kMarkCap] in LDS
    uint32_t n;   // wave-uniform

    __device__ __forceinline__ void push(bool hit, A a, int lane)
    {
        const uint64_t b = __ballot(hit);
        if (b == 0) return;
        if (hit) at[n + (uint32_t)__popcll(b & ((1ull << lane) - 1ull))] = a;
        n += (uint32_t)__popcll(b);
    }

    template <bool kBricked>
    __device__ __forceinline__ void flush(const Cells<kBricked>& cells, int lane)
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t i = (uint32_t)lane; i < n; i += kWave) cells.mark(at[i]);
        n = 0;
        __builtin_amdgcn_wave_barrier();
    }
};

// Bricked addresses.  A brick holds 2^e[0] x 2^e[1] x 2^e[2] cells (512 where
// the grid is large enough); a cell's address has the low bits of its
// coordinates in the lowest bits and the rest above, x and y padded to powers
// of two, so a coordinate's bits sit in two fields: bits [0, e) at p0, the
// rest at p1.  Such a dilated coordinate moves by a dilated increment with one
// add, the bits outside its fields being ones to carry across, and the
// address is the AND of the three.
struct Bricks {
    uint32_t e[3], p0[3], p1[3];
    uint64_t mask[3];        // the fields of each axis (z: everything from its p1 up)
    uint64_t words;          // 32-cell words of a bitmap
    uint32_t n[3];           // bricks that hold cells of the grid
    uint32_t log2words;      // words of a brick
    uint32_t used;           // words of those bricks
};

Bricks bricks_of(const Geom& g)
{
    Bricks b{};
    uint32_t full[3];   // bits of each axis
    for (int k = 0; k < 3; ++k) {
        full[k] = 0;
        while ((1ull << full[k]) < (uint64_t)g.dims[k]) ++full[k];
        b.e[k] = 0;
    }
    // nine bits dealt out evenly, x first, short axes leaving theirs to the others
    for (int left = 9, k = 0, dry = 0; left > 0 && dry < 3; k = (k + 1) % 3) {
        if (b.e[k] < full[k]) {
            ++b.e[k];
            --left;
            dry = 0;
        } else {
            ++dry;
        }
    }
    uint32_t p = 0;
    for (int k = 0; k < 3; ++k) {
        b.p0[k] = p;
        p += b.e[k];
    }
    for (int k = 0; k < 3; ++k) {
        b.p1[k] = p;
        if (k < 2) p += full[k] - b.e[k];
    }
    for (int k = 0; k < 3; ++k) {
        const uint64_t lo = ((1ull << b.e[k]) - 1ull) << b.p0[k];
        const uint64_t hi = k < 2 ? ((1ull << (full[k] - b.e[k])) - 1ull) << b.p1[k] : ~0ull << b.p1[2];
        b.mask[k] = lo | hi;
    }
    const uint64_t nz = ((uint64_t)g.dims[2] + (1ull << b.e[2]) - 1) >> b.e[2];
    b.words = ((nz << b.p1[2]) + 31) / 32;
    const uint32_t bits = b.e[0] + b.e[1] + b.e[2];
    b.log2words = bits > 5 ? bits - 5 : 0;
    for (int k = 0; k < 3; ++k) b.n[k] = (uint32_t)(((uint64_t)g.dims[k] + (1ull << b.e[k]) - 1) >> b.e[k]);
    // (each axis grows to less than twice its cells: below 2^35 of them)
    b.used = (uint32_t)(((uint64_t)b.n[0] * b.n[1] * b.n[2]) << b.log2words);
    return b;
}

// the dilated form of a (signed) number along an axis, zero outside its fields
template <typename A>
__device__ __forceinline__ A dilate(int32_t v, uint32_t e, uint32_t p0, uint32_t p1, A mask)
{
    const A x = (A)(int64_t)v;   // sign-extended
    return (((x & (((A)1 << e) - 1)) << p0) | ((A)((int64_t)v >> e) << p1)) & mask;
}

struct CastArgs {
    Pose pose;
    Geom g;
    Bricks br;
    int32_t s[3];            // the sensor's voxel
    CellWord* brick;         // occupancy and cells on a ray (occupied ones only), in bricks
    const uint32_t* bits;    // or the occupancy index
    uint32_t* ray;           // and the marks beside it
    const uint32_t* list;    // the points that cast a line
    const uint32_t* count;   // their number
    uint32_t* next;          // the next batch's number, cleared here
};

// coordinate v along axis k (0, 1, 2; per lane) as a part of an address: in
// bricks dilated, zero outside its fields, else times the axis' stride
template <typename A, bool kBricked>
__device__ __forceinline__ A along(const CastArgs& a, int32_t k, int32_t v)
{
    if (!kBricked) {
        const uint32_t nx = (uint32_t)a.g.dims[0];
        return (A)(uint32_t)v * (A)(k == 0 ? 1u : (k == 1 ? nx : nx * (uint32_t)a.g.dims[1]));
    }
    const Bricks& br = a.br;
    return dilate<A>(v, k == 0 ? br.e[0] : (k == 1 ? br.e[1] : br.e[2]),
                     k == 0 ? br.p0[0] : (k == 1 ? br.p0[1] : br.p0[2]),
                     k == 0 ? br.p1[0] : (k == 1 ? br.p1[1] : br.p1[2]),
                     (A)(k == 0 ? br.mask[0] : (k == 1 ? br.mask[1] : br.mask[2])));
}

// the ones outside axis k's fields that a step's add carries across
template <typename A, bool kBricked>
__device__ __forceinline__ A outside(const CastArgs& a, int32_t k)
{
    return kBricked ? ~(A)(k == 0 ? a.br.mask[0] : (k == 1 ? a.br.mask[1] : a.br.mask[2])) : (A)0;
}

// the address of three such parts (with the ones outside their fields)
template <typename A, bool kBricked>
__device__ __forceinline__ A address(A m, A u, A w)
{
    return kBricked ? m & u & w : m + u + w;
}

// bits [key, key + n) of the occupancy index, n <= 32
__device__ __forceinline__ uint32_t cells_at(const uint32_t* __restrict__ bits, uint32_t key, uint32_t n)
{
    const uint32_t b = key & 31u;
    uint32_t v = bits[key >> 5] >> b;
    if (b + n > 32u) v |= bits[(key >> 5) + 1u] << (32u - b);
    return n < 32u ? v & ((1u << n) - 1u) : v;
}

// The i-th word of the bricks that hold cells: the padding to powers of two is
// neither written nor read (a grid of 2100x2100x60 cells takes 33.5M words with
// it and 8.9M without).
__device__ __forceinline__ uint64_t used_word(const Bricks& br, uint32_t i)
{
    const uint32_t b = i >> br.log2words, w = i & ((1u << br.log2words) - 1u);
    const uint32_t by = b / br.n[0], bx = b - by * br.n[0], bz = by / br.n[1];
    const uint64_t at = (uint64_t)bx << br.p1[0] | (uint64_t)(by - bz * br.n[1]) << br.p1[1] | (uint64_t)bz << br.p1[2];
    return (at >> 5) + w;   // (a grid of less than a word is one brick, at 0)
}

// the cell at an address (z may lie past the grid, x and y in the padding)
__device__ __forceinline__ void cell_of(const Bricks& br, uint64_t at, uint32_t c[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t lo = (uint32_t)(at >> br.p0[k]) & ((1u << br.e[k]) - 1u);
        c[k] = lo | (uint32_t)((at & br.mask[k]) >> br.p1[k]) << br.e[k];
    }
}

// a point's voxel (floor division of the fixed-point coordinate), false for
// non-finite points or points absurdly far away (the negated test also
// rejects NaN)
__device__ __forceinline__ bool end_of(const float* __restrict__ xyz, int64_t i, const Pose& pose, const Geom& g,
                                       int64_t e[3])
{
    const double px = (double)xyz[3 * i + 0];
    const double py = (double)xyz[3 * i + 1];
    const double pz = (double)xyz[3 * i + 2];
    const double wx = fma(pose.R[2], pz, fma(pose.R[1], py, fma(pose.R[0], px, pose.t[0])));
    const double wy = fma(pose.R[5], pz, fma(pose.R[4], py, fma(pose.R[3], px, pose.t[1])));
    const double wz = fma(pose.R[8], pz, fma(pose.R[7], py, fma(pose.R[6], px, pose.t[2])));
    const double fx = floor((wx - g.origin[0]) * g.inv_q);
    const double fy = floor((wy - g.origin[1]) * g.inv_q);
    const double fz = floor((wz - g.origin[2]) * g.inv_q);
    if (!(fx >= -1e15 && fx <= 1e15 && fy >= -1e15 && fy <= 1e15 && fz >= -1e15 && fz <= 1e15)) return false;
    e[0] = (int64_t)fx >> 20;
    e[1] = (int64_t)fy >> 20;
    e[2] = (int64_t)fz >> 20;
    return true;
}

constexpr int kEndPoints = 4;
constexpr uint32_t kEndTile = kEndPoints * kBlock;
// One workgroup per compute unit: a point finds its cell set, and makes no
// device atomic, only if an earlier one's atomic has returned (1M points: 76
// us; all tiles at once 133-145 us, 512 workgroups 113 us).
constexpr int kEndBlocks = 256;

// The first `pblocks` workgroups take the points of the batch (indices below
// 2^32), the others, on the first batch of the bricked form, the words: their
// cells are rows of up to 2^e[0] cells along x.
template <typename A, bool kBricked>
__global__ void __launch_bounds__(kBlock) k_clear_prepare(const float* __restrict__ xyz, uint32_t n, Pose pose, Geom g,
                                                          Bricks br, uint32_t pblocks,
                                                          const uint32_t* __restrict__ bits,
                                                          CellWord* __restrict__ cells, uint32_t* ends,
                                                          uint32_t* __restrict__ list, uint32_t* __restrict__ count)
{
    if (blockIdx.x < pblocks) {
        // a tile's points, kEndPoints per thread: their reads and their atomics
        // are in flight together, and the tile takes its list positions with
        // one atomic (one per wave took 200 us for 1M points)
        __shared__ uint32_t wsum[kBlock / kWave];
        __shared__ uint32_t s_base;
        const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
        for (uint64_t t0 = (uint64_t)blockIdx.x * kEndTile; t0 < n; t0 += (uint64_t)pblocks * kEndTile) {
            A at[kEndPoints];
            bool first[kEndPoints], in[kEndPoints];
            uint32_t word[kEndPoints];
#pragma unroll
            for (int j = 0; j < kEndPoints; ++j) {
                const uint64_t i = t0 + (uint32_t)(j * kBlock) + threadIdx.x;
                int64_t e[3];
                first[j] = i < n && end_of(xyz, (int64_t)i, pose, g, e);
                in[j] = first[j] && e[0] >= 0 && e[1] >= 0 && e[2] >= 0 && e[0] < g.dims[0] && e[1] < g.dims[1] &&
                        e[2] < g.dims[2];
                at[j] = 0;
                if (!kBricked && in[j])
                    at[j] = (A)((uint32_t)e[0] + (uint32_t)g.dims[0] * ((uint32_t)e[1] + (uint32_t)g.dims[1] * (uint32_t)e[2]));
#pragma unroll
                for (int k = 0; kBricked && k < 3; ++k)
                    if (in[j]) at[j] |= dilate<A>((int32_t)e[k], br.e[k], br.p0[k], br.p1[k], (A)br.mask[k]);
            }
            // a plain read first: most points find their cell set
#pragma unroll
            for (int j = 0; j < kEndPoints; ++j)
                word[j] = __hip_atomic_load(&ends[at[j] >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
#pragma unroll
            for (int j = 0; j < kEndPoints; ++j) {
                const uint32_t bit = 1u << ((uint32_t)at[j] & 31u);
                if (in[j] && !(word[j] & bit)) word[j] = atomicOr(&ends[at[j] >> 5], bit);
            }
            uint32_t cnt = 0;
#pragma unroll
            for (int j = 0; j < kEndPoints; ++j) {
                if (in[j]) first[j] = !((word[j] >> ((uint32_t)at[j] & 31u)) & 1u);
                cnt += first[j] ? 1u : 0u;
            }
            uint32_t inc = cnt;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t o = __shfl_up(inc, d, kWave);
                if (lane >= d) inc += o;
            }
            if (lane == kWave - 1) wsum[wave] = inc;
            __syncthreads();
            uint32_t pos = inc - cnt, tot = 0;
#pragma unroll
            for (int w = 0; w < kBlock / kWave; ++w) {
                pos += w < wave ? wsum[w] : 0u;
                tot += wsum[w];
            }
            if (threadIdx.x == 0) s_base = tot ? atomicAdd(count, tot) : 0u;
            __syncthreads();
            pos += s_base;
#pragma unroll
            for (int j = 0; j < kEndPoints; ++j)
                if (first[j]) list[pos++] = (uint32_t)t0 + (uint32_t)(j * kBlock) + threadIdx.x;
            __syncthreads();   // wsum and s_base are reused by the next tile
        }
        return;
    }
    const uint32_t NX = (uint32_t)g.dims[0], NY = (uint32_t)g.dims[1], NZ = (uint32_t)g.dims[2];
    const uint32_t le = min(br.e[0], 5u), len = 1u << le;
    for (uint32_t i = (blockIdx.x - pblocks) * kBlock + threadIdx.x; i < br.used; i += (gridDim.x - pblocks) * kBlock) {
        const uint64_t w = used_word(br, i);
        uint32_t v = 0;
        for (uint32_t r = 0; r < 32u; r += len) {
            uint32_t c[3];
            cell_of(br, w * 32u + r, c);
            if (c[0] < NX && c[1] < NY && c[2] < NZ)
                v |= cells_at(bits, c[0] + NX * (c[1] + NY * c[2]), min(len, NX - c[0])) << r;
        }
        cells[w] = {v, 0u};
    }
}

// The Bresenham walk has a closed form: after k steps along the driving axis
// m, a minor axis with extent d has moved floor((2 d k + dm) / (2 dm)) times
// (the error-term rule, a step when the term reaches zero, unrolled).  The
// walk leaves the grid at the first step where some coordinate does (each
// moves one way only); that step is computed up front per axis, so every lane
// knows where to stop.

// A line too long for the 32-bit walk below (dm >= kFarSteps), by the whole
// wave: lane l takes steps l, l + 64, ... and keeps each minor coordinate as a
// quotient and remainder, advanced by the constant increments of 64 steps.
constexpr int64_t kFarSteps = 1 << 24;

template <typename A, bool kBricked>
__device__ __forceinline__ void walk_far(const CastArgs& a, const Cells<kBricked>& cells, int lane, int64_t dm, int64_t du, int64_t dw, int64_t nsteps,
                                         int m, int gm, int gu, int gw)
{
    const int u = m == 2 ? 0 : m + 1, w = m == 0 ? 2 : m - 1;
    const int64_t two_dm = 2 * dm;
    int64_t k = lane;
    const int64_t nu = 2 * du * lane + dm, nw = 2 * dw * lane + dm;
    int64_t U = nu / two_dm, ru = nu % two_dm, W = nw / two_dm, rw = nw % two_dm;
    const int64_t iu = 2 * du * kWave, iw = 2 * dw * kWave;
    const int64_t qu = iu / two_dm, pu = iu % two_dm, qw = iw / two_dm, pw = iw % two_dm;
    const A om = outside<A, kBricked>(a, m), ou = outside<A, kBricked>(a, u), ow = outside<A, kBricked>(a, w);
    for (; k < nsteps; k += kWave) {
        cells.mark(address<A, kBricked>(along<A, kBricked>(a, m, a.s[m] + gm * (int32_t)k) | om,
                                        along<A, kBricked>(a, u, a.s[u] + gu * (int32_t)U) | ou,
                                        along<A, kBricked>(a, w, a.s[w] + gw * (int32_t)W) | ow));
        U += qu;
        ru += pu;
        if (ru >= two_dm) {
            ++U;
            ru -= two_dm;
        }
        W += qw;
        rw += pw;
        if (rw >= two_dm) {
            ++W;
            rw -= two_dm;
        }
    }
}

// n / d and its remainder for n < 2^29, d >= 2 and a quotient of at most 16
// (the estimate from a 24-bit reciprocal is at most one off)
__device__ __forceinline__ void small_div(uint32_t n, uint32_t d, float rcp, uint32_t* q_out, uint32_t* r_out)
{
    uint32_t q = (uint32_t)((float)n * rcp);
    int32_t r = (int32_t)(n - q * d);
    if (r < 0) {
        --q;
        r += (int32_t)d;
    }
    if (r >= (int32_t)d) {
        ++q;
        r -= (int32_t)d;
    }
    *q_out = q;
    *r_out = (uint32_t)r;
}

// first step at which a coordinate starting at c and moving by g per move
// leaves [0, D), in steps of the driving axis: moves = floor((2 d k + dm) / (2 dm))
__device__ __forceinline__ int64_t exit_step(int64_t c, int32_t g, int64_t D, int64_t d, int64_t dm)
{
    const int64_t L = g > 0 ? D - c : c + 1;   // moves that stay inside
    if (d == 0) return (int64_t)0x7FFFFFFFFFFFFFFFll;
    return (2 * dm * L - dm + 2 * d - 1) / (2 * d);
}

// Lanes per line in the walk: a line of the 4x4x2 m map has some 200 steps, so
// 16 lanes waste a twentieth of their last round (64 would waste a fifth), and
// the setup that a walking lane does per line is shared by four lines.
constexpr int kRayLanes = 16;
constexpr int kStepBatch = 4;   // rounds of steps whose reads are in flight together

// the largest of the wave's lines (uniform within each group of kRayLanes lanes)
__device__ __forceinline__ int32_t wave_max(int32_t v)
{
    int32_t m = 0;
#pragma unroll
    for (int g = 0; g < kWave / kRayLanes; ++g) m = max(m, __builtin_amdgcn_readlane(v, g * kRayLanes));
    return m;
}

// A: the addresses' type (64 bits where the padded grid has 2^32 cells or more)
template <typename A, bool kBricked>
__global__ void __launch_bounds__(kBlock, 6) k_clear_cast(const float* __restrict__ xyz, CastArgs a)
{
    const int64_t n = *a.count;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.next = 0u;
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane % kRayLanes, grp = lane / kRayLanes;
    const int32_t NX = a.g.dims[0], NY = a.g.dims[1], NZ = a.g.dims[2];
    __shared__ A mark_lds[kBlock / kWave][kMarkCap];
    MarkList<A> marks{mark_lds[threadIdx.x / kWave], 0u};
    const Cells<kBricked> cells{a.brick, a.bits, a.ray};
    // the wave's contiguous share of the points, 64 at a time
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    const int64_t w = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const int64_t i1 = n * (w + 1) / waves;
    for (int64_t i0 = n * w / waves; i0 < i1; i0 += kWave) {
        // ---- the lane's own point and line ----
        const int64_t i = i0 + lane;
        int32_t m = 0, nsteps = 0;   // driving axis; steps (0: no line)
        int64_t dm = 0, du = 0, dw = 0, steps = 0;
        bool neg_m = false, neg_u = false, neg_w = false;
        if (i < i1) {
            int64_t e[3];
            if (end_of(xyz, (int64_t)a.list[i], a.pose, a.g, e)) {
                const int64_t e0 = e[0], e1 = e[1], e2 = e[2];
                // Bresenham on (driving axis m, minor axes u = m+1, w = m+2 mod 3)
                const int64_t d0 = e0 - a.s[0], d1 = e1 - a.s[1], d2 = e2 - a.s[2];
                const int64_t ad0 = d0 < 0 ? -d0 : d0, ad1 = d1 < 0 ? -d1 : d1, ad2 = d2 < 0 ? -d2 : d2;
                if (ad1 > ad0) m = 1;
                if (ad2 > (m == 0 ? ad0 : ad1)) m = 2;
                dm = m == 0 ? ad0 : (m == 1 ? ad1 : ad2);
                du = m == 0 ? ad1 : (m == 1 ? ad2 : ad0);
                dw = m == 0 ? ad2 : (m == 1 ? ad0 : ad1);
                neg_m = (m == 0 ? d0 : (m == 1 ? d1 : d2)) < 0;
                neg_u = (m == 0 ? d1 : (m == 1 ? d2 : d0)) < 0;
                neg_w = (m == 0 ? d2 : (m == 1 ? d0 : d1)) < 0;
                const int64_t Dm = m == 0 ? NX : (m == 1 ? NY : NZ);
                const int64_t Du = m == 0 ? NY : (m == 1 ? NZ : NX);
                const int64_t Dw = m == 0 ? NZ : (m == 1 ? NX : NY);
                const int64_t cm = m == 0 ? a.s[0] : (m == 1 ? a.s[1] : a.s[2]);
                const int64_t cu = m == 0 ? a.s[1] : (m == 1 ? a.s[2] : a.s[0]);
                const int64_t cw = m == 0 ? a.s[2] : (m == 1 ? a.s[0] : a.s[1]);
                if (dm > 0) {
                    steps = min(dm, neg_m ? cm + 1 : Dm - cm);
                    steps = min(steps, exit_step(cu, neg_u ? -1 : 1, Du, du, dm));
                    steps = min(steps, exit_step(cw, neg_w ? -1 : 1, Dw, dw, dm));
                }
                if (dm < kFarSteps) nsteps = (int32_t)steps;
            }
        }
        // the walk's increments over kRayLanes steps (quotients and remainders
        // of 2 d kRayLanes by 2 dm), and its axis and signs in one word
        const uint32_t two_dm = (uint32_t)(2 * dm);
        uint32_t pu = 0, pw = 0, qs = 0;
        if (nsteps > 0) {
            const float rcp = 1.0f / (float)two_dm;
            uint32_t qu, qw;
            small_div(2u * kRayLanes * (uint32_t)du, two_dm, rcp, &qu, &pu);
            small_div(2u * kRayLanes * (uint32_t)dw, two_dm, rcp, &qw, &pw);
            qs = qu | (qw << 8) | ((uint32_t)m << 16) | (neg_m ? 1u << 20 : 0u) | (neg_u ? 1u << 21 : 0u) |
                 (neg_w ? 1u << 22 : 0u);
        }
        // ---- the wave's lines, kWave / kRayLanes at a time ----
        for (int j = 0; j < kRayLanes; ++j) {
            const int src = j * (kWave / kRayLanes) + grp;
            const int32_t ns = __shfl(nsteps, src, kWave);
            if (__ballot(ns > 0) == 0) continue;
            const uint32_t tdm = __shfl(two_dm, src, kWave);
            const uint32_t sdu = (uint32_t)__shfl((int32_t)du, src, kWave), sdw = (uint32_t)__shfl((int32_t)dw, src, kWave);
            const uint32_t spu = __shfl(pu, src, kWave), spw = __shfl(pw, src, kWave), q = __shfl(qs, src, kWave);
            const int32_t ax = (int32_t)((q >> 16) & 3u);
            const int32_t gm = (q >> 20) & 1u ? -1 : 1, gu = (q >> 21) & 1u ? -1 : 1, gw = (q >> 22) & 1u ? -1 : 1;
            // the three dilated coordinates after `sub` steps, ones outside
            // their fields, and their increments (a minor axis: without and
            // with the remainder's carry)
            uint32_t U = 0, W = 0, ru = 0, rw = 0;
            if (ns > 0) {
                const float rcp = 1.0f / (float)tdm;
                small_div(2u * sdu * (uint32_t)sub + (tdm >> 1), tdm, rcp, &U, &ru);
                small_div(2u * sdw * (uint32_t)sub + (tdm >> 1), tdm, rcp, &W, &rw);
            }
            const int32_t ux = ax == 2 ? 0 : ax + 1, wx = ax == 0 ? 2 : ax - 1;
            const A om = outside<A, kBricked>(a, ax), ou = outside<A, kBricked>(a, ux), ow = outside<A, kBricked>(a, wx);
            A am = along<A, kBricked>(a, ax, (ax == 0 ? a.s[0] : (ax == 1 ? a.s[1] : a.s[2])) + gm * sub) | om;
            A au = along<A, kBricked>(a, ux, (ux == 0 ? a.s[0] : (ux == 1 ? a.s[1] : a.s[2])) + gu * (int32_t)U) | ou;
            A aw = along<A, kBricked>(a, wx, (wx == 0 ? a.s[0] : (wx == 1 ? a.s[1] : a.s[2])) + gw * (int32_t)W) | ow;
            const int32_t qu = (int32_t)(q & 255u), qw = (int32_t)((q >> 8) & 255u);
            const A im = along<A, kBricked>(a, ax, gm * kRayLanes);
            const A iu0 = along<A, kBricked>(a, ux, gu * qu), iu1 = along<A, kBricked>(a, ux, gu * (qu + 1));
            const A iw0 = along<A, kBricked>(a, wx, gw * qw), iw1 = along<A, kBricked>(a, wx, gw * (qw + 1));
            // (every lane of the wave runs the longest line's rounds: the marks
            // are placed by a ballot)
            const int32_t nmax = wave_max(ns);
            for (int32_t k = sub; k - sub < nmax; k += kStepBatch * kRayLanes) {
                A at[kStepBatch];
                CellWord word[kStepBatch];
#pragma unroll
                for (int b = 0; b < kStepBatch; ++b) {
                    at[b] = address<A, kBricked>(am, au, aw);
                    word[b] = {0u, 0u};
                    if (k + b * kRayLanes < ns) word[b] = cells.at(at[b]);
                    am = (am + im) | om;
                    ru += spu;
                    rw += spw;
                    const bool cu = ru >= tdm, cw = rw >= tdm;
                    au = (au + (cu ? iu1 : iu0)) | ou;
                    aw = (aw + (cw ? iw1 : iw0)) | ow;
                    ru -= cu ? tdm : 0u;
                    rw -= cw ? tdm : 0u;
                }
#pragma unroll
                for (int b = 0; b < kStepBatch; ++b)
                    marks.push(unmarked(word[b], 1u << ((uint32_t)at[b] & 31u)), at[b], lane);
                if (marks.n > kMarkCap - kStepBatch * kWave) marks.flush(cells, lane);
            }
        }
        marks.flush(cells, lane);
        // ---- lines too long for the 32-bit walk, one after another ----
        for (uint64_t far = __ballot(steps > 0 && dm >= kFarSteps); far; far &= far - 1) {
            const int src = __ffsll((long long)far) - 1;
            auto bc = [&](int64_t v) { return (int64_t)__shfl((long long)v, src, kWave); };
            const int32_t ax = __shfl(m, src, kWave);
            const int32_t sm = __shfl((int)neg_m, src, kWave) ? -1 : 1, su = __shfl((int)neg_u, src, kWave) ? -1 : 1,
                          sw = __shfl((int)neg_w, src, kWave) ? -1 : 1;
            walk_far<A>(a, cells, lane, bc(dm), bc(du), bc(dw), bc(steps), __builtin_amdgcn_readfirstlane(ax), sm, su, sw);
        }
    }
}

template <bool kBricked>
__global__ void __launch_bounds__(kBlock) k_clear_apply(Geom g, Bricks br, Hash h, uint32_t* __restrict__ bits,
                                                        const CellWord* __restrict__ brick, uint32_t* __restrict__ ray,
                                                        uint32_t* __restrict__ ends, DevCounters* __restrict__ ctr)
{
    uint32_t removed = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) ctr->rays[0] = ctr->rays[1] = 0u;   // for the next call
    const uint32_t n = kBricked ? br.used : g.nwords;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint64_t w = kBricked ? used_word(br, i) : i;
        const uint32_t k = ends[w], r = kBricked ? brick[w].ray : ray[w];
        if (k) ends[w] = 0u;
        if (!kBricked && r) ray[w] = 0u;
        uint32_t c = r & ~k;   // (only occupied cells are marked)
        removed += (uint32_t)__popc(c);
        if (!kBricked && c) bits[w] &= ~c;
        while (c) {
            const uint32_t j = (uint32_t)__ffs(c) - 1u;
            c &= c - 1u;
            uint32_t key = (uint32_t)w * 32u + j;
            if (kBricked) {
                uint32_t at[3];
                cell_of(br, w * 32u + j, at);
                key = at[0] + (uint32_t)g.dims[0] * (at[1] + (uint32_t)g.dims[1] * at[2]);
                // a word of the occupancy index belongs to several bricks
                atomicAnd(&bits[key >> 5], ~(1u << (key & 31u)));
            }
            const uint32_t s = hash_find(h, key);
            if (s == kEmpty) continue;   // cannot happen for an occupied cell
            Slot* sl = &h.slot[s];
            sl->cnt = 0u;
            sl->sum[0] = 0ull;
            sl->sum[1] = 0ull;
            sl->sum[2] = 0ull;
        }
    }
    // one pair of atomics per block: occupied -= removed, cleared += removed
    __shared__ uint32_t part[kBlock / kWave];
    uint32_t t = removed;
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) t += __shfl_xor(t, d, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long tot = 0;
        for (int q = 0; q < (int)(blockDim.x / kWave); ++q) tot += part[q];
        if (tot) {
            atomicAdd(&ctr->occupied, 0ull - tot);
            atomicAdd(&ctr->cleared, tot);
        }
    }
}

}  // namespace

uint64_t clear_words(const Geom& g) { return bricks_of(g).words; }

// Whether n rays are worth the bricks: the steps of rays across half the grid
// against the passes over its words.  Measured in both forms, a call of 10k and
// of 50k rays takes, in the grid's order and in bricks: 400x400x200 cells 39 / 42
// and 72 / 57 us, 800x800x400 81 / 112 and 293 / 146, 2100x2100x60 138 / 140 and
// 664 / 208, 1500x1500x700 236 / 658 and 807 / 742, 200x200x100 30 / 32 and 42 /
// 41.  Rays of a grid that is long in one direction only pass along its lines
// in either order (4000x1x1 cells 54 / 61 and 80 / 99).
bool bricks_pay(const Geom& g, int64_t n)
{
    const int64_t x = g.dims[0], y = g.dims[1], z = g.dims[2];
    const int64_t longest = std::max(x, std::max(y, z)), second = std::max(std::min(x, y), std::min(std::max(x, y), z));
    return second >= 8 && n >= (6000000 + (int64_t)g.nwords + g.nwords / 4 + longest - 1) / longest;
}

namespace {
template <typename A, bool kBricked>
hipError_t clear_rays(const float* xyz, int64_t n, CastArgs a, const Hash& h, uint32_t* bits, uint32_t* ends,
                      uint32_t* list, uint32_t list_cap, DevCounters* ctr, hipStream_t s)
{
    uint32_t turn = 0;
    for (int64_t done = 0; done < n; done += list_cap, turn ^= 1u) {
        const uint32_t m = (uint32_t)(n - done < (int64_t)list_cap ? n - done : (int64_t)list_cap);
        a.list = list;
        a.count = &ctr->rays[turn];
        a.next = &ctr->rays[turn ^ 1u];
        const int pb = grid_for(m, (int)kEndTile, kEndBlocks);
        const int wb = !kBricked || done ? 0 : grid_for(a.br.used, kBlock, 4096);
        k_clear_prepare<A, kBricked><<<pb + wb, kBlock, 0, s>>>(xyz + 3 * done, m, a.pose, a.g, a.br, (uint32_t)pb, bits,
                                                                a.brick, ends, list, &ctr->rays[turn]);
        // resident workgroups (six per compute unit), but no more than give
        // every wave the four lines it walks together (1000 rays in a grid of
        // 400x400x200: 134 us with 64 lines to a wave, 39 so in bricks, 31 without)
        k_clear_cast<A, kBricked><<<grid_for(m, kBlock / kRayLanes, 256 * 6), kBlock, 0, s>>>(xyz + 3 * done, a);
    }
    k_clear_apply<kBricked><<<grid_for(kBricked ? a.br.used : a.g.nwords), kBlock, 0, s>>>(a.g, a.br, h, bits, a.brick, a.ray,
                                                                                          ends, ctr);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_clear_rays(const float* xyz, int64_t n, const Pose& pose, const Geom& g, const int32_t sensor[3],
                             const Hash& h, uint32_t* bits, uint32_t* marks, uint32_t* bricks, uint32_t* list,
                             uint32_t list_cap, DevCounters* ctr, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    CastArgs a{};
    a.pose = pose;
    a.g = g;
    a.br = bricks_of(g);
    a.s[0] = sensor[0];
    a.s[1] = sensor[1];
    a.s[2] = sensor[2];
    a.bits = bits;
    a.ray = marks;
    if (!bricks) return clear_rays<uint32_t, false>(xyz, n, a, h, bits, marks + g.nwords, list, list_cap, ctr, s);
    a.brick = reinterpret_cast<CellWord*>(bricks);
    uint32_t* ends = bricks + 2 * a.br.words;
    return a.br.words < (1ull << 27) ? clear_rays<uint32_t, true>(xyz, n, a, h, bits, ends, list, list_cap, ctr, s)
                                     : clear_rays<uint64_t, true>(xyz, n, a, h, bits, ends, list, list_cap, ctr, s);
}

}  // namespace vm
