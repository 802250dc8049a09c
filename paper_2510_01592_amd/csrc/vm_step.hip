// vm_step.hip -- steppable point classification (Sec. III-C, Eq. (3)-(4))
// and the clustering of steppable points with Alg. 1's distance and
// normal-angle gates.
//
//   k_step_means:    the Eq. (1) mean of every occupied voxel, by rank
//                    (one hash lookup each);
//   k_step_classify: a thread per voxel gathers the means of the occupied
//                    voxels within `radius` cells, in ascending key order:
//                    their mean, then their scatter matrix (fp64), its cyclic
//                    Jacobi eigenvectors, the unit normal of the smallest
//                    eigenvalue oriented to +z, and the Eq. (4) test.  The
//                    neighbours in a row of cells have consecutive ranks, so a
//                    row costs two occupancy words and one rank whatever its
//                    width, and all rows' reads are in flight together;
//   k_step_runs:     steppable voxels that pass both gates with the one before
//                    them in x (rank r - 1) are linked; a run of links within
//                    a wave starts as one set;
//   k_step_hook:     union-find over the steppable voxels: each unites with
//                    its other 12 neighbours of smaller key that pass both
//                    gates (they are symmetric, so every edge is seen once),
//                    but for the edges that links and other edges imply;
//                    hooks put the larger root under the smaller, so each
//                    root is its component's smallest key, Alg. 1's fixed
//                    point from L_i = i;
//   k_step_flatten:  every voxel takes its root; steppable roots count their
//                    voxels (the grouping then keeps components of at least
//                    min_cluster voxels; voxels that are not steppable count
//                    nothing and join no cluster).
// The fp64 arithmetic is written operation by operation (no contraction), so
// the normals and decisions are the same bits as the definition computes.
//
// Measured on a 400x400x200 map of 916k voxels: classification 243 -> 114 us
// (cell by cell, each with its own word, rank and branch, before; now bound by
// the eigenvectors' fp64 divisions and roots), links and hooks 471 -> 112 us,
// roots and counts 62 -> 13 us.
#include "vm_common.h"
#include "vm_dev.h"

#include <math.h>

namespace vm {
namespace {

__device__ __forceinline__ uint32_t ld_rel(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// path-halving and flattening stores are device-scope (written through to
// memory), as in the unconditional labelling's union-find
__device__ __forceinline__ void st_rel(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a moves to the root of its set and b to the root of its own, with path
// halving (parents only ever move to ancestors); a step of one and a step of
// the other wait for memory together
__device__ __forceinline__ void find_roots(uint32_t* parent, uint32_t& a, uint32_t& b)
{
    while (a != b) {
        const uint32_t pa = ld_rel(&parent[a]), pb = ld_rel(&parent[b]);
        const uint32_t ga = ld_rel(&parent[pa]), gb = ld_rel(&parent[pb]);
        const bool ra = ga == pa, rb = gb == pb;   // pa (pb) is a root
        if (!ra) st_rel(&parent[a], ga);
        if (!rb) st_rel(&parent[b], gb);
        a = ga;
        b = gb;
        if (ra && rb) return;
    }
}

// union of the sets of a and b: the larger root is hooked under the smaller
__device__ __forceinline__ void unite(uint32_t* parent, uint32_t a, uint32_t b)
{
    find_roots(parent, a, b);
    while (a != b) {
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        const uint32_t old = atomicCAS(&parent[a], a, b);
        if (old == a) return;
        a = old;
        find_roots(parent, a, b);
    }
}

__global__ void __launch_bounds__(kBlock) k_step_means(Geom g, Hash h, const DevCounters* __restrict__ ctr,
                                                       const uint32_t* __restrict__ occ_key, float4* __restrict__ mean)
{
    const uint32_t V = ctr->n_occ;
    const uint32_t nx = (uint32_t)g.dims[0], ny = (uint32_t)g.dims[1];
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += gridDim.x * blockDim.x) {
        const uint32_t k = occ_key[r];
        // linear probing as in hash_find, with the whole slot in one read
        uint32_t s = hash_slot(k, h.log2cap);
        Slot sl = h.slot[s];
        for (uint32_t p = 1; sl.key != k && sl.key != kEmpty && p < kMaxProbe && p <= h.mask; ++p) {
            s = (s + 1) & h.mask;
            sl = h.slot[s];
        }
        float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
        if (sl.key == k) {
            m.x = voxel_mean_axis(k % nx, sl.sum[0], sl.cnt, g.voxel_size, g.origin[0]);
            m.y = voxel_mean_axis((k / nx) % ny, sl.sum[1], sl.cnt, g.voxel_size, g.origin[1]);
            m.z = voxel_mean_axis(k / (nx * ny), sl.sum[2], sl.cnt, g.voxel_size, g.origin[2]);
        }
        mean[r] = m;
    }
}

// the cyclic Jacobi method on a symmetric 3x3 matrix: rotations in the planes
// (0,1), (0,2), (1,2) in turn, sweeps until the off-diagonal part is
// negligible against the diagonal (at most 16); V receives the eigenvectors
__device__ __forceinline__ void jacobi3(double A[3][3], double V[3][3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) V[i][j] = (i == j) ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 16; ++sweep) {
        const double off = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
        const double dia = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2];
        if (off <= 1e-30 * dia) break;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int p = r < 2 ? 0 : 1, q = r == 0 ? 1 : 2;
            const double apq = A[p][q];
            if (apq == 0.0) continue;
            const double tau = (A[q][q] - A[p][p]) / (2.0 * apq);
            const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            const double c = 1.0 / sqrt(1.0 + t * t);
            const double s = t * c;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double akp = A[k][p], akq = A[k][q];
                A[k][p] = c * akp - s * akq;
                A[k][q] = s * akp + c * akq;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double apk = A[p][k], aqk = A[q][k];
                A[p][k] = c * apk - s * aqk;
                A[q][k] = s * apk + c * aqk;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double vkp = V[k][p], vkq = V[k][q];
                V[k][p] = c * vkp - s * vkq;
                V[k][q] = s * vkp + c * vkq;
            }
        }
    }
}

struct StepArgs {
    const uint32_t* bits;
    const uint32_t* wrank;
    const uint32_t* occ_key;
    float4* mean;         // [cap] xyz, w: kStep and kLink (k_step_runs)
    int32_t nx, ny, nz;
    uint32_t n_th;
    double cos_th;
    double d_th;
    float4* normal;       // [cap] xyz + pad
    uint8_t* step;        // [cap]
};

constexpr uint32_t kStep = 1, kLink = 2;   // flags in a mean's fourth word

// The occupied cells of a row, |cell - x| <= kR, at (y, z): bit j of `bits` is
// cell x - kR + j, and the first of them has rank `rank` (the others follow).
struct Row {
    uint32_t bits, rank;
};

template <int kR>
__device__ __forceinline__ Row row_at(const StepArgs& a, int x, int y, int z)
{
    const bool ok = y >= 0 && z >= 0 && y < a.ny && z < a.nz;
    const uint32_t base = ok ? (uint32_t)a.nx * ((uint32_t)y + (uint32_t)a.ny * (uint32_t)z) : 0u;
    const int lo = max(x - kR, 0), hi = min(x + kR, a.nx - 1);
    const uint32_t k0 = base + (uint32_t)lo, k1 = base + (uint32_t)hi, sh = k0 & 31u;
    const uint32_t w0 = a.bits[k0 >> 5], w1 = a.bits[k1 >> 5], wr = a.wrank[k0 >> 5];
    const uint32_t f = (uint32_t)((((uint64_t)w1 << 32) | w0) >> sh) & ((1u << (hi - lo + 1)) - 1u);
    return {ok ? f << (lo - (x - kR)) : 0u, wr + (uint32_t)__popc(w0 & ((1u << sh) - 1u))};
}

// rank of the row's cell j (an occupied one); `other` for the rest, so that a
// read needs no branch
__device__ __forceinline__ uint32_t row_rank(const Row& w, int j, uint32_t other)
{
    return (w.bits >> j) & 1u ? w.rank + (uint32_t)__popc(w.bits & ((1u << j) - 1u)) : other;
}

// Eq. (3)-(4) for every occupied voxel.  A cell that is not occupied adds
// +0 to sums that are never -0, which leaves them as they are.  The means are
// read again for the second pass, a layer at a time, and the registers held to
// four waves per SIMD: with all 27 in registers two waves fit (108 us at
// radius 1, but spills at radius 2), without the bound two as well (132 us).
template <int kR>
__global__ void __launch_bounds__(kBlock, 4) k_step_classify(StepArgs a, const DevCounters* __restrict__ ctr)
{
    constexpr int kW = 2 * kR + 1;   // layers, rows per layer, cells per row
    const uint32_t V = ctr->n_occ;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += gridDim.x * blockDim.x) {
        const uint32_t key = a.occ_key[r];
        const int x = (int)(key % (uint32_t)a.nx), y = (int)((key / (uint32_t)a.nx) % (uint32_t)a.ny),
                  z = (int)(key / ((uint32_t)a.nx * (uint32_t)a.ny));
        // fn(occupied, mean) for the neighbourhood's cells in ascending key
        // order, a layer's reads in flight together
        const auto each = [&](auto fn) {
#pragma unroll 1
            for (int dz = -kR; dz <= kR; ++dz) {
                Row row[kW];
                float4 p[kW][kW];
#pragma unroll
                for (int q = 0; q < kW; ++q) row[q] = row_at<kR>(a, x, y + q - kR, z + dz);
#pragma unroll
                for (int q = 0; q < kW; ++q)
#pragma unroll
                    for (int j = 0; j < kW; ++j) p[q][j] = a.mean[row_rank(row[q], j, r)];
#pragma unroll
                for (int q = 0; q < kW; ++q)
#pragma unroll
                    for (int j = 0; j < kW; ++j) fn((row[q].bits >> j) & 1u, p[q][j]);
            }
        };
        // pass 1: the neighbours' mean
        double sx = 0.0, sy = 0.0, sz = 0.0;
        uint32_t cnt = 0;
        each([&](bool in, const float4& p) {
            sx += in ? (double)p.x : 0.0;
            sy += in ? (double)p.y : 0.0;
            sz += in ? (double)p.z : 0.0;
            cnt += in;
        });
        const double mx = sx / (double)cnt, my = sy / (double)cnt, mz = sz / (double)cnt;
        // pass 2: their scatter matrix about that mean (same order)
        double A[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
        each([&](bool in, const float4& p) {
            const double ex = in ? (double)p.x - mx : 0.0, ey = in ? (double)p.y - my : 0.0,
                         ez = in ? (double)p.z - mz : 0.0;
            A[0][0] += ex * ex;
            A[0][1] += ex * ey;
            A[0][2] += ex * ez;
            A[1][1] += ey * ey;
            A[1][2] += ey * ez;
            A[2][2] += ez * ez;
        });
        A[1][0] = A[0][1];
        A[2][0] = A[0][2];
        A[2][1] = A[1][2];
        double Vv[3][3];
        jacobi3(A, Vv);
        int m = 0;
        if (A[1][1] < A[m][m]) m = 1;
        if (A[2][2] < A[m][m]) m = 2;
        double nx = m == 0 ? Vv[0][0] : (m == 1 ? Vv[0][1] : Vv[0][2]);
        double ny = m == 0 ? Vv[1][0] : (m == 1 ? Vv[1][1] : Vv[1][2]);
        double nz = m == 0 ? Vv[2][0] : (m == 1 ? Vv[2][1] : Vv[2][2]);
        const double len = sqrt(nx * nx + ny * ny + nz * nz);
        nx /= len;
        ny /= len;
        nz /= len;
        // the orientation as one flag and a product with -1 or +1 (exact; +0
        // becomes -0 as under negation): no branches, whose nested short
        // circuits the device compiler has been seen to resolve for nz >= 0
        // without the inner tests
        const bool flip = (nz < 0.0) | ((nz == 0.0) & ((ny < 0.0) | ((ny == 0.0) & (nx < 0.0))));
        const double sg = flip ? -1.0 : 1.0;
        nx *= sg;
        ny *= sg;
        nz *= sg;
        a.normal[r] = make_float4((float)nx, (float)ny, (float)nz, 0.f);
        a.step[r] = (cnt >= a.n_th && nz >= a.cos_th) ? 1 : 0;
    }
}

// Alg. 1's gates between two steppable voxels
__device__ __forceinline__ bool gates(const StepArgs& a, const float4& pi, const float4& ni, const float4& pj,
                                      const float4& nj)
{
    const double ddx = (double)pi.x - (double)pj.x, ddy = (double)pi.y - (double)pj.y,
                 ddz = (double)pi.z - (double)pj.z;
    const double dot = (double)ni.x * (double)nj.x + (double)ni.y * (double)nj.y + (double)ni.z * (double)nj.z;
    return ddx * ddx + ddy * ddy + ddz * ddz < a.d_th * a.d_th && dot > a.cos_th;
}

// Links in x and the parents they give: a voxel's parent is the first of its
// run within the wave's 64 ranks.
__global__ void __launch_bounds__(kBlock) k_step_runs(StepArgs a, const DevCounters* __restrict__ ctr,
                                                      uint32_t* __restrict__ parent)
{
    const uint32_t V = ctr->n_occ;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t b0 = blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); b0 < V; b0 += stride) {
        const uint32_t r = b0 + (uint32_t)lane, i = min(r, V - 1u), j = i ? i - 1u : 0u;
        const uint32_t key = a.occ_key[i];
        const bool st = a.step[i] != 0;
        const bool link = r < V && i > 0 && st && a.step[j] && a.occ_key[j] + 1u == key && key % (uint32_t)a.nx != 0u &&
                          gates(a, a.mean[i], a.normal[i], a.mean[j], a.normal[j]);
        const uint64_t first = ~__ballot(link) | 1ull;
        if (r < V) {
            parent[r] = b0 + 63u - (uint32_t)__clzll((long long)(first & (~0ull >> (63 - lane))));
            a.mean[r].w = __uint_as_float((st ? kStep : 0u) | (link ? kLink : 0u));
        }
    }
}

// Union-find over the steppable voxels with Alg. 1's gates (parent = rank).
// An edge is left out where the others imply it.  Let c-, c0, c+ be a row's
// cells at x - 1, x and x + 1, and o the voxel before this one in x, in the
// same wave and linked to it:
//   to c-: when o has its edge to its own c0 (the same cell);
//   to c0: when o has its edge to its own c+, or when this voxel has an edge to
//          c- and c- and c0 are linked;
//   to c+: when this voxel has an edge to c0 and c0 and c+ are linked.
// Each edge is implied by links and by edges of earlier lanes, or earlier ones
// of this lane, so the chain of reasons ends at edges that are united.
__global__ void __launch_bounds__(kBlock) k_step_hook(StepArgs a, const DevCounters* __restrict__ ctr,
                                                      uint32_t* parent)
{
    const uint32_t V = ctr->n_occ;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t stride = gridDim.x * blockDim.x;
    // every lane runs the same iterations (the shuffles need them all)
    for (uint32_t b0 = blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); b0 < V; b0 += stride) {
        const uint32_t r = min(b0 + (uint32_t)lane, V - 1u);
        const uint32_t key = a.occ_key[r];
        const int x = (int)(key % (uint32_t)a.nx), y = (int)((key / (uint32_t)a.nx) % (uint32_t)a.ny),
                  z = (int)(key / ((uint32_t)a.nx * (uint32_t)a.ny));
        const float4 pi = a.mean[r], ni = a.normal[r];
        const uint32_t fl = __float_as_uint(pi.w);
        const bool st = b0 + (uint32_t)lane < V && (fl & kStep);
        const bool link = st && (fl & kLink);
        if (__ballot(st) == 0) continue;
        uint32_t left = link && lane == 0 ? 1u << 12 : 0u;   // edges to unite: 3 q + j, and the link into the wave
        // the rows of smaller keys: dz = -1 (dy = -1, 0, 1), and dz = 0, dy = -1
        Row row[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) row[q] = row_at<1>(a, x, q < 3 ? y + q - 1 : y - 1, q < 3 ? z - 1 : z);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t rk[3];
            float4 pj[3], nj[3];
            bool e[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                rk[j] = row_rank(row[q], j, r);
                pj[j] = a.mean[rk[j]];
                nj[j] = a.normal[rk[j]];
            }
#pragma unroll
            for (int j = 0; j < 3; ++j)
                e[j] = st && ((row[q].bits >> j) & 1u) && (__float_as_uint(pj[j].w) & kStep) &&
                       gates(a, pi, ni, pj[j], nj[j]);
            const uint32_t own = (e[1] ? 1u : 0u) | (e[2] ? 2u : 0u);
            const uint32_t up = __shfl_up(own, 1, kWave);
            const uint32_t before = link && lane > 0 ? up : 0u;
            const bool l0 = __float_as_uint(pj[1].w) & kLink, l1 = __float_as_uint(pj[2].w) & kLink;
            const uint32_t keep = (e[0] && !(before & 1u) ? 1u : 0u) | (e[1] && !(before & 2u) && !(e[0] && l0) ? 2u : 0u) |
                                  (e[2] && !(e[1] && l1) ? 4u : 0u);
            left |= keep << (3 * q);
        }
        // a round takes one edge of every lane that has one left (an edge's
        // own site for each of the 13 had the wave wait for up to 13 unions)
        for (; left; left &= left - 1u) {
            const int i = __ffs(left) - 1, q = i / 3;
            const Row w = q == 0 ? row[0] : q == 1 ? row[1] : q == 2 ? row[2] : row[3];
            unite(parent, r, i == 12 ? r - 1u : row_rank(w, i - 3 * q, r));
        }
    }
}

// Every voxel takes its root (a read-only walk, then its own store); steppable
// voxels add one to their root's count.  A floor is one root: an atomic per
// wave on its count took most of the kernel's time (14k of them, 63 us), so
// a workgroup gathers the counts of its roots in LDS first.
constexpr int kFlatBlock = 1024;
constexpr uint32_t kFlatSlots = 64;

__global__ void __launch_bounds__(kFlatBlock) k_step_flatten(const DevCounters* __restrict__ ctr,
                                                             const uint8_t* __restrict__ step, uint32_t* parent,
                                                             uint32_t* csize)
{
    __shared__ uint32_t root_of[kFlatSlots], count[kFlatSlots];
    const uint32_t V = ctr->n_occ;
    const int lane = threadIdx.x & (kWave - 1);
    if (threadIdx.x < kFlatSlots) {
        root_of[threadIdx.x] = kEmpty;
        count[threadIdx.x] = 0;
    }
    __syncthreads();
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t b0 = blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); b0 < V; b0 += stride) {
        const uint32_t r = b0 + (uint32_t)lane;
        uint32_t x = r;
        bool cs = false;
        if (r < V) {
            cs = step[r] != 0;
            uint32_t p = ld_rel(&parent[r]);
            while (p != x) {
                x = p;
                p = ld_rel(&parent[x]);
            }
            st_rel(&parent[r], x);
        }
        uint64_t pending = __ballot(cs);
        while (pending) {
            const int leader = __ffsll((long long)pending) - 1;
            const uint32_t root = __shfl(x, leader, kWave);
            const uint64_t same = __ballot(cs && x == root);
            if (lane == leader) {
                const uint32_t n = (uint32_t)__popcll(same), at = (root * 0x9E3779B1u) >> 26;
                const uint32_t old = atomicCAS(&root_of[at], kEmpty, root);
                if (old == kEmpty || old == root) atomicAdd(&count[at], n);
                else atomicAdd(&csize[root], n);   // another root has the slot
            }
            pending &= ~same;
        }
    }
    __syncthreads();
    if (threadIdx.x < kFlatSlots && count[threadIdx.x]) atomicAdd(&csize[root_of[threadIdx.x]], count[threadIdx.x]);
}
static_assert(kFlatSlots == 1u << (32 - 26), "the slot is a hash's top bits");

// labels in ascending key order: the root's key, kEmpty where not steppable
__global__ void __launch_bounds__(kBlock) k_step_labels(const DevCounters* __restrict__ ctr,
                                                        const uint32_t* __restrict__ parent,
                                                        const uint8_t* __restrict__ step,
                                                        const uint32_t* __restrict__ occ_key, uint32_t* __restrict__ labels)
{
    const uint32_t V = ctr->n_occ;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += gridDim.x * blockDim.x)
        labels[r] = step[r] ? occ_key[parent[r]] : kEmpty;
}

// the classification as three floats and one byte per voxel (caller's buffers)
__global__ void __launch_bounds__(kBlock) k_step_export(const DevCounters* __restrict__ ctr,
                                                        const float4* __restrict__ normal,
                                                        const uint8_t* __restrict__ step, float* __restrict__ n_out,
                                                        uint8_t* __restrict__ s_out)
{
    const uint32_t V = ctr->n_occ;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < V; r += gridDim.x * blockDim.x) {
        if (n_out) {
            const float4 n = normal[r];
            n_out[3 * (size_t)r + 0] = n.x;
            n_out[3 * (size_t)r + 1] = n.y;
            n_out[3 * (size_t)r + 2] = n.z;
        }
        if (s_out) s_out[r] = step[r];
    }
}

}  // namespace

hipError_t launch_steppable(const Geom& g, const Hash& h, const uint32_t* bits, SegBuffers& b, uint32_t cap,
                            const StepBuffers& sb, uint32_t radius, uint32_t n_th, double cos_th, double d_th,
                            float* d_normal, uint8_t* d_steppable, DevCounters* ctr, hipStream_t s)
{
    const int grid = grid_for(cap);
    k_step_means<<<grid, kBlock, 0, s>>>(g, h, ctr, b.occ_key, sb.mean);
    StepArgs a;
    a.bits = bits;
    a.wrank = b.wrank;
    a.occ_key = b.occ_key;
    a.mean = sb.mean;
    a.nx = g.dims[0];
    a.ny = g.dims[1];
    a.nz = g.dims[2];
    a.n_th = n_th;
    a.cos_th = cos_th;
    a.d_th = d_th;
    a.normal = sb.normal;
    a.step = sb.step;
    if (radius == 1) k_step_classify<1><<<grid, kBlock, 0, s>>>(a, ctr);
    else k_step_classify<2><<<grid, kBlock, 0, s>>>(a, ctr);
    k_step_runs<<<grid, kBlock, 0, s>>>(a, ctr, b.parent);
    k_step_hook<<<grid, kBlock, 0, s>>>(a, ctr, b.parent);
    k_step_flatten<<<grid_for(cap, kFlatBlock, 1024), kFlatBlock, 0, s>>>(ctr, sb.step, b.parent, b.csize);
    if (d_normal || d_steppable) k_step_export<<<grid, kBlock, 0, s>>>(ctr, sb.normal, sb.step, d_normal, d_steppable);
    return hipGetLastError();
}

hipError_t launch_step_labels(const SegBuffers& b, const StepBuffers& sb, uint32_t cap, DevCounters* ctr,
                              uint32_t* d_labels, hipStream_t s)
{
    k_step_labels<<<grid_for(cap), kBlock, 0, s>>>(ctr, b.parent, sb.step, b.occ_key, d_labels);
    return hipGetLastError();
}

}  // namespace vm
