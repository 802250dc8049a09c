// vm_tilescan.h -- two-kernel exclusive scans whose values are computed on the
// fly and whose results are consumed in place, so that a
// "flag -> scan -> use" sequence takes two launches and no flag arrays.
//
//   k_tile_reduce:  tile t sums f(i) over its kTsTile items into blk[t];
//   k_tile_down:    tile t adds up blk[0, t) (a block-wide sum over a few
//                   thousand words from L2), scans its own items (wave by
//                   wave, consecutive lanes on consecutive items) and calls
//                   g(i, f(i), exclusive prefix) for every item whose
//                   values are not all zero; the tile holding the last item
//                   (or tile 0 when there are no items) calls g.total(sum of
//                   all).
// Items are i < n with n = min(*d_n, n_fixed) (or n_fixed when d_n is null).
// Launch through tile_scan(); blk needs N * ts_tiles(n_fixed) words.  f and
// g are small structs of device pointers, passed by value.
#pragma once
#include "vm_common.h"

namespace vm {

template <int N>
struct Vec {
    uint32_t v[N];
};

template <int N>
__device__ __forceinline__ Vec<N> vzero()
{
    Vec<N> r;
#pragma unroll
    for (int q = 0; q < N; ++q) r.v[q] = 0u;
    return r;
}

template <int N>
__device__ __forceinline__ Vec<N> vadd(const Vec<N>& a, const Vec<N>& b)
{
    Vec<N> r;
#pragma unroll
    for (int q = 0; q < N; ++q) r.v[q] = a.v[q] + b.v[q];
    return r;
}

constexpr int kTsItems = 4;                      // items per thread (small tiles: many workgroups)
constexpr uint32_t kTsTile = kBlock * kTsItems;  // items per tile (1024)
// Up to this many tiles, a tile sums the tile totals before it itself;
// beyond, one workgroup scans the totals in between.
constexpr uint32_t kTsDirectTiles = 16384;

inline uint32_t ts_tiles(uint64_t n_fixed)
{
    const uint64_t t = (n_fixed + kTsTile - 1) / kTsTile;
    return (uint32_t)(t ? t : 1);
}

// exclusive prefix of x over the block (thread order); *total = block sum.
// lds needs kBlock / kWave entries.
template <int N>
__device__ __forceinline__ Vec<N> ts_block_excl(Vec<N> x, Vec<N>* lds, Vec<N>* total)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    Vec<N> inc = x;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t o = __shfl_up(inc.v[q], d, kWave);
            if (lane >= d) inc.v[q] += o;
        }
    }
    if (lane == kWave - 1) lds[wave] = inc;
    __syncthreads();
    Vec<N> off = vzero<N>(), tot = vzero<N>();
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) {
        const Vec<N> t = lds[w];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            off.v[q] += (w < wave) ? t.v[q] : 0u;
            tot.v[q] += t.v[q];
        }
    }
    __syncthreads();
    *total = tot;
    Vec<N> r;
#pragma unroll
    for (int q = 0; q < N; ++q) r.v[q] = off.v[q] + inc.v[q] - x.v[q];
    return r;
}

template <int N, class F>
__global__ void __launch_bounds__(kBlock) k_tile_reduce(F f, const uint32_t* d_n, uint32_t n_fixed,
                                                        Vec<N>* __restrict__ blk)
{
    __shared__ Vec<N> lds[kBlock / kWave];
    const uint32_t n = d_n ? min(*d_n, n_fixed) : n_fixed;
    const uint64_t base = (uint64_t)blockIdx.x * kTsTile;
    if (base >= n) {
        if (threadIdx.x == 0) blk[blockIdx.x] = vzero<N>();
        return;
    }
    Vec<N> s = vzero<N>();
#pragma unroll 4
    for (int j = 0; j < kTsItems; ++j) {
        const uint64_t i = base + (uint64_t)j * kBlock + threadIdx.x;
        if (i < n) s = vadd(s, f((uint32_t)i));
    }
    Vec<N> tot;
    ts_block_excl(s, lds, &tot);
    if (threadIdx.x == 0) blk[blockIdx.x] = tot;
}

template <int N>
__device__ __forceinline__ Vec<N> ts_wave_incl(Vec<N> x, int lane)
{
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t o = __shfl_up(x.v[q], d, kWave);
            if (lane >= d) x.v[q] += o;
        }
    }
    return x;
}

template <int N>
__device__ __forceinline__ Vec<N> ts_shfl(const Vec<N>& x, int src)
{
    Vec<N> r;
#pragma unroll
    for (int q = 0; q < N; ++q) r.v[q] = __shfl(x.v[q], src, kWave);
    return r;
}

// Wave w of the tile handles items base + w * kTsWaveSpan + j * 64 + lane
// (j < kTsItems), so consecutive lanes handle consecutive items in every
// step and the consumer's reads and writes coalesce.
constexpr uint32_t kTsWaveSpan = kWave * kTsItems;

template <int N, class F, class G>
__global__ void __launch_bounds__(kBlock) k_tile_down(F f, G g, const uint32_t* d_n, uint32_t n_fixed,
                                                      const Vec<N>* __restrict__ blk, bool scanned)
{
    __shared__ Vec<N> lds[kBlock / kWave];
    __shared__ Vec<N> wsum[kBlock / kWave];
    const uint32_t n = d_n ? min(*d_n, n_fixed) : n_fixed;
    const uint64_t base = (uint64_t)blockIdx.x * kTsTile;
    if (base >= n) {
        if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) g.total(vzero<N>());
        return;
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // prefix of this tile: the sum of the tiles before it (or the scanned totals)
    Vec<N> tile_pre;
    if (scanned) {
        tile_pre = blk[blockIdx.x];
    } else {
        Vec<N> pre = vzero<N>();
        for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kBlock) pre = vadd(pre, blk[t]);
        ts_block_excl(pre, lds, &tile_pre);
    }
    const uint64_t wbase = base + (uint64_t)wave * kTsWaveSpan;
    Vec<N> xs[kTsItems];
    Vec<N> s = vzero<N>();
    bool some[kTsItems], any = false;   // (uniform over the wave)
#pragma unroll
    for (int j = 0; j < kTsItems; ++j) {
        const uint64_t i = wbase + (uint64_t)j * kWave + lane;
        xs[j] = i < n ? f((uint32_t)i) : vzero<N>();
        s = vadd(s, xs[j]);
    }
#pragma unroll
    for (int j = 0; j < kTsItems; ++j) {
        uint32_t o = 0;
#pragma unroll
        for (int q = 0; q < N; ++q) o |= xs[j].v[q];
        some[j] = __ballot(o != 0u) != 0;
        any |= some[j];
    }
    // Wave totals, then each wave's starting prefix.  Roots are few, so most
    // rounds of a wave and most waves hold zeros only, and nothing is scanned
    // there: the chains of lane shifts, not the reads, are what the kernel
    // waited for (cluster roots among 0.9 M voxels: 8.0 -> 5.9 us, among
    // 7.9 M: 32 -> 21 us).
    if (any) s = ts_shfl(ts_wave_incl(s, lane), kWave - 1);
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    Vec<N> run = tile_pre, all = tile_pre;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) {
        if (w < wave) run = vadd(run, wsum[w]);
        all = vadd(all, wsum[w]);
    }
#pragma unroll
    for (int j = 0; j < kTsItems; ++j) {
        if (!some[j]) continue;
        const uint64_t i = wbase + (uint64_t)j * kWave + lane;
        const Vec<N> inc = ts_wave_incl(xs[j], lane);
        Vec<N> ex;
        uint32_t o = 0;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            ex.v[q] = run.v[q] + inc.v[q] - xs[j].v[q];
            o |= xs[j].v[q];
        }
        if (o) g((uint32_t)i, xs[j], ex);
        run = vadd(run, ts_shfl(inc, kWave - 1));
    }
    if (threadIdx.x == 0 && base + kTsTile >= n) g.total(all);
}

// Exclusive scan of the tile totals in place (one workgroup), for grids of
// many tiles; with d_n only those that hold the *d_n items (7.9M items
// in room for 33M: 105 us over all tiles, 256 a step, 6.5 us so).  One
// workgroup waits for memory, so a thread asks for all its words of a round
// (32 K words) at once, four to a read, and the waves share one barrier a
// round (31 K totals: 19.6 us reading a thread's four words a round -> 6.8).
// blk starts on 16 bytes and its length is rounded up to 4 words.
template <int N>
__global__ void __launch_bounds__(kOneBlockThreads) k_tile_totals(Vec<N>* blk, uint32_t ntiles,
                                                                  const uint32_t* d_n = nullptr)
{
    constexpr int kReads = 8, kPer = 4 / N;   // reads a thread, tiles a read
    constexpr uint32_t kSpan = kWave * 4 * kReads, kRound = kSpan * (kOneBlockThreads / kWave);
    __shared__ Vec<N> wsum[2][kOneBlockThreads / kWave];
    const uint32_t used = d_n ? min((uint32_t)(((uint64_t)*d_n + kTsTile - 1) / kTsTile), ntiles) : ntiles;
    const uint32_t words = used * N;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint4* p = reinterpret_cast<uint4*>(blk);
    Vec<N> carry = vzero<N>();
    int half = 0;
    for (uint32_t c0 = 0; c0 < words; c0 += kRound, half ^= 1) {
        const uint32_t w0 = c0 + wave * kSpan + lane * 4;
        union Four {
            uint4 u;
            Vec<N> t[kPer];
            uint32_t w[4];
        } x[kReads];
#pragma unroll
        for (int j = 0; j < kReads; ++j) x[j].u = p[min(w0 + j * kWave * 4, words - 1) / 4];
        Vec<N> sum[kReads], inc[kReads], s = carry;
        const bool live = c0 + wave * kSpan < words;   // (uniform over the wave)
#pragma unroll
        for (int j = 0; j < kReads; ++j) {
            sum[j] = inc[j] = vzero<N>();
            if (!live) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) x[j].w[k] = w0 + j * kWave * 4 + k < words ? x[j].w[k] : 0u;
#pragma unroll
            for (int k = 0; k < kPer; ++k) sum[j] = vadd(sum[j], x[j].t[k]);
            inc[j] = ts_wave_incl(sum[j], lane);
        }
        Vec<N> all = vzero<N>();
#pragma unroll
        for (int j = 0; j < kReads; ++j) all = vadd(all, ts_shfl(inc[j], kWave - 1));
        if (lane == 0) wsum[half][wave] = all;
        __syncthreads();   // (the next round writes the other half)
#pragma unroll
        for (int w = 0; w < kOneBlockThreads / kWave; ++w) {
            const Vec<N> t = wsum[half][w];
            if (w < wave) s = vadd(s, t);
            carry = vadd(carry, t);
        }
#pragma unroll
        for (int j = 0; j < kReads; ++j) {
            Vec<N> e;
#pragma unroll
            for (int q = 0; q < N; ++q) e.v[q] = s.v[q] + inc[j].v[q] - sum[j].v[q];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const Vec<N> t = x[j].t[k];
                x[j].t[k] = e;
                e = vadd(e, t);
            }
            const uint32_t w = w0 + j * kWave * 4;
            if (w < words) p[w / 4] = x[j].u;
            s = vadd(s, ts_shfl(inc[j], kWave - 1));
        }
    }
}

// The two (or three) launches of a fused scan over n_fixed item slots.
template <int N, class F, class G>
inline void tile_scan(F f, G g, const uint32_t* d_n, uint32_t n_fixed, Vec<N>* blk, hipStream_t s)
{
    const uint32_t nt = ts_tiles(n_fixed);
    const bool scanned = nt > kTsDirectTiles;
    k_tile_reduce<N><<<nt, kBlock, 0, s>>>(f, d_n, n_fixed, blk);
    if (scanned) k_tile_totals<N><<<1, kOneBlockThreads, 0, s>>>(blk, nt, d_n);
    k_tile_down<N><<<nt, kBlock, 0, s>>>(f, g, d_n, n_fixed, blk, scanned);
}

}  // namespace vm
