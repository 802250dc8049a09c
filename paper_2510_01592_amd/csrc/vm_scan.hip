// vm_scan.hip -- device-wide exclusive scan, with the element count read on
// the device so that no stage of a frame waits for the host.
#include "vm_common.h"

namespace vm {
namespace {

constexpr int kScanItems = 16;                      // per thread
constexpr int kScanTile = kBlock * kScanItems;      // 4096 values per block

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, int lane)
{
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(v, d, kWave);
        if (lane >= d) v += o;
    }
    return v;
}

// Block-wide exclusive scan of one value per thread; returns the prefix and
// writes the block total to *total.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds4, uint32_t* total)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t inc = wave_incl_scan(v, lane);
    if (lane == kWave - 1) lds4[wave] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) {
        const uint32_t t = lds4[w];
        off += (w < wave) ? t : 0u;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__global__ void __launch_bounds__(kBlock) k_scan_reduce(const uint32_t* __restrict__ in, const uint32_t* d_n,
                                                        uint32_t n_fixed, uint32_t* __restrict__ blk)
{
    __shared__ uint32_t lds[kBlock / kWave];
    const uint32_t n = d_n ? min(*d_n, n_fixed) : n_fixed;
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    if (base >= n) {
        if (threadIdx.x == 0) blk[blockIdx.x] = 0;
        return;
    }
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const uint64_t i = base + (uint64_t)j * kBlock + threadIdx.x;
        if (i < n) s += in[i];
    }
    uint32_t tot;
    block_excl_scan(s, lds, &tot);
    if (threadIdx.x == 0) blk[blockIdx.x] = tot;
}

// Down-sweep: each tile adds up the totals of the tiles before it (a block-
// wide sum over at most a few thousand words, read from L2), so the scan
// needs no pass over the totals of its own and no workgroup waits on another.
__global__ void __launch_bounds__(kBlock) k_scan_down(const uint32_t* in, uint32_t* out, const uint32_t* d_n,
                                                      uint32_t n_fixed, const uint32_t* __restrict__ blk,
                                                      uint32_t* d_total)
{
    __shared__ uint32_t lds[kBlock / kWave];
    const uint32_t n = d_n ? min(*d_n, n_fixed) : n_fixed;
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    if (base >= n) {
        if (blockIdx.x == 0 && threadIdx.x == 0 && d_total) *d_total = 0;   // n == 0
        return;
    }
    uint32_t pre = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kBlock) pre += blk[i];
    // blocked arrangement: thread t owns values [t*I, t*I + I) of the tile
    uint32_t v[kScanItems];
    uint32_t s = 0;
    const uint64_t mine = base + (uint64_t)threadIdx.x * kScanItems;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const uint64_t i = mine + j;
        v[j] = i < n ? in[i] : 0u;
        s += v[j];
    }
    uint32_t prefix;
    block_excl_scan(pre, lds, &prefix);   // block total of the partial sums = prefix of this tile
    uint32_t tot;
    uint32_t run = block_excl_scan(s, lds, &tot) + prefix;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const uint64_t i = mine + j;
        if (i < n) out[i] = run;
        run += v[j];
    }
    if (d_total && threadIdx.x == 0 && base + kScanTile >= n) *d_total = prefix + tot;
}

// Short arrays (per-cluster counts) are scanned by one workgroup in one
// launch; a two-kernel scan would cost a second launch, which is most of its
// time at these sizes.
__global__ void __launch_bounds__(kOneBlockThreads) k_scan_small(const uint32_t* in, uint32_t* out,
                                                                 const uint32_t* d_n, uint32_t n_fixed,
                                                                 uint32_t* d_total)
{
    const uint32_t n = d_n ? min(*d_n, n_fixed) : n_fixed;
    uint32_t total[1];
    one_block_scan<kOneBlockThreads, 4, 1>(
        n, [&](uint32_t i, uint32_t(&v)[1]) { v[0] = in[i]; }, [&](uint32_t i, const uint32_t(&e)[1]) { out[i] = e[0]; },
        total);
    if (threadIdx.x == 0 && d_total) *d_total = total[0];
}

}  // namespace

size_t scan_blk_words(uint64_t n_cap)
{
    return (size_t)((n_cap + kScanTile - 1) / kScanTile) + 64;
}

hipError_t scan_exclusive_dev(const uint32_t* in, uint32_t* out, const uint32_t* d_n, uint32_t n_cap,
                              uint32_t* d_total, uint32_t* blk, hipStream_t s)
{
    if (n_cap <= kOneBlockMax) {
        k_scan_small<<<1, kOneBlockThreads, 0, s>>>(in, out, d_n, n_cap, d_total);
        return hipGetLastError();
    }
    uint32_t nblk = (uint32_t)((uint64_t(n_cap) + kScanTile - 1) / kScanTile);
    if (nblk == 0) nblk = 1;   // still writes the total (0)
    k_scan_reduce<<<nblk, kBlock, 0, s>>>(in, d_n, n_cap, blk);
    k_scan_down<<<nblk, kBlock, 0, s>>>(in, out, d_n, n_cap, blk, d_total);
    return hipGetLastError();
}

}  // namespace vm
