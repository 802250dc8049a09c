// vm_dev.h -- device functions shared by the library's kernels (gfx950):
// the counter-based generator and the hypothesis plane of Sec. III-C (a), the
// inlier test of (b), and the in-plane projection, orientation test and
// monotone-chain building blocks of the boundary polygons.
#pragma once
#include "vm_common.h"

#include <math.h>

namespace vm {
namespace dev {

// The 128-bit product of two 64-bit words from four 32 x 32 -> 64 bit
// multiply-adds (the high and the low half of one product; computing them
// as separate 64-bit operations repeats partial products).
__device__ __forceinline__ void mul_64x64_128(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo)
{
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
    const uint64_t p00 = (uint64_t)a0 * b0;
    const uint64_t t = (uint64_t)a0 * b1 + (p00 >> 32);             // < 2^64
    const uint64_t t2 = (uint64_t)a1 * b0 + (uint32_t)t;            // < 2^64
    lo = (t2 << 32) | (uint32_t)p00;
    hi = (uint64_t)a1 * b1 + (t >> 32) + (t2 >> 32);
}

__device__ __forceinline__ void philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                              uint64_t k1, uint64_t out[4])
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t hi0, lo0, hi1, lo1;
        mul_64x64_128(M0, c0, hi0, lo0);
        mul_64x64_128(M1, c2, hi1, lo1);
        const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += W0;
        k1 += W1;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// Sec. III-C (a): hypothesis h of a cluster of n points (pointers at its
// first point): three distinct points drawn with Philox4x64-10, key (seed, 0)
// and counter (h, tag, frame, 0); the plane through them in fp64 (unit
// normal with +z first, then +y, then +x; offset from the first point),
// rounded to float32.  Degenerate triples (and n < 3) give a NaN plane.
__device__ __forceinline__ float4 hyp_plane(const float* __restrict__ X, const float* __restrict__ Y,
                                            const float* __restrict__ Z, uint64_t n, uint32_t h, uint32_t tag,
                                            uint32_t frame, uint64_t seed)
{
    const float qnan = __builtin_nanf("");
    float4 pl = make_float4(qnan, qnan, qnan, qnan);
    if (n >= 3) {
        uint64_t r[4];
        philox4x64_10(h, tag, frame, 0, seed, 0, r);
        const uint64_t u0 = r[0] >> 32, u1 = r[1] >> 32, u2 = r[2] >> 32;
        const uint64_t ia = (u0 * n) >> 32;
        uint64_t ib = (u1 * (n - 1)) >> 32;
        if (ib >= ia) ib += 1;
        uint64_t ic = (u2 * (n - 2)) >> 32;
        const uint64_t lo = ia < ib ? ia : ib, hi = ia < ib ? ib : ia;
        if (ic >= lo) ic += 1;
        if (ic >= hi) ic += 1;
        const double ax = X[ia], ay = Y[ia], az = Z[ia];
        const double e1x = (double)X[ib] - ax, e1y = (double)Y[ib] - ay, e1z = (double)Z[ib] - az;
        const double e2x = (double)X[ic] - ax, e2y = (double)Y[ic] - ay, e2z = (double)Z[ic] - az;
        double nx = e1y * e2z - e1z * e2y;
        double ny = e1z * e2x - e1x * e2z;
        double nz = e1x * e2y - e1y * e2x;
        const double nn = nx * nx + ny * ny + nz * nz;
        if (nn >= 1e-24) {
            const double inv = 1.0 / sqrt(nn);
            nx = nx * inv;
            ny = ny * inv;
            nz = nz * inv;
            // one flag and a product with -1 or +1 (exact, and +0 becomes -0 as
            // under negation): the nested short-circuit form was compiled so
            // that for nz = 0 the inner tests were lost
            const bool flip = (nz < 0.0) | ((nz == 0.0) & ((ny < 0.0) | ((ny == 0.0) & (nx < 0.0))));
            const double sg = flip ? -1.0 : 1.0;
            nx = nx * sg;
            ny = ny * sg;
            nz = nz * sg;
            const double d = -(nx * ax + ny * ay + nz * az);
            pl = make_float4((float)nx, (float)ny, (float)nz, (float)d);
        }
    }
    return pl;
}

// Sec. III-C (b): the inlier test of a point against a plane, as specified
__device__ __forceinline__ bool inlier_test(const float4 pl, float x, float y, float z, float eps)
{
    return fabsf(fmaf(pl.z, z, fmaf(pl.y, y, fmaf(pl.x, x, pl.w)))) < eps;
}

// ---- inlier counting on the matrix cores ------------------------------------------
// The test's distance is the chain fma(nz, z, fma(ny, y, fma(nx, x, d))).
// v_mfma_f32_16x16x1 (four blocks, K = 1) adds one product to each of its
// 1024 accumulators with a single rounding, so three of them from an
// accumulator holding d give that chain bit for bit (the tests hold the counts
// to a plain fmaf chain's over subnormal, ordinary, huge, infinite and NaN
// coordinates and thresholds).  The columns are a
// wave's 64 planes (block b holds planes 16b .. 16b + 15), the rows 16 of its
// 64 points, broadcast to all four blocks (cbsz 2, abid the group of 16): lane
// l gets planes 16b + l % 16 against points 4 (l / 16) .. + 3.
// Why: on this chip a VALU instruction with a scalar-register operand issues
// at half rate (4.1 cycles per wave against 2.2-2.7), and a ballot form needs
// two scalar instructions per 64 tests besides; here every operand is a
// vector register, the three multiply-adds take 7.1 cycles per 64 tests and
// counting two 2-cycle VALU instructions more.  A loop of these tests over
// rows read from memory reaches 14.0 T tests/s with two plane groups per wave
// and 13.2 T with one; the ballot form with the planes (or eps) in scalar
// registers 8.6-9.1 T.
typedef float f32x16 __attribute__((ext_vector_type(16)));

// |d| < eps as 1 or 0: (eps - |d|) * big in one fma, clamped to [0, 1], with
// big = 2^(26 - e) for eps = m 2^e (0.5 <= m < 1).  eps * big is exact, the
// fma's sign is exact, and the smallest positive eps - |d| is 2^(e - 25), so
// a passing test gives at least 2 before the clamp; NaN clamps to 0.  For
// eps below kMinFloatEps big would overflow: those calls compare instead.
constexpr float kMinFloatEps = 0x1p-90f;

struct EpsTest {
    float eps, big, scaled;
};

inline __host__ __device__ EpsTest eps_test(float eps)
{
    EpsTest t;
    t.eps = eps;
    int e = 0;
    if (eps >= kMinFloatEps) (void)frexpf(eps, &e);
    t.big = ldexpf(1.0f, 26 - e);
    t.scaled = eps * t.big;
    return t;
}

__device__ __forceinline__ float vector_reg(float v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// G groups of 64 planes on one wave and their running counts (whole numbers
// in fp32: a lane adds at most a tile's points).
template <int G>
struct PlaneGroups {
    float nx[G], ny[G], nz[G];
    f32x16 d[G];
    float cnt[G][4];

    // planes h0 .. h1 - 1 (at most 64 G of them) of the cluster's list; the
    // rest are NaN and pass no test
    __device__ __forceinline__ void load(const float4* __restrict__ hk, uint32_t h0, uint32_t h1, int lane)
    {
        const float qnan = __builtin_nanf("");
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t h = h0 + (uint32_t)(g * kWave + lane);
            const float4 p = h < h1 ? hk[h] : make_float4(qnan, qnan, qnan, qnan);
            nx[g] = p.x;
            ny[g] = p.y;
            nz[g] = p.z;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float w = __shfl(p.w, 16 * b + (lane & 15), kWave);
#pragma unroll
                for (int i = 0; i < 4; ++i) d[g][4 * b + i] = w;
                cnt[g][b] = 0.0f;
            }
        }
    }

    // points 16 A .. 16 A + 15 of the wave's row of 64
    template <int A, bool kFloat>
    __device__ __forceinline__ void step(float x, float y, float z, const EpsTest& t)
    {
        f32x16 r[G];
#pragma unroll
        for (int g = 0; g < G; ++g) r[g] = __builtin_amdgcn_mfma_f32_16x16x1f32(x, nx[g], d[g], 2, A, 0);
#pragma unroll
        for (int g = 0; g < G; ++g) r[g] = __builtin_amdgcn_mfma_f32_16x16x1f32(y, ny[g], r[g], 2, A, 0);
#pragma unroll
        for (int g = 0; g < G; ++g) r[g] = __builtin_amdgcn_mfma_f32_16x16x1f32(z, nz[g], r[g], 2, A, 0);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = r[g][4 * b + i];
                    if (kFloat) cnt[g][b] += fminf(fmaxf(fmaf(-fabsf(v), t.big, t.scaled), 0.0f), 1.0f);
                    else cnt[g][b] += fabsf(v) < t.eps ? 1.0f : 0.0f;
                }
    }

    template <bool kFloat>
    __device__ __forceinline__ void row(float x, float y, float z, const EpsTest& t)
    {
        step<0, kFloat>(x, y, z, t);
        step<1, kFloat>(x, y, z, t);
        step<2, kFloat>(x, y, z, t);
        step<3, kFloat>(x, y, z, t);
    }

    // n points (n > 0) at X/Y/Z, a row of 64 at a time with the next kAhead
    // rows' loads in flight (a row's 8 G matrix steps take about a
    // microsecond beside the other waves', a read from HBM two; the loads are
    // unconditional, from the last point past the end: a branch around them
    // would make the row before wait for them); points past the end are NaN
    template <bool kFloat>
    __device__ __forceinline__ void sweep(const float* __restrict__ X, const float* __restrict__ Y,
                                          const float* __restrict__ Z, uint32_t n, EpsTest t, int lane)
    {
        constexpr uint32_t kAhead = 4;
        t.eps = vector_reg(t.eps);
        t.big = vector_reg(t.big);
        t.scaled = vector_reg(t.scaled);
        float x[kAhead], y[kAhead], z[kAhead];
        auto fetch = [&](uint32_t j, uint32_t r) {
            const uint32_t q = min(r + (uint32_t)lane, n - 1u);
            x[j] = X[q];
            y[j] = Y[q];
            z[j] = Z[q];
        };
#pragma unroll
        for (uint32_t j = 0; j < kAhead; ++j) fetch(j, j * kWave);
        uint32_t r = 0;
        for (; r + kAhead * kWave <= n; r += kAhead * kWave) {
#pragma unroll
            for (uint32_t j = 0; j < kAhead; ++j) {
                row<kFloat>(x[j], y[j], z[j], t);
                fetch(j, r + (j + kAhead) * kWave);
            }
        }
        // the last rows: only the groups of 16 that hold points
#pragma unroll
        for (uint32_t j = 0; j < kAhead; ++j, r += kWave) {
            if (r >= n) break;
            const uint32_t m = n - r;
            if ((uint32_t)lane >= m) x[j] = __builtin_nanf("");
            step<0, kFloat>(x[j], y[j], z[j], t);
            if (m > 16) step<1, kFloat>(x[j], y[j], z[j], t);
            if (m > 32) step<2, kFloat>(x[j], y[j], z[j], t);
            if (m > 48) step<3, kFloat>(x[j], y[j], z[j], t);
        }
    }

    // lane l's count of plane 64 g + l: a plane's tests lie on the four lanes
    // that share l % 16
    __device__ __forceinline__ uint32_t count(int g, int lane) const
    {
        float v = 0.0f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float s = cnt[g][b];
            s += __shfl_xor(s, 16, kWave);
            s += __shfl_xor(s, 32, kWave);
            v = (lane >> 4) == b ? s : v;
        }
        return (uint32_t)v;
    }
};

__device__ __forceinline__ bool p2_less(double au, double av, uint32_t ai, double bu, double bv, uint32_t bi)
{
    if (au != bu) return au < bu;
    if (av != bv) return av < bv;
    return ai < bi;
}

__device__ __forceinline__ double cross3(double ou, double ov, double au, double av, double bu, double bv)
{
    return (au - ou) * (bv - ov) - (av - ov) * (bu - ou);
}

struct Basis {
    double u[3], v[3];
};

__device__ __forceinline__ Basis plane_basis(float4 pl)
{
    Basis b;
    const double n0 = pl.x, n1 = pl.y, n2 = pl.z;
    double a[3] = {0.0, 0.0, 0.0};
    if (fabs(n0) < 0.9) a[0] = 1.0;
    else a[1] = 1.0;
    const double c0 = a[1] * n2 - a[2] * n1;
    const double c1 = a[2] * n0 - a[0] * n2;
    const double c2 = a[0] * n1 - a[1] * n0;
    const double inv = 1.0 / sqrt(c0 * c0 + c1 * c1 + c2 * c2);
    b.u[0] = c0 * inv;
    b.u[1] = c1 * inv;
    b.u[2] = c2 * inv;
    b.v[0] = n1 * b.u[2] - n2 * b.u[1];
    b.v[1] = n2 * b.u[0] - n0 * b.u[2];
    b.v[2] = n0 * b.u[1] - n1 * b.u[0];
    return b;
}

// per-cluster constants of the passes over inliers
struct ClusterFrame {
    uint32_t ib, m, pb, nk;   // inlier offset/count, point offset/count
    Basis B;
    double ox, oy, oz;        // origin = first inlier
};

__device__ __forceinline__ void project(const ClusterFrame& f, float x, float y, float z, double* pu, double* pv)
{
    const double dx = (double)x - f.ox, dy = (double)y - f.oy, dz = (double)z - f.oz;
    *pu = f.B.u[0] * dx + f.B.u[1] * dy + f.B.u[2] * dz;
    *pv = f.B.v[0] * dx + f.B.v[1] * dy + f.B.v[2] * dz;
}

__device__ __forceinline__ void swap3(double* U, double* V, uint32_t* I, uint32_t a, uint32_t b)
{
    const double tu = U[a], tv = V[a];
    const uint32_t ti = I[a];
    U[a] = U[b];
    V[a] = V[b];
    I[a] = I[b];
    U[b] = tu;
    V[b] = tv;
    I[b] = ti;
}

// One thread's chain over the points idx[0..m) (indices into U, V) in that
// order: a point pops the stack top while it does not turn left of the top
// two (collinear and repeated points too); the kept indices go to out[0..h)
// and h is returned.  out may be idx itself (a store lands at or below the
// read position).  The two top entries' coordinates stay in registers, the
// next point's coordinates and the index after it are loaded a step ahead, so
// a step waits for one LDS load at most when it does not pop.
template <typename S>
__device__ __forceinline__ uint32_t chain_run(const double* U, const double* V, const S* idx, uint32_t m, S* out)
{
    uint32_t h = 0;
    double au = 0.0, av = 0.0, bu = 0.0, bv = 0.0;   // out[h - 2], out[h - 1]
    uint32_t i1 = m > 0 ? (uint32_t)idx[0] : 0u;
    double u1 = m > 0 ? U[i1] : 0.0, v1 = m > 0 ? V[i1] : 0.0;
    uint32_t i2 = m > 1 ? (uint32_t)idx[1] : 0u;
    for (uint32_t j = 0; j < m; ++j) {
        const uint32_t i = i1;
        const double iu = u1, iv = v1;
        if (j + 1 < m) {
            i1 = i2;
            u1 = U[i1];
            v1 = V[i1];
        }
        if (j + 2 < m) i2 = idx[j + 2];
        while (h >= 2) {
            if (!(cross3(au, av, bu, bv, iu, iv) <= 0.0)) break;
            --h;
            bu = au;
            bv = av;
            if (h >= 2) {
                const uint32_t a = out[h - 2];
                au = U[a];
                av = V[a];
            }
        }
        out[h] = (S)i;
        if (h >= 1) {
            au = bu;
            av = bv;
        }
        bu = iu;
        bv = iv;
        ++h;
    }
    return h;
}

// ---- monotone chains by elimination ------------------------------------------------
// A chain (lower or upper) over sorted points drops, round after round and all
// at once, every point that lies on the inner side of the segment between its
// two neighbours by more than a tolerance far above the fp64 rounding of a
// cross product at the set's scale: such a point is no vertex of the hull of
// any set holding those three.  When a round drops nothing and every corner
// turns left by more than the tolerance, the points left are the plain
// chain's output; otherwise (collinear, coincident or nearly collinear
// points) the plain chain runs over the points left and decides among them.
// Usually a few rounds suffice, where the serial chain takes a dependent step
// of some 200 cycles per point.  (Checked on the CPU against the plain chain
// on 800k random, lattice, circular and nearly collinear sets: the same
// output on every one.)
constexpr int kMaxRounds = 32;   // then the plain chain takes over

__device__ __forceinline__ double chain_tolerance(double span) { return 1e-12 * span * span + 1e-300; }

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// largest k < K with off[k] <= x (off does not decrease, off[0] <= x), found by a
// whole wave, 64 probes at a time: two dependent reads for up to 4096 entries,
// three for 262144, where a bisection takes 12 and 18
__device__ __forceinline__ uint32_t last_at_or_below(const uint32_t* __restrict__ off, uint32_t K, uint32_t x)
{
    const uint32_t lane = threadIdx.x & (kWave - 1);
    uint32_t lo = 0, n = K;
    while (n > 1) {
        const uint32_t step = (n + kWave - 1) / kWave, i = lo + lane * step;
        const bool le = lane * step < n && off[min(i, K - 1u)] <= x;
        lo += ((uint32_t)__popcll(__ballot(le)) - 1u) * step;
        n = min(step, K - lo);
    }
    return lo;
}

__device__ __forceinline__ double wave_max_d(double v)
{
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d, kWave));
    return v;
}

// One wave's hull of at most 64 points, one per lane (u, v and i = the
// point's position in its list; lanes >= ns hold +inf and 0xFFFFFFFF): the
// points are sorted across the lanes by (u, v, i) with a bitonic network on
// shuffles, then both chains are found by elimination on lane masks.
// su/sv/si (64 entries) and st (2*64+2) are this wave's LDS scratch.  Returns
// the vertex count h and the shoelace area (on every lane) and, for lane < h,
// the sorted position vi of vertex `lane` (counter-clockwise from the smallest
// point): its list position is si[vi].
struct WaveHull {
    uint32_t h, vi;
    double area;
};

__device__ __forceinline__ WaveHull wave_hull(double u, double v, uint32_t i, uint32_t ns, int lane, double* su,
                                              double* sv, uint32_t* si, uint8_t* st)
{
    WaveHull r;
    for (int kk = 2; kk <= kWave; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
            const double ou = __shfl_xor(u, j, kWave), ov = __shfl_xor(v, j, kWave);
            const uint32_t oi = __shfl_xor(i, j, kWave);
            const bool up = (lane & kk) == 0, low = (lane & j) == 0;
            const bool mine_less = p2_less(u, v, i, ou, ov, oi);
            if ((low == up) != mine_less) {
                u = ou;
                v = ov;
                i = oi;
            }
        }
    }
    su[lane] = u;
    sv[lane] = v;
    si[lane] = i;
    wave_sync();
    const bool valid = (uint32_t)lane < ns;
    const double span = wave_max_d(valid ? fmax(u - su[0], fabs(v - sv[0])) : 0.0);
    const double tol = chain_tolerance(span);
    const uint64_t below = (1ull << lane) - 1ull, above = ~below & ~(1ull << lane);
    const uint64_t all = ns >= 64 ? ~0ull : (1ull << ns) - 1ull;
    uint64_t lo = all, up = all;   // the points left of the lower and the upper chain
    bool settled = ns < 3;
    for (int round = 0; !settled && round < kMaxRounds; ++round) {
        // (a point's neighbours among those left; the end points stay)
        const bool inner = valid && lane != 0 && (uint32_t)lane + 1u != ns;
        double cl = INFINITY, cu = INFINITY;
        if (inner && ((lo >> lane) & 1ull)) {
            const int p = 63 - __clzll((long long)(lo & below)), n = __ffsll((long long)(lo & above)) - 1;
            cl = cross3(su[p], sv[p], u, v, su[n], sv[n]);
        }
        if (inner && ((up >> lane) & 1ull)) {   // the upper chain runs from the last point to the first
            const int p = __ffsll((long long)(up & above)) - 1, n = 63 - __clzll((long long)(up & below));
            cu = cross3(su[p], sv[p], u, v, su[n], sv[n]);
        }
        const uint64_t dl = __ballot(cl < -tol), du = __ballot(cu < -tol);
        lo &= ~dl;
        up &= ~du;
        if ((dl | du) == 0) {
            settled = __ballot(!(cl > tol) || !(cu > tol)) == 0;
            break;
        }
    }
    uint32_t hl, hu;
    if (settled) {
        hl = (uint32_t)__popcll(lo);
        hu = (uint32_t)__popcll(up);
        if ((lo >> lane) & 1ull) st[__popcll(lo & below)] = (uint8_t)lane;
        if ((up >> lane) & 1ull) st[kWave + 1 + __popcll(up & above)] = (uint8_t)lane;
    } else {
        // the plain chains over the points left, the lower on lane 0 and the
        // upper on lane 1 at the same time, in place
        if ((lo >> lane) & 1ull) st[__popcll(lo & below)] = (uint8_t)lane;
        if ((up >> lane) & 1ull) st[kWave + 1 + __popcll(up & above)] = (uint8_t)lane;
        wave_sync();
        uint32_t h = 0;
        if (lane < 2) {
            uint8_t* s = st + (lane ? kWave + 1 : 0);
            h = chain_run(su, sv, s, (uint32_t)__popcll(lane ? up : lo), s);
        }
        hl = __shfl(h, 0, kWave);
        hu = __shfl(h, 1, kWave);
    }
    wave_sync();
    // the polygon: the lower chain, then the upper one without its end
    // points (the lower chain's last and first points)
    const uint32_t h = hl + (hu >= 2 ? hu - 2 : 0u);
    auto vertex = [&](uint32_t p) -> uint32_t {
        return p < hl ? st[p] : st[kWave + 1 + (p - hl + 1)];
    };
    double term = 0.0;
    uint32_t vi = 0;
    if ((uint32_t)lane < h) {
        vi = vertex((uint32_t)lane);
        const uint32_t v1 = vertex((uint32_t)lane + 1 == h ? 0u : (uint32_t)lane + 1);
        term = su[vi] * sv[v1] - su[v1] * sv[vi];
    }
    // shoelace sum over the vertices (a wave reduction)
#pragma unroll
    for (int dd = kWave / 2; dd >= 1; dd >>= 1) term += __shfl_xor(term, dd, kWave);
    r.h = h;
    r.vi = vi;
    r.area = h >= 3 ? 0.5 * term : 0.0;
    return r;
}

constexpr int kChainBlock = 512;   // threads of block_chain: the first half takes the lower chain

// LDS scratch of block_chain for up to Cap points.
template <int Cap>
struct ChainLds {
    double su[Cap];
    double sv[Cap];
    uint32_t si[Cap];
    uint16_t list[2][2][Cap];   // [lower, upper][two buffers]: points left, in chain order
    uint32_t cnt[2];
    uint32_t wsum[kChainBlock / kWave];
    uint32_t flag[2];           // a point was dropped; a corner does not clearly turn left
    double red[kChainBlock / kWave];
};

// The hull of 1 <= ns <= Cap points by one workgroup of kChainBlock threads:
// the points (load(t, &u, &v, &i) gives point t) are sorted in L by (u, v, i)
// -- one point per thread with shuffles for short distances, or a bitonic
// network in LDS -- then the two halves of the workgroup find the two chains
// by elimination.  emit(q, p) receives vertex q (counter-clockwise from the
// smallest point) as sorted position p (list position L.si[p]); thread 0 gets
// the shoelace area.  Returns the vertex count.
template <int Cap, class Load, class Emit>
__device__ __forceinline__ uint32_t block_chain(ChainLds<Cap>& L, uint32_t ns, Load load, Emit emit, double* area)
{
    uint32_t N = 1;
    while (N < ns) N <<= 1;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (N <= (uint32_t)kChainBlock) {
        // one point per thread: bitonic stages over distances below 64
        // are shuffles inside a wave, the others go through LDS
        const uint32_t t = threadIdx.x;
        double u = INFINITY, v = INFINITY;
        uint32_t id = 0xFFFFFFFFu;
        if (t < ns) load(t, &u, &v, &id);
        for (uint32_t size = 2; size <= N; size <<= 1) {
            for (uint32_t j = size >> 1; j > 0; j >>= 1) {
                double ou, ov;
                uint32_t oi;
                if (j >= (uint32_t)kWave) {
                    L.su[t] = u;
                    L.sv[t] = v;
                    L.si[t] = id;
                    __syncthreads();
                    ou = L.su[t ^ j];
                    ov = L.sv[t ^ j];
                    oi = L.si[t ^ j];
                    __syncthreads();
                } else {
                    ou = __shfl_xor(u, (int)j, kWave);
                    ov = __shfl_xor(v, (int)j, kWave);
                    oi = __shfl_xor(id, (int)j, kWave);
                }
                const bool up = (t & size) == 0, low = (t & j) == 0;
                if ((low == up) != p2_less(u, v, id, ou, ov, oi)) {
                    u = ou;
                    v = ov;
                    id = oi;
                }
            }
        }
        L.su[t] = u;
        L.sv[t] = v;
        L.si[t] = id;
        __syncthreads();
    } else {
        for (uint32_t t = threadIdx.x; t < N; t += kChainBlock) {
            if (t < ns) {
                load(t, &L.su[t], &L.sv[t], &L.si[t]);
            } else {
                L.su[t] = INFINITY;
                L.sv[t] = INFINITY;
                L.si[t] = 0xFFFFFFFFu;
            }
        }
        __syncthreads();
        for (uint32_t size = 2; size <= N; size <<= 1) {
            for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
                for (uint32_t t = threadIdx.x; t < N / 2; t += kChainBlock) {
                    const uint32_t a = 2 * t - (t & (stride - 1)), b = a + stride;
                    const bool upw = (a & size) == 0;
                    if (p2_less(L.su[b], L.sv[b], L.si[b], L.su[a], L.sv[a], L.si[a]) == upw) swap3(L.su, L.sv, L.si, a, b);
                }
                __syncthreads();
            }
        }
    }
    // the set's scale, and both lists: the sorted points, forward and backward
    double span = 0.0;
    for (uint32_t t = threadIdx.x; t < ns; t += kChainBlock) {
        span = fmax(span, fmax(L.su[t] - L.su[0], fabs(L.sv[t] - L.sv[0])));
        L.list[0][0][t] = (uint16_t)t;
        L.list[1][0][t] = (uint16_t)(ns - 1u - t);
    }
    span = wave_max_d(span);
    if (lane == 0) L.red[wave] = span;
    if (threadIdx.x < 2) {
        L.cnt[threadIdx.x] = ns;
        L.flag[threadIdx.x] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kChainBlock / kWave; ++w) span = fmax(span, L.red[w]);
    const double tol = chain_tolerance(span);
    constexpr uint32_t kHalf = kChainBlock / 2;
    constexpr int kHalfWaves = (int)kHalf / kWave;
    const uint32_t half = threadIdx.x / kHalf, t = threadIdx.x % kHalf;
    uint32_t n = ns;
    int buf = 0;
    bool settled = ns < 3;
    for (int round = 0; !settled && round < kMaxRounds; ++round) {
        const uint16_t* src = L.list[half][buf];
        uint16_t* dst = L.list[half][buf ^ 1];
        const uint32_t most = max(L.cnt[0], L.cnt[1]);
        uint32_t kept = 0;
        bool drop = false, odd = false;
        for (uint32_t p0 = 0; p0 < most; p0 += kHalf) {   // uniform over the workgroup
            const uint32_t p = p0 + t;
            bool keep = p < n;
            uint32_t me = 0;
            if (keep) {
                me = src[p];
                if (p > 0 && p + 1 < n) {
                    const uint32_t a = src[p - 1], b = src[p + 1];
                    const double c = cross3(L.su[a], L.sv[a], L.su[me], L.sv[me], L.su[b], L.sv[b]);
                    if (c < -tol) {
                        keep = false;
                        drop = true;
                    } else if (!(c > tol)) {
                        odd = true;
                    }
                }
            }
            const uint64_t bal = __ballot(keep);
            if (lane == 0) L.wsum[wave] = (uint32_t)__popcll(bal);
            __syncthreads();
            uint32_t pos = kept + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull)), tot = 0;
#pragma unroll
            for (int w = 0; w < kHalfWaves; ++w) {
                const uint32_t x = L.wsum[half * kHalfWaves + w];
                pos += w < wave % kHalfWaves ? x : 0u;
                tot += x;
            }
            if (keep) dst[pos] = (uint16_t)me;
            kept += tot;
            __syncthreads();   // wsum is reused, dst is read by the next round
        }
        n = kept;
        if (t == 0) L.cnt[half] = n;
        if (drop) L.flag[0] = 1;
        if (odd) L.flag[1] = 1;
        __syncthreads();
        const bool any_drop = L.flag[0] != 0, any_odd = L.flag[1] != 0;
        buf ^= 1;
        __syncthreads();
        if (threadIdx.x < 2) L.flag[threadIdx.x] = 0;
        if (!any_drop) {
            settled = !any_odd;
            break;
        }
        __syncthreads();
    }
    __syncthreads();
    if (!settled && t == 0) L.cnt[half] = chain_run(L.su, L.sv, L.list[half][buf], n, L.list[half][buf]);
    __syncthreads();
    // hull = lower chain, then the upper chain without its end points
    // (they are the lower chain's last and first points); the
    // vertices and the shoelace terms are taken in parallel
    {
        const uint32_t hl = L.cnt[0], hu = L.cnt[1];
        const uint32_t h = hl + (hu >= 2 ? hu - 2 : 0u);
        auto vertex = [&](uint32_t q) -> uint32_t { return q < hl ? L.list[0][buf][q] : L.list[1][buf][q - hl + 1]; };
        double term = 0.0;
        for (uint32_t q = threadIdx.x; q < h; q += kChainBlock) {
            const uint32_t p0 = vertex(q), p1 = vertex(q + 1 == h ? 0u : q + 1);
            term += L.su[p0] * L.sv[p1] - L.su[p1] * L.sv[p0];
            emit(q, p0);   // vertex q is sorted point p0
        }
#pragma unroll
        for (int dd = kWave / 2; dd >= 1; dd >>= 1) term += __shfl_xor(term, dd, kWave);
        if (lane == 0) L.red[wave] = term;
        __syncthreads();
        if (threadIdx.x == 0) {
            double tot = 0.0;
            for (int w2 = 0; w2 < kChainBlock / kWave; ++w2) tot += L.red[w2];
            *area = h >= 3 ? 0.5 * tot : 0.0;
        }
        return h;
    }
}

}  // namespace dev
}  // namespace vm
