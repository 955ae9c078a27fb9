// Particle loss of the learned correction and its adjoint on the mesh, by tile ownership.
//
//   L = sum_p |r_p|^2 / D,  r_p = g1_p + G[dF]_p - g3_p,  D = sum_p |g3_p - g1_p|^2
//   d_dF = dL / d(dF) = G^T (2 r / D)       (G: CIC gather at absolute positions on a dense n^3 mesh)
//
// G^T is a deposit of three values per particle.  With float atomics to HBM (k_lc_loss, for callers
// without scratch) 24 of them per particle bound the pass: 1558 us for 128^3 particles on 128^3 cells,
// about 32 atomics per nanosecond.  Here the particles are sorted by tile as in the density deposit and
// each tile is accumulated in LDS and written once:
//   resid    r_p, the loss, the largest |r| component, count and rank per key
//   scan     of the counts
//   scatter  32-byte records {cell, fractions, r} in key order
//   tile     accumulation, d_dF written (no clear before)
// 128^3 particles on 128^3 cells: 112 + 14 + 22 + 52 us.
//
// The LDS sums are 64-bit fixed point, 2^-b of the largest |r| per unit: LDS integer atomics run at tens of
// times the rate of float ones.  b = 62 - log2(particles) up to 40, so no sum can overflow; a term is rounded
// to at most 2^-b of the largest, below float rounding of the sums except where they are 2^-16 of it.
// A loss with an infinite or NaN residual (or D = 0) takes float atomics in LDS, which keep such values in
// the cells that they reach.

#include <algorithm>
#include <cmath>

#include "cola_internal.h"
#include "lc_internal.h"
#include "lc_cic.h"
#include "tile_pull.h"
#include "wave_ops.h"

namespace cola {

namespace {

constexpr int kLossCells = 1024;  // most cells of a tile: three 64-bit sums each

struct LossSort {
    float4* resid;    // per particle: r, rank in its key
    float4* sorted;   // two per particle, in key order
    uint32_t *count, *start, *block_sums;
    uint32_t* rmax;   // bits of the largest |r| component
    size_t total;
};

// Tiles of at most kLossCells cells: those of a mesh with at least a particle per cell.
TileGeom loss_tiles(int n, long np) { return make_tiles(n, std::max(np, (long)n * n * n)); }

LossSort carve_loss(void* base, long np, const TileGeom& tg) {
    LossSort w{};
    char* b = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = b ? b + off : nullptr;
        off += lc_align(bytes);
        return p;
    };
    w.resid = reinterpret_cast<float4*>(take((size_t)np * 16));
    w.sorted = reinterpret_cast<float4*>(take((size_t)np * 32));
    w.count = reinterpret_cast<uint32_t*>(take(((size_t)tg.nkeys + 1) * 4));
    w.start = reinterpret_cast<uint32_t*>(take(((size_t)tg.nkeys + 1) * 4));
    w.block_sums = reinterpret_cast<uint32_t*>(take(((size_t)tg.nkeys / 1024 + 2) * 4));
    w.rmax = reinterpret_cast<uint32_t*>(take(4));
    w.total = off;
    return w;
}

struct Ptr3 {
    const float* p[3];
};

__global__ void __launch_bounds__(256) k_loss_resid(Ptr3 pos, long np, int n, float inv_h, Ptr3 df, Ptr3 g1, Ptr3 g3,
                                                    TileGeom tg, double* stats, uint32_t* count, uint32_t* rmax,
                                                    float4* resid) {
    __shared__ double red[256];
    __shared__ uint32_t top;
    if (threadIdx.x == 0) top = 0u;
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = p < np;
    double l2 = 0.0;
    uint32_t key = 0, big = 0;
    float r0 = 0.0f, r1 = 0.0f, r2 = 0.0f;
    if (valid) {
        LossCell c;
        loss_cell(pos.p[0][p], pos.p[1][p], pos.p[2][p], inv_h, n, c);
        loss_resid(c, n, df.p, g1.p, g3.p, p, r0, r1, r2);
        const double inv = 1.0 / stats[1];
        l2 = ((double)r0 * r0 + (double)r1 * r1 + (double)r2 * r2) * inv;
        big = max(__float_as_uint(fabsf(r0)), max(__float_as_uint(fabsf(r1)), __float_as_uint(fabsf(r2))));
        int local;
        key = tile_key(tg, c.i[0][0], c.i[1][0], c.i[2][0], local);
    }
    const uint32_t rank = wave_increment(count, key, valid);
    if (valid) resid[p] = make_float4(r0, r1, r2, __uint_as_float(rank));
    for (int off = 32; off > 0; off >>= 1) big = max(big, (uint32_t)__shfl_xor((int)big, off));
    red[threadIdx.x] = l2;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicMax(&top, big);
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicAdd(&stats[0], red[0]);
        atomicMax(rmax, top);
    }
}

__global__ void __launch_bounds__(256) k_loss_scatter(Ptr3 pos, long np, int n, float inv_h, TileGeom tg,
                                                      const uint32_t* start, const float4* resid, float4* sorted) {
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    LossCell c;
    loss_cell(pos.p[0][p], pos.p[1][p], pos.p[2][p], inv_h, n, c);
    const float4 r = resid[p];
    int local;
    const uint32_t key = tile_key(tg, c.i[0][0], c.i[1][0], c.i[2][0], local);
    float4* dst = sorted + 2 * (size_t)(start[key] + __float_as_uint(r.w));
    dst[0] = make_float4(__int_as_float(local), c.f[0], c.f[1], c.f[2]);
    dst[1] = make_float4(r.x, r.y, r.z, 0.0f);
}

__global__ void __launch_bounds__(256) k_loss_tile(TileGeom tg, const uint32_t* start, const float4* recs, int bits,
                                                   const uint32_t* rmax, const double* stats, float* ddf) {
    __shared__ unsigned long long acc[3 * kLossCells];
    __shared__ PullRanges pr;
    float* const facc = reinterpret_cast<float*>(acc);
    const int ncell = tg.tx * tg.ty * tg.tz;
    const TileBox tb = tile_box(tg, blockIdx.x);
    uint32_t b, e;
    request_pulls(tg, tb, start, b, e);
    for (int i = threadIdx.x; i < 3 * ncell; i += blockDim.x) acc[i] = 0ull;
    finish_pulls(pr, b, e);
    const float top = __uint_as_float(*rmax);
    const float s = (float)(2.0 * (1.0 / stats[1]));
    const bool fixed = top <= 3.0e38f && fabsf(s) <= 3.0e38f;  // neither infinite nor NaN
    const double to_fixed = top > 0.0f ? ldexp(1.0, bits) / (double)top : 0.0;
    const double from_fixed = (double)top * ldexp(1.0, -bits);
    __syncthreads();
    const uint32_t total = pr.len[14];
    const PullStarts ps = pull_starts(pr);
    const uint32_t chunk = (total + blockDim.x - 1) / blockDim.x;  // lanes far apart in the order, as in the deposit
    const uint32_t i0 = threadIdx.x * chunk;
    const uint32_t i1 = min(total, i0 + chunk);
    for (uint32_t i = i0; i < i1; ++i) {
        int dx, dy, dz;
        const float4* src = recs + 2 * (size_t)pulled_record(pr, ps, i, dx, dy, dz);
        const float4 rec = src[0], rv = src[1];
        int hx, hy, hz;
        pulled_cell(tg, __float_as_int(rec.x), dx, dy, dz, hx, hy, hz);
        const float wx[2] = {1.0f - rec.y, rec.y}, wy[2] = {1.0f - rec.z, rec.z}, wz[2] = {1.0f - rec.w, rec.w};
        const double q[3] = {rv.x * to_fixed, rv.y * to_fixed, rv.z * to_fixed};
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
            const int ux = hx + cx;
            if (ux < 0 || ux >= tb.nx) continue;
#pragma unroll
            for (int cy = 0; cy < 2; ++cy) {
                const int uy = hy + cy;
                if (uy < 0 || uy >= tb.ny) continue;
#pragma unroll
                for (int cz = 0; cz < 2; ++cz) {
                    const int uz = hz + cz;
                    if (uz < 0 || uz >= tb.nz) continue;
                    const int cell = (((ux << tg.ly) + uy) << tg.lz) + uz;
                    const float w = wx[cx] * wy[cy] * wz[cz];
                    if (fixed) {
#pragma unroll
                        for (int d = 0; d < 3; ++d)
                            atomicAdd(&acc[d * ncell + cell], (unsigned long long)__double2ll_rn((double)w * q[d]));
                    } else {
                        const float ws = w * s;
                        atomicAdd(&facc[cell], ws * rv.x);
                        atomicAdd(&facc[ncell + cell], ws * rv.y);
                        atomicAdd(&facc[2 * ncell + cell], ws * rv.z);
                    }
                }
            }
        }
    }
    __syncthreads();
    const long V = (long)tg.n * tg.n * tg.n;
    for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
        const int uz = i & (tg.tz - 1), uy = (i >> tg.lz) & (tg.ty - 1), ux = i >> (tg.lz + tg.ly);
        if (ux >= tb.nx || uy >= tb.ny || uz >= tb.nz) continue;
        const long o = ((long)(tb.x0 + ux) * tg.n + (tb.y0 + uy)) * tg.n + (tb.z0 + uz);
#pragma unroll
        for (int d = 0; d < 3; ++d)
            ddf[d * V + o] = fixed ? (float)((double)(long long)acc[d * ncell + i] * from_fixed) * s : facc[d * ncell + i];
    }
}

}  // namespace

size_t lc_loss_bytes(int n, long np) {
    const TileGeom tg = loss_tiles(n, np);
    return tg.nkeys + 1 > (long)INT32_MAX ? 0 : carve_loss(nullptr, np, tg).total;
}

hipError_t lc_loss_tiled(const float* const pos[3], long np, int n, double box, const float* const df[3],
                         const float* const g1[3], const float* const g3[3], double* stats, float* ddf, void* scratch,
                         hipStream_t st) {
    const TileGeom tg = loss_tiles(n, np);
    const LossSort w = carve_loss(scratch, np, tg);
    const float inv_h = (float)(n / box);
    const Ptr3 P{{pos[0], pos[1], pos[2]}};
    int lg = 0;
    while ((1L << lg) < np) ++lg;
    const int bits = std::min(40, 62 - lg);
    hipError_t e = lc_loss_denominator(g1, g3, np, stats, st);
    if (e != hipSuccess) return e;
    if ((e = launch_fill(reinterpret_cast<float*>(w.count), tg.nkeys + 1, 0.0f, st)) != hipSuccess) return e;
    if ((e = launch_fill(reinterpret_cast<float*>(w.rmax), 1, 0.0f, st)) != hipSuccess) return e;
    ProfScope ps(PROF_LC_MISC, st);
    const dim3 grid((unsigned)((np + 255) / 256));
    hipLaunchKernelGGL(k_loss_resid, grid, dim3(256), 0, st, P, np, n, inv_h, Ptr3{{df[0], df[1], df[2]}},
                       Ptr3{{g1[0], g1[1], g1[2]}}, Ptr3{{g3[0], g3[1], g3[2]}}, tg, stats, w.count, w.rmax, w.resid);
    if ((e = scan_counts(w.count, w.start, nullptr, w.block_sums, tg.nkeys, 0, 1, (uint32_t)np, false, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_loss_scatter, grid, dim3(256), 0, st, P, np, n, inv_h, tg, w.start, w.resid, w.sorted);
    hipLaunchKernelGGL(k_loss_tile, dim3((unsigned)tg.ntiles), dim3(256), 0, st, tg, w.start, w.sorted, bits, w.rmax,
                       stats, ddf);
    return hipGetLastError();
}

}  // namespace cola
