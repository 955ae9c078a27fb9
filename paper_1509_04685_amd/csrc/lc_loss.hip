// Particle loss of the learned correction and its adjoint on the mesh, by tile ownership.
//
//   L = sum_p |r_p|^2 / D,  r_p = g1_p + G[dF]_p - g3_p,  D = sum_p |g3_p - g1_p|^2
//   d_dF = dL / d(dF) = G^T (2 r / D)       (G: CIC gather at absolute positions on a dense n^3 mesh)
//
// G^T is a deposit of three values per particle.  With float atomics to HBM (k_lc_loss, for callers
// without scratch) 24 of them per particle bound the pass: 1558 us for 128^3 particles on 128^3 cells,
// about 32 atomics per nanosecond.  Here the particles are sorted by tile as in the density deposit and
// each tile is accumulated in LDS and written once:
//   resid    r_p, the loss, count and rank per key
//   scan     of the counts
//   scatter  32-byte records {cell, fractions, r} in key order
//   tile     accumulation, d_dF written (no clear before)
// 128^3 particles on 128^3 cells in a training step: 111 + 5 + 22 + 62 us.
//
// The LDS sums are 64-bit fixed point: LDS integer atomics run at tens of times the rate of float ones.  The unit is
// 2^-b of the power of two above the tile's largest term, b = min(52, 62 - ceil(log2 records)), so that no sum
// can overflow.  c terms are then off by c / 2 units at most, less than c float32 additions where the result has 2^25
// units; the few smaller results of a tile are summed again in float64.  Where they are many, or a term would
// be lost, because residuals of very different size meet in the tile, all its sums are formed again with a unit
// for each cell and component, 2^-b above its own largest term.  (One unit for all, 2^-40 of the largest
// |r| of the call, left residuals 1e6 below it 18 bits.)  A tile that meets an infinite or NaN term
// takes float atomics in LDS, which keep such values in the cells that they reach, and so does a loss with D = 0.

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
constexpr uint32_t kSmallSums = 32;  // most sums of a tile that are formed again one by one

struct LossSort {
    float4* resid;    // per particle: r, rank in its key
    float4* sorted;   // two per particle, in key order
    uint32_t *count, *start, *block_sums;
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
    w.total = off;
    return w;
}

struct Ptr3 {
    const float* p[3];
};

__global__ void __launch_bounds__(256) k_loss_resid(Ptr3 pos, long np, int n, float inv_h, Ptr3 df, Ptr3 g1, Ptr3 g3,
                                                    TileGeom tg, double* stats, uint32_t* count, float4* resid) {
    __shared__ double red[256];
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = p < np;
    double l2 = 0.0;
    uint32_t key = 0;
    float r0 = 0.0f, r1 = 0.0f, r2 = 0.0f;
    if (valid) {
        LossCell c;
        loss_cell(pos.p[0][p], pos.p[1][p], pos.p[2][p], inv_h, n, c);
        loss_resid(c, n, df.p, g1.p, g3.p, p, r0, r1, r2);
        const double inv = 1.0 / stats[1];
        l2 = ((double)r0 * r0 + (double)r1 * r1 + (double)r2 * r2) * inv;
        int local;
        key = tile_key(tg, c.i[0][0], c.i[1][0], c.i[2][0], local);
    }
    const uint32_t rank = wave_increment(count, key, valid);
    if (valid) resid[p] = make_float4(r0, r1, r2, __uint_as_float(rank));
    red[threadIdx.x] = l2;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(&stats[0], red[0]);
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

// Calls f(cell, weight, r) for every corner inside the tile of the records i0 .. i1 - 1 of those that it pulls, the next
// record in flight meanwhile.
template <class F>
__device__ __forceinline__ void each_corner(const TileGeom& tg, const TileBox& tb, const PullRanges& pr, const PullStarts& ps,
                                            const float4* recs, uint32_t i0, uint32_t i1, F f) {
    int dx = 0, dy = 0, dz = 0;
    float4 next = make_float4(0.f, 0.f, 0.f, 0.f), next_r = next;
    auto load = [&](uint32_t i) {
        const float4* src = recs + 2 * (size_t)pulled_record(pr, ps, i, dx, dy, dz);
        next = src[0];
        next_r = src[1];
    };
    if (i0 < i1) load(i0);
    for (uint32_t i = i0; i < i1; ++i) {
        const float4 rec = next;
        const float r[3] = {next_r.x, next_r.y, next_r.z};
        int hx, hy, hz;
        pulled_cell(tg, __float_as_int(rec.x), dx, dy, dz, hx, hy, hz);
        if (i + 1 < i1) load(i + 1);
        const float wx[2] = {1.0f - rec.y, rec.y}, wy[2] = {1.0f - rec.z, rec.z}, wz[2] = {1.0f - rec.w, rec.w};
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
                    f((((ux << tg.ly) + uy) << tg.lz) + uz, wx[cx] * wy[cy] * wz[cz], r);
                }
            }
        }
    }
}

// Binary exponent of the unit of sums whose largest |term| has the upper word `top` (as a double), `bits` below the
// power of two above it.  Terms are products of two floats: above 2^-300 or zero.
__device__ __forceinline__ int unit_exponent(uint32_t top, int bits) { return (int)max(top >> 20, 200u) - 1022 - bits; }
__device__ __forceinline__ double exp2_of(int k) { return __hiloint2double((1023 + k) << 20, 0); }

// Bound by LDS atomics (24 of 64 bits per record) and, in a tile of many records, by the latency of their loads, hence
// blocks of 512.
__global__ void __launch_bounds__(512) k_loss_tile(TileGeom tg, const uint32_t* start, const float4* recs,
                                                   const double* stats, float* ddf) {
    __shared__ unsigned long long acc[3 * kLossCells];
    __shared__ uint32_t tile_top, small_sums, small[kSmallSums];
    __shared__ double exact[kSmallSums];
    __shared__ PullRanges pr;
    float* const facc = reinterpret_cast<float*>(acc);
    const int ncell = tg.tx * tg.ty * tg.tz;
    const TileBox tb = tile_box(tg, blockIdx.x);
    uint32_t b, e;
    request_pulls(tg, tb, start, b, e);
    for (int i = threadIdx.x; i < 3 * ncell; i += blockDim.x) acc[i] = 0ull;
    if (threadIdx.x == 0) tile_top = small_sums = 0u;
    if (threadIdx.x < kSmallSums) exact[threadIdx.x] = 0.0;
    finish_pulls(pr, b, e);
    const double s = 2.0 * (1.0 / stats[1]);
    __syncthreads();
    const uint32_t total = pr.len[14];
    const PullStarts ps = pull_starts(pr);
    const int bits = min(52, 30 + __clz((int)max(total, 2u) - 1));  // 62 - ceil(log2 total)
    const uint32_t chunk = (total + blockDim.x - 1) / blockDim.x;  // lanes far apart in the order, as in the deposit
    const uint32_t i0 = threadIdx.x * chunk;
    const uint32_t i1 = min(total, i0 + chunk);
    uint32_t most = 0, least = 0x7f800000u;  // float bits of the largest |w r| that a record can have, the smallest but 0
    for (uint32_t i = threadIdx.x; i < total; i += blockDim.x) {  // neighbours here, whole lines for the loads
        int dx, dy, dz;
        const float4* src = recs + 2 * (size_t)pulled_record(pr, ps, i, dx, dy, dz);
        const float4 rec = src[0], rv = src[1];
        const float f[3] = {fabsf(rec.y), fabsf(rec.z), fabsf(rec.w)};
        const float g[3] = {fabsf(1.0f - rec.y), fabsf(1.0f - rec.z), fabsf(1.0f - rec.w)};
        float hi = 1.0f, lo = 1.0f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float m = fminf(f[d], g[d]);
            hi *= fmaxf(f[d], g[d]);
            lo *= m > 0.0f ? m : 1.0f;
        }
        const float r[3] = {rv.x, rv.y, rv.z};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            most = max(most, __float_as_uint(fabsf(hi * r[d])));
            if (r[d] != 0.0f) least = min(least, __float_as_uint(fabsf(lo * r[d])));
        }
    }
    for (int off = 32; off > 0; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
    if ((threadIdx.x & 63) == 0 && most) atomicMax(&tile_top, most);
    __syncthreads();
    most = tile_top;
    const bool fixed = most < 0x7f800000u && fabs(s) <= 3.0e38;  // neither infinite nor NaN
    int k = 0;
    bool again = false;
    if (fixed && total > 0) {
        k = (int)(most >> 23) - 126 - bits;
        const double per_unit = exp2_of(-k);
        // a term would be lost, or the largest is nearer to zero than floats can tell
        again = __syncthreads_or((double)__uint_as_float(least) * per_unit < 1.0 || most < 0x00800000u);
        if (!again)
            each_corner(tg, tb, pr, ps, recs, i0, i1, [&](int cell, float w, const float (&r)[3]) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double t = (double)w * (double)r[d];
                    atomicAdd(&acc[d * ncell + cell], (unsigned long long)__double2ll_rn(t * per_unit));
                }
            });
        __syncthreads();
        for (int i = threadIdx.x; i < 3 * ncell; i += blockDim.x)
            if (acc[i] + (1ull << 25) < 1ull << 26 && acc[i] != 0ull) {
                const uint32_t q = atomicAdd(&small_sums, 1u);
                if (q < kSmallSums) small[q] = (uint32_t)i;
            }
        __syncthreads();
        again = again || small_sums > kSmallSums;
        if (!again && small_sums > 0)
            each_corner(tg, tb, pr, ps, recs, i0, i1, [&](int cell, float w, const float (&r)[3]) {
                for (uint32_t q = 0; q < small_sums; ++q) {
                    const int d = (int)small[q] / ncell;
                    if ((int)small[q] - d * ncell == cell)
                        atomicAdd(&exact[q], (double)w * (double)(d == 0 ? r[0] : d == 1 ? r[1] : r[2]));
                }
            });
    }
    const long V = (long)tg.n * tg.n * tg.n;
    auto place = [&](int i) {  // of cell i of the tile in the mesh, -1 outside
        const int uz = i & (tg.tz - 1), uy = (i >> tg.lz) & (tg.ty - 1), ux = i >> (tg.lz + tg.ly);
        return ux < tb.nx && uy < tb.ny && uz < tb.nz
                   ? ((long)(tb.x0 + ux) * tg.n + (tb.y0 + uy)) * tg.n + (tb.z0 + uz) : -1L;
    };
    if (again) {  // a component at a time, so that the upper words of the largest |term| fit beside its sums
        uint32_t* const top = reinterpret_cast<uint32_t*>(acc + ncell);
        for (int d = 0; d < 3; ++d) {
            __syncthreads();
            for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
                acc[i] = 0ull;
                top[i] = 0u;
            }
            __syncthreads();
            each_corner(tg, tb, pr, ps, recs, i0, i1, [&](int cell, float w, const float (&r)[3]) {
                const uint32_t t = (uint32_t)__double2hiint(fabs((double)w * (double)(d == 0 ? r[0] : d == 1 ? r[1] : r[2])));
                if (__hip_atomic_load(top + cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < t)
                    atomicMax(top + cell, t);
            });
            __syncthreads();
            each_corner(tg, tb, pr, ps, recs, i0, i1, [&](int cell, float w, const float (&r)[3]) {
                const double t = (double)w * (double)(d == 0 ? r[0] : d == 1 ? r[1] : r[2]);
                atomicAdd(&acc[cell], (unsigned long long)__double2ll_rn(t * exp2_of(-unit_exponent(top[cell], bits))));
            });
            __syncthreads();
            for (int i = threadIdx.x; i < ncell; i += blockDim.x)
                if (const long o = place(i); o >= 0)
                    ddf[d * V + o] = (float)((double)(long long)acc[i] * exp2_of(unit_exponent(top[i], bits)) * s);
        }
        return;
    }
    if (!fixed) {
        each_corner(tg, tb, pr, ps, recs, i0, i1, [&](int cell, float w, const float (&r)[3]) {
            const float ws = w * (float)s;
#pragma unroll
            for (int d = 0; d < 3; ++d) atomicAdd(&facc[d * ncell + cell], ws * r[d]);
        });
    }
    __syncthreads();
    const double unit = exp2_of(k);
    for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
        const long o = place(i);
        if (o < 0) continue;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int j = d * ncell + i;
            ddf[d * V + o] = fixed ? (float)((double)(long long)acc[j] * unit * s) : facc[j];
        }
    }
    if (small_sums == 0) return;
    __syncthreads();
    if (threadIdx.x < small_sums) {
        const int j = (int)small[threadIdx.x], d = j / ncell;
        ddf[d * V + place(j - d * ncell)] = (float)(exact[threadIdx.x] * s);
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
    hipError_t e = lc_loss_denominator(g1, g3, np, stats, st);
    if (e != hipSuccess) return e;
    if ((e = launch_fill(reinterpret_cast<float*>(w.count), tg.nkeys + 1, 0.0f, st)) != hipSuccess) return e;
    ProfScope ps(PROF_LC_MISC, st);
    const dim3 grid((unsigned)((np + 255) / 256));
    hipLaunchKernelGGL(k_loss_resid, grid, dim3(256), 0, st, P, np, n, inv_h, Ptr3{{df[0], df[1], df[2]}},
                       Ptr3{{g1[0], g1[1], g1[2]}}, Ptr3{{g3[0], g3[1], g3[2]}}, tg, stats, w.count, w.resid);
    if ((e = scan_counts(w.count, w.start, nullptr, w.block_sums, tg.nkeys, 0, 1, (uint32_t)np, false, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_loss_scatter, grid, dim3(256), 0, st, P, np, n, inv_h, tg, w.start, w.resid, w.sorted);
    hipLaunchKernelGGL(k_loss_tile, dim3((unsigned)tg.ntiles), dim3(512), 0, st, tg, w.start, w.sorted, stats, ddf);
    return hipGetLastError();
}

}  // namespace cola
