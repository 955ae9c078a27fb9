// Cloud-in-cell mass assignment by tile ownership (Sec. 2.2: CIC onto the force mesh; Sec. 2.5:
// CIC onto the P(k) mesh), without atomics to HBM and without clearing the mesh first.
//
// The mesh is cut into tiles of TX x TY x TZ cells.  Each particle gets a key
//   key = tile(home cell) * 8 + category,   category = 4 [x on the tile's upper face]
//                                                      + 2 [y on it] + [z on it],
// where the home cell is the lower CIC corner.  A particle's eight corners land in its own tile
// and, only along axes where its category bit is set, in the next tile up.  After a counting sort
// by key, the block that owns tile M reads its own bin and, from each of the seven tiles M - d
// (d in {0,1}^3, d != 0), just the categories that contain d -- the particles whose corners reach
// into M.  It accumulates the corners that fall inside M in LDS and writes every cell of M once,
// already converted to delta = rho * scale + offset.
//
// Passes: bin (wave-aggregated counts per key, which leave each particle its rank in its key), exclusive scan of the
// counts, place (the record of every particle, formed again from its position, at its key's start plus its
// rank), tile accumulation.  Particles drifted on the fly, whose positions are not kept, are binned with key and
// record, which a scatter pass moves.  Records keep the CIC fractions exactly as computed from the lattice index and
// displacement.

#include <algorithm>

#include "cola_internal.h"
#include "force_gather.h"
#include "lattice.h"
#include "tile_pull.h"
#include "wave_ops.h"

namespace cola {

// Tiles of 8 x 8 x tz cells; a mesh side that a tile side does not divide ends in a narrower tile.  tz is
// the largest of 64, 32, 16 that pads the side by at most an eighth and holds no more than about 1024
// particles on average -- on a mesh with a particle per cell (PM_grid 1) the 4096-particle tiles of
// 8 x 8 x 64 made the tile pass and the sort counters (many waves on one key) slower: 0.19 + 0.25 ms
// against 0.13 + 0.16 ms for 8 x 8 x 16.  Meshes of several particles per cell take smaller tiles, until
// one holds about 4096 particles, so that there are keys and blocks enough (uniform points in no
// order, 2.1e6 on 28^3: 485 -> 354 us, 1.7e6 on 64^3: 487 -> 285 us; 3e6 on 7^3 with tiles of 2 x 2 x 4 cells
// 2600, of single cells 530).
// Tiles that divide the side, as before, fell to 2 x 2 x 2 and to single cells for sides of 2 b and odd
// sides: 1e6 points on 250^3 took 2389 us, and past 256^3 single-cell tiles are more blocks than a
// grid holds.
TileGeom make_tiles(int n, long n_particles) {
    TileGeom t;
    t.n = n;
    const double per_cell = (double)n_particles / ((double)n * n * n);
    t.tx = 8;
    t.tz = 16;
    for (int c : {64, 32})
        if ((n + c - 1) / c * c - n <= n / 8 && (double)t.tx * t.tx * c * per_cell <= 1024.0) { t.tz = c; break; }
    while ((double)t.tx * t.tx * t.tz * per_cell > 4096.0 && t.tx * t.tz > 1) {
        if (t.tx > 4 || (t.tz <= 4 && t.tx > 1)) t.tx /= 2;
        else t.tz /= 2;
    }
    t.ty = t.tx;
    t.ntx = (n + t.tx - 1) / t.tx;
    t.nty = (n + t.ty - 1) / t.ty;
    t.ntz = (n + t.tz - 1) / t.tz;
    t.ntiles = (long)t.ntx * t.nty * t.ntz;
    t.nkeys = t.ntiles * 8;
    auto lg = [](int v) { int l = 0; while ((1 << l) < v) ++l; return l; };
    t.lx = lg(t.tx);
    t.ly = lg(t.ty);
    t.lz = lg(t.tz);
    return t;
}

namespace {


// The per-particle key and record arrays are written once and read once, in particle order:
// non-temporal, so that they do not evict mesh and count lines from L2 (the tile pass also
// stores the mesh this way).
__device__ __forceinline__ void store_rec_stream(float4* p, float4 v) {
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
    __builtin_nontemporal_store(v.z, &p->z);
    __builtin_nontemporal_store(v.w, &p->w);
}
__device__ __forceinline__ float4 load_rec_stream(const float4* p) {
    float4 v;
    v.x = __builtin_nontemporal_load(&p->x);
    v.y = __builtin_nontemporal_load(&p->y);
    v.z = __builtin_nontemporal_load(&p->z);
    v.w = __builtin_nontemporal_load(&p->w);
    return v;
}

// Binning of the particles onto the mesh of dg (counts per key).  MODE 0: at their positions; 1: drifted
// on the fly (kick with the force gathered from fg's
// meshes, then the drift of kd) without changing the state -- outputs between nodes and the
// redshift-space mapping; 2: the step's gather, kick and drift, written back to p and x, then
// binned at the new positions for the next force evaluation (dg = fg).
// Modes 0 and 2 leave each particle's rank in its key, from which, with its position, k_dep_place
// forms the record again: 4 bytes written and 16 read per particle instead of 20 and 20, and no
// atomics in the second pass (256^3 particles and cells: 439 + 171 -> 390 + 142 us; both bound by their
// memory traffic, the second by its scattered 16-byte stores).  The drifted positions of mode 1 are not kept, so it stores key and record.
template <int MODE>
__global__ void __launch_bounds__(256) k_dep_bin(ParticlePtrs P, long npr, LatticeGeom dg, TileGeom tg,
                                                 LatticeGeom fg, const float* F, KickDrift kd, SortBufs sb) {
    constexpr bool DRIFT = MODE != 0;
    const LatticeSite site = lattice_site(dg);
    const int r = blockIdx.z;
    const bool valid = site.valid;
    const long gid = (long)r * npr + site.p;
    uint32_t key = 0;
    if (valid) {
        float x[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) x[d] = __builtin_nontemporal_load(P.x[d] + gid);
        // x is issued first: loads complete in order, so the gather, whose addresses need only x,
        // waits for these three and not for the nine below
        __builtin_amdgcn_sched_barrier(0);
        if (DRIFT) {
            // The particle arrays are read before the force gather, so both are in flight together.
            // All nine are loaded without a branch: loads guarded per axis (by the line of sight)
            // made the compiler wait for each axis's loads before issuing the next, which added a
            // memory round trip to every wave.
            float s1[3], s2[3], pv[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                s1[d] = __builtin_nontemporal_load(P.psi1[d] + gid);
                s2[d] = __builtin_nontemporal_load(P.psi2[d] + gid);
                pv[d] = __builtin_nontemporal_load(P.p[d] + gid);
            }
            float g[3] = {0.0f, 0.0f, 0.0f};
            if (kd.kick != 0.0f) {  // no force mesh is read for a pure drift (redshift-space mapping)
                LatticeCell c[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) c[d] = lattice_cell(fg, site.i[d], x[d]);
                gather_interleaved(F + (long)r * fg.mesh_bstride, fg.row, fg.n_mesh, c[0].m, c[1].m, c[2].m, c[0].f,
                                   c[1].f, c[2].f, g);
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if (kd.los >= 0 && d != kd.los) continue;
                const float ph = pv[d] + kd.kick * (g[d] - kd.d1 * s1[d] - kd.d2m * s2[d]);
                x[d] = x[d] + ph * kd.drift + kd.dd1 * s1[d] + kd.dd2 * s2[d];
                if (MODE == 2) {
                    __builtin_nontemporal_store(ph, P.p[d] + gid);
                    __builtin_nontemporal_store(x[d], P.x[d] + gid);
                }
            }
        }
        LatticeCell c[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) c[d] = lattice_cell(dg, site.i[d], x[d]);
        int local;
        key = tile_key(tg, c[0].m, c[1].m, c[2].m, local);
        if (MODE == 1) {
            __builtin_nontemporal_store(key, sb.keys + gid);
            store_rec_stream(sb.recs + gid, make_float4(__int_as_float(local), c[0].f, c[1].f, c[2].f));
        }
    }
    const uint32_t rank = wave_increment(sb.count + (long)r * sb.kstride, key, valid);
    if (MODE != 1 && valid) __builtin_nontemporal_store(rank, sb.keys + gid);
}

// The record of every particle at its key's start plus its rank.
__global__ void __launch_bounds__(256) k_dep_place(ParticlePtrs P, long npr, LatticeGeom dg, TileGeom tg, SortBufs sb) {
    const LatticeSite site = lattice_site(dg);
    if (!site.valid) return;
    const int r = blockIdx.z;
    const long gid = (long)r * npr + site.p;
    LatticeCell c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) c[d] = lattice_cell(dg, site.i[d], __builtin_nontemporal_load(P.x[d] + gid));
    const uint32_t rank = __builtin_nontemporal_load(sb.keys + gid);
    int local;
    const uint32_t key = tile_key(tg, c[0].m, c[1].m, c[2].m, local);
    sb.sorted[(long)r * npr + sb.start[(long)r * sb.kstride + key] + rank] =
        make_float4(__int_as_float(local), c[0].f, c[1].f, c[2].f);
}

// Absolute positions (the component entry points): the cell of a coordinate is floor(pos n / L) modulo
// the mesh.  Two passes over the positions: the first counts per key and keeps each point's rank in its
// key (the counter's old value), the second forms the cell record again and stores it at its key's start
// plus that rank.  Both are bound by the counters' atomics where the points come in no order (about 20 per
// nanosecond on the whole chip, against one per run of equal keys in lattice order), so the second pass
// has none, and no key and record arrays pass through HBM between the two: 1e6 clustered points in no order,
// 250^3 cells, 89 + 83 us with atomics in both and records in between, 74 + 25 us so; 1e7 uniform ones on
// 200^3 1162 -> 864 us for the whole deposit.
struct AbsCells {
    LatticeCell c[3];
};
__device__ __forceinline__ AbsCells abs_cells(const float* px, const float* py, const float* pz, long p, int n_mesh,
                                              float inv_h) {
    const float* ps[3] = {px, py, pz};
    AbsCells a;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        // the cell of the rounded product, the fraction of the exact one (a fused multiply-add):
        // where the product rounds up to a node the fraction is about -1e-7 of it, a weight that
        // the tile pass clamps at 0
        const float v = __builtin_nontemporal_load(ps[d] + p);
        const float fl = floorf(v * inv_h);
        a.c[d].f = fmaf(v, inv_h, -fl);
        int m = (int)fl % n_mesh;
        m = m < 0 ? m + n_mesh : m;
        a.c[d].m = min(max(m, 0), n_mesh - 1);
    }
    return a;
}

constexpr int kOddRecord = (int)0x80000000;

// Whether all fractions are those of a finite position near enough for its float32 cell coordinate to hold them:
// within a quarter of [0, 1], which up to 2^22 cells from the origin they are.
__device__ __forceinline__ bool regular(const AbsCells& a) {
    return fabsf(a.c[0].f - 0.5f) <= 0.75f && fabsf(a.c[1].f - 0.5f) <= 0.75f && fabsf(a.c[2].f - 0.5f) <= 0.75f;
}

__global__ void __launch_bounds__(256) k_abs_count(const float* px, const float* py, const float* pz, long n,
                                                   int n_mesh, float inv_h, TileGeom tg, uint32_t* count,
                                                   uint32_t* rank) {
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = p < n;
    uint32_t key = 0;
    if (valid) {
        const AbsCells a = abs_cells(px, py, pz, p, n_mesh, inv_h);
        int local;
        key = tile_key(tg, a.c[0].m, a.c[1].m, a.c[2].m, local);
    }
    const uint32_t r = wave_increment<true>(count, key, valid);
    if (valid) __builtin_nontemporal_store(r, rank + p);
}

// MARK: the cell of a point that is not regular has its sign set.
template <bool MARK>
__global__ void __launch_bounds__(256) k_abs_scatter(const float* px, const float* py, const float* pz, long n,
                                                     int n_mesh, float inv_h, TileGeom tg, const uint32_t* start,
                                                     const uint32_t* rank, float4* sorted) {
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t r = __builtin_nontemporal_load(rank + p);
    const AbsCells a = abs_cells(px, py, pz, p, n_mesh, inv_h);
    int local;
    const uint32_t key = tile_key(tg, a.c[0].m, a.c[1].m, a.c[2].m, local);
    if (MARK && !regular(a)) local |= kOddRecord;
    sorted[start[key] + r] = make_float4(__int_as_float(local), a.c[0].f, a.c[1].f, a.c[2].f);
}

// Exclusive scan of the key counts in at most two launches (three for more than 4096 blocks of keys).  At a
// few microseconds a launch is what these passes cost on most meshes, so they are few: per block of 4096
// keys one sum, then every block adds up the sums before it and scans its own keys; one block does all
// where it can.  Blocks of 1024 keys, a pass for their sums and one to add them took three launches
// on every mesh: 10 steps of 32^3 particles 1218 -> 1170 us; 16.8e6 cells of friends-of-friends 94 -> 35 us
// (four-key vectors in rows of a wave; with a thread's 16 keys next to each other 210 us).
constexpr int kScanKeys = 16;                     // keys of a thread: four of each of its wave's four rows of 256
constexpr int kScanBlock = 256 * kScanKeys;       // keys of a block of 256
constexpr int kScanOne = 1024 * kScanKeys;        // up to these, one block of 1024 threads
constexpr int kScanSums = 4096;                   // up to these blocks, each adds up the sums before it

__device__ __forceinline__ long scan_key(int row) {  // the thread's first key of a row (a multiple of 4)
    return ((long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (64 * kScanKeys) + row * 256 +
           (threadIdx.x & 63) * 4;
}
__device__ __forceinline__ uint4 load_counts(const uint32_t* count, long k, long nkeys) {
    if (k + 3 < nkeys) return *reinterpret_cast<const uint4*>(count + k);
    return make_uint4(k < nkeys ? count[k] : 0u, k + 1 < nkeys ? count[k + 1] : 0u, k + 2 < nkeys ? count[k + 2] : 0u, 0u);
}
__device__ __forceinline__ void store_keys(uint32_t* out, long k, long nkeys, uint4 v) {
    if (k + 3 < nkeys) {
        *reinterpret_cast<uint4*>(out + k) = v;
    } else {
        if (k < nkeys) out[k] = v.x;
        if (k + 1 < nkeys) out[k + 1] = v.y;
        if (k + 2 < nkeys) out[k + 2] = v.z;
    }
}

__device__ __forceinline__ uint32_t wave_prefix(uint32_t s) {  // inclusive
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(s, off);
        s += lane >= off ? t : 0u;
    }
    return s;
}

// Sum over the earlier waves of the block (at most 16) of their s, the same in all lanes of a wave; `all` is the
// block's sum.
__device__ __forceinline__ uint32_t waves_before(uint32_t s, uint32_t& all) {
    __shared__ uint32_t wave_sum[16];
    const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    __syncthreads();  // an earlier use has been read
    if ((threadIdx.x & 63) == 0) wave_sum[wave] = s;
    __syncthreads();
    uint32_t before = 0;
    all = 0;
    for (int w = 0; w < waves; ++w) {
        before += w < wave ? wave_sum[w] : 0u;
        all += wave_sum[w];
    }
    return before;
}

__global__ void __launch_bounds__(256) k_scan_sums(const uint32_t* count, uint32_t* sums, long nkeys, long kstride,
                                                   int nblocks) {
    const int r = blockIdx.y;
    uint32_t s = 0, all;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint4 v = load_counts(count + (long)r * kstride, scan_key(j), nkeys);
        s += v.x + v.y + v.z + v.w;
    }
    waves_before(__shfl(wave_prefix(s), 63), all);
    if (threadIdx.x == 0) sums[(long)r * nblocks + blockIdx.x] = all;
}

// The block sums' exclusive prefix, in place (more than kScanSums blocks).
__global__ void __launch_bounds__(1024) k_scan_totals(uint32_t* sums, int nblocks) {
    sums += (long)blockIdx.y * nblocks;
    const int per = (nblocks + 1023) / 1024;
    const int b0 = min(nblocks, (int)threadIdx.x * per), b1 = min(nblocks, b0 + per);
    uint32_t s = 0, all;
    for (int b = b0; b < b1; ++b) s += sums[b];
    const uint32_t incl = wave_prefix(s);
    uint32_t run = waves_before(__shfl(incl, 63), all) + incl - s;
    for (int b = b0; b < b1; ++b) {
        const uint32_t v = sums[b];
        sums[b] = run;
        run += v;
    }
}

// start[k] = sum of the counts before k, cursor[k] the same (null: not wanted), start[nkeys] = total; clear: the
// counts become zero, for the next binning.  prefix: the sums are already prefixes.
__global__ void __launch_bounds__(1024) k_scan_keys(uint32_t* count, uint32_t* start, uint32_t* cursor,
                                                    const uint32_t* sums, bool prefix, bool clear, long nkeys,
                                                    long kstride, int nblocks, uint32_t total) {
    const int r = blockIdx.y;
    count += (long)r * kstride;
    start += (long)r * kstride;
    sums += (long)r * nblocks;
    uint4 v[4];
    uint32_t incl[4], sum = 0, base = 0, all;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = load_counts(count, scan_key(j), nkeys);
    if (prefix) {
        base = sums[blockIdx.x];
    } else if (blockIdx.x > 0) {
        uint32_t s = 0;
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += blockDim.x) s += sums[b];
        waves_before(__shfl(wave_prefix(s), 63), base);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        incl[j] = wave_prefix(v[j].x + v[j].y + v[j].z + v[j].w);
        sum += __shfl(incl[j], 63);
    }
    uint32_t row = base + waves_before(sum, all);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const long k = scan_key(j);
        const uint32_t a = row + incl[j] - (v[j].x + v[j].y + v[j].z + v[j].w);
        const uint4 o = make_uint4(a, a + v[j].x, a + v[j].x + v[j].y, a + v[j].x + v[j].y + v[j].z);
        store_keys(start, k, nkeys, o);
        if (cursor) store_keys(cursor + (long)r * kstride, k, nkeys, o);
        if (clear) store_keys(count, k, nkeys, make_uint4(0u, 0u, 0u, 0u));
        row += __shfl(incl[j], 63);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) start[nkeys] = total;
}

// All passes before the tiles for a few points on few keys, by one block with the counts in LDS: the four launches
// of the general path cost more than their work (density of 1000 points 28 -> 19 us, fields of 16^3 particles on 16^3
// cells 73 -> 61).  Beyond 4096 points the positions' memory round trips, in one block one after the other, cost more.
constexpr long kSmallPoints = 4096, kSmallKeys = 8192;
template <bool MARK>
__global__ void __launch_bounds__(1024) k_abs_small(const float* px, const float* py, const float* pz, int n, int n_mesh,
                                                    float inv_h, TileGeom tg, uint32_t* start, float4* sorted) {
    extern __shared__ uint32_t cnt[];
    const int nkeys = (int)tg.nkeys, per = (nkeys + 1023) / 1024;
    for (int k = threadIdx.x; k < nkeys; k += 1024) cnt[k] = 0u;
    __syncthreads();
    for (int p = threadIdx.x; p < n; p += 1024) {
        const AbsCells a = abs_cells(px, py, pz, p, n_mesh, inv_h);
        int local;
        atomicAdd(&cnt[tile_key(tg, a.c[0].m, a.c[1].m, a.c[2].m, local)], 1u);
    }
    __syncthreads();
    const int k0 = min(nkeys, (int)threadIdx.x * per), k1 = min(nkeys, k0 + per);
    uint32_t s = 0, all;
    for (int k = k0; k < k1; ++k) s += cnt[k];
    const uint32_t incl = wave_prefix(s);
    uint32_t run = waves_before(__shfl(incl, 63), all) + incl - s;
    for (int k = k0; k < k1; ++k) {
        const uint32_t c = cnt[k];
        cnt[k] = start[k] = run;  // the next free place of the key
        run += c;
    }
    if (threadIdx.x == 0) start[nkeys] = (uint32_t)n;
    __syncthreads();
    for (int p = threadIdx.x; p < n; p += 1024) {
        const AbsCells a = abs_cells(px, py, pz, p, n_mesh, inv_h);
        int local;
        const uint32_t key = tile_key(tg, a.c[0].m, a.c[1].m, a.c[2].m, local);
        if (MARK && !regular(a)) local |= kOddRecord;
        sorted[atomicAdd(&cnt[key], 1u)] = make_float4(__int_as_float(local), a.c[0].f, a.c[1].f, a.c[2].f);
    }
}

__global__ void k_dep_scatter(long npr, SortBufs sb) {
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    const bool valid = p < npr;
    const long gid = (long)r * npr + p;
    uint32_t key = valid ? __builtin_nontemporal_load(sb.keys + gid) : 0u;
    float4 rec = valid ? load_rec_stream(sb.recs + gid) : make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t slot = wave_increment(sb.cursor + (long)r * sb.kstride, key, valid);
    if (valid) sb.sorted[(long)r * npr + slot] = rec;
}

// A CIC weight w in [0, 1] in 32.32 fixed point (rounded; a negative one, see above, is 0).
__device__ __forceinline__ unsigned long long fixed_weight(float w) {
    const float t = __builtin_rintf(fmaxf(w, 0.0f) * 4294967296.0f);
    const bool whole = t >= 4294967296.0f;
    return (unsigned long long)(whole ? 1u : 0u) << 32 | (whole ? 0u : (uint32_t)t);
}

// A 32.32 fixed-point sum as float, rounded once: its 32 leading bits, the last of them also set for any
// bit below (round to nearest even of the conversion then sees them).
__device__ __forceinline__ float mass_of(unsigned long long v) {
    const uint32_t hi = (uint32_t)(v >> 32);
    const int s = hi ? __clz((int)hi) : 32;
    const unsigned long long t = v << s;
    return ldexpf((float)((uint32_t)(t >> 32) | min((uint32_t)t, 1u)), -s);
}

// One block per tile: pull the records whose corners reach into the tile, accumulate in LDS,
// write every cell of the tile once as delta = rho * scale + offset.  The 14 record ranges are
// fetched in parallel first, then all threads sweep their concatenation, the next record in flight
// while one is added.  The pass is bound by the vector ALU as much as by its stores (1135
// instructions per wave, 121 of 130 us, with 64-bit conversions of every weight and cell and 64-bit
// addresses, on 256^3 cells and particles), hence 32-bit arithmetic for both: 121 us there; 653 -> 636 us for
// 256^3 particles on 768^3 cells, where the chain of loads of a tile is longer than its arithmetic.
//
// Cell masses accumulate in fixed point in 64-bit integers: LDS integer atomics run at tens of times the
// rate of LDS float atomics on this hardware, and integer sums do not depend on the order of the adds
// (the deposit is bitwise reproducible).  32.32 for FRAC = 0: a CIC weight is rounded to 2^-32, a negative one
// is 0, a cell overflows only beyond 2^32 particles.  A mesh with many more cells than particles multiplies
// that rounding by their ratio, and the fields of the learned correction had float sums, with 24 bits of a weight
// of any size and its sign.  So theirs (FRAC = 1) are signed, with `frac` = 61 - ceil(log2 particles) bits after the
// point where cells are more than three to two particles (rounded to cells 2^-61 a term, in units of the mean
// density), and 32 otherwise (rounded to 2^-32; the contrast itself is rounded to 2^-25; the bits of cic_density).
// Points that are not regular are left out of the sums and added to the finished tile with float atomics:
// NaN and infinite weights reach the cells that they have there, as in a mesh of float sums.
template <bool FRAC>
__global__ void __launch_bounds__(256) k_dep_tile(TileGeom tg, SortBufs sb, long npr, float* mesh, long row,
                                                  long mesh_bstride, float scale, float offset, int frac) {
    extern __shared__ unsigned long long acc[];
    __shared__ PullRanges pr;
    const int r = blockIdx.y;
    const int ncell = tg.tx * tg.ty * tg.tz;
    const TileBox tb = tile_box(tg, blockIdx.x);
    const float4* recs = sb.sorted + (long)r * npr;
    // The range bounds are requested first, so that their latency overlaps the LDS clear.
    uint32_t b, e;
    request_pulls(tg, tb, sb.start + (long)r * sb.kstride, b, e);
    // 8 bytes per lane and store: with 16 the whole pass took 767 instead of 636 us on 768^3
    for (int i = threadIdx.x; i < ncell; i += 256) acc[i] = 0ull;
    finish_pulls(pr, b, e);
    __syncthreads();
    const uint32_t total = pr.len[14];
    const PullStarts ps = pull_starts(pr);
    const float units = ldexpf(1.0f, frac);  // of a weight of 1
    auto fixed = [&](float w) { return FRAC ? (unsigned long long)__float2ll_rn(w * units) : fixed_weight(w); };
    auto cell = [&](unsigned long long v) { return fmaf(FRAC ? (float)(long long)v : mass_of(v), scale, offset); };
    // Each thread sweeps a contiguous chunk of the concatenated records, so that the lanes of a
    // wave work on records far apart in the sorted order: records of one key range are in
    // Lagrangian order, and neighbouring particles hit the same cells -- consecutive records on
    // consecutive lanes would serialise the LDS atomics.
    const uint32_t chunk = (total + blockDim.x - 1) / blockDim.x;
    const uint32_t i0 = threadIdx.x * chunk;
    const uint32_t i1 = min(total, i0 + chunk);
    int dx = 0, dy = 0, dz = 0;
    bool odd = false;
    float4 next = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i0 < i1) next = recs[pulled_record(pr, ps, i0, dx, dy, dz)];
    for (uint32_t i = i0; i < i1; ++i) {
        const float4 rec = next;
        int hx, hy, hz;
        pulled_cell(tg, __float_as_int(rec.x), dx, dy, dz, hx, hy, hz);
        if (i + 1 < i1) next = recs[pulled_record(pr, ps, i + 1, dx, dy, dz)];
        if (FRAC && (__float_as_int(rec.x) & kOddRecord)) {
            odd = true;
            continue;
        }
        const float wx[2] = {1.0f - rec.y, rec.y}, wy[2] = {1.0f - rec.z, rec.z}, wz[2] = {1.0f - rec.w, rec.w};
        const bool okx[2] = {hx >= 0, hx + 1 < tb.nx}, oky[2] = {hy >= 0, hy + 1 < tb.ny}, okz[2] = {hz >= 0, hz + 1 < tb.nz};
        const int cell0 = ((hx << tg.ly) + hy) * (1 << tg.lz) + hz;  // of the lower corner (an index, not yet a cell)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx)
#pragma unroll
            for (int cy = 0; cy < 2; ++cy) {
                if (!(okx[cx] && oky[cy])) continue;
                const float wxy = wx[cx] * wy[cy];
                const int c = cell0 + (((cx << tg.ly) + cy) << tg.lz);
                if (okz[0]) atomicAdd(&acc[c], fixed(wxy * wz[0]));
                if (okz[1]) atomicAdd(&acc[c + 1], fixed(wxy * wz[1]));
            }
    }
    if (FRAC) odd = __syncthreads_or(odd);
    else __syncthreads();
    float* out = mesh + (long)r * mesh_bstride + ((long)tb.x0 * tg.n + tb.y0) * row + tb.z0;
    const uint32_t row32 = (uint32_t)row;  // offsets within a tile: below 8 1536 rows of 1568 floats
    if (((tg.tz | tg.n | (int)row) & 3) == 0) {  // rows of the tile are whole, aligned float4s
        for (int i4 = threadIdx.x; i4 < (ncell >> 2); i4 += 256) {
            const int i = i4 << 2;
            const int uz = i & (tg.tz - 1), uy = (i >> tg.lz) & (tg.ty - 1), ux = i >> (tg.lz + tg.ly);
            if (ux >= tb.nx || uy >= tb.ny || uz >= tb.nz) continue;
            const ulonglong2 u = reinterpret_cast<const ulonglong2*>(acc)[i >> 1],
                             v = reinterpret_cast<const ulonglong2*>(acc)[(i >> 1) + 1];
            const float4 a = make_float4(cell(u.x), cell(u.y), cell(v.x), cell(v.y));
            const uint32_t o = __umul24(__umul24(ux, tg.n) + uy, row32) + uz;
            store_rec_stream(reinterpret_cast<float4*>(out + o), a);
        }
    } else {
        for (int i = threadIdx.x; i < ncell; i += 256) {
            const int uz = i & (tg.tz - 1), uy = (i >> tg.lz) & (tg.ty - 1), ux = i >> (tg.lz + tg.ly);
            if (ux >= tb.nx || uy >= tb.ny || uz >= tb.nz) continue;
            out[__umul24(__umul24(ux, tg.n) + uy, row32) + uz] = cell(acc[i]);
        }
    }
    if (!FRAC || !odd) return;
    __syncthreads();
    const float back = scale * units;  // the scale of a weight
    for (uint32_t i = threadIdx.x; i < total; i += 256) {
        const float4 rec = recs[pulled_record(pr, ps, i, dx, dy, dz)];
        const int local = __float_as_int(rec.x);
        if (!(local & kOddRecord)) continue;
        int h[3];
        pulled_cell(tg, local & ~kOddRecord, dx, dy, dz, h[0], h[1], h[2]);
        const float f[3] = {rec.y, rec.z, rec.w};
        for (int c = 0; c < 8; ++c) {
            const int ux = h[0] + (c >> 2), uy = h[1] + (c >> 1 & 1), uz = h[2] + (c & 1);
            if (ux < 0 || uy < 0 || uz < 0 || ux >= tb.nx || uy >= tb.ny || uz >= tb.nz) continue;
            const float w = (c >> 2 ? f[0] : 1.0f - f[0]) * (c >> 1 & 1 ? f[1] : 1.0f - f[1]) * (c & 1 ? f[2] : 1.0f - f[2]);
            atomicAdd(out + __umul24(__umul24(ux, tg.n) + uy, row32) + uz, w * back);
        }
    }
}

}  // namespace

hipError_t scan_counts(uint32_t* count, uint32_t* start, uint32_t* cursor, uint32_t* block_sums, long nkeys,
                       long kstride, int n_real, uint32_t total, bool clear, hipStream_t st) {
    const bool one = nkeys <= kScanOne;
    const int threads = one ? (int)((nkeys + 64 * kScanKeys - 1) / (64 * kScanKeys)) * 64 : 256;
    const int nblocks = one ? 1 : (int)((nkeys + kScanBlock - 1) / kScanBlock);
    const bool prefix = nblocks > kScanSums;
    if (!one)
        hipLaunchKernelGGL(k_scan_sums, dim3(nblocks, n_real), dim3(256), 0, st, count, block_sums, nkeys, kstride,
                           nblocks);
    if (prefix) hipLaunchKernelGGL(k_scan_totals, dim3(1, n_real), dim3(1024), 0, st, block_sums, nblocks);
    hipLaunchKernelGGL(k_scan_keys, dim3(nblocks, n_real), dim3(threads), 0, st, count, start, cursor, block_sums, prefix,
                       clear, nkeys, kstride, nblocks, total);
    return hipGetLastError();
}

size_t sort_bytes(long n_particles_per_real, const TileGeom& tg, int n_real) {
    size_t nkp = (size_t)tg.nkeys + 1;
    size_t nblocks = (size_t)((tg.nkeys + 1023) / 1024);
    size_t per = (size_t)n_particles_per_real * (4 + 16 + 16) + nkp * 4 * 3 + nblocks * 4 + 256 * 6;
    return per * (size_t)n_real + 1024;
}

SortBufs carve_sort(void* base, long npr, const TileGeom& tg, int n_real) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    char* b = static_cast<char*>(base);
    SortBufs s;
    s.kstride = tg.nkeys + 4;  // nkeys + 1 entries, every realization's aligned to 16 bytes (nkeys is a multiple of 8)
    size_t off = 0;
    s.keys = reinterpret_cast<uint32_t*>(b + off); off = al(off + (size_t)npr * n_real * 4);
    s.recs = reinterpret_cast<float4*>(b + off); off = al(off + (size_t)npr * n_real * 16);
    s.sorted = reinterpret_cast<float4*>(b + off); off = al(off + (size_t)npr * n_real * 16);
    s.count = reinterpret_cast<uint32_t*>(b + off); off = al(off + (size_t)s.kstride * n_real * 4);
    s.start = reinterpret_cast<uint32_t*>(b + off); off = al(off + (size_t)s.kstride * n_real * 4);
    s.cursor = reinterpret_cast<uint32_t*>(b + off); off = al(off + (size_t)s.kstride * n_real * 4);
    s.block_sums = reinterpret_cast<uint32_t*>(b + off);
    return s;
}

namespace {
// Tile accumulation of the sorted records.  frac: bits after the point of the signed sums, 0: 32.32.
hipError_t run_tiles(long npr, int n_real, const TileGeom& tg, const SortBufs& sb, float* mesh, long row,
                     long mesh_bstride, float scale, float offset, int frac, hipStream_t st) {
    ProfScope ps(PROF_DEP_TILE, st);
    size_t lds = (size_t)tg.tx * tg.ty * tg.tz * sizeof(unsigned long long);
    const dim3 grid((unsigned)tg.ntiles, n_real);
    if (frac)
        hipLaunchKernelGGL(k_dep_tile<true>, grid, dim3(256), lds, st, tg, sb, npr, mesh, row, mesh_bstride,
                           ldexpf(scale, -frac), offset, frac);
    else
        hipLaunchKernelGGL(k_dep_tile<false>, grid, dim3(256), lds, st, tg, sb, npr, mesh, row, mesh_bstride, scale,
                           offset, 0);
    return hipGetLastError();
}

// Scan of the key counts, records into key order, tile accumulation: the passes after the binning.
// drifted: key and record of every particle are in keys and recs, else its rank is in keys.
hipError_t sort_and_tile(const ParticlePtrs& P, long npr, int n_real, const LatticeGeom& dg, bool drifted,
                         const TileGeom& tg, const SortBufs& sb, float* mesh, float scale, float offset,
                         hipStream_t st) {
    {
        ProfScope ps(PROF_DEP_SORT, st);
        hipError_t e = scan_counts(sb.count, sb.start, drifted ? sb.cursor : nullptr, sb.block_sums, tg.nkeys, sb.kstride,
                                   n_real, (uint32_t)npr, true, st);
        if (e != hipSuccess) return e;
        if (drifted)
            hipLaunchKernelGGL(k_dep_scatter, dim3((unsigned)((npr + 255) / 256), n_real), dim3(256), 0, st, npr, sb);
        else
            hipLaunchKernelGGL(k_dep_place, lattice_grid(dg.n_part, n_real), dim3(256), 0, st, P, npr, dg, tg, sb);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return run_tiles(npr, n_real, tg, sb, mesh, dg.row, dg.mesh_bstride, scale, offset, 0, st);
}
}  // namespace

size_t abs_sort_bytes(long n, const TileGeom& tg) {
    const size_t nblocks = (size_t)((tg.nkeys + 1023) / 1024);
    return (size_t)n * (4 + 16) + ((size_t)tg.nkeys + 1) * 4 * 2 + nblocks * 4 + 256 * 5;
}

hipError_t sorted_deposit_absolute(const float* const pos[3], long n, int n_mesh, float inv_h, const TileGeom& tg,
                                   void* scratch, float* mesh, long row, float scale, float offset, bool full_weights,
                                   hipStream_t st) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    char* b = static_cast<char*>(scratch);
    SortBufs sb;
    sb.kstride = tg.nkeys + 1;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = b + off;
        off = al(off + bytes);
        return p;
    };
    sb.sorted = reinterpret_cast<float4*>(take((size_t)n * 16));
    uint32_t* rank = reinterpret_cast<uint32_t*>(take((size_t)n * 4));
    sb.count = reinterpret_cast<uint32_t*>(take((size_t)sb.kstride * 4));
    sb.start = reinterpret_cast<uint32_t*>(take((size_t)sb.kstride * 4));
    sb.block_sums = reinterpret_cast<uint32_t*>(take((size_t)(tg.nkeys + 1023) / 1024 * 4));
    hipError_t e = hipSuccess;
    if (n <= kSmallPoints && tg.nkeys <= kSmallKeys) {
        ProfScope ps(PROF_DEPOSIT, st);
        hipLaunchKernelGGL(full_weights ? k_abs_small<true> : k_abs_small<false>, dim3(1), dim3(1024),
                           (size_t)tg.nkeys * 4, st, pos[0], pos[1], pos[2], (int)n, n_mesh, inv_h, tg, sb.start, sb.sorted);
    } else {
        if ((e = launch_fill(reinterpret_cast<float*>(sb.count), sb.kstride, 0.0f, st)) != hipSuccess) return e;
        const dim3 grid((unsigned)((n + 255) / 256));
        {
            ProfScope ps(PROF_DEPOSIT, st);
            hipLaunchKernelGGL(k_abs_count, grid, dim3(256), 0, st, pos[0], pos[1], pos[2], n, n_mesh, inv_h, tg, sb.count,
                               rank);
        }
        ProfScope ps(PROF_DEP_SORT, st);
        if ((e = scan_counts(sb.count, sb.start, nullptr, sb.block_sums, tg.nkeys, 0, 1, (uint32_t)n, false, st)) !=
            hipSuccess)
            return e;
        hipLaunchKernelGGL(full_weights ? k_abs_scatter<true> : k_abs_scatter<false>, grid, dim3(256), 0, st, pos[0],
                           pos[1], pos[2], n, n_mesh, inv_h, tg, sb.start, rank, sb.sorted);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int lg = 0;
    while ((1L << lg) < n) ++lg;
    const bool sparse = (double)n_mesh * n_mesh * n_mesh > 1.5 * (double)n;
    const int frac = full_weights ? (sparse ? 61 - lg : std::min(32, 61 - lg)) : 0;
    return run_tiles(n, 1, tg, sb, mesh, row, 0, scale, offset, frac, st);
}

hipError_t sorted_deposit(const ParticlePtrs& P, long npr, int n_real, const LatticeGeom& dg, bool drift,
                          const LatticeGeom& fg, const float* F, const KickDrift& kd, const TileGeom& tg,
                          const SortBufs& sb, float* mesh, float scale, float offset, hipStream_t st) {
    const dim3 pgrid = lattice_grid(dg.n_part, n_real);
    hipError_t e = launch_fill(reinterpret_cast<float*>(sb.count), sb.kstride * n_real, 0.0f, st);
    if (e != hipSuccess) return e;
    {
        ProfScope ps(drift ? PROF_PK_DEPOSIT : PROF_DEPOSIT, st);
        if (drift)
            hipLaunchKernelGGL(k_dep_bin<1>, pgrid, dim3(256), 0, st, P, npr, dg, tg, fg, F, kd, sb);
        else
            hipLaunchKernelGGL(k_dep_bin<0>, pgrid, dim3(256), 0, st, P, npr, dg, tg, fg, F, kd, sb);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return sort_and_tile(P, npr, n_real, dg, drift, tg, sb, mesh, scale, offset, st);
}

hipError_t gather_kick_drift_bin(const ParticlePtrs& P, long npr, int n_real, const LatticeGeom& fg, const float* F,
                                 const LatticeGeom& dg, const KickDrift& kd, const TileGeom& tg, const SortBufs& sb,
                                 bool counts_zero, hipStream_t st) {
    if (!counts_zero)
        if (hipError_t e = launch_fill(reinterpret_cast<float*>(sb.count), sb.kstride * n_real, 0.0f, st); e != hipSuccess)
            return e;
    KickDrift k = kd;
    k.los = -1;
    ProfScope ps(PROF_GKD, st);
    hipLaunchKernelGGL(k_dep_bin<2>, lattice_grid(dg.n_part, n_real), dim3(256), 0, st, P, npr, dg, tg, fg, F, k, sb);
    return hipGetLastError();
}

hipError_t sorted_deposit_binned(const ParticlePtrs& P, long npr, int n_real, const LatticeGeom& dg, const TileGeom& tg,
                                 const SortBufs& sb, float* mesh, float scale, float offset, hipStream_t st) {
    return sort_and_tile(P, npr, n_real, dg, false, tg, sb, mesh, scale, offset, st);
}

}  // namespace cola
