// Friends-of-friends haloes (Sec. 2.1: linking length 0.2 of the mean inter-particle separation,
// after Davis et al. 1985), their catalogue and the binned Warren mass function (Sec. 2.5).
//
// Two particles are friends when their periodic distance is below the linking length b; groups
// are the connected components of the friendship graph, labelled by their smallest particle
// index.  The decision is taken in float32 with every operation rounded on its own:
//   d = x_j - x_i;  d -= L if d > L/2;  d += L if d < -L/2      (per axis)
//   d2 = (dx*dx + dy*dy) + dz*dz;   friends iff d2 < b2,  b2 = float32(b) * float32(b).
//
// Passes (one stream, all device work):
//   bin      cell of every particle on a grid of cells no smaller than b, counts per cell and the
//            particle's rank in its cell (the counter's old value);
//   scan     exclusive scan of the counts (shared with the tiled deposit);
//   scatter  particle records {x, y, z, index} in cell order, at the cell's start plus the rank;
//   local    the pairs of records of one block that follow each other in a row of cells, joined in
//            LDS; every particle's first parent is the smallest index of its set so far;
//   link     one thread per record: the other pairs with the records after it in its own cell and with
//            those of the 13 "forward" neighbour cells (each unordered pair of cells once) that lie within
//            reach; a friend pair joins its two trees in a lock-free union-find;
//   finish   every particle's root, written back as its label (full compression), and the
//            group sizes at the roots (sizes start at 1: only members below a root count themselves).
//
// Union-find invariant: a root is only hooked under a smaller root (compare-and-swap on the
// root's own entry) and path halving only replaces a parent by one of its ancestors, so every
// non-root entry holds a smaller index than its own.  Walks therefore end, no cycle can form,
// and the root of each tree is the smallest index in it.  Each failed compare-and-swap means
// another thread completed a hook, and at most n - 1 hooks exist, so every thread exits.
//
// Cost: the link pass tests every pair in each cell and between the neighbours within a linking length of a
// particle's own cell, so its time grows with the square of the particles per cell.  At the mean density there is about one
// particle per cell; the densest cells of the z = 0 runs hold a few hundred.  Positions that
// pile a large fraction of all particles into one cell (a degenerate input) make the pass
// quadratic in n.

#include <algorithm>
#include <cmath>

#include "cola_internal.h"
#include "lc_internal.h"
#include "wave_ops.h"

namespace cola {

namespace {

constexpr int kFofMaxBins = 64;

struct FofGrid {
    int nc;          // cells per side
    float inv_cell;  // nc / L
    float reach;     // linking length in cells, with the margin of the float32 cell coordinate
    long ncell;
};

struct MassBins {
    int nb;
    int32_t lo[kFofMaxBins + 1];  // particle-count edges: bin b holds lo[b] <= N < lo[b + 1]
};

__device__ __forceinline__ int wrap_cell(float fl, int nc) {
    int c = (int)fl;
    if ((unsigned)c >= (unsigned)nc) {  // outside the box: periodic
        c %= nc;
        c = c < 0 ? c + nc : c;
        c = min(max(c, 0), nc - 1);  // a non-finite coordinate still maps into the grid
    }
    return c;
}

__device__ __forceinline__ int cell1(float x, float inv_cell, int nc) { return wrap_cell(floorf(x * inv_cell), nc); }

// The cell of a coordinate, and whether a friend can sit in the next one up or down: only within `reach`
// of that face.  A cell coordinate is rounded by at most 2.4e-4 below 4096, which the margin of `reach`
// covers twice over; farther out every neighbour counts.
struct CellReach {
    int c;
    bool up, down;
};
__device__ __forceinline__ CellReach cell_reach(float x, const FofGrid& g) {
    const float u = x * g.inv_cell, fl = floorf(u), f = u - fl;
    const bool far = !(fabsf(u) < 4096.0f);
    CellReach r;
    r.c = wrap_cell(fl, g.nc);
    r.up = far || f + g.reach >= 1.0f;
    r.down = far || f - g.reach <= 0.0f;
    return r;
}

__device__ __forceinline__ uint32_t cell3(float x, float y, float z, const FofGrid& g) {
    const int cx = cell1(x, g.inv_cell, g.nc), cy = cell1(y, g.inv_cell, g.nc), cz = cell1(z, g.inv_cell, g.nc);
    return (uint32_t)(((long)cx * g.nc + cy) * g.nc + cz);
}

__device__ __forceinline__ int32_t ld_parent(const int32_t* p, int32_t x) {
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_parent(int32_t* p, int32_t x, int32_t v) {
    __hip_atomic_store(p + x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x with path halving.
__device__ __forceinline__ int32_t fof_find(int32_t* parent, int32_t x) {
    while (true) {
        const int32_t p = ld_parent(parent, x);
        if (p == x) return x;
        const int32_t gp = ld_parent(parent, p);
        if (gp != p) st_parent(parent, x, gp);
        x = gp;
    }
}

// A parent entry as this compute unit last saw it.  Every value that an entry ever held is an ancestor of
// it for good (sets only join), so a stale one still proves that two particles share a set.
__device__ __forceinline__ int32_t ld_parent_near(const int32_t* p, int32_t x) {
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Joins the sets of a and b (any members); returns a root of the joined set.
__device__ __forceinline__ int32_t fof_union(int32_t* parent, int32_t a, int32_t b) {
    while (true) {
        int32_t ra = fof_find(parent, a), rb = fof_find(parent, b);
        if (ra == rb) return ra;
        if (ra > rb) {
            const int32_t t = ra;
            ra = rb;
            rb = t;
        }
        if (atomicCAS(parent + rb, rb, ra) == rb) return ra;  // rb was still a root: hooked
        a = ra;
        b = rb;
    }
}

__device__ __forceinline__ float min_image(float d, float box, float half) {
    if (d > half) return d - box;
    if (d < -half) return d + box;
    return d;
}

__device__ __forceinline__ float d2_of(float4 a, float4 b, float box, float half) {
#pragma clang fp contract(off)  // each product and sum rounded on its own, no fused multiply-add
    const float dx = min_image(b.x - a.x, box, half);
    const float dy = min_image(b.y - a.y, box, half);
    const float dz = min_image(b.z - a.z, box, half);
    const float sxy = dx * dx + dy * dy;
    return sxy + dz * dz;
}

// d2_of of particles whose differences need no minimum image, the usual case: `far` is set where one does
// (beyond half the box on some axis), and the value is then not to be used.
__device__ __forceinline__ float d2_near(float4 a, float4 b, float half, bool& far) {
#pragma clang fp contract(off)
    const float dx = b.x - a.x, dy = b.y - a.y, dz = b.z - a.z;
    far = far || fmaxf(fmaxf(fabsf(dx), fabsf(dy)), fabsf(dz)) > half;
    const float sxy = dx * dx + dy * dy;
    return sxy + dz * dz;
}

__global__ void k_fof_ones(int32_t* size, long n) {  // every particle a group of one
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) size[i] = 1;
}

// Points with about one per cell have few runs of equal cells, so the counters' atomics bound this pass; the
// scatter has none of its own, as the rank is kept (256^3 particles: 320 + 477 us with atomics in both, 340 + 204
// us so).
__global__ void k_fof_bin(const float* __restrict__ px, const float* __restrict__ py, const float* __restrict__ pz,
                          long n, FofGrid g, uint32_t* rank, uint32_t* count) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;  // every lane takes part in the wave-level counting
    const uint32_t c = valid ? cell3(px[i], py[i], pz[i], g) : 0u;
    const uint32_t r = wave_increment(count, c, valid);
    if (valid) rank[i] = r;
}

__global__ void k_fof_scatter(const float* __restrict__ px, const float* __restrict__ py,
                              const float* __restrict__ pz, long n, FofGrid g, const uint32_t* rank,
                              const uint32_t* start, float4* recs) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = px[i], y = py[i], z = pz[i];
    recs[start[cell3(x, y, z, g)] + rank[i]] = make_float4(x, y, z, __int_as_float((int)i));
}

// First record of row (cx, cy) cell z.
__device__ __forceinline__ uint32_t row_start(const FofGrid& g, const uint32_t* start, int cx, int cy, int z) {
    return start[((uint32_t)cx * g.nc + cy) * g.nc + z];
}

// Roots in LDS: entries are slots of the block's records, a root is hooked under the root of the smaller
// particle index.
__device__ __forceinline__ int local_find(int* parent, int x) {
    while (true) {
        const int p = __hip_atomic_load(parent + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (p == x) return x;
        const int gp = __hip_atomic_load(parent + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (gp != p) __hip_atomic_store(parent + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        x = gp;
    }
}
__device__ __forceinline__ int local_union(int* parent, const float4* recs, int a, int b) {
    while (true) {
        a = local_find(parent, a);
        b = local_find(parent, b);
        if (a == b) return a;
        if (__float_as_int(recs[a].w) > __float_as_int(recs[b].w)) {
            const int t = a;
            a = b;
            b = t;
        }
        int expected = b;
        if (__hip_atomic_compare_exchange_strong(parent + b, &expected, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            return a;
    }
}

// The records of a halo sit together in record order, so most of its hooks can be made in LDS, where one
// costs some hundred cycles instead of several memory round trips across the chip.
constexpr int kFofBlock = 256;
__global__ void __launch_bounds__(kFofBlock) k_fof_local(const float4* __restrict__ recs, long n, FofGrid g,
                                                         const uint32_t* __restrict__ start, float box, float link2,
                                                         int32_t* parent) {
    __shared__ float4 r[kFofBlock];
    __shared__ int up[kFofBlock];
    const long t0 = (long)xcd_block() * kFofBlock, t = t0 + threadIdx.x;
    const int s = threadIdx.x;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (t < n) a = recs[t];
    r[s] = a;
    up[s] = s;
    int end = 0;  // slots of the block that this record is tested with: s + 1 .. end - 1
    if (t < n) {
        const CellReach z = cell_reach(a.z, g);  // the own cell, and the next in z where it is in reach and no wrap
        const int z1 = min(z.c + (z.up ? 1 : 0), g.nc - 1);
        const uint32_t last = row_start(g, start, cell1(a.x, g.inv_cell, g.nc), cell1(a.y, g.inv_cell, g.nc), z1 + 1);
        end = (int)min((long)last - t0, (long)kFofBlock);
    }
    __syncthreads();
    const float half = 0.5f * box;
    // First the nearest friends only, which joins most of a halo; then, with every entry pointing at its
    // root, the rest of the records, whose entries mostly compare equal (with entries some hooks behind their
    // root nearly every friend pair led to find walks).
    int root = s, known = s, k = s + 1;  // a root of the own set, the last other entry joined to it
    auto step = [&]() {
        int pk[4];
        float d2[4];
        bool far = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) d2[u] = d2_near(a, r[min(k + u, end - 1)], half, far);
        if (far)
            for (int u = 0; u < 4; ++u) d2[u] = d2_of(a, r[min(k + u, end - 1)], box, half);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            pk[u] = k + u < end && d2[u] < link2
                        ? __hip_atomic_load(up + k + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                        : root;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (pk[u] == root || pk[u] == known) continue;
            known = pk[u];
            root = local_union(up, r, root, pk[u]);
        }
        k += 4;
    };
    if (k < end) step();
    __syncthreads();
    const int flat = local_find(up, s);
    __syncthreads();
    up[s] = flat;
    __syncthreads();
    root = known = flat;
    while (k < end) step();
    __syncthreads();
    if (t < n) parent[__float_as_int(a.w)] = __float_as_int(r[local_find(up, s)].w);
}

// The cells after the own one, (ox, oy, oz) in {-1, 0, 1}^3 lexicographically after (0, 0, 0), are 13; cells
// consecutive in z are consecutive in record order, so they are five ranges: the rest of the own cell with the
// next in z (from the end of the block on, see k_fof_local), and up to three cells in z of (0, 1), (1, -1), (1, 0),
// (1, 1).  At the two z ends of the grid the wrapped cells are five ranges more.
//
// Cells are several linking lengths wide (one particle per cell on average; 5 at b = 0.2), so most neighbours
// are out of reach: a range is cut to the cells whose face is within reach (cell_reach), which leaves about
// 1.4 records per particle of 13.5 at the mean density.  The pass was bound by the vector ALU: testing all of
// them, with their minimum images, took 4000 instructions per wave.  256^3 particles, a fifth of them in
// clumps: one pass over 14 cells 4980 us, the two passes 600 + 1220 us.
//
// The ranges are walked as one sequence, kFofStep records in flight.  In a halo nearly every pair tested is a
// friend pair whose sets are joined already: the parents of the friends among the kFofStep records are requested
// together (from this unit's own cache level, see ld_parent_near) and compared with the root of the thread's set
// and the kFofKnown parents that it last found joined to it.  Only another one leads to find walks, and the pair
// (root, parent) to those of one thread of the block: the others of a halo meet the same pairs, find them in the
// block's table of pairs and go on (the sets are joined by the time the kernel ends).
constexpr int kFofStep = 8;
constexpr int kFofKnown = 3;
constexpr int kFofPairs = 512;  // entries of the table, addressed by a 9-bit hash of the pair

__global__ void __launch_bounds__(kFofBlock) k_fof_link(const float4* __restrict__ recs, long n, FofGrid g,
                                                        const uint32_t* __restrict__ start, float box, float link2,
                                                        int32_t* parent) {
    __shared__ unsigned long long pairs[kFofPairs];
    for (int k = threadIdx.x; k < kFofPairs; k += kFofBlock) pairs[k] = ~0ull;
    __syncthreads();
    const int block = xcd_block();
    const long t = (long)block * kFofBlock + threadIdx.x;
    if (t >= n) return;
    const float4 a = recs[t];
    const int32_t i = __float_as_int(a.w);
    const float half = 0.5f * box;
    const uint32_t block_end = (uint32_t)min(((long)block + 1) * kFofBlock, n);
    const CellReach x = cell_reach(a.x, g), y = cell_reach(a.y, g), z = cell_reach(a.z, g);
    const int xp = x.c + 1 == g.nc ? 0 : x.c + 1, yp = y.c + 1 == g.nc ? 0 : y.c + 1, ym = y.c ? y.c - 1 : g.nc - 1;
    const int rx[5] = {x.c, x.c, xp, xp, xp}, ry[5] = {y.c, yp, ym, y.c, yp};
    const bool grid = g.nc >= 3;  // a grid of a single cell has its rest of the own cell and nothing else
    const bool use[5] = {true, grid && y.up, grid && x.up && y.down, grid && x.up, grid && x.up && y.up};
    const int32_t first = ld_parent(parent, i);
    int32_t root = first;  // an ancestor of i, or i
    int32_t known[kFofKnown];  // entries of the same set
#pragma unroll
    for (int u = 0; u < kFofKnown; ++u) known[u] = root;
    for (int pass = 0; pass < 2; ++pass) {
        // pass 0: the ranges up to the ends of the grid in z; pass 1: those across (for the own row upwards only)
        const bool low = z.c == 0 && z.down, high = z.c == g.nc - 1 && z.up;
        if (pass == 1 && !(grid && (low || high))) break;
        const int w = z.c ? 0 : g.nc - 1;
        const int z0 = pass ? w : max(z.c - (z.down ? 1 : 0), 0), z1 = pass ? w : min(z.c + (z.up ? 1 : 0), g.nc - 1);
        uint32_t rb[5], re[5];  // every bound is requested before the first is used
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            rb[q] = re[q] = 0u;
            if (use[q]) {
                rb[q] = row_start(g, start, rx[q], ry[q], z0);
                re[q] = row_start(g, start, rx[q], ry[q], z1 + 1);
            }
        }
        if (pass == 0) rb[0] = block_end;
        else if (z.c == 0) re[0] = 0u;
        // record i of the ranges walked as one sequence is i + the offset of its range
        uint32_t end[5], off[5], total = 0;
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            off[q] = rb[q] - total;
            total += re[q] > rb[q] ? re[q] - rb[q] : 0u;
            end[q] = total;
        }
        const uint32_t e0 = end[0], e1 = end[1], e2 = end[2], e3 = end[3];
        const uint32_t d1 = off[1] - off[0], d2 = off[2] - off[1], d3 = off[3] - off[2], d4 = off[4] - off[3];
        const uint32_t base = off[0];
        auto record = [&](uint32_t q) {
            return q + base + (q >= e0 ? d1 : 0u) + (q >= e1 ? d2 : 0u) + (q >= e2 ? d3 : 0u) + (q >= e3 ? d4 : 0u);
        };
        for (uint32_t k = 0; k < total; k += kFofStep) {
            int32_t j[kFofStep], pj[kFofStep];
            float4 b[kFofStep];
#pragma unroll
            for (int u = 0; u < kFofStep; ++u) b[u] = recs[record(min(k + u, total - 1))];
            float d2[kFofStep];
            bool far = false;
#pragma unroll
            for (int u = 0; u < kFofStep; ++u) d2[u] = d2_near(a, b[u], half, far);
            if (far) {
#pragma unroll
                for (int u = 0; u < kFofStep; ++u) d2[u] = d2_of(a, b[u], box, half);
            }
#pragma unroll
            for (int u = 0; u < kFofStep; ++u) j[u] = k + u < total && d2[u] < link2 ? __float_as_int(b[u].w) : -1;
#pragma unroll
            for (int u = 0; u < kFofStep; ++u) pj[u] = j[u] >= 0 ? ld_parent_near(parent, j[u]) : root;
#pragma unroll
            for (int u = 0; u < kFofStep; ++u) {
                bool joined = pj[u] == root;
#pragma unroll
                for (int v = 0; v < kFofKnown; ++v) joined |= pj[u] == known[v];
                if (joined) continue;
#pragma unroll
                for (int v = kFofKnown - 1; v > 0; --v) known[v] = known[v - 1];
                known[0] = pj[u];
                const uint32_t lo = (uint32_t)min(root, pj[u]), hi = (uint32_t)max(root, pj[u]);
                const unsigned long long pair = (unsigned long long)hi << 32 | lo;
                const uint32_t slot = (lo * 2654435761u + hi * 2246822519u) >> 23;
                if (atomicExch(&pairs[slot], pair) == pair) continue;  // another thread joins these two
                root = fof_union(parent, root, pj[u]);
            }
        }
    }
    // other threads compare the parent of i with theirs; i is no root any more where this is another
    if (root != first && root != i) st_parent(parent, i, root);
}

// Every entry becomes its root (writes of an ancestor over a parent keep the forest valid for
// concurrent walks); sizes are counted at the roots.
__global__ void k_fof_finish(int32_t* parent, long n, int32_t* size) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;  // every lane takes part in the wave-level counting
    int32_t r = (int32_t)i;
    while (valid) {
        const int32_t p = ld_parent(parent, r);
        if (p == r) break;
        r = p;
    }
    const bool member = valid && r != (int32_t)i;
    if (member) {
        st_parent(parent, (int32_t)i, r);
        size[i] = 0;
    }
    // one atomic per run of members of one root: neighbours in index often are in one group
    (void)wave_increment(reinterpret_cast<uint32_t*>(size), (uint32_t)r, member);
}

// ---- catalogue

constexpr int kCatItems = 1024;  // particles per block of the halo scan (four per thread)

// Haloes per block of kCatItems particles.
__global__ void __launch_bounds__(256) k_cat_count(const int32_t* size, long n, int32_t n_min, uint32_t* sums) {
    __shared__ uint32_t total;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    uint32_t mine = 0;
    for (int q = 0; q < 4; ++q) {
        const long i = (long)blockIdx.x * kCatItems + q * 256 + threadIdx.x;
        mine += (uint32_t)__popcll(__ballot(i < n && size[i] >= n_min));
    }
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&total, mine);
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Exclusive scan of the block sums in place; their total.
__global__ void __launch_bounds__(1024) k_cat_offsets(uint32_t* sums, long nblocks, int64_t* n_halos) {
    __shared__ uint32_t sh[1024];
    const long per = (nblocks + 1023) / 1024, b0 = threadIdx.x * per;
    uint32_t s = 0;
    for (long i = b0; i < min(b0 + per, nblocks); ++i) s += sums[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t t = threadIdx.x >= off ? sh[threadIdx.x - off] : 0u;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    uint32_t run = sh[threadIdx.x] - s;
    for (long i = b0; i < min(b0 + per, nblocks); ++i) {
        const uint32_t v = sums[i];
        sums[i] = run;
        run += v;
    }
    if (threadIdx.x == 1023) *n_halos = (int64_t)sh[1023];
}

// The haloes in index order: hidx[root] = position in the catalogue (only at the roots of haloes).
__global__ void __launch_bounds__(256) k_cat_fill(const int32_t* size, long n, int32_t n_min, const uint32_t* offsets,
                                                  double m_p, uint32_t* hidx, int32_t* root, int32_t* count,
                                                  double* mass, double* cx, double* cy, double* cz) {
    __shared__ uint32_t waves[4][4];  // haloes per quarter and wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long hit[4];
    int32_t sz[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const long i = (long)blockIdx.x * kCatItems + q * 256 + threadIdx.x;
        sz[q] = i < n ? size[i] : 0;
        hit[q] = __ballot(i < n && sz[q] >= n_min);
        if (lane == 0) waves[q][wave] = (uint32_t)__popcll(hit[q]);
    }
    __syncthreads();
    uint32_t before = offsets[blockIdx.x];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t h = before;
        for (int w = 0; w < 4; ++w) {
            if (w < wave) h += waves[q][w];
            before += waves[q][w];
        }
        if (!(hit[q] >> lane & 1)) continue;
        const long i = (long)blockIdx.x * kCatItems + q * 256 + threadIdx.x;
        h += (uint32_t)__popcll(hit[q] & ((1ull << lane) - 1ull));
        const double N = (double)sz[q];
        hidx[i] = h;
        root[h] = (int32_t)i;
        count[h] = sz[q];
        mass[h] = m_p * N * (1.0 - pow(N, -0.6));
        cx[h] = 0.0;
        cy[h] = 0.0;
        cz[h] = 0.0;
    }
}

// Sums of the members' offsets from the root particle.  Neighbours in index often are in one halo: a
// run of lanes with one root is summed by lane shifts and adds once (256^3 particles: 461 -> 222 us).
__global__ void __launch_bounds__(256) k_cat_sum(const float* __restrict__ px, const float* __restrict__ py,
                                                 const float* __restrict__ pz, long n, const int32_t* group,
                                                 const int32_t* size, int32_t n_min, const uint32_t* hidx, float box,
                                                 double* cx, double* cy, double* cz) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    int32_t r = i < n ? group[i] : -1;
    if (r < 0 || r >= n || size[r] < n_min) r = -1;  // a label outside the particle range is ignored
    if (__ballot(r >= 0) == 0ull) return;
    double d[3] = {0.0, 0.0, 0.0};
    if (r >= 0) {
        const float half = 0.5f * box;
        d[0] = (double)min_image(px[i] - px[r], box, half);
        d[1] = (double)min_image(py[i] - py[r], box, half);
        d[2] = (double)min_image(pz[i] - pz[r], box, half);
    }
    const int32_t prev = __shfl_up(r, 1);
    const bool head = lane == 0 || prev != r;
    const unsigned long long heads = __ballot(head);
    const unsigned long long after = lane == 63 ? 0ull : heads >> (lane + 1) << (lane + 1);
    const int end = after ? __ffsll((long long)after) - 1 : 64;  // first lane of the next run
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double v = __shfl_down(d[a], off);
            if (lane + off < end) d[a] += v;
        }
    if (!head || r < 0) return;
    const uint32_t h = hidx[r];
    atomicAdd(cx + h, d[0]);
    atomicAdd(cy + h, d[1]);
    atomicAdd(cz + h, d[2]);
}

__device__ __forceinline__ double wrap_box(double c, double box) {
    return c >= box ? c - box : (c < 0.0 ? c + box : c);
}

__global__ void k_cat_com(const float* __restrict__ px, const float* __restrict__ py, const float* __restrict__ pz,
                          const int64_t* n_halos, const int32_t* root, const int32_t* count, double box, double* cx,
                          double* cy, double* cz) {
    const long h = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= *n_halos) return;
    const int32_t i = root[h];
    const double N = (double)count[h];
    cx[h] = wrap_box((double)px[i] + cx[h] / N, box);
    cy[h] = wrap_box((double)py[i] + cy[h] / N, box);
    cz[h] = wrap_box((double)pz[i] + cz[h] / N, box);
}

// ---- mass histogram

// Counts are summed in LDS over a block's share of the particles (added to memory one group at a time, the few
// hot counters took 79 us for 16.8e6 particles; 31 us so).
__global__ void __launch_bounds__(256) k_fof_hist(const int32_t* size, long n, MassBins mb, unsigned long long* counts) {
    __shared__ uint32_t sh[kFofMaxBins];
    if (threadIdx.x < kFofMaxBins) sh[threadIdx.x] = 0u;
    __syncthreads();
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const int32_t s = size[i];
        if (s < mb.lo[0] || s >= mb.lo[mb.nb]) continue;
        int b = 0;
        while (b + 1 < mb.nb && s >= mb.lo[b + 1]) ++b;
        atomicAdd(&sh[b], 1u);
    }
    __syncthreads();
    if ((int)threadIdx.x < mb.nb && sh[threadIdx.x]) atomicAdd(counts + threadIdx.x, (unsigned long long)sh[threadIdx.x]);
}

__global__ void k_zero_u64(unsigned long long* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

unsigned blocks_of(long n) { return (unsigned)((n + 255) / 256); }

// Cells per side: cells of side L / nc no smaller than b (with a margin of 1e-3 for the float32
// cell coordinate), at most ceil(cbrt(n)) per side; grids of fewer than 3 cells collapse to one
// cell so that the 13 forward neighbours are distinct cells.
FofGrid fof_grid(long n, double box, double link) {
    FofGrid g;
    const double by_link = std::floor(box / (link * 1.001));
    const double by_count = std::ceil(std::cbrt((double)std::max(1L, n)));
    int nc = (int)std::max(1.0, std::min(std::min(by_link, by_count), 1290.0));
    if (nc < 3) nc = 1;
    g.nc = nc;
    g.inv_cell = (float)(nc / box);
    g.reach = (float)(link * nc / box * 1.001 + 1e-3);
    g.ncell = (long)nc * nc * nc;
    return g;
}

struct FofWs {
    uint32_t* rank;     // n + 1
    float4* recs;       // n
    uint32_t* count;    // keys + 1
    uint32_t* start;    // keys + 1 (catalogue: the halo index of each root)
    uint32_t* block_sums;
    size_t total;
};

// keys: the cells of the grid, or n + 1 for the halo index, whichever is larger.
FofWs fof_ws(long n, const FofGrid& g, void* base) {
    FofWs w{};
    char* b = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = b ? b + off : nullptr;
        off += lc_align(bytes);
        return p;
    };
    const long keys = std::max(g.ncell, n + 1);
    w.rank = reinterpret_cast<uint32_t*>(take((size_t)(n + 1) * 4));
    w.recs = reinterpret_cast<float4*>(take((size_t)n * 16));
    w.count = reinterpret_cast<uint32_t*>(take((size_t)(keys + 1) * 4));
    w.start = reinterpret_cast<uint32_t*>(take((size_t)(keys + 1) * 4));
    w.block_sums = reinterpret_cast<uint32_t*>(take((size_t)((keys + 1023) / 1024 + 1) * 4));
    w.total = off;
    return w;
}

bool pos_ok(const float* const pos[3], long n) {
    return pos && pos[0] && pos[1] && pos[2] && n >= 1 && n <= (long)INT32_MAX - 1;
}

double warren(double N, double m_p) { return m_p * N * (1.0 - std::pow(N, -0.6)); }

// Smallest N >= 1 whose Warren mass reaches m (INT32_MAX if no N below it does).
int32_t first_n_reaching(double m, double m_p) {
    long lo = 1, hi = (long)INT32_MAX - 1;
    if (warren(1.0, m_p) >= m) return 1;
    if (!(warren((double)hi, m_p) >= m)) return INT32_MAX;
    while (hi - lo > 1) {  // warren(lo) < m <= warren(hi); the mass increases with N
        const long mid = lo + (hi - lo) / 2;
        if (warren((double)mid, m_p) >= m) hi = mid;
        else lo = mid;
    }
    return (int32_t)hi;
}

}  // namespace

}  // namespace cola

using namespace cola;

#define FOF_TRY(expr)                                        \
    do {                                                     \
        hipError_t _e = (expr);                              \
        if (_e != hipSuccess) return hip_fail(_e, #expr);    \
    } while (0)

extern "C" {

size_t cola_fof_workspace_bytes(int64_t n, double box, double link) {
    if (n < 1 || n > (int64_t)INT32_MAX - 1 || !std::isfinite(box) || !(box > 0.0) || !std::isfinite(link) ||
        !(link > 0.0))
        return 0;
    return fof_ws((long)n, fof_grid((long)n, box, link), nullptr).total;
}

int cola_fof(const float* pos[3], int64_t n, double box, double link, int32_t* group, int32_t* group_size, void* ws,
             size_t ws_bytes, void* stream) {
    if (!std::isfinite(box) || !std::isfinite(link)) return COLA_ERR_NONFINITE;
    if (!pos_ok(pos, (long)n) || !std::isfinite(box) || !(box > 0.0) || !std::isfinite(link) || !(link > 0.0) ||
        !(link < 0.5 * box) || !group || !group_size || !ws)
        return COLA_ERR_INVALID_ARG;
    const FofGrid g = fof_grid((long)n, box, link);
    const FofWs w = fof_ws((long)n, g, ws);
    if (ws_bytes < w.total) return COLA_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ws_forget(ws);
    (void)hipGetLastError();
    const float link2 = (float)link * (float)link;
    ProfScope ps(PROF_FOF, st, g.nc);
    FOF_TRY(launch_fill(reinterpret_cast<float*>(w.count), g.ncell, 0.0f, st));
    hipLaunchKernelGGL(k_fof_ones, dim3(blocks_of(n)), dim3(256), 0, st, group_size, (long)n);
    hipLaunchKernelGGL(k_fof_bin, dim3(blocks_of(n)), dim3(256), 0, st, pos[0], pos[1], pos[2], (long)n, g,
                       w.rank, w.count);
    FOF_TRY(hipGetLastError());
    FOF_TRY(scan_counts(w.count, w.start, nullptr, w.block_sums, g.ncell, 0, 1, (uint32_t)n, false, st));
    hipLaunchKernelGGL(k_fof_scatter, dim3(blocks_of(n)), dim3(256), 0, st, pos[0], pos[1], pos[2], (long)n, g,
                       w.rank, w.start, w.recs);
    const unsigned blocks = (unsigned)(((long)n + kFofBlock - 1) / kFofBlock);
    hipLaunchKernelGGL(k_fof_local, dim3(blocks), dim3(kFofBlock), 0, st, w.recs, (long)n, g, w.start, (float)box,
                       link2, group);
    hipLaunchKernelGGL(k_fof_link, dim3(blocks), dim3(kFofBlock), 0, st, w.recs, (long)n, g, w.start, (float)box,
                       link2, group);
    hipLaunchKernelGGL(k_fof_finish, dim3(blocks_of(n)), dim3(256), 0, st, group, (long)n, group_size);
    FOF_TRY(hipGetLastError());
    return COLA_OK;
}

int cola_fof_catalogue(const float* pos[3], int64_t n, double box, const int32_t* group, const int32_t* group_size,
                       int32_t n_min, double particle_mass, int64_t max_halos, int32_t* halo_root, int32_t* halo_n,
                       double* halo_mass, double* halo_com[3], int64_t* n_halos, void* ws, size_t ws_bytes,
                       void* stream) {
    if (!std::isfinite(box) || !std::isfinite(particle_mass)) return COLA_ERR_NONFINITE;
    if (!pos_ok(pos, (long)n) || !std::isfinite(box) || !(box > 0.0) || !group || !group_size || n_min < 1 ||
        !std::isfinite(particle_mass) || !(particle_mass > 0.0) || !halo_root || !halo_n || !halo_mass ||
        !halo_com || !halo_com[0] || !halo_com[1] || !halo_com[2] || !n_halos || !ws)
        return COLA_ERR_INVALID_ARG;
    if (max_halos < n / n_min) return COLA_ERR_INVALID_ARG;  // room for every possible halo
    // the halo-index scan needs n + 1 keys, which every workspace of cola_fof_workspace_bytes has
    const FofWs w = fof_ws((long)n, FofGrid{1, 1.0f, 1.0f, 1}, ws);
    if (ws_bytes < w.total) return COLA_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ws_forget(ws);
    (void)hipGetLastError();
    ProfScope ps(PROF_FOF, st, -1);
    uint32_t* hidx = w.start;
    const long nb = ((long)n + kCatItems - 1) / kCatItems;
    hipLaunchKernelGGL(k_cat_count, dim3((unsigned)nb), dim3(256), 0, st, group_size, (long)n, n_min, w.block_sums);
    hipLaunchKernelGGL(k_cat_offsets, dim3(1), dim3(1024), 0, st, w.block_sums, nb, n_halos);
    hipLaunchKernelGGL(k_cat_fill, dim3((unsigned)nb), dim3(256), 0, st, group_size, (long)n, n_min, w.block_sums,
                       particle_mass, hidx, halo_root, halo_n, halo_mass, halo_com[0], halo_com[1], halo_com[2]);
    hipLaunchKernelGGL(k_cat_sum, dim3(blocks_of(n)), dim3(256), 0, st, pos[0], pos[1], pos[2], (long)n, group,
                       group_size, n_min, hidx, (float)box, halo_com[0], halo_com[1], halo_com[2]);
    hipLaunchKernelGGL(k_cat_com, dim3(blocks_of(n / n_min + 1)), dim3(256), 0, st, pos[0], pos[1], pos[2], n_halos,
                       halo_root, halo_n, box, halo_com[0], halo_com[1], halo_com[2]);
    FOF_TRY(hipGetLastError());
    return COLA_OK;
}

int cola_fof_mass_histogram(const int32_t* group_size, int64_t n, int32_t n_min, double particle_mass,
                            const double* log10_mass_edges, int32_t n_bins, uint64_t* counts, void* stream) {
    if (!std::isfinite(particle_mass)) return COLA_ERR_NONFINITE;
    if (!group_size || n < 1 || n > (int64_t)INT32_MAX - 1 || n_min < 1 || !std::isfinite(particle_mass) ||
        !(particle_mass > 0.0) || !log10_mass_edges || n_bins < 1 || n_bins > kFofMaxBins || !counts)
        return COLA_ERR_INVALID_ARG;
    MassBins mb{};
    mb.nb = n_bins;
    for (int b = 0; b <= n_bins; ++b) {
        const double e = log10_mass_edges[b];
        if (!std::isfinite(e)) return COLA_ERR_NONFINITE;
        if (b > 0 && !(e > log10_mass_edges[b - 1])) return COLA_ERR_INVALID_ARG;
        mb.lo[b] = std::max(first_n_reaching(std::pow(10.0, e), particle_mass), n_min);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    (void)hipGetLastError();
    ProfScope ps(PROF_FOF, st, -2);
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(kFofMaxBins), 0, st, reinterpret_cast<unsigned long long*>(counts),
                       n_bins);
    hipLaunchKernelGGL(k_fof_hist, dim3(std::min(blocks_of(n), 1024u)), dim3(256), 0, st, group_size, (long)n, mb,
                       reinterpret_cast<unsigned long long*>(counts));
    FOF_TRY(hipGetLastError());
    return COLA_OK;
}

double cola_particle_mass(const cola_cosmology* cosmo, double box, int32_t n_part) {
    // Omega_m times the critical density today (2.775e11 h^2 M_sun Mpc^-3) per particle volume
    if (!cosmo || !(box > 0.0) || n_part < 1) return 0.0;
    const double cell = box / n_part;
    return cosmo->omega_m * 2.775e11 * cell * cell * cell;
}

}  // extern "C"
