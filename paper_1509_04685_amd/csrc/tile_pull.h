// Device side of the tile-sorted particle-to-mesh passes (the deposit, the adjoint of the learned
// correction's loss): the key of a cell, and the record ranges that a tile pulls.
#pragma once

#include "cola_internal.h"

namespace cola {

// Key and tile-local cell of the cell (mx, my, mz).  Tile sides are powers of two; the upper face of a
// tile is its last layer, which in the last tile of a side is the mesh's last layer.
__device__ __forceinline__ uint32_t tile_key(const TileGeom& tg, int mx, int my, int mz, int& local) {
    const int lx = mx & (tg.tx - 1), ly = my & (tg.ty - 1), lz = mz & (tg.tz - 1), last = tg.n - 1;
    const uint32_t tile = ((uint32_t)(mx >> tg.lx) * tg.nty + (my >> tg.ly)) * tg.ntz + (mz >> tg.lz);
    const uint32_t cat = ((lx == tg.tx - 1 || mx == last) ? 4 : 0) | ((ly == tg.ty - 1 || my == last) ? 2 : 0) |
                         ((lz == tg.tz - 1 || mz == last) ? 1 : 0);
    local = (((lx << tg.ly) + ly) << tg.lz) + lz;
    return tile * 8 + cat;
}

// The 14 (offset d, category range) pairs a tile pulls: from tile M - d, the categories c with
// (c & d) == d, grouped into contiguous runs [c_lo, c_hi).
struct Pull {
    int d, c_lo, c_hi;
};
__device__ constexpr Pull kPulls[14] = {{0, 0, 8}, {4, 4, 8}, {2, 2, 4}, {2, 6, 8}, {1, 1, 2}, {1, 3, 4}, {1, 5, 6},
                                {1, 7, 8}, {6, 6, 8}, {5, 5, 6}, {5, 7, 8}, {3, 3, 4}, {3, 7, 8}, {7, 7, 8}};
// The offsets d of kPulls packed 3 bits each (entry q at bits 3q), for a register lookup.
constexpr unsigned long long pack_pull_offsets() {
    const int d[14] = {0, 4, 2, 2, 1, 1, 1, 1, 6, 5, 5, 3, 3, 7};
    unsigned long long v = 0;
    for (int q = 0; q < 14; ++q) v |= (unsigned long long)d[q] << (3 * q);
    return v;
}
constexpr unsigned long long kPullOffsets = pack_pull_offsets();

struct PullRanges {
    uint32_t begin[14];  // first record of each range
    uint32_t len[15];    // exclusive prefix of the range lengths; [14]: their sum
};
struct PullStarts {
    uint32_t rl[14];
};

// The cells of a tile: origin and number along each axis (the last tile of a side may be narrower).
struct TileBox {
    int tx, ty, tz;
    int x0, y0, z0;
    int nx, ny, nz;
};
__device__ __forceinline__ TileBox tile_box(const TileGeom& tg, long tile) {
    TileBox t;
    t.tz = (int)(tile % tg.ntz);
    t.ty = (int)((tile / tg.ntz) % tg.nty);
    t.tx = (int)(tile / ((long)tg.ntz * tg.nty));
    t.x0 = t.tx * tg.tx;
    t.y0 = t.ty * tg.ty;
    t.z0 = t.tz * tg.tz;
    t.nx = min(tg.tx, tg.n - t.x0);
    t.ny = min(tg.ty, tg.n - t.y0);
    t.nz = min(tg.tz, tg.n - t.z0);
    return t;
}

// Bounds of the 14 ranges, one per thread of the first wave: requested here, used by finish_pulls.
__device__ __forceinline__ void request_pulls(const TileGeom& tg, const TileBox& t, const uint32_t* start, uint32_t& b,
                                              uint32_t& e) {
    b = e = 0;
    if (threadIdx.x < 14) {
        const Pull pl = kPulls[threadIdx.x];
        const int dx = (pl.d >> 2) & 1, dy = (pl.d >> 1) & 1, dz = pl.d & 1;
        const int sx = t.tx - dx < 0 ? tg.ntx - 1 : t.tx - dx;
        const int sy = t.ty - dy < 0 ? tg.nty - 1 : t.ty - dy;
        const int sz = t.tz - dz < 0 ? tg.ntz - 1 : t.tz - dz;
        const long src = ((long)sx * tg.nty + sy) * tg.ntz + sz;
        b = start[src * 8 + pl.c_lo];
        e = start[src * 8 + pl.c_hi];
    }
}
// Exclusive prefix of the range lengths by a lane scan in the first wave (a barrier must follow).
__device__ __forceinline__ void finish_pulls(PullRanges& pr, uint32_t b, uint32_t e) {
    if (threadIdx.x >= 64) return;
    const uint32_t len = threadIdx.x < 14 ? e - b : 0u;
    uint32_t inc = len;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        const uint32_t y = __shfl_up(inc, off);
        if ((int)threadIdx.x >= off) inc += y;
    }
    if (threadIdx.x < 14) {
        pr.begin[threadIdx.x] = b;
        pr.len[threadIdx.x] = inc - len;
    }
    if (threadIdx.x == 13) pr.len[14] = inc;
}
// Register copy of the range starts in the concatenation (non-decreasing).
__device__ __forceinline__ PullStarts pull_starts(const PullRanges& pr) {
    PullStarts s;
#pragma unroll
    for (int k = 0; k < 14; ++k) s.rl[k] = pr.len[k];
    return s;
}
// Index of the i-th pulled record, and the offset d = (dx, dy, dz) of the tile that it comes from.
__device__ __forceinline__ uint32_t pulled_record(const PullRanges& pr, const PullStarts& s, uint32_t i, int& dx,
                                                  int& dy, int& dz) {
    int q = 0;  // the last range starting at or before i (empty ranges share their start)
#pragma unroll
    for (int k = 1; k < 14; ++k) q += i >= s.rl[k] ? 1 : 0;
    const int d = (int)((kPullOffsets >> (3 * q)) & 7u);
    dx = (d >> 2) & 1;
    dy = (d >> 1) & 1;
    dz = d & 1;
    return pr.begin[q] + (i - pr.len[q]);
}
// Home cell of a pulled record relative to this tile: a record of the tile below sits on that
// tile's upper face.
__device__ __forceinline__ void pulled_cell(const TileGeom& tg, int local, int dx, int dy, int dz, int& hx, int& hy,
                                            int& hz) {
    hx = dx ? -1 : local >> (tg.lz + tg.ly);
    hy = dy ? -1 : (local >> tg.lz) & (tg.ty - 1);
    hz = dz ? -1 : local & (tg.tz - 1);
}

}  // namespace cola
