// Lattice index and mesh cell of a particle, for the passes over the particle arrays.
//
// Integer division by a run-time number takes some 20 vector instructions, a modulus more; with two cells of
// three axes per particle they were most of the instructions of the gather/kick/drift pass (556 per wave,
// 237 of its 445 us at 256^3 particles on 256^3 cells).  So the grid gives the lattice plane, one float
// product the row, and the lattice's own mesh (n_mesh a multiple of n_part) needs no division at all:
// 258 instructions, 408 us (390 without the records that the pass then wrote); on 768^3 cells 1163 -> 1096 us.
#pragma once

#include "cola_internal.h"

namespace cola {

struct LatticeSite {
    int i[3];
    long p;      // index in the realization
    bool valid;
};

// Grid of a pass over the particles: 256 of one lattice plane per block, planes along y, realizations along z.
inline dim3 lattice_grid(int n_part, int n_real) {
    return dim3((unsigned)(((long)n_part * n_part + 255) / 256), (unsigned)n_part, (unsigned)n_real);
}
__device__ __forceinline__ LatticeSite lattice_site(const LatticeGeom& g) {
    const int np = g.n_part, np2 = np * np;
    const int r = (int)(blockIdx.x * 256 + threadIdx.x);
    LatticeSite s;
    s.valid = r < np2;
    int j = (int)((float)r * g.inv_np);  // r < 2^24: off by one at most
    j -= j * np > r ? 1 : 0;
    j += (j + 1) * np <= r ? 1 : 0;
    s.i[0] = (int)blockIdx.y;
    s.i[1] = j;
    s.i[2] = r - j * np;
    s.p = (long)blockIdx.y * np2 + r;
    return s;
}

struct LatticeCell {
    int m;    // lower node, wrapped into [0, n)
    float f;  // fraction towards m + 1
};

// The cell coordinate is an exact integer part from the lattice index and a small float part from the
// displacement: u = (i n_mesh) / N_p + [((i n_mesh) mod N_p) / N_p + qoff + x n_mesh / L].  32-bit arithmetic:
// i n_mesh < 1536^2.
__device__ __forceinline__ LatticeCell lattice_cell(const LatticeGeom& g, int i, float x) {
    int q;
    float base;
    if (g.pm) {
        q = i * g.pm;
        base = g.qoff;
    } else {
        const uint32_t a = (uint32_t)i * (uint32_t)g.n_mesh;
        q = (int)(a / (uint32_t)g.n_part);
        base = (float)(int)(a - (uint32_t)q * (uint32_t)g.n_part) / (float)g.n_part + g.qoff;
    }
    const float w = fmaf(x, g.inv_h, base), fl = floorf(w);
    LatticeCell c;
    c.f = w - fl;
    int m = q + (int)fl;
    if ((unsigned)m >= (unsigned)g.n_mesh) {
        m = m < 0 ? m + g.n_mesh : m - g.n_mesh;
        if ((unsigned)m >= (unsigned)g.n_mesh) {  // a displacement of more than a box, or a non-finite one
            m %= g.n_mesh;
            m = m < 0 ? m + g.n_mesh : m;
            m = min(max(m, 0), g.n_mesh - 1);
        }
    }
    c.m = m;
    return c;
}

}  // namespace cola
