// CIC gather of a dense vector mesh at absolute positions: the residual of the learned correction's loss.
#pragma once

#include <hip/hip_runtime.h>

namespace cola {

__device__ __forceinline__ void cic_abs(float pos, float inv_h, int n, int& i0, int& i1, float& f) {
    const float u = pos * inv_h;
    const float fl = floorf(u);
    f = u - fl;
    int m = (int)fl % n;
    m = m < 0 ? m + n : m;
    m = min(max(m, 0), n - 1);  // a non-finite position still maps inside the mesh
    i0 = m;
    i1 = m + 1 == n ? 0 : m + 1;
}

struct LossCell {
    int i[3][2];  // lower and upper node per axis
    float f[3];
};
__device__ __forceinline__ void loss_cell(float x, float y, float z, float inv_h, int n, LossCell& c) {
    cic_abs(x, inv_h, n, c.i[0][0], c.i[0][1], c.f[0]);
    cic_abs(y, inv_h, n, c.i[1][0], c.i[1][1], c.f[1]);
    cic_abs(z, inv_h, n, c.i[2][0], c.i[2][1], c.f[2]);
}

// r = g1 + G[dF] - g3 at particle p.
__device__ __forceinline__ void loss_resid(const LossCell& c, int n, const float* const df[3], const float* const g1[3],
                                           const float* const g3[3], long p, float& r0, float& r1, float& r2) {
    const float wx[2] = {1.0f - c.f[0], c.f[0]}, wy[2] = {1.0f - c.f[1], c.f[1]}, wz[2] = {1.0f - c.f[2], c.f[2]};
    float a0 = 0.f, a1 = 0.f, a2 = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const long v = ((long)c.i[0][a] * n + c.i[1][b]) * n + c.i[2][d];
                const float w = wx[a] * wy[b] * wz[d];
                a0 += w * df[0][v];
                a1 += w * df[1][v];
                a2 += w * df[2][v];
            }
    r0 = g1[0][p] + a0 - g3[0][p];
    r1 = g1[1][p] + a1 - g3[1][p];
    r2 = g1[2][p] + a2 - g3[2][p];
}

}  // namespace cola
