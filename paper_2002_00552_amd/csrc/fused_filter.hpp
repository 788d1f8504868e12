// The single-kernel forward path's copy of the transformed filter (fused.hip reads it, transforms.hip writes it).
#pragma once

#include "plan.hpp"

namespace dwm {

// (G_l g)[i] with the 2-tap case run as 3 taps with a zero third tap.
__device__ __forceinline__ float fused_g_row(int l, int i, float v0, float v1, float v2)
{
    if (l == 1) return v0;
    switch (i) {
        case 0: return v0;
        case 1: return 0.5f * (v0 + v1 + v2);
        case 2: return 0.5f * (v0 - v1 + v2);
        default: return v2;
    }
}

// ---------------------------------------------------------------------------------
// Filter copy for this path: UF[class][slice][plane][row][i][half], filter = 32*slice +
// 16*half + i; zero for filters >= K, padding rows and frequencies a part does not have.
// One thread per (row, filter).
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void fused_filter(const DevPlan& P, const FusedArgs& F, const FilterSource& Q, const float* __restrict__ w,
                                             float* __restrict__ U, int row, int k)
{
    if (row >= F.rows_total) return;
    int fi = 0;
    while (fi + 1 < F.nfc && row >= F.fc[fi + 1].row0) ++fi;
    const FusedClass fc = F.fc[fi];
    const unsigned desc = F.rowdesc[row];
    const bool real = (desc >> 15) != 0 && k < P.K;
    const DevPiece hp = P.ph[desc & 15], wp = P.pw[(desc >> 4) & 15];
    const int c = (desc >> 8) & 127;
    float g[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            float v = 0.f;
            if (real && i < hp.l && j < wp.l) {
                const int r = P.s * (hp.j + i) + hp.p, q = P.s * (wp.j + j) + wp.p;
                v = w[Q.base + k * Q.sk + c * Q.sc + r * Q.sr + q * Q.ss];
            }
            g[i][j] = v;
        }
    float t[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) t[i][j] = fused_g_row(hp.l, i, g[0][j], g[1][j], g[2][j]);
    const int slice = k >> 5, half = (k >> 4) & 1, ki = k & 15;
    float* dst = U + fc.uf_off + ((size_t)slice * fc.nfh * fc.nfw * fc.rows + (row - fc.row0)) * 32 + ki * 2 + half;
#pragma unroll
    for (int fh = 0; fh < 4; ++fh)
#pragma unroll
        for (int fw = 0; fw < 4; ++fw)
            if (fh < fc.nfh && fw < fc.nfw) {
                const float u = fused_g_row(wp.l, fw, t[fh][0], t[fh][1], t[fh][2]);
                dst[(size_t)(fh * fc.nfw + fw) * fc.rows * 32] = (real && fh <= hp.l && fw <= wp.l) ? u : 0.f;
            }
}

}  // namespace dwm
