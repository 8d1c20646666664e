// One tile of the value prior (Sec. 4.3), shared by the launch of its own (value_prior.hip) and
// by the fp32 row-statistics launch, which appends the tiles to its own workgroups.
#pragma once

#include "aha_dev.h"
#include "aha_host.h"

namespace aha {

// gamma = average pool of ||V||^2 for the kVTileRows tokens of tile `tile` of problem z, written
// to `gamma`, and the tile's largest gamma to gblockmax[z * n_vtiles + tile]; called by all 256
// threads of a workgroup.
template <int ESIZE>
__device__ __forceinline__ void value_prior_tile(const ScoreGeom &g, int z, int tile, int n_vtiles,
                                                 float *gamma, float *gblockmax, int tid) {
    __shared__ float s_nu[kVTileRows + 256];
    __shared__ float s_max[4];
    const int b = z / g.Hkv, h = z % g.Hkv;
    const char *vbase =
        (const char *)g.v + (int64_t)ESIZE * (b * g.vs[0] + h * g.vs[1]);
    const int half = (g.pool - 1) / 2;
    const int t0 = tile * kVTileRows;
    const int lo = max(0, t0 - half);
    const int hi = min(g.n, t0 + kVTileRows + half);  // exclusive
    value_norms_to_lds<ESIZE>(vbase, g.vs[2], g.d, lo, hi, s_nu, tid);
    __syncthreads();

    const int j = t0 + tid;
    float gam = 0.f;
    if (j < g.n) {
        const int a = max(0, j - half), e = min(g.n - 1, j + half);
        float s = 0.f;
        for (int t = a; t <= e; ++t) s += s_nu[t - lo];
        gam = s / (float)(e - a + 1);
        gamma[(int64_t)z * g.n + j] = gam;
    }
    float m = wave_max(gam);
    if ((tid & 63) == 0) s_max[tid >> 6] = m;
    __syncthreads();
    if (tid == 0)
        gblockmax[z * n_vtiles + tile] = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
}

}  // namespace aha
