// Value prior (Sec. 4.3): nu_j = ||V_j||^2, gamma = average pool of nu over
// tokens (odd width, stride 1, mean over the in-range taps), and the per-tile
// maxima of gamma from which the consumers form gamma / max(gamma).
//
// HBM-bound: V is read exactly once (plus (pool-1)/2 halo rows per tile).
// The windowed bf16 scores form the prior inside their one launch (score_window.hip,
// score_given.hip) or, in two, inside the row statistics (score_bf16.hip, up to 128 rows), fp32
// inputs as extra workgroups of theirs (score_f32.hip); this kernel serves full accumulation
// (where it also zeroes the scores; without a prior the row statistics do), pool widths above 17, chosen rows, larger tiles whose workspace
// holds two launches only, and given normalisers in two launches (which it converts for the
// column-sum pass).
#include "value_tile.h"

namespace aha {

// One workgroup = kVTileRows consecutive tokens of one (batch, KV head).
// 16-byte loads; LPR lanes cover one row.
template <int ESIZE>
__global__ __launch_bounds__(256) void vprior_kernel(ScoreGeom g, int n_vtiles, float *gamma,
                                                     float *gblockmax,
                                                     float *zero_scores, const float *lse,
                                                     float *row_stats, int rows_pad, int pr) {
    const int z = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
    if (lse) {
        // the caller's row normalisers (natural log, [batch, Hq, window]) -> log2 domain, in
        // the order of each KV head's places, pr per query head (those without a row: unused)
        const int b = z / g.Hkv, h = z % g.Hkv;
        for (uint32_t at = tile * 256 + tid; at < (uint32_t)rows_pad; at += gridDim.x * 256) {
            const int gi = at / (uint32_t)pr, ii = at - gi * pr;
            const bool row = gi < g.G && ii < g.r;
            row_stats[(int64_t)z * rows_pad + at] = row ? lse[((int64_t)b * g.Hq + h * g.G + gi) * g.r + ii] * kLog2e : 0.f;
        }
    }
    if (zero_scores && tile < n_vtiles) {
        // full accumulation adds tile contributions atomically: the scores start from zero
        const int j = tile * kVTileRows + tid;
        if (j < g.n) zero_scores[(int64_t)z * g.n + j] = 0.f;
    }
    if (!g.value_prior || tile >= n_vtiles) return;
    value_prior_tile<ESIZE>(g, z, tile, n_vtiles, gamma, gblockmax, tid);
}

hipError_t launch_value_prior(const ScoreGeom &g, const PrefillPlan &pl, void *ws,
                              float *scores, const float *lse, bool prior_here, hipStream_t st) {
    char *w = (char *)ws;
    float *gamma = (float *)(w + pl.off_gamma);
    float *gbm = (float *)(w + pl.off_gblockmax);
    if (!prior_here && !lse) return hipSuccess;  // nothing for this launch to do
    // bf16 full accumulation (several query tiles) needs zeroed scores (without this launch the row statistics zero them)
    float *zero_scores = (g.dtype == AHA_BF16 && pl.n_qtiles > 1) ? scores : nullptr;
    ScoreGeom gl = g;
    gl.value_prior = prior_here ? 1 : 0;
    const int vt = (prior_here || zero_scores) ? pl.n_vtiles : 1;
    dim3 grid(vt, pl.Z);
    // where pass 2 reads the row statistics: one chunk per (problem, tile, row) on the bf16
    // path (rows padded to whole tiles), one value per row on the fp32 path
    float *row_stats = (float *)(w + (g.dtype == AHA_BF16 ? pl.off_partial : pl.off_rowL));
    const int rows_pad = g.dtype == AHA_BF16 ? pl.full_tiles * pl.qtile : g.R, pr = g.dtype == AHA_BF16 ? pl.full_pr : g.r;
    if (g.dtype == AHA_BF16)
        hipLaunchKernelGGL(vprior_kernel<2>, grid, dim3(256), 0, st, gl, pl.n_vtiles, gamma, gbm,
                           zero_scores, lse, row_stats, rows_pad, pr);
    else
        hipLaunchKernelGGL(vprior_kernel<4>, grid, dim3(256), 0, st, gl, pl.n_vtiles, gamma, gbm,
                           zero_scores, lse, row_stats, rows_pad, pr);
    return hipGetLastError();
}

}  // namespace aha
