// fp32 dots of 32 keys and 32 query rows on the matrix core, and what brings them there.
//
// v_mfma_f32_32x32x2_f32, keys on M and query rows on N as in score_bf16.hip: fp32 products and
// sums at twice the vector ALU's rate, and none of the vector-ALU kernels' lane exchanges or LDS
// reads per product.  A lane holds the 16-byte chunks 2 i + lane / 32 of its row; element e of chunk i of the
// two half-waves is one contraction step (channels 8 i + e and 8 i + 4 + e).  The steps are dealt to
// eight accumulators, so that no sum is a longer chain (D / 8 products) than in the kernels above
// and the rounding error stays theirs
// (against float64, 32 heads x 256 rows x 2206 keys, d = 64: 1.5e-7 of the scores' norm, 2.1e-7 there).
// Both passes of that problem 147 -> 112 us, at d = 128 258 -> 189; 32 heads x 128 rows x 1108
// keys, d = 128, 110 -> 73.
#pragma once

#include "score_tile.h"

namespace aha {

template <int D>
__device__ __forceinline__ f32x16 f32_block_dots(const f32x4 (&a)[D / 8], const float *sq) {
    f32x16 acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
#pragma unroll
    for (int i = 0; i < D / 8; ++i) {
        const f32x4 q = *(const f32x4 *)(sq + 8 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[(4 * i + e) & 7] =
                __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], q[e], acc[(4 * i + e) & 7], 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
        acc[0][v] = ((acc[0][v] + acc[1][v]) + (acc[2][v] + acc[3][v])) +
                    ((acc[4][v] + acc[5][v]) + (acc[6][v] + acc[7][v]));
    return acc[0];
}
// key rows of a block of 32 from kb on; past the last key: the last one (its results are dropped)
template <int D>
__device__ __forceinline__ void f32_load_keys(const float *kbase, int64_t stride, int kb, int last,
                                              int lane, f32x4 (&a)[D / 8]) {
    const float *row = kbase + (int64_t)min(kb + (lane & 31), last) * stride + 4 * (lane >> 5);
#pragma unroll
    for (int i = 0; i < D / 8; ++i) a[i] = *(const f32x4 *)(row + 8 * i);
}
constexpr int f32_ld(int d) { return d + 4; }  // padded row of a query block in LDS (floats)

// THREADS lanes bring the 32 query rows from rho0 on (past the last one: the last) to LDS; request
// and commit apart, so that whatever else the block needs travels with them
template <int D, int THREADS>
struct F32QueryBlock {
    static constexpr int CPR = D / 4, N = 32 * CPR / THREADS;
    f32x4 w[N];
    __device__ __forceinline__ void request(const ScoreGeom &g, const RowMap &rm, int b, int h,
                                            int rho0, int t0) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int t = t0 + u * THREADS, rho = min(rho0 + t / CPR, g.R - 1);
            w[u] = *(const f32x4 *)((const float *)g.q + b * g.qs[0] +
                                    (int64_t)(h * g.G + rm.head(rho)) * g.qs[1] +
                                    (int64_t)rm.pos(rho) * g.qs[2] + 4 * (t % CPR));
        }
    }
    __device__ __forceinline__ void commit(int t0, float *sq) const {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int t = t0 + u * THREADS;
            *(f32x4 *)(sq + (t / CPR) * f32_ld(D) + 4 * (t % CPR)) = w[u];
        }
    }
};

}  // namespace aha
