// What the bf16 score kernels do with a block product: the row statistics and the column sums of
// a 64-key x 32-row block, and the squared norms of value rows that were loaded like keys.
#pragma once

#include "score_tile.h"

namespace aha {

// Online max / sum-of-exp2 of one 64 x 32 block for this lane's query column.
// The scale is non-negative, so the maximum of the scaled logits is the scale
// times the maximum raw dot.
// With ENT the first moment u = sum of exp2(t - m) * (t - m) is kept beside the sum: the
// row's entropy is ln 2 * (log2 s - u / s) (Sec. 4.2, entropy of a softmax row).
template <bool MASK, bool ENT, bool LAZY = false>
__device__ __forceinline__ void stats_update(const f32x16 (&acc)[kMB], float lam, int pos, int kb,
                                             int lane, float &m, float &s, float &u) {
    if (MASK) asm volatile("" ::: "memory");
    if constexpr (!MASK && LAZY) {
        // (LAZY: full accumulation, where this loop is the kernel; in the windowed kernel the
        // second code path costs registers that spill.)
        // Unmasked blocks: `m` is a REFERENCE that sum and moment are relative to, not
        // necessarily the running maximum (the final statistics m + log2 s and u / s do not
        // depend on it).  As long as every lane has one, the block is summed against it as it
        // stands - no maximum over the block's 32 elements - and the reference is only moved
        // (by the exact update below, which also redoes this block) when a block's sum says
        // that it has fallen more than 40 binades behind: fp32 has room for that, and a
        // reference never lies above the largest logit seen, so nothing underflows that the
        // exact update would have kept.
        if (__builtin_amdgcn_ballot_w64(m == -INFINITY) == 0) {
            float sum[4] = {0.f, 0.f, 0.f, 0.f}, mom[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float x = fmaf(acc[mb][v], lam, -m);
                    const float e = fast_exp2(x);
                    sum[v & 3] += e;
                    if (ENT) mom[v & 3] = fmaf(e, x, mom[v & 3]);
                }
            const float bs = (sum[0] + sum[1]) + (sum[2] + sum[3]);
            if (__builtin_amdgcn_ballot_w64(!(bs < 0x1p40f)) == 0) {  // (also: not a NaN)
                s += bs;
                if (ENT) u += (mom[0] + mom[1]) + (mom[2] + mom[3]);
                return;
            }
        }
    }
    float amax = -INFINITY;
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float x = acc[mb][v];
            if (MASK && acc_key(kb, mb, v, lane) > pos) x = -INFINITY;
            amax = fmaxf(amax, x);
        }
    const float tmax = amax == -INFINITY ? -INFINITY : amax * lam;
    const float mn = fmaxf(m, tmax);
    const float mref = mn == -INFINITY ? 0.f : mn;
    // four partial sums: independent chains, so that the exponentials' result latency is
    // covered by other work instead of wait states
    float sum[4] = {0.f, 0.f, 0.f, 0.f}, mom[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float x = fmaf(acc[mb][v], lam, -mref);
            float e = fast_exp2(x);
            if (MASK && acc_key(kb, mb, v, lane) > pos) e = 0.f;
            sum[v & 3] += e;
            // (e = 0 for masked or far-away keys: 0 * x, x finite, adds nothing)
            if (ENT) mom[v & 3] = fmaf(e, x, mom[v & 3]);
        }
    const float f = fast_exp2(m - mref);  // 0 while the row has seen no key
    if (ENT) {
        const float dm = m == -INFINITY ? 0.f : m - mref;
        u = (u + dm * s) * f + ((mom[0] + mom[1]) + (mom[2] + mom[3]));
    }
    s = s * f + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
    m = mn;
}

template <bool MASK>
__device__ __forceinline__ void colsum_update(const f32x16 (&acc)[kMB], float lam, float L,
                                              int pos, int kb, int lane, f32x16 (&col)[kMB]) {
    // The empty asm keeps the masked and the unmasked instantiation apart: without it the
    // compiler merges the two branches and every block pays the per-element compare/select.
    if (MASK) asm volatile("" ::: "memory");
    if constexpr (!MASK) {
        // Four elements at a time - their scaled logits, their exponentials, their sums - and
        // the instructions kept in that order: scheduled by register pressure alone, every
        // exponential is followed at once by the addition that needs it, with a wait state
        // (an issue slot of the wave) in between.
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
            for (int v0 = 0; v0 < 16; v0 += 4) {
                float t[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = fmaf(acc[mb][v0 + i], lam, -L);
                asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = fast_exp2(t[i]);
                asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
#pragma unroll
                for (int i = 0; i < 4; ++i) col[mb][v0 + i] += t[i];
            }
        return;
    }
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float p = fast_exp2(fmaf(acc[mb][v], lam, -L));
            if (MASK && acc_key(kb, mb, v, lane) > pos) p = 0.f;
            col[mb][v] += p;
        }
    if (MASK) asm volatile("" ::: "memory");
}

// Value prior (Sec. 4.3) inside pass 1.  The value rows of the 64 keys a wave multiplies in a
// step are loaded with the addressing of the key fragments into the register buffer that is
// idle in the first half of the step (the next key block is requested at mid-step instead of
// at the start): a lane then holds one half (the channels of its half-wave) of two value rows.

// nu = ||V_row||^2 of those rows: squares summed in-lane, one exchange between the half-waves.
// M: of the first M groups of 32 rows.
template <int D, int M = kMB>
__device__ __forceinline__ void fragment_row_norms(const bf16x8 (&a)[kMB][D / 16],
                                                   float (&nu)[kMB]) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int mb = 0; mb < M; ++mb) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            const bf16x8 w = a[mb][ks];
            const bf16x2 p0 = {w[0], w[1]}, p1 = {w[2], w[3]}, p2 = {w[4], w[5]}, p3 = {w[6], w[7]};
            s0 = __builtin_amdgcn_fdot2_f32_bf16(p0, p0, s0, false);
            s1 = __builtin_amdgcn_fdot2_f32_bf16(p1, p1, s1, false);
            s0 = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, s0, false);
            s1 = __builtin_amdgcn_fdot2_f32_bf16(p3, p3, s1, false);
        }
        const float h = s0 + s1;
        nu[mb] = combine_lane_xor<32>(h, OpSum{});
    }
}

constexpr int kPriorPiece = 512;   // keys whose norms are staged for pooling at a time
constexpr int kPriorMaxHalo = 32;  // rows on both sides together
// Pooling halo of a key range [kbeg, kend): the (pool - 1) / 2 value rows below and above it,
// one per group of d / 8 lanes (at most 256 / (d / 8) rows: the host checks the pool width).
// Requested right after the main loop, squared when the range is pooled.
template <int D>
struct PriorHalo {
    static constexpr int CPR = D / 8;  // 16-byte chunks per value row
    u32x4 w;
    int pos;     // token of this thread's halo row
    bool valid;  // the row exists (inside the sequence, inside the halo)
    bool below;
    __device__ __forceinline__ void request(const ScoreGeom &g, const __bf16 *vbase, int kbeg,
                                            int kend, int tid) {
        const int half = (g.pool - 1) / 2, hrow = tid / CPR;
        below = hrow < half;
        pos = below ? kbeg - half + hrow : kend + hrow - half;
        valid = hrow < 2 * half && pos >= 0 && pos < g.n;
        w = u32x4{0u, 0u, 0u, 0u};
        if (valid) w = *(const u32x4 *)(vbase + (int64_t)pos * g.vs[2] + (tid % CPR) * 8);
    }
    // ||row||^2 in the first lane of the row's group (every lane takes part)
    __device__ __forceinline__ float norm() const {
        float hn = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float x = bf16_lo(w[c]), y = bf16_hi(w[c]);
            hn = fmaf(x, x, fmaf(y, y, hn));
        }
        return reduce_lanes<1, CPR>(hn, OpSum{});
    }
};

}  // namespace aha
