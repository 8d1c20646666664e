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
template <bool MASK, bool ENT>
__device__ __forceinline__ void stats_update(const f32x16 (&acc)[kMB], float lam, int pos, int kb,
                                             int lane, float &m, float &s, float &u) {
    if (MASK) asm volatile("" ::: "memory");
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

// A block's products with keys that a row does not see become -inf, which counts as nothing in the update that follows, given
// a scale above 0; `room`: the row's position less the key of accumulator element 0.  A scale of (almost) 0 goes into
// the products instead.
constexpr float kLeastScale = 1e-30f;
__device__ __forceinline__ void hide_unseen(f32x16 (&acc)[kMB], int room, float &lam) {
    asm volatile("" ::: "memory");  // (else the branch that leads here becomes a choice per element in every block)
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(lam < kLeastScale) != 0, 0)) {
        const float f = lam < kLeastScale ? lam / kLeastScale : 1.f;
        lam = fmaxf(lam, kLeastScale);
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][v] *= f;
    }
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (mb * 32 + 8 * (v >> 2) + (v & 3) > room) acc[mb][v] = -INFINITY;  // (acc_key)
}
// stats_update() that leaves the block's exponentials in the place of its products, relative to `ref`, the running maximum (-inf: no
// key seen yet), so that a column sum takes one multiplication per element.
__device__ __forceinline__ void stats_weights(f32x16 (&acc)[kMB], float lam, float &m, float &s, float &ref) {
    float amax = -INFINITY;
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) amax = fmaxf(amax, acc[mb][v]);
    const float tmax = amax == -INFINITY ? -INFINITY : amax * lam;
    ref = fmaxf(m, tmax);
    const float mref = ref == -INFINITY ? 0.f : ref;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[mb][v] = fast_exp2(fmaf(acc[mb][v], lam, -mref));
            sum[v & 3] += acc[mb][v];
        }
    s = s * fast_exp2(m - mref) + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
    m = ref;
}
// Weights whose row has no factor (`none`: NaN or infinite): the keys that the row sees get NaN, the others nothing; `room`: the
// row's position less the key of element 0.
__device__ __forceinline__ void weights_without_factor(f32x16 (&acc)[kMB], int room, bool none, float &f) {
    asm volatile("" ::: "memory");
    f = none ? 1.f : f;
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (none) acc[mb][v] = mb * 32 + 8 * (v >> 2) + (v & 3) <= room ? __builtin_nanf("") : 0.f;  // (acc_key)
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

// Value prior (Sec. 4.3).  The value rows of the keys a wave multiplies in a step pass through the
// register buffer that the next key block does not need yet.  Loaded with the addressing of the key
// fragments (two tiles of the two-sweep kernel), a lane holds one half (the
// channels of its half-wave) of a value row per group of 32.

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

// Value prior of the one-launch kernels, a template argument: none, value rows through the caches, past them.
constexpr int kNoValues = 0, kValuesCached = 1, kValuesOnce = 2;
// The same for value rows that a wave loads as they lie in memory, D / 8 lanes to a row and 512 / D rows to
// an instruction.  M: 32 rows each.  ONCE: past the caches.
template <int D, bool ONCE, int M = kMB>
__device__ __forceinline__ void load_rows(const __bf16 *vbase, int64_t v_tstride, int kb, int end, int lane,
                                          bf16x8 (&w)[kMB][D / 16]) {
    constexpr int CPR = D / 8, RPI = 64 / CPR;
    int row = kb + lane / CPR;
    const __bf16 *p = vbase + (int64_t)min(row, end - 1) * v_tstride + (lane % CPR) * 8;
#pragma unroll
    for (int u = 0; u < M * D / 16; ++u) {
        bf16x8 &x = w[u / (D / 16)][u % (D / 16)];
        if constexpr (ONCE) x = __builtin_nontemporal_load((const bf16x8 *)p);
        else x = *(const bf16x8 *)p;
        row += RPI;
        if (row < end) p += RPI * v_tstride;  // (past the end: a row that is there once more)
    }
}
// Recursive halving over M, M / 2, .. 1: of N per-lane values the sums over those lanes, one value in each; `u`: which.
template <int M, int N>
__device__ __forceinline__ float fold_rows(float (&x)[N], int lane, int &u) {
    const bool hi = lane & M;
    if constexpr (N > 1) {
        float y[N / 2];
#pragma unroll
        for (int t = 0; t < N / 2; ++t) {
            const float send = hi ? x[t] : x[t + N / 2], keep = hi ? x[t + N / 2] : x[t];
            y[t] = keep + from_lane_xor<M>(send);
        }
        u += hi ? N / 2 : 0;
        if constexpr (M > 1) return fold_rows<M / 2>(y, lane, u);
        else return y[0];
    } else {
        const float y = x[0] + from_lane_xor<M>(x[0]);
        if constexpr (M > 1) {
            float z[1] = {y};
            return fold_rows<M / 2>(z, lane, u);
        } else return y;
    }
}
// ||V_row||^2 of one of those rows, row kb + `row`: in each lane (M = 1: pair of lanes) another one.
template <int D, int M = kMB>
__device__ __forceinline__ float loaded_row_norm(const bf16x8 (&w)[kMB][D / 16], int lane, int &row) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    constexpr int CPR = D / 8, RPI = 64 / CPR, U = M * D / 16;
    static_assert(U <= CPR, "no more rows than lanes");
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bf16x8 v = w[u / (D / 16)][u % (D / 16)];
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 8; c += 2) {
            const bf16x2 pr = {v[c], v[c + 1]};
            s = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, s, false);
        }
        x[u] = s;
    }
    int u = 0;
    const float nu = fold_rows<CPR / 2>(x, lane, u);
    row = u * RPI + lane / CPR;
    return nu;
}

constexpr int kPriorPiece = 512;   // keys whose norms are staged for pooling at a time (unless there is more LDS)
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

// gamma (Sec. 4.3) of the keys [kbeg, kend), whose norms and pooling halo are in s_nu[t - lo],
// lo = max(0, kbeg - half), into s_gam[key - kbeg]; returns this thread's largest.
__device__ __forceinline__ float pool_norms(const ScoreGeom &g, int kbeg, int kend, const float *s_nu,
                                            float *s_gam, int tid, int nthreads) {
    const int half = (g.pool - 1) / 2, lo = max(0, kbeg - half);
    float gmax = 0.f;
    for (int j = kbeg + tid; j < kend; j += nthreads) {
        const int a = max(0, j - half), e = min(g.n - 1, j + half);
        float s = 0.f;
        for (int t = a; t <= e; ++t) s += s_nu[t - lo];
        const float gam = s / (float)(e - a + 1);
        s_gam[j - kbeg] = gam;
        gmax = fmaxf(gmax, gam);
    }
    return gmax;
}

// gamma of the keys [kbeg, kend) from the norms the workgroup's waves left in nu_g, in pieces staged in
// s_nu, to use(key, gamma); returns this thread's largest.  The caller has passed a barrier since the last norm
// was written, and nobody uses s_nu any more.
template <int D, int THREADS, int PIECE = kPriorPiece, class Use>
__device__ __forceinline__ float pool_norms_of_range(const ScoreGeom &g, int z, int kbeg, int kend,
                                                     const float *nu_g, const PriorHalo<D> &halo,
                                                     float *s_nu, int tid, Use &&use) {
    const int half = (g.pool - 1) / 2;
    const float hn = halo.norm();
    float gmax = 0.f;
    for (int t0 = kbeg; t0 < kend; t0 += PIECE) {
        const int t1 = min(kend, t0 + PIECE);
        const int lo = max(0, t0 - half), hi = min(g.n, t1 + half);  // hi exclusive
        for (int t = max(lo, kbeg) + tid; t < min(hi, kend); t += THREADS) s_nu[t - lo] = nu_g[(int64_t)z * g.n + t];
        // the halo rows that touch this piece (the first piece below, the last one above)
        if (halo.valid && tid % PriorHalo<D>::CPR == 0 && (halo.below ? t0 == kbeg : t1 == kend))
            s_nu[halo.pos - lo] = hn;
        __syncthreads();
        for (int j = t0 + tid; j < t1; j += THREADS) {
            const int a = max(0, j - half), e = min(g.n - 1, j + half);
            float s = 0.f;
            for (int t = a; t <= e; ++t) s += s_nu[t - lo];
            const float gam = s / (float)(e - a + 1);
            use(j, gam);
            gmax = fmaxf(gmax, gam);
        }
        __syncthreads();
    }
    return gmax;
}

// Work split of several query tiles (score_full.hip, and pass 1 for the row statistics' output).  Query tile `pair` is
// teamed with tile T-1-pair: a tile of late rows sees many keys, its partner few, together
// about the same as any other pair.  The pair's work is laid out on a line - the first
// tile's key steps, the set-up of the partner (`set_up` steps' worth; every workgroup pays
// one set-up anyway, only a second one counts), the partner's steps - and the line is cut into `nparts` equal ranges.  Segment `seg` (0: first tile,
// 1: partner) of a workgroup is the part of its range that falls on that tile's steps.
// A single tile (windowed scores, or the middle tile of an odd count) is cut into equal
// ranges of steps.
struct Segment {
    int qt;          // query tile, -1: no such segment
    int kbeg, kend;  // keys [kbeg, kend); empty when kbeg >= kend
};
template <class Map>
__device__ __forceinline__ Segment pair_segment(const Map &rm, int rows, int T, int pair,
                                                int part, int nparts, int seg,
                                                int step = kWgKeys, int set_up = 1) {
    const int tA = pair, tB = T - 1 - pair;
    const bool two = tB != tA;
    // (chosen accumulator rows - a single tile - may sit anywhere: the whole sequence)
    const int endA = rm.rows ? rm.n : rm.max_pos(tA * rows, (tA + 1) * rows) + 1;
    const int endB = two ? rm.max_pos(tB * rows, (tB + 1) * rows) + 1 : 0;
    const int sA = (endA + step - 1) / step, sB = (endB + step - 1) / step;
    // positions on the line: first tile's steps start at oA, the partner's at oB
    const int oA = 0, oB = sA + set_up, V = two ? sA + sB + set_up : sA;
    const int v0 = (int)((int64_t)part * V / nparts), v1 = (int)((int64_t)(part + 1) * V / nparts);
    Segment r;
    if (seg == 0) {
        r.qt = tA;
        r.kbeg = (max(v0, oA) - oA) * step;
        r.kend = min(endA, (min(v1, oA + sA) - oA) * step);
    } else {
        r.qt = two ? tB : -1;
        r.kbeg = (max(v0, oB) - oB) * step;
        r.kend = min(endB, (min(v1, oB + sB) - oB) * step);
    }
    return r;
}

// Log2-sum-exp2 of one query row from the per-chunk log2-sum-exp2 values that pass 1 left.
// A batch of values is requested at once (request), so that it travels together with the
// other loads of the tile set-up, and merged later (merge) into the running (M, sum) with
// sum = sum over chunks of exp2(value - M).  Both go by groups of eight and skip the
// groups past the last chunk.
template <int BATCH>
__device__ __forceinline__ void chunk_request(const float *src, int stride, int c0, int nchunks,
                                              float (&e)[BATCH]) {
    static_assert(BATCH % 8 == 0, "groups of eight");
#pragma unroll
    for (int g8 = 0; g8 < BATCH; g8 += 8) {
        if (c0 + g8 >= nchunks) break;  // uniform
        // entries past the last chunk re-read it (branch-free, back-to-back loads) and are
        // neutralised in the merge
#pragma unroll
        for (int t = g8; t < g8 + 8; ++t) e[t] = src[(int64_t)min(c0 + t, nchunks - 1) * stride];
    }
}
template <int BATCH>
__device__ __forceinline__ void chunk_merge(const float (&e)[BATCH], int count, float &M,
                                            float &sum) {
    float bm = -INFINITY;
#pragma unroll
    for (int g8 = 0; g8 < BATCH; g8 += 8) {
        if (g8 >= count) break;  // uniform
#pragma unroll
        for (int t = g8; t < g8 + 8; ++t) bm = fmaxf(bm, t < count ? e[t] : -INFINITY);
    }
    const float mn = fmaxf(M, bm);
    const float mref = mn == -INFINITY ? 0.f : mn;
    sum *= fast_exp2(M - mref);
#pragma unroll
    for (int g8 = 0; g8 < BATCH; g8 += 8) {
        if (g8 >= count) break;
#pragma unroll
        for (int t = g8; t < g8 + 8; ++t) sum += t < count ? fast_exp2(e[t] - mref) : 0.f;
    }
    M = mn;
}

}  // namespace aha
