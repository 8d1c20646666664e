// fp32 eviction scores (Sec. 4.1 - 4.3; Alg. 1 Prefill), vector-ALU kernels for small problems and
// matrix-core kernels for larger ones.  This is the small-problem, high-accuracy path (fp32 Q/K/V); the
// bf16 path in score_bf16.hip carries the throughput.
//
// Pass 1: a workgroup finds max_j and log2-sum-exp2 of t_ij = s_i * log2(e) * (Q_i . K_j) over
//         j <= i for one or four observed query rows; extra workgroups of the same launch form
//         the value prior.
// Pass 2: a workgroup sums exp2(t_ij - L_i) over the observed rows i >= j for its 16 or 64 keys,
//         the rows dealt to its four waves.
//
// In both passes FOUR lanes share a dot product: lane p of a quad holds the 16-byte chunks
// p, p + 4, ... of its key rows (a quad reads 64 contiguous bytes at a time, and a row takes a
// quarter of the registers of one thread), and two exchanges inside the quad sum the parts.  Four
// products of a quad then leave one exponential per lane: four rows of one key in pass 1, four
// keys of one row in pass 2.  The small variants (one row, 16 keys per workgroup) leave that
// factor unused for four times as many workgroups: the path's own problem (2 heads x 512 keys x
// 32 rows, head_dim 64) is bound by latency, and one thread per key gave it four workgroups that
// each walked all rows.  Measured there: pass 2 25.5 -> 5.5 us, pass 1 and the prior (two
// launches, 7.2 + 4.5 us) -> 5.6 us.
#include "f32_tile.h"
#include "value_tile.h"

namespace aha {

// A running statistic (m, s, u) of scaled logits t: m = max t, s = sum exp2(t - m),
// u = sum exp2(t - m) (t - m).  The row's entropy is ln 2 * (log2 s - u / s) (Sec. 4.2).
// Re-referenced to a maximum M >= m it is (M, s f, (u + (m - M) s) f) with f = 2^(m - M).
__device__ __forceinline__ void reref_stat(float m, float M, float &s, float &u) {
    if (m == -INFINITY) { s = 0.f; u = 0.f; return; }
    const float f = exp2f(m - M);
    u = (u + (m - M) * s) * f;
    s *= f;
}
// the statistic of the union of two key sets
__device__ __forceinline__ void merge_stat(float &m, float &s, float &u, float m2, float s2,
                                           float u2) {
    const float M = fmaxf(m, m2);
    reref_stat(m, M, s, u);
    reref_stat(m2, M, s2, u2);
    m = M;
    s += s2;
    u += u2;
}

// Sum over the four lanes of a quad.
__device__ __forceinline__ float quad_sum(float x) { return reduce_lanes<1, 4>(x, OpSum{}); }
// x[part] without a dynamically indexed array.  The elements go through an opaque move: otherwise
// the compiler sees through the choice and keeps the array in memory, indexed - in LDS, at an address
// formed from the workgroup's size, which is read from the dispatch packet in the host's memory (14
// us of latency: 64 heads x 32 rows x 40 keys 19.3 us instead of 5), or in scratch.
__device__ __forceinline__ float pick4(const float (&x)[4], int part) {
    float x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
    asm volatile("" : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3));
    const float a = part & 1 ? x1 : x0, b = part & 1 ? x3 : x2;
    return part & 2 ? b : a;
}

// A lane's share of a row: chunks part, part + 4, ... of 16 bytes.
template <int D>
struct QuadRow {
    f32x4 c[D / 16];
    __device__ __forceinline__ void load(const float *row, int part) {
#pragma unroll
        for (int t = 0; t < D / 16; ++t) c[t] = *(const f32x4 *)(row + 4 * (part + 4 * t));
    }
    __device__ __forceinline__ float dot(const QuadRow &o) const {  // this lane's part
        float w[2] = {0.f, 0.f};
#pragma unroll
        for (int t = 0; t < D / 16; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[t & 1] = fmaf(c[t][e], o.c[t][e], w[t & 1]);
        return w[0] + w[1];
    }
};

// RQ observed rows (1 or 4) per workgroup; workgroups past the row blocks take the value tiles.
// `lse_out` / `ent_out` (either may be null): natural-log normaliser and entropy of every
// observed row, dense [batch, Hq, window].
template <int D, int RQ>
__global__ __launch_bounds__(256) void f32_pass1_kernel(ScoreGeom g, int row_blocks, int n_vtiles,
                                                        float *gamma, float *gblockmax, float *rowL,
                                                        float *lse_out, float *ent_out) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Workgroups go to the XCDs in turn: a problem's, which read the same keys, are dealt to one of
    // them (64 heads x 4 rows x 3000 keys, d = 128: 60 -> 21 us).
    int z = blockIdx.y, blk = blockIdx.x;
    if (gridDim.x < 1u << 15) {  // (32-bit indexes)
        const uint32_t per = gridDim.x * gridDim.y / kXcds, id = blockIdx.y * gridDim.x + blockIdx.x;
        const uint32_t wg = id < per * kXcds ? id % kXcds * per + id / kXcds : id;
        z = (int)(wg / gridDim.x);
        blk = (int)(wg % gridDim.x);
    }
    if (blk >= row_blocks) {  // (workgroup-uniform)
        value_prior_tile<4>(g, z, blk - row_blocks, n_vtiles, gamma, gblockmax, tid);
        return;
    }
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int rho0 = blk * RQ, part = tid & 3, kk = tid >> 2;
    const RowMap rm{g.n, g.r, g.R,
                    g.rows ? g.rows + ((int64_t)b * g.Hq + (int64_t)h * g.G) * g.r : nullptr};
    const float *kbase = (const float *)g.k + b * g.ks[0] + h * g.ks[1];
    __shared__ float s_m[4][RQ], s_s[4][RQ], s_u[4][RQ];

    // (rows past the last one stand for the last; their results are dropped)
    QuadRow<D> q[RQ];
    int last = 0;  // the largest position of the rows
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
        const int rho = min(rho0 + r, g.R - 1), i = rm.pos(rho);
        last = max(last, i);
        q[r].load((const float *)g.q + b * g.qs[0] + (int64_t)(h * g.G + rm.head(rho)) * g.qs[1] +
                      (int64_t)i * g.qs[2], part);
    }
    // the row whose statistic this lane keeps
    const int my_rho = min(rho0 + (RQ == 4 ? part : 0), g.R - 1), my_i = rm.pos(my_rho);
    const float lam = row_scale_log2(g.scale_mode, g.fixed_scale, g.lambda_floor, my_i + 1,
                                     g.budget, g.d);

    float m = -INFINITY, s = 0.f, u = 0.f;
    constexpr int U = RQ == 4 || D == 128 ? 2 : 4;  // keys per quad requested together
    for (int j0 = 0; j0 <= last; j0 += 64 * U) {
        QuadRow<D> k[U];
#pragma unroll
        for (int t = 0; t < U; ++t)
            k[t].load(kbase + (int64_t)min(j0 + t * 64 + kk, last) * g.ks[2], part);
        __builtin_amdgcn_sched_barrier(0);  // (all requested before the first is used)
#pragma unroll
        for (int t = 0; t < U; ++t) {
            float w[RQ];
#pragma unroll
            for (int r = 0; r < RQ; ++r) w[r] = quad_sum(q[r].dot(k[t]));
            float x;
            if constexpr (RQ == 4) x = pick4(w, part);
            else x = w[0];
            // (no branch around the quad's exchanges: its lanes may keep rows that end apart)
            const bool sees = j0 + t * 64 + kk <= my_i;
            const float tt = x * lam, mn = sees ? fmaxf(m, tt) : m, dt = sees ? tt - mn : 0.f;
            reref_stat(m, mn, s, u);
            const float e = sees ? exp2f(dt) : 0.f;
            s += e;
            u = fmaf(e, dt, u);
            m = mn;
        }
    }
    // over the keys of the wave (lanes with the same part), then over the waves
#pragma unroll
    for (int o = 4; o < 64; o <<= 1)
        merge_stat(m, s, u, __shfl_xor(m, o), __shfl_xor(s, o), __shfl_xor(u, o));
    if (lane < RQ) { s_m[wave][lane] = m; s_s[wave][lane] = s; s_u[wave][lane] = u; }
    __syncthreads();
    const int rho = rho0 + tid;
    if (tid < RQ && rho < g.R) {
        m = s_m[0][tid]; s = s_s[0][tid]; u = s_u[0][tid];
#pragma unroll
        for (int t = 1; t < 4; ++t) merge_stat(m, s, u, s_m[t][tid], s_s[t][tid], s_u[t][tid]);
        const float L = m + log2f(s);
        rowL[(int64_t)z * g.R + rho] = L;
        const int64_t o = ((int64_t)b * g.Hq + h * g.G + rm.head(rho)) * g.r + (rho % g.r);
        const float kLn2 = 0.69314718055994531f;
        if (lse_out) lse_out[o] = L * kLn2;
        if (ent_out) ent_out[o] = fmaxf(0.f, (log2f(s) - u / s) * kLn2);
    }
}

constexpr int kF32QRows = 64;  // query rows staged in LDS per step of pass 2

// KPL keys (1 or 4) per quad: 16 KPL keys per workgroup.
template <int D, int KPL>
__global__ __launch_bounds__(256) void f32_pass2_kernel(ScoreGeom g, const float *rowL,
                                                        const float *gamma,
                                                        const float *gblockmax, int n_vtiles,
                                                        float *scores) {
    constexpr int KEYS = 16 * KPL;
    const int z = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = lane & 3, kk = lane >> 2;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const RowMap rm{g.n, g.r, g.R,
                    g.rows ? g.rows + ((int64_t)b * g.Hq + (int64_t)h * g.G) * g.r : nullptr};
    const float *kbase = (const float *)g.k + b * g.ks[0] + h * g.ks[1];

    __shared__ __attribute__((aligned(16))) float s_q[kF32QRows][D];
    __shared__ float s_lam[kF32QRows], s_L[kF32QRows], s_acc[4][KEYS];
    __shared__ int s_pos[kF32QRows];

    const int j_lo = blockIdx.x * KEYS;        // smallest key of this workgroup
    const int j = j_lo + kk * KPL + (KPL == 4 ? part : 0);  // the key whose sum this lane keeps
    QuadRow<D> k[KPL];
#pragma unroll
    for (int t = 0; t < KPL; ++t)
        k[t].load(kbase + (int64_t)min(j_lo + kk * KPL + t, g.n - 1) * g.ks[2], part);
    // the prior of this workgroup's keys and the tiles' maxima travel with the keys
    float gm = 0.f, gam = 1.f;
    if (g.value_prior) {
        for (int t = lane; t < n_vtiles; t += 64) gm = fmaxf(gm, gblockmax[z * n_vtiles + t]);
        gam = gamma[(int64_t)z * g.n + min(j_lo + tid % KEYS, g.n - 1)];
    }

    float acc = 0.f;
    for (int r0 = 0; r0 < g.R; r0 += kF32QRows) {
        // rows of this step; skip steps whose rows all lie before the block's keys
        if (rm.max_pos(r0, r0 + kF32QRows) < j_lo) continue;
        const int rows = min(kF32QRows, g.R - r0);
        __syncthreads();
        for (int t = tid; t < rows * (D / 4); t += 256) {
            const int rr = t / (D / 4), c = t % (D / 4), rho = r0 + rr;
            *(f32x4 *)&s_q[rr][4 * c] =
                *(const f32x4 *)((const float *)g.q + b * g.qs[0] +
                                 (int64_t)(h * g.G + rm.head(rho)) * g.qs[1] +
                                 (int64_t)rm.pos(rho) * g.qs[2] + 4 * c);
        }
        if (tid < rows) {
            const int rho = r0 + tid, i = rm.pos(rho);
            s_pos[tid] = i;
            s_lam[tid] = row_scale_log2(g.scale_mode, g.fixed_scale, g.lambda_floor, i + 1,
                                        g.budget, g.d);
            s_L[tid] = rowL[(int64_t)z * g.R + rho];
        }
        __syncthreads();
#pragma unroll 2
        for (int rr = wave; rr < rows; rr += 4) {
            QuadRow<D> q;
            q.load(s_q[rr], part);
            float w[KPL];
#pragma unroll
            for (int t = 0; t < KPL; ++t) w[t] = quad_sum(q.dot(k[t]));
            float x;
            if constexpr (KPL == 4) x = pick4(w, part);
            else x = w[0];
            const float p = exp2f(fmaf(x, s_lam[rr], -s_L[rr]));
            acc += (j <= s_pos[rr]) ? p : 0.f;
        }
    }
    // over the waves; one thread per key writes
    if (KPL == 4) s_acc[wave][lane % KEYS] = acc;
    else if (part == 0) s_acc[wave][kk % KEYS] = acc;
    __syncthreads();
    gm = wave_max(gm);  // (every lane takes part)
    if (tid < KEYS && j_lo + tid < g.n) {
        float out = (s_acc[0][tid] + s_acc[1][tid]) + (s_acc[2][tid] + s_acc[3][tid]);
        if (g.value_prior) {
            out = gm > 0.f ? out * (gam / gm) : out;  // all-zero values: no prior
        }
        scores[(int64_t)z * g.n + j_lo + tid] = out;
    }
}

// ---- larger problems: the dots on the matrix core (f32_tile.h) ----
// Pass 1: a workgroup takes 32 rows and one of nparts key ranges, its waves 32 keys in turn; each
// row's maximum and sum over the range go to partial[problem][row block][range][row] (as a pair:
// pass 2 forms exp2(t - maximum) / sum, free of the rounding of a log-sum-exp2 of some tens).
// Workgroups past row_blocks * nparts take the value tiles.
template <int D>
__global__ __launch_bounds__(256, 2) void f32_mfma_pass1_kernel(ScoreGeom g, int row_blocks, int nparts,
                                                                int n_vtiles, float *gamma,
                                                                float *gblockmax, float2 *partial) {
    const int z = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    if ((int)blockIdx.x >= row_blocks * nparts) {  // (workgroup-uniform)
        value_prior_tile<4>(g, z, (int)blockIdx.x - row_blocks * nparts, n_vtiles, gamma, gblockmax, tid);
        return;
    }
    const int b = z / g.Hkv, h = z % g.Hkv, rb = blockIdx.x / nparts, part = blockIdx.x % nparts;
    const int rho = rb * 32 + (lane & 31);
    const RowMap rm{g.n, g.r, g.R,
                    g.rows ? g.rows + ((int64_t)b * g.Hq + (int64_t)h * g.G) * g.r : nullptr};
    const float *kbase = (const float *)g.k + b * g.ks[0] + h * g.ks[1];
    __shared__ __attribute__((aligned(16))) float s_q[32 * f32_ld(D)];
    __shared__ float s_m[4][32], s_s[4][32];
    F32QueryBlock<D, 256> qb;
    qb.request(g, rm, b, h, rb * 32, tid);
    const int pos = rm.pos(rho);  // -1 past the last row
    const int end = rm.max_pos(rb * 32, rb * 32 + 32) + 1, steps = (end + 127) / 128;
    const int k0 = (int)((int64_t)part * steps / nparts) * 128;
    const int k1 = min(end, (int)((int64_t)(part + 1) * steps / nparts) * 128);
    const float lam = row_scale_log2(g.scale_mode, g.fixed_scale, g.lambda_floor, max(pos, 0) + 1,
                                     g.budget, g.d);
    f32x4 a[D / 8];
    f32_load_keys<D>(kbase, g.ks[2], k0 + wave * 32, max(k1, 1) - 1, lane, a);
    qb.commit(tid, s_q);
    __syncthreads();
    const float *sq = s_q + (lane & 31) * f32_ld(D) + 4 * (lane >> 5);
    float m = -INFINITY, s = 0.f;
    for (int kb = k0 + wave * 32; kb < k1; kb += 128) {
        if (kb >= k0 + 128) f32_load_keys<D>(kbase, g.ks[2], kb, k1 - 1, lane, a);
        f32x16 t = f32_block_dots<D>(a, sq);
        float mx = m;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = acc_key(kb, 0, v, lane);
            t[v] = key <= pos && key < k1 ? t[v] * lam : -INFINITY;
            mx = fmaxf(mx, t[v]);
        }
        const float mref = mx == -INFINITY ? 0.f : mx;
#pragma unroll
        for (int v = 0; v < 16; ++v) t[v] = exp2f(t[v] - mref);
#pragma unroll
        for (int o = 8; o; o >>= 1)
#pragma unroll
            for (int v = 0; v < o; ++v) t[v] += t[v + o];
        s = fmaf(s, exp2f(m - mref), t[0]);
        m = mx;
    }
    float u = 0.f;
    merge_stat(m, s, u, __shfl_xor(m, 32), __shfl_xor(s, 32), 0.f);
    if (lane < 32) { s_m[wave][lane] = m; s_s[wave][lane] = s; }
    __syncthreads();
    if (tid < 32) {
        m = s_m[0][tid]; s = s_s[0][tid];
#pragma unroll
        for (int w = 1; w < 4; ++w) merge_stat(m, s, u, s_m[w][tid], s_s[w][tid], 0.f);
        // (-inf, 0 for a row that saw no key of the range)
        partial[(((int64_t)z * row_blocks + rb) * nparts + part) * 32 + tid] = make_float2(m, s);
    }
}

// Pass 2: a workgroup takes 4 / wpk blocks of 32 keys; wpk waves share one, the blocks of query rows
// dealt among them.  `rowL`, when not null, holds the rows' normalisers ([problem][row]).
template <int D>
__global__ __launch_bounds__(256, 2) void f32_mfma_pass2_kernel(ScoreGeom g, int row_blocks, int nparts,
                                                                int wpk, const float2 *partial,
                                                                const float *rowL, const float *gamma,
                                                                const float *gblockmax, int n_vtiles,
                                                                float *scores) {
    extern __shared__ __attribute__((aligned(16))) float s_q[];  // a query block per wave
    __shared__ float s_acc[4][32];
    const int z = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int b = z / g.Hkv, h = z % g.Hkv, kw = 4 / wpk;
    const RowMap rm{g.n, g.r, g.R,
                    g.rows ? g.rows + ((int64_t)b * g.Hq + (int64_t)h * g.G) * g.r : nullptr};
    const float *kbase = (const float *)g.k + b * g.ks[0] + h * g.ks[1];
    const int kb = ((int)blockIdx.x * kw + wave / wpk) * 32;
    f32x4 a[D / 8];
    f32_load_keys<D>(kbase, g.ks[2], kb, g.n - 1, lane, a);
    float gm = 0.f;
    if (g.value_prior)
        for (int t = lane; t < n_vtiles; t += 64) gm = fmaxf(gm, gblockmax[z * n_vtiles + t]);
    gm = wave_max(gm);
    float *sq_wave = s_q + wave * 32 * f32_ld(D);
    const float *sq = sq_wave + (lane & 31) * f32_ld(D) + 4 * (lane >> 5);
    f32x16 col;
#pragma unroll
    for (int v = 0; v < 16; ++v) col[v] = 0.f;
    for (int rb = kb < g.n ? wave % wpk : row_blocks; rb < row_blocks; rb += wpk) {
        if (rm.max_pos(rb * 32, rb * 32 + 32) < kb) continue;  // no row of the block sees these keys
        F32QueryBlock<D, 64> qb;
        qb.request(g, rm, b, h, rb * 32, lane);
        const int rho = rb * 32 + (lane & 31), pos = rm.pos(rho);
        float M, inv = 1.f;  // the row's reference and the reciprocal of its sum
        if (rowL) {
            M = rowL[(int64_t)z * g.R + min(rho, g.R - 1)];
        } else {
            const float2 *pl = partial + ((int64_t)z * row_blocks + rb) * nparts * 32 + (lane & 31);
            M = pl[0].x;
            float sum = pl[0].y;
            for (int c = 1; c < nparts; ++c) {
                const float2 e = pl[c * 32];
                const float mn = fmaxf(M, e.x);
                const float mref = mn == -INFINITY ? 0.f : mn;  // (ranges behind the row's last key)
                sum = fmaf(sum, exp2f(M - mref), e.y * exp2f(e.x - mref));
                M = mn;
            }
            inv = 1.f / sum;
        }
        const float lam = row_scale_log2(g.scale_mode, g.fixed_scale, g.lambda_floor, max(pos, 0) + 1,
                                         g.budget, g.d);
        // (the wave's own copy: no other wave reads it, and a wave's LDS accesses stay in order)
        qb.commit(lane, sq_wave);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        const f32x16 t = f32_block_dots<D>(a, sq);
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = exp2f(fmaf(t[v], lam, -M)) * inv;
            col[v] += acc_key(kb, 0, v, lane) <= pos ? p : 0.f;
        }
    }
    const float tot = fold16_over32(col, lane);
    const int my_v = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
    if ((lane & 1) == 0) s_acc[wave][acc_key(0, 0, my_v, lane)] = tot;
    __syncthreads();
    const int j = (int)blockIdx.x * kw * 32 + tid;
    if (tid < kw * 32 && j < g.n) {
        float out = 0.f;
        for (int w = 0; w < wpk; ++w) out += s_acc[tid / 32 * wpk + w][tid % 32];
        if (g.value_prior) out = gm > 0.f ? out * (gamma[(int64_t)z * g.n + j] / gm) : out;  // all-zero values: no prior
        scores[(int64_t)z * g.n + j] = out;
    }
}

// Four rows / keys per quad once the small variants would put more than about eight workgroups
// on every CU: from there the vector ALU bounds the passes and the spare factor four counts.
constexpr int64_t kF32ManyWgs = 2048;

template <int D>
static void launch_pass1(const ScoreGeom &g, const PrefillPlan &pl, void *ws, bool prior, float *lse,
                         float *entropy, hipStream_t st) {
    char *w = (char *)ws;
    float *gamma = (float *)(w + pl.off_gamma), *gbm = (float *)(w + pl.off_gblockmax);
    float *rowL = (float *)(w + pl.off_rowL);
    const int vt = prior ? pl.n_vtiles : 0;
    if ((int64_t)g.R * pl.Z >= kF32ManyWgs) {
        const int rb = (g.R + 3) / 4;
        hipLaunchKernelGGL((f32_pass1_kernel<D, 4>), dim3(rb + vt, pl.Z), dim3(256), 0, st, g, rb,
                           pl.n_vtiles, gamma, gbm, rowL, lse, entropy);
    } else {
        hipLaunchKernelGGL((f32_pass1_kernel<D, 1>), dim3(g.R + vt, pl.Z), dim3(256), 0, st, g, g.R,
                           pl.n_vtiles, gamma, gbm, rowL, lse, entropy);
    }
}

template <int D>
static void launch_pass2(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores,
                         hipStream_t st) {
    char *w = (char *)ws;
    const float *rowL = (float *)(w + pl.off_rowL);
    const float *gamma = (const float *)(w + pl.off_gamma);
    const float *gbm = (const float *)(w + pl.off_gblockmax);
    if ((int64_t)((g.n + 15) / 16) * pl.Z >= kF32ManyWgs)
        hipLaunchKernelGGL((f32_pass2_kernel<D, 4>), dim3((g.n + 63) / 64, pl.Z), dim3(256), 0, st,
                           g, rowL, gamma, gbm, pl.n_vtiles, scores);
    else
        hipLaunchKernelGGL((f32_pass2_kernel<D, 1>), dim3((g.n + 15) / 16, pl.Z), dim3(256), 0, st,
                           g, rowL, gamma, gbm, pl.n_vtiles, scores);
}

template <int D>
static hipError_t launch_mfma(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores,
                              hipStream_t st, hipEvent_t mid, bool have_lse) {
    char *w = (char *)ws;
    float *gamma = (float *)(w + pl.off_gamma), *gbm = (float *)(w + pl.off_gblockmax);
    float2 *partial = (float2 *)(w + pl.off_partial);
    constexpr size_t smem = (size_t)4 * 32 * f32_ld(D) * sizeof(float);
    static DeviceOnce once;
    const hipError_t ea = device_once(once, [] {
        return hipFuncSetAttribute((const void *)f32_mfma_pass2_kernel<D>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    });
    if (ea != hipSuccess) return ea;
    const int rb = (g.R + 31) / 32;
    if (!have_lse) {
        hipLaunchKernelGGL(f32_mfma_pass1_kernel<D>, dim3(rb * pl.nchunks + (g.value_prior ? pl.n_vtiles : 0), pl.Z),
                           dim3(256), 0, st, g, rb, pl.nchunks, pl.n_vtiles, gamma, gbm, partial);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (mid) (void)hipEventRecord(mid, st);
    const int wpk = rb >= 4 ? 4 : rb >= 2 ? 2 : 1, keys = 4 / wpk * 32;
    hipLaunchKernelGGL(f32_mfma_pass2_kernel<D>, dim3((g.n + keys - 1) / keys, pl.Z), dim3(256), smem, st, g,
                       rb, pl.nchunks, wpk, partial, have_lse ? (const float *)(w + pl.off_rowL) : nullptr,
                       gamma, gbm, pl.n_vtiles, scores);
    return hipGetLastError();
}

hipError_t launch_score_f32(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores,
                            hipStream_t st, hipEvent_t mid, bool have_lse) {
    if (pl.f32_mfma)
        return g.d == 64 ? launch_mfma<64>(g, pl, ws, scores, st, mid, have_lse)
                         : launch_mfma<128>(g, pl, ws, scores, st, mid, have_lse);
    // (with the caller's row normalisers the prior comes from launch_value_prior)
    if (!have_lse) {
        if (g.d == 64) launch_pass1<64>(g, pl, ws, g.value_prior, nullptr, nullptr, st);
        else launch_pass1<128>(g, pl, ws, g.value_prior, nullptr, nullptr, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (mid) (void)hipEventRecord(mid, st);
    if (g.d == 64) launch_pass2<64>(g, pl, ws, scores, st);
    else launch_pass2<128>(g, pl, ws, scores, st);
    return hipGetLastError();
}

hipError_t launch_row_stats_f32(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *lse,
                                float *entropy, hipStream_t st) {
    if (g.d == 64) launch_pass1<64>(g, pl, ws, false, lse, entropy, st);
    else launch_pass1<128>(g, pl, ws, false, lse, entropy, st);
    return hipGetLastError();
}

}  // namespace aha
