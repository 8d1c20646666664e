// bf16 eviction scores of up to 256 rows in two launches on the gfx950 matrix cores (Sec. 4.1 - 4.3;
// Alg. 1 Prefill), and the row statistics' output of any number.  Two passes, both recomputing tiles of K Q^T with
// v_mfma_f32_32x32x16_bf16 (keys on M, queries on N); the n x n probability
// matrix never exists in memory.
//
//   pass 1: per observed query row, max and sum of exp2 over its keys
//           (log2 domain, scale applied in fp32 after the MFMA);
//   pass 2: per key, sum over the observed rows of exp2(t - L_row), times the
//           value prior.
//
// With keys on M the 32x32 accumulator gives every lane ONE query column
// (lane % 32) and 16 key rows, so the per-row scale, maximum and log-sum-exp
// are per-lane scalars in both passes; pass 1 reduces over keys in-lane, and
// pass 2 accumulates over query blocks in-lane and folds the 32 lanes of a
// half-wave once per key block.
//
// Work split: a workgroup keeps one tile of query rows (up to 256 flattened
// rows of a KV head's query group) in LDS as the B operand; each of its four
// waves owns 64-key blocks whose A fragments it loads straight from global
// memory into registers (each K byte is fetched once per tile), so waves run
// independently between the tile barriers; the A fragments are double-buffered so
// that the next key block is in flight while the current one multiplies.
#include "score_block.h"

namespace aha {

// ---------------------------------------------------------------- pass 1 --
constexpr int kNoPrior = 0, kPriorFold = 1;  // value prior inside pass 1 (below)

// The prior of a key range formed AFTER the main loop (see bf16_pass1_kernel): value rows of the keys [kbeg, kend) of problem z are streamed in a phase
// of their own: nu = ||V||^2 of the range and its pooling halo into
// LDS, gamma = edge-truncated mean over the pool window, written to `gamma`; returns (in
// every thread) the largest gamma of the range.  Works through the range in pieces of
// kPriorPiece keys so that the LDS it borrows (the query tile's, free at that time) stays
// small.  Ends with a barrier: the LDS may be reused at once.
// value rows a lane requests before it uses the first (9 and 33 measured slower here)
constexpr int kPriorLoads = 17;
constexpr size_t kPriorTailSmem = (kPriorPiece + 256 + 4) * sizeof(float);
__device__ __forceinline__ float value_prior_of_range(const ScoreGeom &g, int b, int h, int z,
                                                      int kbeg, int kend, float *s_nu,
                                                      float *gamma, int tid) {
    const char *vbase = (const char *)g.v + (int64_t)2 * (b * g.vs[0] + h * g.vs[1]);
    const int half = (g.pool - 1) / 2;
    float *s_max = s_nu + kPriorPiece + 256;
    float gmax = 0.f;
    for (int t0 = kbeg; t0 < kend; t0 += kPriorPiece) {
        const int t1 = min(kend, t0 + kPriorPiece);
        const int lo = max(0, t0 - half), hi = min(g.n, t1 + half);  // hi exclusive
        value_norms_to_lds<2, kPriorLoads>(vbase, g.vs[2], g.d, lo, hi, s_nu, tid);
        __syncthreads();
        for (int j = t0 + tid; j < t1; j += 256) {
            const int a = max(0, j - half), e = min(g.n - 1, j + half);
            float s = 0.f;
            for (int t = a; t <= e; ++t) s += s_nu[t - lo];
            const float gam = s / (float)(e - a + 1);
            gamma[(int64_t)z * g.n + j] = gam;
            gmax = fmaxf(gmax, gam);
        }
        __syncthreads();
    }
    gmax = wave_max(gmax);
    if ((tid & 63) == 0) s_max[tid >> 6] = gmax;
    __syncthreads();
    gmax = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    __syncthreads();
    return gmax;
}

// PRIOR (windowed scores of up to four row blocks with the value prior, the sizes that score_window.hip
// leaves): the workgroup also forms the prior of its key range and leaves the range's maximum in
// gblockmax[z * nparts + part]: one launch less than a value-prior kernel of its own.
// The steps are too short to hide value rows under (the key prefetch would have half a
// step to arrive), and the kernel is bound by the key stream: the value rows are streamed
// in a phase of their own after the statistics (16K tokens x 128 heads x 64 rows: 183 us
// against 215 us interleaved).
// ENT: the chunk's mean scaled logit under its own probabilities, E_c[t] = m + u / s, is
// written to `partial_mean` beside the chunk's log2-sum-exp2; row_stats_merge_kernel turns the
// chunks of a row into its entropy.
template <int D, int NB, bool ENT, bool ROWS = false, int PRIOR = kNoPrior>
__global__ __launch_bounds__(256, 2) void bf16_pass1_kernel(ScoreGeom g, int n_qtiles, int nparts,
                                                            int total_wgs, float *partial,
                                                            float *partial_mean, float *gamma,
                                                            float *gblockmax) {
    using S = TileSmem<D, NB>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __bf16 *sQ = (__bf16 *)smem;
    float *sLam = (float *)(smem + S::q_bytes);
    int *sPos = (int *)(sLam + S::ROWS);
    int *sBlk = sPos + 2 * S::ROWS;
    float4 *sRed = (float4 *)smem;  // reuses the query tile after the main loop

    // logical workgroup index -> (part, tile pair, problem)
    const int wg = logical_wg_index(total_wgs, n_qtiles > 1);
    if (wg >= total_wgs) return;
    const int npairs = (n_qtiles + 1) / 2;
    const int part = wg % nparts, pair = (wg / nparts) % npairs, z = wg / (nparts * npairs);
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const RowMap rm{g.n, g.r, g.R,
                    ROWS ? g.rows + ((int64_t)b * g.Hq + (int64_t)h * g.G) * g.r : nullptr};
    const __bf16 *kbase = (const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1];

    for (int seg = 0; seg < 2; ++seg) {
        const Segment sg = pair_segment(rm, S::ROWS, n_qtiles, pair, part, nparts, seg);
        if (sg.qt < 0) break;
        const int qt = sg.qt, rho0 = qt * S::ROWS;
        const int64_t my_off = ((int64_t)(z * n_qtiles + qt) * nparts + part) * S::ROWS;
        float *my_partial = partial + my_off;
        const int key_begin = sg.kbeg, key_end = sg.kend;
        if (key_begin >= key_end) {
            // none of this part's steps fall on this tile: leave neutral statistics
            if (tid < S::ROWS) {
                my_partial[tid] = -INFINITY;
                if (ENT) partial_mean[my_off + tid] = 0.f;
            }
            if (PRIOR != kNoPrior && tid == 0) gblockmax[z * nparts + part] = 0.f;  // no keys, no prior
            continue;
        }
        if (seg) __syncthreads();  // the previous tile (and its reduction buffer) is done with
        // The query tile (served by the L2 after its first touch) is requested first and the
        // first key block (from HBM, behind every other workgroup's) right after it: loads
        // return in order, so the tile is in LDS and the barrier passed while the keys are
        // still on their way.
        // The first tile of a pair walks its 256-key steps upwards, the partner downwards.
        // Step i of the pair's common clock is then key step i for every workgroup still on
        // its first tile and key step (steps of a full sequence) - i for every workgroup on
        // its partner tile, whatever the pair: the workgroups of a problem, which share an
        // XCD, read the same two key blocks at any time and find them in the L2.
        const int nsteps = (key_end - key_begin + kWgKeys - 1) / kWgKeys;
        const int kdir = seg ? -kWgKeys : kWgKeys;
        const int k_at0 = (seg ? key_begin + (nsteps - 1) * kWgKeys : key_begin) + wave * kWaveKeys;
        // this wave's key block of step i; past the last step: rows clamped to the range's end
        auto kb_of = [&](int i) { return i < nsteps ? k_at0 + i * kdir : key_end; };
        bf16x8 a0[kMB][D / 16], a1[kMB][D / 16];  // the next key block loads while one multiplies
        {
            // (the thread index goes through an opaque move: the set-up's addresses are then
            // recomputed per tile instead of being kept across the main loop, where they
            // would be spilled and their reload would wait for every load in flight)
            int tid_s = tid;
            asm volatile("" : "+v"(tid_s));
            QTileRegs<D, NB> qt_regs;
            q_tile_request<D, NB, ROWS>(g, b, h, rho0, tid_s, qt_regs);
            const float lam_req = q_tile_scale<D, NB>(g, rm, rho0, tid_s);
            __builtin_amdgcn_sched_barrier(0);  // the key block is requested last
            load_a<D>(kbase, g.ks[2], kb_of(0), key_end, lane, a0);
            q_tile_meta<D, NB>(g, rm, rho0, tid_s, lam_req, sLam, sPos, sBlk);
            q_tile_commit<D, NB>(qt_regs, tid_s, sQ);
        }
        __syncthreads();

        float lam[NB], m[NB], s[NB], u[ENT ? NB : 1];
        int pos[NB], bmax[NB], bmin[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            lam[nb] = sLam[nb * 32 + (lane & 31)];
            pos[nb] = sPos[nb * 32 + (lane & 31)];
            bmax[nb] = uniform(sBlk[nb]);
            bmin[nb] = uniform(sBlk[NB + nb]);
            m[nb] = -INFINITY;
            s[nb] = 0.f;
            u[ENT ? nb : 0] = 0.f;
        }

        const int tile_min = ROWS ? tile_min_pos<NB>(sBlk) : rm.min_pos(rho0, rho0 + S::ROWS);
        // blocks [nb0, nb1) of the tile against the 64 keys at kb
        auto blocks = [&](const bf16x8 (&a)[kMB][D / 16], int kb, int nb0, int nb1) {
            if (kb >= key_end) return;  // (a wave past the range's ragged end)
            if (kb + kWaveKeys - 1 <= tile_min) {
                // every row of the tile sees all 64 keys: no masks, no skipped blocks
                bf16x8 qf = query_fragment<D, NB>(sQ, nb0, 0, lane);
#pragma unroll
                for (int nb = nb0; nb < nb1; ++nb) {
                    f32x16 acc[kMB];
                    mma_block_stream<D, NB>(a, sQ, nb, nb + 1 < nb1 ? nb + 1 : nb0, lane, qf, acc);
                    stats_update<false, ENT>(acc, lam[nb], 0, kb, lane, m[nb], s[nb], u[ENT ? nb : 0]);
                }
                return;
            }
#pragma unroll
            for (int nb = nb0; nb < nb1; ++nb) {
                if (bmax[nb] < kb) continue;  // nothing of this block sees these keys
                f32x16 acc[kMB];
                mma_block<D, NB>(a, sQ, nb, lane, acc);
                if (kb + kWaveKeys - 1 > bmin[nb])
                    stats_update<true, ENT>(acc, lam[nb], pos[nb], kb, lane, m[nb], s[nb], u[ENT ? nb : 0]);
                else
                    stats_update<false, ENT>(acc, lam[nb], pos[nb], kb, lane, m[nb], s[nb], u[ENT ? nb : 0]);
            }
        };
        // One step: the key block in `a` against the whole tile, while `nx` receives the next
        // key block.  The loads are issued unconditionally (past the range they re-read
        // clamped rows that are never used): behind a branch the compiler can no longer tell
        // how many loads are in flight and would wait for the prefetch itself.
        auto step = [&](const bf16x8 (&a)[kMB][D / 16], bf16x8 (&nx)[kMB][D / 16], int kb,
                        int kb_next) {
            load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            blocks(a, kb, 0, NB);
        };
        for (int i = 0; i < nsteps; i += 2) {
            step(a0, a1, kb_of(i), kb_of(i + 1));
            if (i + 1 >= nsteps) break;
            step(a1, a0, kb_of(i + 1), kb_of(i + 2));
        }
        // fold the two half-waves (same query column, different key rows); a statistic
        // (m, s, u) re-referenced to a maximum M >= m is (M, s f, (u + (m - M) s) f), f = 2^(m - M)
        auto reref = [](float m_, float mref, float &s_, float &u_) {
            const float f = fast_exp2(m_ - mref);
            if (ENT) u_ = (u_ + (m_ == -INFINITY ? 0.f : m_ - mref) * s_) * f;
            s_ *= f;
        };
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float m2 = __shfl_xor(m[nb], 32), s2 = __shfl_xor(s[nb], 32);
            float u1 = u[ENT ? nb : 0], u2 = ENT ? __shfl_xor(u1, 32) : 0.f;
            const float mn = fmaxf(m[nb], m2);
            const float mref = mn == -INFINITY ? 0.f : mn;
            reref(m[nb], mref, s[nb], u1);
            reref(m2, mref, s2, u2);
            s[nb] += s2;
            u[ENT ? nb : 0] = u1 + u2;
            m[nb] = mn;
        }
        __syncthreads();  // everyone is done reading the query tile
        if (lane < 32) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                sRed[wave * S::ROWS + nb * 32 + lane] =
                    make_float4(m[nb], s[nb], u[ENT ? nb : 0], 0.f);
        }
        __syncthreads();
        if (tid < S::ROWS) {
            float M = -INFINITY;
#pragma unroll
            for (int w = 0; w < 4; ++w) M = fmaxf(M, sRed[w * S::ROWS + tid].x);
            const float mref = M == -INFINITY ? 0.f : M;
            float sum = 0.f, mom = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float4 e = sRed[w * S::ROWS + tid];
                float sw = e.y, uw = e.z;
                reref(e.x, mref, sw, uw);
                sum += sw;
                mom += uw;
            }
            my_partial[tid] = M + log2f(sum);  // -inf for a row that saw no key
            if (ENT) partial_mean[my_off + tid] = sum > 0.f ? mref + mom / sum : 0.f;
        }
        if constexpr (PRIOR == kPriorFold) {
            __syncthreads();  // the reduction buffer is done with
            const float gm = value_prior_of_range(g, b, h, z, key_begin, key_end, (float *)smem,
                                                  gamma, tid);
            if (tid == 0) gblockmax[z * nparts + part] = gm;
        }
    }
}

// ---------------------------------------------------------------- pass 2 --
// All observed rows fit one query tile, which is loaded once; the workgroup walks over several 256-key steps and the A
// fragments of the next step load while the current one multiplies; every score is written exactly once.
template <int D, int NB, bool ROWS = false>
__global__ __launch_bounds__(256, 2) void bf16_pass2_kernel(ScoreGeom g, int total_wgs, int wg_keys, int nchunks,
                                                            const float *partial,
                                                            const float *gamma,
                                                            const float *gblockmax,
                                                            int n_vtiles, float *scores) {
    using S = TileSmem<D, NB>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __bf16 *sQ = (__bf16 *)smem;
    float *sLam = (float *)(smem + S::q_bytes);
    int *sPos = (int *)(sLam + S::ROWS);
    float *sL = (float *)(sPos + S::ROWS);
    int *sBlk = (int *)(sL + S::ROWS);
    __shared__ float s_gmax[4];

    // logical workgroup index -> (key range, problem)
    const int wg = logical_wg_index(total_wgs, false);
    if (wg >= total_wgs) return;
    const int per_problem = total_wgs / (g.batch * g.Hkv);
    const int z = wg / per_problem, wg_in_z = wg % per_problem;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const RowMap rm{g.n, g.r, g.R,
                    ROWS ? g.rows + ((int64_t)b * g.Hq + (int64_t)h * g.G) * g.r : nullptr};
    const __bf16 *kbase = (const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1];
    const int key_begin = wg_in_z * wg_keys, key_end = min(g.n, key_begin + wg_keys);

    bf16x8 a0[kMB][D / 16];
    // (the windowed pass walks its key range from the last step to the first)
    const int last_step = key_begin + (key_end - key_begin - 1) / kWgKeys * kWgKeys;

    // this thread's share of the value prior's per-tile maxima (requested here, reduced
    // during the first tile set-up)
    float gm = (g.value_prior && tid < n_vtiles) ? gblockmax[z * n_vtiles + tid] : 0.f;

    // query tile -> LDS, with the log-sum-exp of its rows folded from pass 1's chunks
    static_assert(S::ROWS <= 256, "one thread folds the statistics of one tile row");
    {
        // tile rows, chunk statistics and scales are requested together, then used
        QTileRegs<D, NB> qt_regs;
        constexpr int kChunkBatch = 64;
        float ch[kChunkBatch];
        const bool row_ok = tid < S::ROWS && tid < g.R;
        // (threads without a row of their own read row 0's statistics and drop them)
        const float *psrc = partial + (int64_t)z * nchunks * S::ROWS + (tid < S::ROWS ? tid : 0);
        q_tile_request<D, NB, ROWS>(g, b, h, 0, tid, qt_regs);
        chunk_request(psrc, S::ROWS, 0, nchunks, ch);
        const float lam_req = q_tile_scale<D, NB>(g, rm, 0, tid);
        __builtin_amdgcn_sched_barrier(0);  // the key block is requested last
        // (right behind the tile's own, L2-served loads, so that those are not queued behind keys from HBM)
        load_a<D>(kbase, g.ks[2], last_step + wave * kWaveKeys, key_end, lane, a0);
        q_tile_meta<D, NB>(g, rm, 0, tid, lam_req, sLam, sPos, sBlk);
        if (g.value_prior) {
            for (int t = tid + 256; t < n_vtiles; t += 256) gm = fmaxf(gm, gblockmax[z * n_vtiles + t]);
            gm = wave_max(gm);
            if (lane == 0) s_gmax[wave] = gm;
        }
        float M = -INFINITY, sum = 0.f;
        chunk_merge(ch, nchunks, M, sum);
        for (int c0 = kChunkBatch; c0 < nchunks; c0 += kChunkBatch) {
            chunk_request(psrc, S::ROWS, c0, nchunks, ch);
            chunk_merge(ch, nchunks - c0, M, sum);
        }
        if (tid < S::ROWS) sL[tid] = row_ok ? M + log2f(sum) : INFINITY;
        q_tile_commit<D, NB>(qt_regs, tid, sQ);
    }
    __syncthreads();
    const int tile_min = ROWS ? tile_min_pos<NB>(sBlk) : rm.min_pos(0, S::ROWS);  // smallest position among the tile's rows
    float lamr[NB], Lr[NB];  // scale and log-sum-exp of this lane's query column, per block
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        lamr[nb] = sLam[nb * 32 + (lane & 31)];
        Lr[nb] = sL[nb * 32 + (lane & 31)];
    }
    // this wave's 64 keys (A fragments a) against the query tile in LDS
    auto tile_times_keys = [&](const bf16x8 (&a)[kMB][D / 16], int kb, f32x16 (&col)[kMB]) {
        if (kb + kWaveKeys - 1 <= tile_min) {
            // all rows of the tile see all 64 keys: no masks, no skipped blocks
            bf16x8 qf = query_fragment<D, NB>(sQ, 0, 0, lane);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                f32x16 acc[kMB];
                mma_block_stream<D, NB>(a, sQ, nb, nb + 1 < NB ? nb + 1 : 0, lane, qf, acc);
                colsum_update<false>(acc, lamr[nb], Lr[nb], 0, kb, lane, col);
            }
            return;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if (uniform(sBlk[nb]) < kb) continue;
            f32x16 acc[kMB];
            mma_block<D, NB>(a, sQ, nb, lane, acc);
            const int pos = sPos[nb * 32 + (lane & 31)];
            if (kb + kWaveKeys - 1 > uniform(sBlk[NB + nb]))
                colsum_update<true>(acc, lamr[nb], Lr[nb], pos, kb, lane, col);
            else
                colsum_update<false>(acc, lamr[nb], Lr[nb], pos, kb, lane, col);
        }
    };
    // The value-prior factors of the (up to two) scores this lane will write are requested
    // when a step starts, so that their latency is hidden behind the step's arithmetic.
    const int my_v = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 +
                     ((lane >> 1) & 1);
    auto request_gamma = [&](int kb, float (&gam)[kMB]) {
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) {
            const int j = acc_key(kb, mb, my_v, lane);
            gam[mb] = (g.value_prior && j < g.n) ? gamma[(int64_t)z * g.n + j] : 1.f;
        }
    };
    // fold the 32 lanes of each half-wave and write the 64 scores of this wave's keys
    auto write_scores = [&](f32x16 (&col)[kMB], int kb, const float (&gam)[kMB]) {
        float ginv = 1.f;
        if (g.value_prior)  // s_gmax was published by the barrier of the first tile load
            ginv = prior_inverse(fmaxf(fmaxf(s_gmax[0], s_gmax[1]), fmaxf(s_gmax[2], s_gmax[3])));
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) {
            const float tot = fold16_over32(col[mb], lane);
            const int j = acc_key(kb, mb, my_v, lane);
            if ((lane & 1) == 0 && j < g.n) scores[(int64_t)z * g.n + j] = tot * prior_factor(gam[mb], ginv);
        }
    };
    auto zero = [&](f32x16 (&col)[kMB]) {
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) col[mb][v] = 0.f;
    };

    bf16x8 a1[kMB][D / 16];
    auto step = [&](const bf16x8 (&a)[kMB][D / 16], int kb0) {
        const int kb = kb0 + wave * kWaveKeys;
        if (kb >= g.n) return;
        float gam[kMB];
        request_gamma(kb, gam);
        f32x16 col[kMB];
        zero(col);
        tile_times_keys(a, kb, col);
        write_scores(col, kb, gam);
    };
    // (unconditional prefetch, as in pass 1)
    for (int kb0 = last_step; kb0 >= key_begin; kb0 -= 2 * kWgKeys) {
        const int k1 = kb0 - kWgKeys, k2 = k1 - kWgKeys;
        // before the range: kb = key_end makes every row read the range's last one
        load_a<D>(kbase, g.ks[2], k1 >= key_begin ? k1 + wave * kWaveKeys : key_end, key_end, lane, a1);
        step(a0, kb0);
        if (k1 < key_begin) break;
        load_a<D>(kbase, g.ks[2], k2 >= key_begin ? k2 + wave * kWaveKeys : key_end, key_end, lane, a0);
        step(a1, k1);
    }
}

// Row statistics out (Sec. 4.2): from pass 1's per-chunk log2-sum-exp2 L_c and mean scaled
// logit E_c, the row's natural-log normaliser lse = ln 2 * L, L = log2 sum_c 2^L_c, and its
// entropy H = ln 2 * (L - sum_c 2^(L_c - L) E_c).  One thread per observed row.
__global__ __launch_bounds__(256) void row_stats_merge_kernel(ScoreGeom g, int rows_tile,
                                                              int n_qtiles, int nparts,
                                                              const float *partial,
                                                              const float *partial_mean,
                                                              float *lse, float *entropy) {
    const int z = blockIdx.y, rho = blockIdx.x * 256 + threadIdx.x;
    if (rho >= g.R) return;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int qt = rho / rows_tile, row = rho % rows_tile;
    const float *pl = partial + ((int64_t)(z * n_qtiles + qt) * nparts) * rows_tile + row;
    const float *pm = partial_mean + ((int64_t)(z * n_qtiles + qt) * nparts) * rows_tile + row;
    float M = -INFINITY;
    for (int c = 0; c < nparts; ++c) M = fmaxf(M, pl[(int64_t)c * rows_tile]);
    float sum = 0.f, mean = 0.f;
    for (int c = 0; c < nparts; ++c) {
        const float wgt = exp2f(pl[(int64_t)c * rows_tile] - M);  // 0 for a chunk without keys
        sum += wgt;
        mean = fmaf(wgt, pm[(int64_t)c * rows_tile], mean);
    }
    const float L = M + log2f(sum);
    const int gi = rho / g.r, ii = rho - gi * g.r;
    const int64_t o = ((int64_t)b * g.Hq + h * g.G + gi) * g.r + ii;
    const float kLn2 = 0.69314718055994531f;
    if (lse) lse[o] = L * kLn2;
    if (entropy) entropy[o] = fmaxf(0.f, (L - mean / sum) * kLn2);
}

// ---------------------------------------------------------------- launch --
template <int D, int NB>
static hipError_t launch_t(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores,
                           hipStream_t st, hipEvent_t mid, bool have_lse, bool fold_prior) {
    using S = TileSmem<D, NB>;
    static_assert(2 * S::bytes <= 160 * 1024, "two workgroups per CU");
    static_assert(S::bytes >= kPriorTailSmem, "the prior's own phase borrows the query tile's LDS");
    char *w = (char *)ws;
    float *partial = (float *)(w + pl.off_partial);
    float *gamma = (float *)(w + pl.off_gamma);
    float *gbm = (float *)(w + pl.off_gblockmax);
    constexpr int kFold = NB <= 4 ? kPriorFold : kNoPrior;  // (larger tiles: value_prior.hip)
    static DeviceOnce once;
    const hipError_t ea = device_once(once, [] {
        const void *kernels[6] = {(const void *)bf16_pass1_kernel<D, NB, false>,
                                  (const void *)bf16_pass1_kernel<D, NB, false, false, kFold>,
                                  (const void *)bf16_pass1_kernel<D, NB, true>,
                                  (const void *)bf16_pass1_kernel<D, NB, false, true>,
                                  (const void *)bf16_pass2_kernel<D, NB>,
                                  (const void *)bf16_pass2_kernel<D, NB, true>};
        for (const void *kf : kernels) {
            const hipError_t e = hipFuncSetAttribute(kf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::bytes);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
    if (ea != hipSuccess) return ea;
    // (part, tile pair, problem), part fastest
    const int64_t wgs1 = (int64_t)pl.nchunks * ((pl.n_qtiles + 1) / 2) * pl.Z;
    // windowed pass 2: (key range, problem)
    const int64_t wgs2 = (int64_t)((g.n + pl.p2_keys - 1) / pl.p2_keys) * pl.Z;
    // with the caller's row normalisers already in place (one "chunk" per row) pass 1 is skipped
    if (!have_lse) {
        if (g.rows)
            hipLaunchKernelGGL((bf16_pass1_kernel<D, NB, false, true>), xcd_grid(wgs1), dim3(256),
                               S::bytes, st, g, pl.n_qtiles, pl.nchunks, (int)wgs1, partial,
                               (float *)nullptr, (float *)nullptr, (float *)nullptr);
        else if (fold_prior)
            hipLaunchKernelGGL((bf16_pass1_kernel<D, NB, false, false, kFold>), xcd_grid(wgs1),
                               dim3(256), S::bytes, st, g, pl.n_qtiles, pl.nchunks, (int)wgs1,
                               partial, (float *)nullptr, gamma, gbm);
        else
            hipLaunchKernelGGL((bf16_pass1_kernel<D, NB, false>), xcd_grid(wgs1), dim3(256),
                               S::bytes, st, g, pl.n_qtiles, pl.nchunks, (int)wgs1, partial,
                               (float *)nullptr, (float *)nullptr, (float *)nullptr);
    }
    const int stat_chunks = have_lse ? 1 : pl.nchunks;
    // the prior's per-range maxima: one per key chunk when pass 1 formed it, else per tile
    const int n_maxima = fold_prior ? pl.nchunks : pl.n_vtiles;
    if (mid) (void)hipEventRecord(mid, st);
    if (g.rows)
        hipLaunchKernelGGL((bf16_pass2_kernel<D, NB, true>), xcd_grid(wgs2), dim3(256), S::bytes, st, g, (int)wgs2, pl.p2_keys,
                           stat_chunks, partial, gamma, gbm, n_maxima, scores);
    else
        hipLaunchKernelGGL((bf16_pass2_kernel<D, NB>), xcd_grid(wgs2), dim3(256), S::bytes, st, g, (int)wgs2, pl.p2_keys,
                           stat_chunks, partial, gamma, gbm, n_maxima, scores);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_d(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores,
                           hipStream_t st, hipEvent_t mid, bool have_lse, bool fold_prior) {
    switch (pl.NB) {
        case 1: return launch_t<D, 1>(g, pl, ws, scores, st, mid, have_lse, fold_prior);
        case 2: return launch_t<D, 2>(g, pl, ws, scores, st, mid, have_lse, fold_prior);
        case 4: return launch_t<D, 4>(g, pl, ws, scores, st, mid, have_lse, fold_prior);
        default: return launch_t<D, 8>(g, pl, ws, scores, st, mid, have_lse, fold_prior);
    }
}

template <int D, int NB>
static hipError_t launch_stats_t(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *lse,
                                 float *entropy, hipStream_t st) {
    using S = TileSmem<D, NB>;
    char *w = (char *)ws;
    float *partial = (float *)(w + pl.off_partial);
    float *partial_mean = (float *)(w + pl.off_partial_mean);
    static DeviceOnce once;
    const hipError_t ea = device_once(once, [] {
        return hipFuncSetAttribute((const void *)bf16_pass1_kernel<D, NB, true>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::bytes);
    });
    if (ea != hipSuccess) return ea;
    const int64_t wgs1 = (int64_t)pl.nchunks * ((pl.n_qtiles + 1) / 2) * pl.Z;
    hipLaunchKernelGGL((bf16_pass1_kernel<D, NB, true>), xcd_grid(wgs1), dim3(256), S::bytes, st,
                       g, pl.n_qtiles, pl.nchunks, (int)wgs1, partial, partial_mean,
                       (float *)nullptr, (float *)nullptr);
    const hipError_t e1 = hipGetLastError();
    if (e1 != hipSuccess) return e1;
    hipLaunchKernelGGL(row_stats_merge_kernel, dim3((g.R + 255) / 256, pl.Z), dim3(256), 0, st, g,
                       pl.qtile, pl.n_qtiles, pl.nchunks, partial, partial_mean, lse, entropy);
    return hipGetLastError();
}

hipError_t launch_row_stats_bf16(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *lse,
                                 float *entropy, hipStream_t st) {
#define AHA_STATS(DD)                                                         \
    switch (pl.NB) {                                                          \
        case 1: return launch_stats_t<DD, 1>(g, pl, ws, lse, entropy, st);    \
        case 2: return launch_stats_t<DD, 2>(g, pl, ws, lse, entropy, st);    \
        case 4: return launch_stats_t<DD, 4>(g, pl, ws, lse, entropy, st);    \
        default: return launch_stats_t<DD, 8>(g, pl, ws, lse, entropy, st);   \
    }
    if (g.d == 64) { AHA_STATS(64) }
    AHA_STATS(128)
#undef AHA_STATS
}

hipError_t launch_score_bf16(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores,
                             hipStream_t st, hipEvent_t mid, bool have_lse, bool fold_prior) {
    return g.d == 64 ? launch_d<64>(g, pl, ws, scores, st, mid, have_lse, fold_prior)
                     : launch_d<128>(g, pl, ws, scores, st, mid, have_lse, fold_prior);
}

}  // namespace aha
