// bf16 eviction scores of more query rows than one tile holds (full accumulation, where every row is
// an accumulator, above all): row statistics, then column sums, each forming K Q^T with
// v_mfma_f32_32x32x16_bf16.
//
// A workgroup of four waves owns a tile of query rows (up to 256) and walks ranges of keys.  A wave keeps
// its 32 NQ rows as fragments in registers for the whole tile; the keys go from global memory straight
// into LDS, 64 rows a step, once for the four waves and three steps ahead, and are read from there
// as fragments one block of 32 keys ahead.  What that leaves free of the register file holds a
// second block of products: while the matrix core forms one, the vector ALU takes the exponentials
// of the one before, in one instruction stream (pipelined()).
//
// The inner loop bounds both kernels: per element a multiply-add, an exponential (two slots of four cycles) and
// an addition, and each product of the matrix core keeps the vector ALU from issuing for some ten of its 32 cycles
// (a loop of these instructions alone: 693 cycles per 64 keys x 32 rows x 128 channels, vector work 521, matrix core 514).  The
// clock is what the power allows, 1.8 GHz in the kernels.  Against tiles of rows in LDS and keys in registers, two buffers
// of them, vector work after the products (us, both kernels, 8 KV heads and 32 query heads x 32768 rows 7960 -> 7600,
// 32 x 4096 167 -> 151, 16 x 2048 52.5 -> 35.8, 8 heads in 1 x 700 to 1000 rows 35 to 40 -> 26 to 29; d = 64, 32 x 4096 113 -> 108).
// Tried: two blocks of products in turn, 64 registers instead of 32 (spills); matrix products of 16 x 16 (less power per
// product, twice as many: 401 and 405 ns per block).
#include "key_stages.h"

namespace aha {

constexpr int kFullStages = 4;   // steps whose keys LDS holds
constexpr int kFullSetup = 2;    // a tile's set-up, in steps

template <int D, int NQ>
struct FullSmem {
    static constexpr int ROWS = 128 * NQ;
    static constexpr int stage = KeyRows<D>::bytes(kFullKeys);
    static constexpr size_t keys = (size_t)kFullStages * stage;
    // column sums: the waves' sums of a step's keys, gamma of the keys, the rows' values
    static constexpr int kGammaRing = 8;
    static constexpr size_t off_col = keys, off_gamma = off_col + 4 * kFullStages * kFullKeys * 4,
                            off_row = off_gamma + kGammaRing * kFullKeys * 4, bytes2 = off_row + 3 * ROWS * 4;
    static_assert(2 * bytes2 <= 160 * 1024, "two workgroups per CU");
};

// Key steps of a workgroup: those of its part of a pair of tiles' line (pair_segment), the first tile's
// upwards, the partner's downwards.
struct FullSteps {
    int qt0, qt1, beg0, beg1, n0, n1;  // tile (-1: none), first key and steps of both segments
    __device__ __forceinline__ FullSteps(const PlaceMap &rm, int rows, int T, int pair, int part, int nparts) {
        const Segment a = pair_segment(rm, rows, T, pair, part, nparts, 0, kFullKeys, kFullSetup);
        const Segment c = pair_segment(rm, rows, T, pair, part, nparts, 1, kFullKeys, kFullSetup);
        qt0 = uniform(a.qt);
        qt1 = uniform(c.qt);
        beg0 = uniform(a.kbeg);
        beg1 = uniform(c.kbeg);
        n0 = uniform(max(0, (a.kend - a.kbeg + kFullKeys - 1) / kFullKeys));
        n1 = c.qt < 0 ? 0 : uniform(max(0, (c.kend - c.kbeg + kFullKeys - 1) / kFullKeys));
    }
    __device__ __forceinline__ int total() const { return n0 + n1; }
    __device__ __forceinline__ int key(int i) const {
        return i < n0 ? beg0 + i * kFullKeys : beg1 + (n0 + n1 - 1 - i) * kFullKeys;
    }
    // of segment t's steps, those whose keys are all at or before position wmin; they come first in an upward segment, last
    // in a downward one
    __device__ __forceinline__ int unmasked(int t, int wmin) const {
        const int beg = t ? beg1 : beg0, n = t ? n1 : n0;
        return wmin < beg ? 0 : min((wmin + 1 - beg) / kFullKeys, n);
    }
};

// ---------------------------------------------------------------- row statistics --
template <int D, int NQ>
__global__ __launch_bounds__(256, 2) void full_stats_kernel(ScoreGeom g, int pr, int n_qtiles, int nparts, int total_wgs,
                                                            float *partial, float *zero) {
    using S = FullSmem<D, NQ>;
    constexpr int KS = D / 16, NI = KeyRequest<D, kFullKeys, 4>::NI, EP = 16 / KS;  // elements per portion
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int wg = logical_wg_index(total_wgs, true);
    if (wg >= total_wgs) return;
    // The scores, to which the column sums are added, start from zero.  (A launch of its own in front, where no prior is to be
    // formed: us with all rows, 32 heads x 4096 keys 156.8 -> 155.9, 8 x 2040 36.7 -> 35.6, 8 x 1024 24.4 -> 23.0, 8 x 2 x 734, d = 64
    // 21.5 -> 19.3.)
    if (zero)
        for (int64_t i = (int64_t)wg * 256 + threadIdx.x; i < (int64_t)g.batch * g.Hkv * g.n; i += (int64_t)total_wgs * 256) zero[i] = 0.f;
    const int npairs = (n_qtiles + 1) / 2;
    const int part = wg % nparts, pair = (wg / nparts) % npairs, z = wg / (nparts * npairs);
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const PlaceMap rm{g.n, g.r, g.G, pr};
    const FullSteps steps(rm, S::ROWS, n_qtiles, pair, part, nparts);
    auto tile_partial = [&](int qt) { return partial + ((int64_t)(z * n_qtiles + qt) * nparts + part) * S::ROWS; };
    // none of this part's steps fall on a tile: neutral statistics
    if (steps.n0 == 0 && tid < S::ROWS) tile_partial(steps.qt0)[tid] = -INFINITY;
    if (steps.n1 == 0 && steps.qt1 >= 0 && tid < S::ROWS) tile_partial(steps.qt1)[tid] = -INFINITY;
    const int total = steps.total();
    if (total == 0) return;

    const KeyRequest<D, kFullKeys, 4> request((const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1], g.ks[2], g.n, lane, wave, smem);
    auto request_step = [&](int i) { request(i < total ? steps.key(i) : 0, i & (kFullStages - 1)); };
    const int place = key_place<D>(lane);
    bf16x8 qf[NQ][KS], kf[KS];
    f32x16 X, Y;  // products in turn
    float lam[NQ], m[NQ], s[NQ];
    int pos[NQ], wmin = 0, wmax = -1, rho0 = 0;

    // Unmasked products P of row block q.  m is a REFERENCE that the sum s is relative to, not necessarily the running maximum
    // (m + log2 s does not depend on it): a block is summed against it as it stands, without a maximum over its
    // elements, and the reference is only moved (by the exact update, which redoes the block) when a block's sum says that it has
    // fallen more than 40 binades behind, or there is none yet.  It never lies above the largest logit seen, so nothing underflows that the
    // exact update would have kept.
    float sum[2], e[EP];
    auto sum_portion = [&](const f32x16 &P, int q, int portion) {
#pragma unroll
        for (int t = 0; t < EP; ++t) {
            const int v = portion * EP + t;
            if (portion) keep_here(sum[t & 1] = v - EP < 2 ? e[t] : sum[t & 1] + e[t]);
            e[t] = fast_exp2(fmaf(P[v], lam[q], -m[q]));
        }
    };
    auto sum_end = [&](const f32x16 &P, int q) {
#pragma unroll
        for (int t = 0; t < EP; ++t) sum[t & 1] += e[t];
        const float bs = sum[0] + sum[1];
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(bs < 0x1p40f)) != 0, 0))  // (also: a NaN)
            exact_stats<false>(P, lam[q], 0, 0, lane, m[q], s[q]);
        else s[q] += bs;
    };
    // the products of a block of 32 keys, the sums of all products but the last formed; `odd`: the second block of a step
    auto block = [&](bool start, bool odd, const char *next) {
        if constexpr (NQ == 2) {
            pipelined<D, true, false>(qf[0], kf, next, place, X, [&](int p) { if (!start) sum_portion(Y, 1, p); });
            if (!start) sum_end(Y, 1);
            pipelined<D, true, true>(qf[1], kf, next, place, Y, [&](int p) { sum_portion(X, 0, p); });
            sum_end(X, 0);
        } else if (odd) {
            pipelined<D, true, true>(qf[0], kf, next, place, Y, [&](int p) { sum_portion(X, 0, p); });
            sum_end(X, 0);
        } else {
            pipelined<D, true, true>(qf[0], kf, next, place, X, [&](int p) { if (!start) sum_portion(Y, 0, p); });
            if (!start) sum_end(Y, 0);
        }
    };
    auto masked_block = [&](const char *keys, int kb) {
        if (kb > wmax) return;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(keys, place, ks);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[q][ks], acc, 0, 0, 0);
            exact_stats<true>(acc, lam[q], pos[q], kb, lane, m[q], s[q]);
        }
    };
    auto begin_tile = [&](int qt) {
        int lane = threadIdx.x & 63;  // (as in the column sums)
        asm volatile("" : "+v"(lane));
        rho0 = qt * S::ROWS + wave * 32 * NQ;
        load_rows_of_wave<D, NQ>(g, rm, b, h, rho0, lane, qf);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int rho = rho0 + 32 * q + (lane & 31);
            pos[q] = rm.pos(rho);
            lam[q] = row_scale_log2_f32(g.scale_mode, g.fixed_scale, g.lambda_floor, max(pos[q], 0) + 1, g.budget, g.d);
            m[q] = -INFINITY;
            s[q] = 0.f;
        }
        wmin = uniform(rm.min_pos(rho0, rho0 + 32 * NQ));
        wmax = uniform(rm.max_pos(rho0, rho0 + 32 * NQ));
        // (waited for here, so that the compiler has no load of its own to wait for in the steps)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[q][ks]));
    };
    auto end_tile = [&](int qt) {
        float *out = tile_partial(qt) + wave * 32 * NQ;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {  // fold the half-waves: one query row, different keys
            const float m2 = __shfl_xor(m[q], 32), s2 = __shfl_xor(s[q], 32);
            const float mn = fmaxf(m[q], m2), mref = mn == -INFINITY ? 0.f : mn;
            const float sum = s[q] * fast_exp2(m[q] - mref) + s2 * fast_exp2(m2 - mref);
            if (lane < 32) out[32 * q + lane] = log2_sum(mn, sum);  // -inf for a row that saw no key
        }
    };

    for (int i = 0; i < kFullStages - 1; ++i) request_step(i);
    wait_vm<NI *(kFullStages - 2)>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    auto stage = [&](int i) { return (const char *)smem + (i & (kFullStages - 1)) * S::stage; };
    // Half way through step i: this wave's loads of step i + 1 have landed (step i + 2's may be in flight); behind the
    // barrier so have all waves', and all are done with step i - 1, whose stage the next request overwrites.
    auto advance = [&](int i) {
        __builtin_amdgcn_sched_barrier(0);
        wait_vm<NI *(kFullStages - 3)>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        request_step(i + kFullStages - 1);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto masked_steps = [&](int i, int end) {
        for (; i < end; ++i) {
            masked_block(stage(i), steps.key(i));
            advance(i);
            masked_block(stage(i) + S::stage / 2, steps.key(i) + 32);
        }
    };
    for (int t = 0; t < 2; ++t) {
        const int first = t ? steps.n0 : 0, end = t ? steps.total() : steps.n0, qt = t ? steps.qt1 : steps.qt0;
        if (first == end) continue;
        begin_tile(qt);
        const int free = steps.unmasked(t, wmin);
        const int i0 = t ? end - free : first, i1 = i0 + free;
        masked_steps(first, i0);
        if (free > 0) {
            int i = i0;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(stage(i), place, ks);
            block(true, false, stage(i) + S::stage / 2);
            advance(i);
            for (;;) {
                block(false, true, stage(i + 1));  // (past the last step: read and not used)
                if (++i == i1) break;
                block(false, false, stage(i) + S::stage / 2);
                advance(i);
            }
            exact_stats<false>(Y, lam[NQ - 1], 0, 0, lane, m[NQ - 1], s[NQ - 1]);
        }
        masked_steps(i1, end);
        end_tile(qt);
    }
    wait_vm<0>();  // (the last requests, past the range, write to LDS)
}

// ---------------------------------------------------------------- column sums --
// The query rows are on M here: a lane owns one key, so that the sum over a wave's rows ends with one
// exchange between the half-waves and one addition in LDS per key; with the keys on M the sums of every
// 32 keys would have to be folded over 32 lanes.  A row's scale (unless it is one for all rows, FIXED) and
// normaliser are then 16 values of a lane per 32 rows, in registers.
template <int D, int NQ, bool FIXED, bool PRIOR>
__global__ __launch_bounds__(256, 2) void full_colsum_kernel(ScoreGeom g, int pr, int n_qtiles, int nparts, int total_wgs,
                                                             int nchunks, const float *partial, const float *gamma,
                                                             const float *gblockmax, int n_vtiles, float *scores) {
    using S = FullSmem<D, NQ>;
    constexpr int KS = D / 16, NI = KeyRequest<D, kFullKeys, 4>::NI + (PRIOR ? 1 : 0), EP = 16 / KS;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    float *sCol = (float *)(smem + S::off_col), *sGamma = (float *)(smem + S::off_gamma);
    float *sL = (float *)(smem + S::off_row), *sLam = sL + S::ROWS;
    int *sPos = (int *)(sLam + S::ROWS);

    const int wg = logical_wg_index(total_wgs, true);
    if (wg >= total_wgs) return;
    const int npairs = (n_qtiles + 1) / 2;
    const int part = wg % nparts, pair = (wg / nparts) % npairs, z = wg / (nparts * npairs);
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const PlaceMap rm{g.n, g.r, g.G, pr};
    const FullSteps steps(rm, S::ROWS, n_qtiles, pair, part, nparts);
    const int total = steps.total();
    if (total == 0) return;

    float ginv = 1.f;
    if constexpr (PRIOR) {
        float gm = 0.f;
        for (int t = lane; t < n_vtiles; t += 64) gm = fmaxf(gm, gblockmax[z * n_vtiles + t]);
        ginv = prior_inverse(wave_max(gm));
    }
    const KeyRequest<D, kFullKeys, 4> request((const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1], g.ks[2], g.n, lane, wave, smem);
    const uint32_t gamma0 = uniform((int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)sGamma);
    auto request_step = [&](int i) {
        const int kb = i < total ? steps.key(i) : 0;
        request(kb, i & (kFullStages - 1));
        if constexpr (PRIOR) {  // (every wave, to the same place: their loads stay equal in number)
            const float *src = gamma + (int64_t)z * g.n + min(kb + lane, g.n - 1);
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                         :
                         : "v"(src), "s"(gamma0 + (i & (S::kGammaRing - 1)) * (kFullKeys * 4))
                         : "memory");
        }
    };
    const int place = key_place<D>(lane);
    bf16x8 qf[NQ][KS], kf[KS];
    f32x16 X, Y;  // products in turn
    f32x4 L[NQ][4], lamr[FIXED ? 1 : NQ][4];
    const float lam_all = row_scale_log2_f32(AHA_SCALE_FIXED, g.fixed_scale, 0.f, 1, 1, g.d);
    int wmin = 0, wmax = -1;

    // (a place per wave: a float atomic in LDS takes 75 cycles, 11 % of the kernel with four waves adding to one place)
    auto put_col = [&](float *to, float c) {
        c = combine_lane_xor<32>(c, OpSum{});
        if (lane < 32) to[lane] = c;
    };
    auto scale = [&](int q, int v) { return FIXED ? lam_all : lamr[FIXED ? 0 : q][v >> 2][v & 3]; };
    float sum[2], e[EP];  // of a block's keys over the wave's rows
    auto sum_portion = [&](const f32x16 &P, int q, int portion) {
#pragma unroll
        for (int t = 0; t < EP; ++t) {
            const int v = portion * EP + t;
            if (portion) keep_here(sum[t & 1] = q == 0 && v - EP < 2 ? e[t] : sum[t & 1] + e[t]);
            e[t] = fast_exp2(fmaf(P[v], scale(q, v), -L[q][v >> 2][v & 3]));
        }
    };
    auto sum_end = [&] {
#pragma unroll
        for (int t = 0; t < EP; ++t) sum[t & 1] += e[t];
    };
    // as in the row statistics; `to`: where the sums of the block before belong
    auto block = [&](bool start, bool odd, const char *next, float *to) {
        auto add = [&] {
            sum_end();
            put_col(to, sum[0] + sum[1]);
        };
        if constexpr (NQ == 2) {
            pipelined<D, false, false>(qf[0], kf, next, place, X, [&](int p) { if (!start) sum_portion(Y, 1, p); });
            if (!start) add();
            pipelined<D, false, true>(qf[1], kf, next, place, Y, [&](int p) { sum_portion(X, 0, p); });
            sum_end();
        } else if (odd) {
            pipelined<D, false, true>(qf[0], kf, next, place, Y, [&](int p) { sum_portion(X, 0, p); });
            add();
        } else {
            pipelined<D, false, true>(qf[0], kf, next, place, X, [&](int p) { if (!start) sum_portion(Y, 0, p); });
            if (!start) add();
        }
    };
    auto masked_block = [&](const char *keys, int kb, float *to) {
        if (kb > wmax) {
            if (lane < 32) to[lane] = 0.f;
            return;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(keys, place, ks);
        float sum = 0.f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[q][ks], kf[ks], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int p = sPos[wave * 32 * NQ + acc_key(0, q, v, lane)];  // (the row's place in the tile)
                const float e = fast_exp2(fmaf(acc[v], scale(q, v), -L[q][v >> 2][v & 3]));
                sum += kb + (lane & 31) <= p ? e : 0.f;
            }
        }
        put_col(to, sum);
    };
    auto begin_tile = [&](int qt) {
        // (through an opaque move: addresses kept across the steps are spilled, and waited for one by one here)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int rho0 = qt * S::ROWS, w0 = rho0 + wave * 32 * NQ;
        load_rows_of_wave<D, NQ>(g, rm, b, h, w0, lane, qf);
        __syncthreads();  // (the values of the tile before are done with)
        if (tid < S::ROWS) {
            constexpr int kBatch = 8;
            float ch[kBatch];
            const int rho = rho0 + tid, p = rm.pos(rho);
            const float *src = partial + ((int64_t)(z * n_qtiles + qt) * nchunks) * S::ROWS + tid;
            float M = -INFINITY, sum = 0.f;
            for (int c0 = 0; c0 < nchunks; c0 += kBatch) {
                chunk_request(src, S::ROWS, c0, nchunks, ch);
                chunk_merge(ch, nchunks - c0, M, sum);
            }
            sL[tid] = p >= 0 ? log2_sum(M, sum) : INFINITY;
            sLam[tid] = row_scale_log2_f32(g.scale_mode, g.fixed_scale, g.lambda_floor, max(p, 0) + 1, g.budget, g.d);
            sPos[tid] = p;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = wave * 32 * NQ + acc_key(0, q, 4 * v, lane);
                L[q][v] = *(const f32x4 *)(sL + at);
                if (!FIXED) lamr[FIXED ? 0 : q][v] = *(const f32x4 *)(sLam + at);
            }
        wmin = uniform(rm.min_pos(w0, w0 + 32 * NQ));
        wmax = uniform(rm.max_pos(w0, w0 + 32 * NQ));
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[q][ks]));
    };
    // step i's sums over the waves -> the scores
    auto flush = [&](int i) {
        const float *c = sCol + (i & (kFullStages - 1)) * (4 * kFullKeys) + lane;
        const float tot = (c[0] + c[kFullKeys]) + (c[2 * kFullKeys] + c[3 * kFullKeys]);
        const float f = PRIOR ? prior_factor(sGamma[(i & (S::kGammaRing - 1)) * kFullKeys + lane], ginv) : 1.f;
        const int j = steps.key(i) + lane;
        if (j < g.n) unsafeAtomicAdd(&scores[(int64_t)z * g.n + j], tot * f);
    };

    for (int i = 0; i < kFullStages - 1; ++i) request_step(i);
    wait_vm<NI *(kFullStages - 2)>();
    __syncthreads();
    auto stage = [&](int i) { return (const char *)smem + (i & (kFullStages - 1)) * S::stage; };
    auto col = [&](int i) { return sCol + (i & (kFullStages - 1)) * (4 * kFullKeys) + wave * kFullKeys; };
    // As in the row statistics; and the sums of step i - 1 are whole.
    auto advance = [&](int i) {
        __builtin_amdgcn_sched_barrier(0);
        wait_vm<NI *(kFullStages - 3)>();
        wait_lds();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (i && (i & 3) == wave) flush(i - 1);
        request_step(i + kFullStages - 1);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto masked_steps = [&](int i, int end) {
        for (; i < end; ++i) {
            masked_block(stage(i), steps.key(i), col(i));
            advance(i);
            masked_block(stage(i) + S::stage / 2, steps.key(i) + 32, col(i) + 32);
        }
    };
    for (int t = 0; t < 2; ++t) {
        const int first = t ? steps.n0 : 0, end = t ? steps.total() : steps.n0, qt = t ? steps.qt1 : steps.qt0;
        if (first == end) continue;
        begin_tile(qt);
        const int free = steps.unmasked(t, wmin);
        const int i0 = t ? end - free : first, i1 = i0 + free;
        masked_steps(first, i0);
        if (free > 0) {
            int i = i0;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(stage(i), place, ks);
            block(true, false, stage(i) + S::stage / 2, nullptr);
            advance(i);
            for (;;) {
                block(false, true, stage(i + 1), col(i));  // (past the last step: read and not used)
                if (++i == i1) break;
                block(false, false, stage(i) + S::stage / 2, col(i - 1) + 32);
                advance(i);
            }
#pragma unroll
            for (int p = 0; p < KS; ++p) sum_portion(Y, NQ - 1, p);
            sum_end();
            put_col(col(i1 - 1) + 32, sum[0] + sum[1]);
        }
        masked_steps(i1, end);
    }
    wait_vm<0>();  // (the last requests, past the range, write to LDS)
    __syncthreads();
    if (wave == 0) flush(total - 1);
}

// ---------------------------------------------------------------- launch --
template <int D, int NQ>
static hipError_t launch_full(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores, hipStream_t st,
                              hipEvent_t mid, bool have_lse) {
    using S = FullSmem<D, NQ>;
    char *w = (char *)ws;
    float *partial = (float *)(w + pl.off_partial);
    const float *gamma = (const float *)(w + pl.off_gamma), *gbm = (const float *)(w + pl.off_gblockmax);
    static DeviceOnce once;
    const hipError_t ea = device_once(once, [] {
        const void *kernels[5] = {(const void *)full_stats_kernel<D, NQ>, (const void *)full_colsum_kernel<D, NQ, true, false>,
                                  (const void *)full_colsum_kernel<D, NQ, true, true>,
                                  (const void *)full_colsum_kernel<D, NQ, false, false>,
                                  (const void *)full_colsum_kernel<D, NQ, false, true>};
        for (const void *kf : kernels) {
            const hipError_t e = hipFuncSetAttribute(kf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::bytes2);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
    if (ea != hipSuccess) return ea;
    const int pr = pl.full_pr, tiles = pl.full_tiles;
    const int64_t pairs = (int64_t)((tiles + 1) / 2) * pl.Z, wgs = pl.full_parts * pairs, wgs2 = pl.full_sum_parts * pairs;
    if (!have_lse)
        hipLaunchKernelGGL((full_stats_kernel<D, NQ>), xcd_grid(wgs), dim3(256), S::keys, st, g, pr, tiles, pl.full_parts, (int)wgs,
                           partial, g.value_prior ? nullptr : scores);
    if (mid) (void)hipEventRecord(mid, st);
    const int stat_chunks = have_lse ? 1 : pl.full_parts;
#define AHA_COLSUM(FIXED, PRIOR)                                                                                         \
    hipLaunchKernelGGL((full_colsum_kernel<D, NQ, FIXED, PRIOR>), xcd_grid(wgs2), dim3(256), S::bytes2, st, g, pr, tiles, \
                       pl.full_sum_parts, (int)wgs2, stat_chunks, partial, gamma, gbm, pl.n_vtiles, scores)
    if (g.scale_mode == AHA_SCALE_FIXED) {
        if (g.value_prior) AHA_COLSUM(true, true);
        else AHA_COLSUM(true, false);
    } else {
        if (g.value_prior) AHA_COLSUM(false, true);
        else AHA_COLSUM(false, false);
    }
#undef AHA_COLSUM
    return hipGetLastError();
}

hipError_t launch_score_full(const ScoreGeom &g, const PrefillPlan &pl, void *ws, float *scores, hipStream_t st,
                             hipEvent_t mid, bool have_lse) {
    if (pl.NB == 8)
        return g.d == 64 ? launch_full<64, 2>(g, pl, ws, scores, st, mid, have_lse)
                         : launch_full<128, 2>(g, pl, ws, scores, st, mid, have_lse);
    return g.d == 64 ? launch_full<64, 1>(g, pl, ws, scores, st, mid, have_lse)
                     : launch_full<128, 1>(g, pl, ws, scores, st, mid, have_lse);
}

}  // namespace aha
