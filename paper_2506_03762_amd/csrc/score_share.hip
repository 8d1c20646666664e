// Windowed bf16 scores of full tiles of 256 and 512 rows in ONE launch, the logits formed twice, by waves that own query rows and share the
// keys (key_stages.h; the exchanges: exchange.h).
//
// A workgroup of eight waves owns a CU and a range of keys.  First sweep: the range's row statistics, which are
// exchanged; second sweep, from the last keys to the first: the column sums, kept in LDS, and beside them the norms of the
// range's value rows (both come from memory or the last-level cache, hardly any from an L2: 203 MB past the L2s at 8 heads x
// 32768 keys x 256 rows, whose keys are 67 MB, and the value rows as much); then the ranges' largest priors are exchanged and the scores written.
// The value rows are left to the second sweep because the first one waits for the keys from memory, and nothing but
// the last factor needs them.
//
// us of the step (scores, top-k, compaction) against waves that keep 64 keys in registers and read the rows from LDS: 8 heads x
// 16384 keys x 512 rows 73.1 -> 59.8 (77.3 -> 66.1 on another box), 8 x 32768 x 256 81.7 -> 77.6.  In the latter (stamps, us): first keys 8, first sweep
// 18, exchange and merge 5 (some 3 since its words carry the data), second sweep 22, prior and its exchange 4; 537 and 690 ns per 64 x 32 block and
// SIMD, where the matrix core and the vector ALU would take 400 together: the sweeps read 200 MB in 40 us besides, a
// barrier per 64 keys.  Steps on the way: value rows three steps of 64 keys ahead instead of one of 128, 81.6 -> 77.6; value
// rows beside the first sweep and the wave-private keys, 84.4 instead of 83.5.
#include <type_traits>

#include "exchange.h"
#include "key_stages.h"

namespace aha {

// RG: groups of 64 query rows; 8 / RG groups of keys, of 64 keys each in a step of the first sweep, of 64 together in one of
// the second.
template <int D, int RG, bool PRIOR>
struct ShareSmem {
    static constexpr int KG = 8 / RG, ROWS = RG * 64;
    static constexpr int STEP = KG * 64, kFirst = 4, stage = KeyRows<D>::bytes(STEP);  // first sweep
    // second sweep: a step's keys, and its value rows, eight per wave
    static constexpr int STEP2 = 64, kSecond = 4, stage2 = KeyRows<D>::bytes(STEP2), wave_values = 8 * D * 2;
    static constexpr int off_values = kSecond * stage2;
    static constexpr int second_bytes = off_values + (PRIOR ? kSecond * 8 * wave_values : 0);
    // [4 steps][8 waves][64 keys]; after the first sweep float2 [KG][ROWS]
    static constexpr int off_col = kFirst * stage > second_bytes ? kFirst * stage : second_bytes;
    static constexpr int off_row = off_col + 4 * 8 * 64 * 4;  // normaliser, scale, position
    static constexpr int off_misc = off_row + 3 * ROWS * 4;
    // between the sweeps: float2 [8][256], in the fourth stage if it is large enough
    static constexpr int red_bytes = 8 * 256 * 8, off_red = red_bytes <= stage2 ? 3 * stage2 : off_misc + 16 * 4;
    static constexpr int off_nu = off_misc + 16 * 4 + (red_bytes <= stage2 ? 0 : red_bytes);
    // ranges of up to KEYS keys keep their norms, prior and sums in LDS, longer ones the norms in the workspace and the sums in the scores
    static constexpr int room = 160 * 1024 - off_nu - kPriorMaxHalo * 4;
    static constexpr int KEYS = !PRIOR ? 0 : room >= 2048 * 12 ? 2048 : room / 12 / 256 * 256;
    static constexpr int off_gam = off_nu + (KEYS + kPriorMaxHalo) * 4, off_sum = off_gam + KEYS * 4;
    static constexpr int bytes = off_sum + KEYS * 4;
    // keys whose norms are pooled at a time, in the stages' place (us of the score stage in pieces of 512 and so: 64 heads x 32768
    // keys x 256 rows 381, 374)
    static constexpr int PIECE = 4096;
    static_assert((PIECE + kPriorMaxHalo) * 4 <= off_col, "the stages");
    static_assert(bytes <= 160 * 1024, "LDS of a CU");
    static_assert(KG * ROWS * 8 <= 4 * 8 * 64 * 4, "the key groups' statistics");
};

template <int D, int RG, bool FIXED, int PRIOR>
__global__ __launch_bounds__(512, 2) void window_share_kernel(ScoreGeom g, int nparts, int part_keys, Exchange x, u32x4 *stats,
                                                              u32x4 *maxima, float *nu_g, float *scores) {
    using W = ShareSmem<D, RG, PRIOR != 0>;
    using R = KeyRows<D>;
    using Request = KeyRequest<D, W::STEP, 8>;
    using Request2 = KeyRequest<D, W::STEP2, 8>;
    constexpr int NQ = 2, KS = D / 16, EP = 16 / KS, NI = Request::NI;
    constexpr int NV = W::wave_values / 1024;  // load instructions for the wave's value rows of a step
    constexpr int NI2 = Request2::NI + (PRIOR ? NV : 0), KEYS2 = W::STEP2 / W::KG;  // (a wave's keys of a step)
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    float *sCol = (float *)(smem + W::off_col), *sL = (float *)(smem + W::off_row), *sLam = sL + W::ROWS;
    int *sPos = (int *)(sLam + W::ROWS);
    float *sMax = (float *)(smem + W::off_misc);
    int *sMissing = (int *)sMax + 8;
    float *sN = (float *)(smem + W::off_nu), *sGam = (float *)(smem + W::off_gam), *sSum = (float *)(smem + W::off_sum);
    const bool in_lds = W::KEYS && part_keys <= W::KEYS;

    const int own = (int)blockIdx.x % nparts, z = (int)blockIdx.x / nparts;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const int wave = uniform((int)threadIdx.x >> 6), rg = wave % RG, kg = wave / RG;
    const PlaceMap rm{g.n, g.r, g.G, g.r};
    const __bf16 *vbase = (const __bf16 *)g.v + b * g.vs[0] + h * g.vs[1];
    const int w0 = rg * 64, wmin = uniform(rm.min_pos(w0, w0 + 64)), wmax = uniform(rm.max_pos(w0, w0 + 64));
    const Request request((const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1], g.ks[2], g.n, (int)threadIdx.x & 63, wave, smem);
    const Request2 request2(request.kbase, g.ks[2], g.n, (int)threadIdx.x & 63, wave, smem);
    const int place = key_place<D>((int)threadIdx.x & 63);

    // the range; its steps in both sweeps, and of those the number without masks for this wave, which have the smallest keys
    int key_begin, key_end, nsteps, free, nsteps2, free2;
    auto set_range = [&](int part) {
        key_begin = part * part_keys;
        key_end = min(g.n, key_begin + part_keys);
        nsteps = (key_end - key_begin + W::STEP - 1) / W::STEP;
        const int past = wmin + 1 - key_begin - (kg + 1) * 64;  // (of the first step's keys of this wave)
        free = past < 0 ? 0 : min(nsteps, past / W::STEP + 1);
        nsteps2 = (key_end - key_begin + W::STEP2 - 1) / W::STEP2;
        const int past2 = wmin + 1 - key_begin - (kg + 1) * KEYS2;
        free2 = past2 < 0 ? 0 : min(nsteps2, past2 / W::STEP2 + 1);
    };
    bf16x8 qf[NQ][KS], kf[KS];
    f32x16 X, Y;  // products in turn
    float sum[2], e[EP];

    // ---- first sweep: row statistics ----
    float lam[NQ], m[NQ], s[NQ];
    int pos[NQ];
    auto first_sweep = [&] {
        const int lane = threadIdx.x & 63;
        auto key = [&](int i) { return key_begin + (i < nsteps ? i : 0) * W::STEP; };
        auto request_step = [&](int i) { request(key(i), i & (W::kFirst - 1)); };
        auto stage = [&](int i) { return (const char *)smem + (i & (W::kFirst - 1)) * W::stage + kg * R::bytes(64); };
        auto advance = [&](int i) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<NI *(W::kFirst - 3)>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            request_step(i + W::kFirst - 1);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto sum_portion = [&](const f32x16 &P, int q, int portion) {
#pragma unroll
            for (int t = 0; t < EP; ++t) {
                const int v = portion * EP + t;
                if (portion) keep_here(sum[t & 1] = v - EP < 2 ? e[t] : sum[t & 1] + e[t]);
                e[t] = fast_exp2(fmaf(P[v], lam[q], -m[q]));
            }
        };
        auto sum_end = [&](const f32x16 &P, int q) {  // (against a reference, as in score_full.hip)
#pragma unroll
            for (int t = 0; t < EP; ++t) sum[t & 1] += e[t];
            const float bs = sum[0] + sum[1];
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(bs < 0x1p40f)) != 0, 0))
                exact_stats<false>(P, lam[q], 0, 0, lane, m[q], s[q]);
            else s[q] += bs;
        };
        auto block = [&](bool start, const char *next) {
            pipelined<D, true, false>(qf[0], kf, next, place, X, [&](int p) { if (!start) sum_portion(Y, 1, p); });
            if (!start) sum_end(Y, 1);
            pipelined<D, true, true>(qf[1], kf, next, place, Y, [&](int p) { sum_portion(X, 0, p); });
            sum_end(X, 0);
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
#pragma unroll
        for (int q = 0; q < NQ; ++q) m[q] = -INFINITY, s[q] = 0.f;
        for (int i = 0; i < W::kFirst - 1; ++i) request_step(i);
        wait_vm<NI *(W::kFirst - 2)>();
        __syncthreads();
        if (free > 0) {
            int i = 0;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(stage(0), place, ks);
            block(true, stage(0) + R::bytes(32));
            advance(0);
            for (;;) {
                block(false, stage(i + 1));  // (past the last step: read and not used)
                if (++i == free) break;
                block(false, stage(i) + R::bytes(32));
                advance(i);
            }
            exact_stats<false>(Y, lam[1], 0, 0, lane, m[1], s[1]);
        }
        for (int i = free; i < nsteps; ++i) {
            masked_block(stage(i), key(i) + kg * 64);
            advance(i);
            masked_block(stage(i) + R::bytes(32), key(i) + kg * 64 + 32);
        }
    };

    // ---- second sweep: column sums, and the value rows' norms ----
    auto key2 = [&](int k) { return key_begin + (k < nsteps2 ? nsteps2 - 1 - k : 0) * W::STEP2; };
    const uint32_t values0 = uniform((int)((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem +
                                           W::off_values + wave * W::wave_values));
    constexpr int kValueStage = 8 * W::wave_values;
    // The wave's eight value rows of a step, as they lie in memory -> a place of its own in LDS.
    auto request_values = [&](int k) {
        const int lane = threadIdx.x & 63, row = key2(k) + wave * 8 + lane / R::CPR;
        const uint32_t dst = values0 + (k & (W::kSecond - 1)) * kValueStage;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const __bf16 *src = vbase + (int64_t)min(row + j * R::RPI, g.n - 1) * g.vs[2] + (lane % R::CPR) * 8;
            if constexpr (PRIOR == kValuesOnce)
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                             :
                             : "v"(src), "s"(dst + j * 1024)
                             : "memory");
            else
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                             :
                             : "v"(src), "s"(dst + j * 1024)
                             : "memory");
        }
    };
    auto store_norms = [&](int k) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        float v[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const bf16x8 w = *(const bf16x8 *)(smem + W::off_values + (k & (W::kSecond - 1)) * kValueStage + wave * W::wave_values +
                                               j * 1024 + lane * 16);
            float a = 0.f;
#pragma unroll
            for (int c = 0; c < 8; c += 2) {
                const bf16x2 pr = {w[c], w[c + 1]};
                a = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, a, false);
            }
            v[j] = a;
        }
        int u = 0;
        const float nu = fold_rows<R::CPR / 2>(v, lane, u);
        const int row = key2(k) + wave * 8 + u * R::RPI + lane / R::CPR;
        if (row >= key_end) return;
        if (in_lds) sN[row - max(0, key_begin - (g.pool - 1) / 2)] = nu;
        else nu_g[(int64_t)z * g.n + row] = nu;
    };
    auto request_second = [&](int k) {
        request2(key2(k), k & (W::kSecond - 1));
        if (PRIOR) request_values(k);
    };
    auto begin_second = [&] {
        for (int k = 0; k < W::kSecond - 1; ++k) request_second(k);
    };
    f32x4 L[NQ][4], lamr[FIXED ? 1 : NQ][4];
    const float lam_all = row_scale_log2_f32(AHA_SCALE_FIXED, g.fixed_scale, 0.f, 1, 1, g.d);
    auto scale = [&](int q, int v) { return FIXED ? lam_all : lamr[FIXED ? 0 : q][v >> 2][v & 3]; };
    auto second_sweep = [&] {
        const int lane = threadIdx.x & 63;
        auto stage = [&](int k) {
            return (const char *)smem + (k & (W::kSecond - 1)) * W::stage2 + (W::KG == 2 ? kg * R::bytes(32) : 0);
        };
        auto col = [&](int k) { return sCol + ((k & 3) * 8 + wave) * 64; };
        auto put_col = [&](float *to, float c) {
            c = combine_lane_xor<32>(c, OpSum{});
            if (lane < 32) to[lane] = c;
        };
        // step k's sums over the waves, one wave's work, in turn
        auto flush = [&](int k) {
            if (wave != (k & 7)) return;
            const float *c = sCol + (k & 3) * 8 * 64 + lane;
            if (W::KG == 2) c += (lane >> 5) * (RG * 64 - 32);
            float tot = (c[0] + c[64]) + (c[128] + c[192]);
            if constexpr (RG == 8) tot += (c[256] + c[320]) + (c[384] + c[448]);
            const int j = key2(k) + lane;
            if (j >= key_end) return;
            if (PRIOR && in_lds) sSum[j - key_begin] = tot;
            else scores[(int64_t)z * g.n + j] = tot;
        };
        // Before step k: the wave's loads of the keys of step k + 1 and of the value rows of step k have landed (what was requested
        // in the step before may be in flight); behind the barrier so have all waves', all are done with step k - 1,
        // whose stage is filled again, and the sums of step k - 2 are whole.
        auto advance = [&](int k) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<NI2>();
            wait_lds();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            request_second(k + W::kSecond - 1);
            if (PRIOR) store_norms(k);
            if (k >= 2) flush(k - 2);
            __builtin_amdgcn_sched_barrier(0);
        };
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
        auto block = [&](bool start, const char *next, float *to) {
            pipelined<D, false, false>(qf[0], kf, next, place, X, [&](int p) { if (!start) sum_portion(Y, 1, p); });
            if (!start) {
                sum_end();
                put_col(to, sum[0] + sum[1]);
            }
            pipelined<D, false, true>(qf[1], kf, next, place, Y, [&](int p) { sum_portion(X, 0, p); });
            sum_end();
        };
        auto masked_block = [&](const char *keys, int kb, float *to) {
            if (kb > wmax) {
                if (lane < 32) to[lane] = 0.f;
                return;
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(keys, place, ks);
            float c = 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[q][ks], kf[ks], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int p = sPos[w0 + acc_key(0, q, v, lane)];  // (the row's place in the tile)
                    const float ev = fast_exp2(fmaf(acc[v], scale(q, v), -L[q][v >> 2][v & 3]));
                    c += kb + (lane & 31) <= p ? ev : 0.f;
                }
            }
            put_col(to, c);
        };
        wait_vm<NI2>();
        __syncthreads();
        const int masked = nsteps2 - free2;
        for (int k = 0; k < masked; ++k) {
            advance(k);
#pragma unroll
            for (int c = 0; c < KEYS2; c += 32) masked_block(stage(k) + R::bytes(c), key2(k) + kg * KEYS2 + c, col(k) + c);
        }
        if (free2 > 0) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = key_fragment(stage(masked), place, ks);
            auto step = [&](bool start, int k) {  // (past the last step: keys read and not used)
                advance(k);
                block(start, KEYS2 == 32 ? stage(k + 1) : stage(k) + R::bytes(32), col(k - 1) + KEYS2 - 32);
                if constexpr (KEYS2 == 64) block(false, stage(k + 1), col(k));
            };
            step(true, masked);
            for (int k = masked + 1; k < nsteps2; ++k) step(false, k);
#pragma unroll
            for (int p = 0; p < KS; ++p) sum_portion(Y, 1, p);
            sum_end();
            put_col(col(nsteps2 - 1) + KEYS2 - 32, sum[0] + sum[1]);
        }
        wait_vm<0>();  // (the last requests, past the range, write to LDS)
        __syncthreads();
        if (nsteps2 >= 2) flush(nsteps2 - 2);
        flush(nsteps2 - 1);
    };

    Count count;
    const Words rows(stats + (int64_t)z * nparts * (W::ROWS / 2), x.tag), priors(maxima + (int64_t)z * nparts, x.tag);
    load_rows_of_wave<D, NQ>(g, rm, b, h, w0, (int)threadIdx.x & 63, qf);
    {
        const int tid = threadIdx.x, lane = tid & 63;
        if (tid < W::ROWS) {
            const int p = rm.pos(tid);
            sPos[tid] = p;
            sLam[tid] = row_scale_log2_f32(g.scale_mode, g.fixed_scale, g.lambda_floor, max(p, 0) + 1, g.budget, g.d);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            pos[q] = sPos[w0 + 32 * q + (lane & 31)];
            lam[q] = sLam[w0 + 32 * q + (lane & 31)];
        }
    }
    for (int part = own;;) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        if (part == 0 && tid == 511) count.look(x, z);
        set_range(part);
        first_sweep();
        if (part == 0 && tid == 511) count.start(x, z);
        // fold the half-waves (same query row, other keys), then the key groups
        float2 *sRed = (float2 *)sCol;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            float m2, s2;
            from_other_half(m[q], s[q], m2, s2);
            merge_stats(m[q], s[q], m2, s2);
            if (lane < 32) sRed[kg * W::ROWS + w0 + 32 * q + lane] = make_float2(m[q], s[q]);
        }
        // the last requests, past the range, write to LDS, where the second sweep begins (and the count is to be there first)
        wait_vm<0>();
        __syncthreads();
        if (tid < W::ROWS) {
            float M = sRed[tid].x, total = sRed[tid].y;
            if constexpr (W::KG == 2) merge_stats(M, total, sRed[W::ROWS + tid].x, sRed[W::ROWS + tid].y);
            put_rows(rows, part * (W::ROWS / 2), tid, log2_sum(M, total));
        }
        // (what the second sweep begins with travels while the others are waited for)
        begin_second();
        sRed = (float2 *)(smem + W::off_red);
        constexpr int MW = RG == 8 ? 4 : 8;  // waves that share 256 rows
        const int tile = RG == 8 ? wave >> 2 : 0;
        int missing = least_missing(merge_parts<256, MW>(rows, tile * 128, W::ROWS / 2, nparts, own, x.looks, sRed + wave * 256,
                                                         wave % MW, lane));
        if (lane == 0) sMissing[wave] = missing;
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < 8; ++wv) missing = min(missing, sMissing[wv]);
        missing = uniform(missing);
        if (missing == INT32_MAX && part == own) break;
        // somebody is not there: done here (and no more waiting); in the end the own part again
        part = missing != INT32_MAX ? missing ^ own : own;
        x.looks = 0;
        wait_vm<0>();
        __syncthreads();
    }
    int tid = threadIdx.x;
    const int lane = tid & 63;
    {
        const float2 *sRed = (const float2 *)(smem + W::off_red);
        constexpr int MW = RG == 8 ? 4 : 8;
        if (tid < W::ROWS) {
            float M = -INFINITY, total = 0.f;
            const float2 *src = sRed + tid / 256 * MW * 256 + tid % 256;
#pragma unroll
            for (int wv = 0; wv < MW; ++wv) merge_stats(M, total, src[wv * 256].x, src[wv * 256].y);
            sL[tid] = tid < g.R ? log2_sum(M, total) : INFINITY;  // (rows past the last one add nothing)
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = w0 + acc_key(0, q, 4 * v, lane);
                L[q][v] = *(const f32x4 *)(sL + at);
                if (!FIXED) lamr[FIXED ? 0 : q][v] = *(const f32x4 *)(sLam + at);
            }
    }
    second_sweep();
    if constexpr (PRIOR != 0) {
        asm volatile("" : "+v"(tid));
        PriorHalo<D> halo;
        halo.request(g, vbase, key_begin, key_end, tid);
        for (int part = own, looks = x.looks;;) {
            float gm;
            if (in_lds) {
                const float hn = halo.norm();
                if (halo.valid && tid % PriorHalo<D>::CPR == 0) sN[halo.pos - max(0, key_begin - (g.pool - 1) / 2)] = hn;
                __syncthreads();
                gm = pool_norms(g, key_begin, key_end, sN, sGam, tid, 512);
            } else {
                __syncthreads();  // (the stages become the norms' LDS)
                gm = pool_norms_of_range<D, 512, W::PIECE>(g, z, key_begin, key_end, nu_g, halo, (float *)smem, tid, [](int, float) {});
            }
            gm = wave_max(gm);
            if (lane == 0) sMax[wave] = gm;
            __syncthreads();
            if (wave == 0) {
                float all = fmaxf(fmaxf(fmaxf(sMax[0], sMax[1]), fmaxf(sMax[2], sMax[3])),
                                  fmaxf(fmaxf(sMax[4], sMax[5]), fmaxf(sMax[6], sMax[7])));
                if (lane == 0) priors.put(part, all, 0.f);
                const int missing = least_missing(largest_of<1>(priors, nparts, own, looks, lane, 64, all));
                if (lane == 0) {
                    *sMissing = missing;
                    sMax[0] = all;
                }
                count.arrived(x);
            }
            __syncthreads();
            const int missing = *sMissing;
            if (missing == INT32_MAX && part == own) break;
            // somebody is not there: its norms are formed here (and no more waiting); in the end the own
            // ones again
            part = missing != INT32_MAX ? missing ^ own : own;
            looks = 0;
            __syncthreads();
            set_range(part);
            halo.request(g, vbase, key_begin, key_end, tid);
            for (int k = 0; k < nsteps2; ++k) {
                request_values(k);
                wait_vm<0>();
                asm volatile("" ::: "memory");
                store_norms(k);
                wait_lds();
            }
        }
        const float ginv = prior_inverse(sMax[0]);
        float *out = scores + (int64_t)z * g.n;
        if (in_lds) {
            for (int j = key_begin + tid; j < key_end; j += 512) out[j] = sSum[j - key_begin] * prior_factor(sGam[j - key_begin], ginv);
        } else {  // (formed once more: no place to keep it)
            pool_norms_of_range<D, 512, W::PIECE>(g, z, key_begin, key_end, nu_g, halo, (float *)smem, tid,
                                        [&](int j, float gam) { out[j] *= prior_factor(gam, ginv); });
        }
    }
    if (tid == 511) count.arrive(x, z);
    if (leave(x, z, nparts, count, tid == 511, sMissing + 1)) {
        Words::take_away(stats + (int64_t)z * nparts * (W::ROWS / 2), nparts * (W::ROWS / 2), tid, 512);
        if (PRIOR) Words::take_away(maxima + (int64_t)z * nparts, nparts, tid, 512);
    }
}

// ---------------------------------------------------------------- launch --
template <int D, int RG, bool FIXED, int PRIOR>
static hipError_t launch_t(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, char *w, float *scores, hipStream_t st) {
    using W = ShareSmem<D, RG, PRIOR != 0>;
    const auto kernel = window_share_kernel<D, RG, FIXED, PRIOR>;
    static DeviceOnce once;
    const hipError_t e = device_once(once, [kernel] {
        return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)W::bytes);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(pl.Z * pl.win_parts)), dim3(512), W::bytes, st, g, pl.win_parts, pl.win_keys, x,
                       (u32x4 *)(w + pl.off_wstats), (u32x4 *)(w + pl.off_wmax), (float *)(w + pl.off_wnu),
                       scores);
    return hipGetLastError();
}

int share_keys_in_lds(int d, int tiles) {
    if (d == 64) return ShareSmem<64, 8, true>::KEYS;
    return tiles == 2 ? ShareSmem<128, 8, true>::KEYS : ShareSmem<128, 4, true>::KEYS;
}

hipError_t launch_score_share(const ScoreGeom &g, const PrefillPlan &pl, void *ws, const ExchangeCall &call, float *scores,
                              hipStream_t st) {
    char *w = (char *)ws;
    const Exchange x{(uint64_t *)(w + pl.off_wwords), call.tag, call.looks, call.replayed};
    auto scaled = [&](auto d, auto rg, auto prior) {
        constexpr int D = decltype(d)::value, RG = decltype(rg)::value, PRIOR = decltype(prior)::value;
        return g.scale_mode == AHA_SCALE_FIXED ? launch_t<D, RG, true, PRIOR>(g, pl, x, w, scores, st)
                                               : launch_t<D, RG, false, PRIOR>(g, pl, x, w, scores, st);
    };
    auto width = [&](auto prior) {
        using std::integral_constant;
        if (g.d == 64) return scaled(integral_constant<int, 64>{}, integral_constant<int, 8>{}, prior);  // (two tiles)
        return pl.win_tiles == 2 ? scaled(integral_constant<int, 128>{}, integral_constant<int, 8>{}, prior)
                                 : scaled(integral_constant<int, 128>{}, integral_constant<int, 4>{}, prior);
    };
    if (!g.value_prior) return width(std::integral_constant<int, kNoValues>{});
    return g.v_once ? width(std::integral_constant<int, kValuesOnce>{}) : width(std::integral_constant<int, kValuesCached>{});
}

}  // namespace aha
