// Windowed bf16 scores from given row normalisers (aha_prefill_scores_lse) in ONE launch.
//
// With the normalisers at hand a key's column sum is final as soon as its products are; only the value
// prior's maximum over all keys is missing.  A workgroup sweeps its range of keys once, multiplies the
// keys and squares the value rows of the same keys beside it, keeps sums and prior in LDS, and exchanges
// the range's largest prior with the other workgroups of its problem (exchange.h) before it writes the
// scores.  Before, a launch formed the prior (V at 5.2 TB/s, nothing to compute under it) and another
// one the sums.  8 heads x 32768 keys x 256 rows: 46.3 -> 39.7 us, bound by the vector ALU and the matrix core
// in turns; 128 x 16384 x 64: 198 -> 172 us, K and V at 6.2 TB/s.
//
// Value rows are loaded as they lie in memory (load_rows) and not with the key fragments' addressing, 32 rows
// x 32 bytes to an instruction: 128 x 16384 x 64 233 -> 212 us.  Ranges are as long as the LDS keeps their
// norms, prior and sums; through the workspace instead the same took 212 us.
#include <type_traits>

#include "exchange.h"
#include "score_block.h"

namespace aha {

// Norms, prior and column sums of a range are in LDS.
template <int D, int NB, bool PRIOR>
struct GivenSmem {
    static constexpr int KEYS = PRIOR ? given_keys(D, NB) : 0;
    static constexpr size_t off_misc = TileSmem<D, NB>::stride;
    static constexpr size_t off_nu = off_misc + 16 * sizeof(float);
    static constexpr size_t off_gam = off_nu + (KEYS + kPriorMaxHalo) * sizeof(float);
    static constexpr size_t off_sum = off_gam + KEYS * sizeof(float);
    static constexpr size_t bytes = off_sum + KEYS * sizeof(float);
    static_assert((NB <= 4 ? 2 : 1) * bytes <= 160 * 1024, "LDS of a CU");
};

// colsum_update with a mask (`room`: the row's position less the key of accumulator element 0), few elements at
// a time: this kernel has no registers to spare for it.
__device__ __forceinline__ void masked_colsum(const f32x16 (&acc)[kMB], float lam, float L, int room, f32x16 (&col)[kMB]) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v0 = 0; v0 < 16; v0 += 4) {
            float t[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                t[i] = fast_exp2(fmaf(acc[mb][v0 + i], lam, -L));
                if (mb * 32 + 2 * v0 + i > room) t[i] = 0.f;  // (acc_key)
            }
            asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
#pragma unroll
            for (int i = 0; i < 4; ++i) col[mb][v0 + i] += t[i];
        }
    asm volatile("" ::: "memory");
}

// WAVES: 4 with up to four row blocks (two workgroups per CU), 8 with more (one).
template <int D, int NB, int WAVES, int PRIOR>
__global__ __launch_bounds__(64 * WAVES, 2) void window_given_kernel(ScoreGeom g, int nparts, int part_keys, Exchange x, u32x4 *maxima,
                                                                     const float *lse, float *scores) {
    using S = TileSmem<D, NB>;
    using W = GivenSmem<D, NB, PRIOR != 0>;
    constexpr int THREADS = 64 * WAVES, STEP = WAVES * kWaveKeys, HALVES = WAVES / 4;
    // With few row blocks a step is too short to pass value rows and next keys through one buffer: the
    // value rows then have a buffer of their own and are a whole step ahead, as the keys' own next
    // block is requested when the last product has read the present one.
    constexpr bool OWN_BUFFER = PRIOR && NB <= 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wave = uniform((int)threadIdx.x >> 6);
    __bf16 *sQ = (__bf16 *)smem;
    float *sLam = (float *)(smem + S::q_bytes);
    int *sPos = (int *)(sLam + S::ROWS);
    float *sL = (float *)(sPos + S::ROWS);
    int *sBlk = (int *)(sL + S::ROWS);
    float *sMax = (float *)(smem + W::off_misc);
    int *sMissing = (int *)sMax + 8;
    float *sN = (float *)(smem + W::off_nu), *sGam = (float *)(smem + W::off_gam), *sSum = (float *)(smem + W::off_sum);

    const int own = (int)blockIdx.x % nparts, z = (int)blockIdx.x / nparts;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const RowMap rm{g.n, g.r, g.R, nullptr};
    const __bf16 *kbase = (const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1];
    const __bf16 *vbase = (const __bf16 *)g.v + b * g.vs[0] + h * g.vs[1];
    const int tile_min = rm.min_pos(0, S::ROWS);

    int key_begin, key_end, nsteps;
    auto kb_of = [&](int i) { return i < nsteps ? key_begin + i * STEP + wave * kWaveKeys : key_end; };
    auto set_range = [&](int part) {
        key_begin = part * part_keys;
        key_end = min(g.n, key_begin + part_keys);
        nsteps = (key_end - key_begin + STEP - 1) / STEP;
    };
    // norms of the wave's value rows of the step at kb, and where they go
    auto store_norms = [&](const bf16x8 (&w)[kMB][D / 16], int kb, int lane) {
        int row;
        const float nu = loaded_row_norm<D>(w, lane, row);
        row += kb;
        if (row < key_end) sN[row - max(0, key_begin - (g.pool - 1) / 2)] = nu;
    };

    // norms of the pooling halo's rows, which `halo` has requested
    auto store_halo = [&](const PriorHalo<D> &halo, int tid) {
        const float hn = halo.norm();
        if (halo.valid && tid % PriorHalo<D>::CPR == 0) sN[halo.pos - max(0, key_begin - (g.pool - 1) / 2)] = hn;
    };

    set_range(own);
    Count count;
    PriorHalo<D> halo;
    if (PRIOR && own == 0 && threadIdx.x == 63) count.look(x, z);
    bf16x8 a0[kMB][D / 16], a1[kMB][D / 16];  // the next key block (or value rows) load while one multiplies
    {
        constexpr int NBL = NB / HALVES;  // row blocks that 256 threads load
        const int tid = threadIdx.x, ht = tid & 255, half = wave >> 2;
        QTileRegs<D, NBL> qt;
        q_tile_request<D, NBL>(g, b, h, half * NBL * 32, ht, qt);
        if (PRIOR) halo.request(g, vbase, key_begin, key_end, tid);
        float L = INFINITY;  // (rows past the last one add nothing)
        if (tid < g.R) {
            const int gi = tid / g.r, ii = tid - gi * g.r;
            L = lse[((int64_t)b * g.Hq + h * g.G + gi) * g.r + ii] * kLog2e;
            if (L == INFINITY) L = NAN;
        }
        const float lam_req = q_tile_scale<D, NB>(g, rm, 0, tid);
        __builtin_amdgcn_sched_barrier(0);  // the keys are requested last
        load_a<D>(kbase, g.ks[2], kb_of(0), key_end, tid & 63, a0);
        if (PRIOR) {
            load_rows<D, PRIOR == kValuesOnce>(vbase, g.vs[2], kb_of(0), key_end, tid & 63, a1);
        }
        if (tid < S::ROWS) sL[tid] = L;
        q_tile_meta<D, NB>(g, rm, 0, tid, lam_req, sLam, sPos, sBlk);
        q_tile_commit<D, NBL>(qt, ht, sQ + half * NBL * 32 * S::LD);
        if (PRIOR) store_halo(halo, tid);
    }
    __syncthreads();

    // (one base for what a lane reads per block: scale, position, normaliser)
    int at = threadIdx.x & 31;
    asm volatile("" : "+v"(at));
    const float *meta = sLam + at;
    // column sums of the blocks [nb0, nb1) on the wave's 64 keys at kb; `after` follows the products of the last
    // one, before its exponentials
    auto blocks = [&](const bf16x8 (&a)[kMB][D / 16], int kb, int nb0, int nb1, f32x16 (&col)[kMB], auto &&after) {
        const int lane = threadIdx.x & 63;
        // (keys past the range's ragged end are never written, those past the last row's position masked)
        const bool all_see = kb + kWaveKeys - 1 <= tile_min;
        bf16x8 qf = query_fragment<D, NB>(sQ, nb0, 0, lane);
#pragma unroll
        for (int nb = nb0; nb < nb1; ++nb) {
            f32x16 acc[kMB];
            const float lam = meta[nb * 32], L = meta[2 * S::ROWS + nb * 32];
            mma_block_stream<D, NB>(a, sQ, nb, nb + 1 < nb1 ? nb + 1 : nb0, lane, qf, acc);
            if (nb + 1 == nb1) after();
            if (all_see) colsum_update<false>(acc, lam, L, 0, kb, lane, col);
            else masked_colsum(acc, lam, L, ((const int *)meta)[S::ROWS + nb * 32] - acc_key(kb, 0, 0, lane), col);
        }
    };
    // step i on the keys in `a`; `nx`: the other buffer
    auto step = [&](bf16x8 (&a)[kMB][D / 16], bf16x8 (&nx)[kMB][D / 16], int i) {
        // (through an opaque move: addresses are formed in each step, not kept and spilled)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int kb = kb_of(i), kb_next = kb_of(i + 1);  // past the range: clamped rows that are never used
        const bool first = i == 0, last = i + 1 >= nsteps;
        f32x16 col[kMB];
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) col[mb][v] = 0.f;
        auto nothing = [] {};
        if constexpr (!PRIOR) {
            load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            blocks(a, kb, 0, NB, col, nothing);
        } else if constexpr (OWN_BUFFER) {
            // (nx: this step's value rows)
            blocks(a, kb, 0, NB, col, [&] { load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, a); });
            __builtin_amdgcn_sched_barrier(0);
            store_norms(nx, kb, lane);
            __builtin_amdgcn_sched_barrier(0);
            load_rows<D, PRIOR == kValuesOnce>(vbase, g.vs[2], kb_next, key_end, lane, nx);
        } else {
            // the first step's value rows came with its keys, so the next keys have most of the step to
            // travel; the last step has no next keys, and its value rows the whole step; in between,
            // value rows travel under the first half and keys under the second
            constexpr int NB1 = NB / 4;
            if (!first) load_rows<D, PRIOR == kValuesOnce>(vbase, g.vs[2], kb, key_end, lane, nx);
            __builtin_amdgcn_sched_barrier(0);
            blocks(a, kb, 0, NB1, col, nothing);
            __builtin_amdgcn_sched_barrier(0);
            if (first) {
                store_norms(nx, kb, lane);
                __builtin_amdgcn_sched_barrier(0);
                load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            }
            __builtin_amdgcn_sched_barrier(0);
            blocks(a, kb, NB1, NB / 2, col, nothing);
            __builtin_amdgcn_sched_barrier(0);
            if (!first && !last) {
                store_norms(nx, kb, lane);
                __builtin_amdgcn_sched_barrier(0);
                load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            }
            __builtin_amdgcn_sched_barrier(0);
            blocks(a, kb, NB / 2, NB, col, nothing);
            __builtin_amdgcn_sched_barrier(0);
            if (!first && last) store_norms(nx, kb, lane);
        }
        const int my_v = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) {
            const float tot = fold16_over32(col[mb], lane);
            const int j = acc_key(kb, mb, my_v, lane);
            if ((lane & 1) || j >= key_end) continue;
            if (PRIOR) sSum[j - key_begin] = tot;
            else scores[(int64_t)z * g.n + j] = tot;
        }
    };
    for (int i = 0; i < nsteps; ++i) {
        step(a0, a1, i);
        if constexpr (!OWN_BUFFER) {
            if (++i >= nsteps) break;
            step(a1, a0, i);
        }
    }
    if constexpr (PRIOR) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const Words priors(maxima + (int64_t)z * nparts, x.tag);
        for (int part = own;;) {
            if (part == 0 && tid == 63) {
                if (own != 0) count.look(x, z);
                count.start(x, z);
            }
            // the prior of the range from its norms, and its largest
            __syncthreads();
            float gm = wave_max(pool_norms(g, key_begin, key_end, sN, sGam, tid, THREADS));
            if (lane == 0) sMax[wave] = gm;
            if (part == 0 && wave == 0) count.started(x);
            __syncthreads();
            if (wave == 0) {
                gm = sMax[0];
#pragma unroll
                for (int wv = 1; wv < WAVES; ++wv) gm = fmaxf(gm, sMax[wv]);
                if (lane == 0) priors.put(part, gm, 0.f);
                const int missing = least_missing(largest_of<1>(priors, nparts, own, x.looks, lane, 64, gm));
                if (lane == 0) {
                    *sMissing = missing;
                    sMax[0] = gm;
                }
                count.arrived(x);
            }
            __syncthreads();
            const int missing = *sMissing;
            if (missing == INT32_MAX && part == own) break;
            // somebody is not there: its norms are formed here (and no more waiting); in the end the own
            // ones again, whose prior the LDS has to hold
            part = missing != INT32_MAX ? missing ^ own : own;
            x.looks = 0;
            __syncthreads();
            set_range(part);
            halo.request(g, vbase, key_begin, key_end, tid);
            for (int i = 0; i < nsteps; ++i) {
                load_rows<D, PRIOR == kValuesOnce>(vbase, g.vs[2], kb_of(i), key_end, lane, a0);
                store_norms(a0, kb_of(i), lane);
            }
            store_halo(halo, tid);
        }
        if (tid == 63) count.arrive(x, z);
        const float ginv = prior_inverse(sMax[0]);
        float *out = scores + (int64_t)z * g.n;
        for (int j = key_begin + tid; j < key_end; j += THREADS)
            out[j] = sSum[j - key_begin] * prior_factor(sGam[j - key_begin], ginv);
        if (leave(x, z, nparts, count, tid == 63, sMissing + 1)) Words::take_away(maxima + (int64_t)z * nparts, nparts, tid, THREADS);
    }
}

// ---------------------------------------------------------------- launch --
template <int D, int NB, int WAVES, int PRIOR>
static hipError_t launch_t(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, u32x4 *maxima, const float *lse, float *scores,
                           hipStream_t st) {
    using W = GivenSmem<D, NB, PRIOR != 0>;
    const auto kernel = window_given_kernel<D, NB, WAVES, PRIOR>;
    if (W::bytes > 64 * 1024) {
        static DeviceOnce once;
        const hipError_t e = device_once(once, [kernel] {
            return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)W::bytes);
        });
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(pl.Z * pl.given_parts)), dim3(64 * WAVES), W::bytes, st, g,
                       pl.given_parts, pl.given_keys, x, maxima, lse, scores);
    return hipGetLastError();
}

template <int D, int PRIOR>
static hipError_t launch_d(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, u32x4 *maxima, const float *lse, float *scores,
                           hipStream_t st) {
    switch (pl.given_nb) {
        case 1: return launch_t<D, 1, 4, PRIOR>(g, pl, x, maxima, lse, scores, st);
        case 2: return launch_t<D, 2, 4, PRIOR>(g, pl, x, maxima, lse, scores, st);
        case 4: return launch_t<D, 4, 4, PRIOR>(g, pl, x, maxima, lse, scores, st);
        case 6: return launch_t<D, 6, 8, PRIOR>(g, pl, x, maxima, lse, scores, st);
        case 8: return launch_t<D, 8, 8, PRIOR>(g, pl, x, maxima, lse, scores, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_score_given(const ScoreGeom &g, const PrefillPlan &pl, void *ws, const ExchangeCall &call,
                              const float *lse, float *scores, hipStream_t st) {
    char *w = (char *)ws;
    const Exchange x{(uint64_t *)(w + pl.off_gwords), call.tag, call.looks, call.replayed};
    u32x4 *maxima = (u32x4 *)(w + pl.off_gmax);
    auto launch = [&](auto prior) {
        constexpr int PRIOR = decltype(prior)::value;
        return g.d == 64 ? launch_d<64, PRIOR>(g, pl, x, maxima, lse, scores, st)
                         : launch_d<128, PRIOR>(g, pl, x, maxima, lse, scores, st);
    };
    if (!g.value_prior) return launch(std::integral_constant<int, kNoValues>{});
    return g.v_once ? launch(std::integral_constant<int, kValuesOnce>{}) : launch(std::integral_constant<int, kValuesCached>{});
}

}  // namespace aha
