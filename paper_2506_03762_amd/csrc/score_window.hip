// Windowed bf16 eviction scores in ONE launch (Sec. 4.1 - 4.3; Alg. 1 Prefill).
//
// A score needs the log-sum-exp of every observed row over ALL keys before any key's column can be
// summed.  The workgroups of a (batch, KV head) problem each own a range of its keys; they exchange
// their ranges' row statistics and prior maxima (exchange.h) and go on to the column sums of their
// own range.  Against two launches this saves the second set-up (query tile, first keys) and, in the
// held form, the second read of the keys and their products.
//
// window_hold_kernel (up to four blocks of 32 rows, eight with two tiles): the exponentials of the range, each block's relative to the
// running maximum of its rows then, stay in the accumulators while the statistics travel, so that a column sum takes a
// multiplication per element; with the logits in them it took the exponential again, and where the range has two steps 9
// registers spilled (now none): us of the step before and after, 128 heads x 16384 keys x 64 rows 336 -> 295, 32 x 4096 x 64 31.1 ->
// 30.6, 12 x 5003 x 120 21.2 -> 20.5; against float64 the scores' rms error over 20 shapes is 0.73 times that from logits.
// 32 heads x 4096 keys x 64 rows in two launches 29 us, so 22; bound by
// the one burst of loads (12 us to the last workgroup's keys), then (stamps, us) statistics and prior 3.5, the exchange 2,
// the column sums 1.6.  128 heads x 16384 x 64: 287 -> 267 us, K read once instead of twice.
// window_stream_kernel (below): more rows or longer ranges, the logits formed twice, 620 ns per 64 x 32 block and SIMD; full
// tiles are score_share.hip's, but for those of 256 rows with d = 64.
//
// Value rows are loaded as they lie in memory (load_rows); with the key fragments' addressing an instruction
// reads 32 bytes of 32 rows.  Where the last-level cache would not keep them anyway they go past the caches.  us
// of the score stage before and after: 48 heads x 6846 keys x 64 rows 59.0, 47.3; 12 x 59081 x 64 108, 92.8; 128 x
// 16384 x 64 259, 252.  110 shapes of 1 to 512 rows 1.027 times as fast on average.
// Two tiles share their value rows, 32 each, and load them like keys (as memory lies was slower).
#include <type_traits>

#include "exchange.h"
#include "score_block.h"

namespace aha {

template <int D, int NB, int NT, int KEYS, bool PRIOR>
struct HoldSmem {
    static constexpr int TROWS = NB * 32, ROWS = NT * TROWS;
    static constexpr size_t off_red = NT * TileSmem<D, NB>::stride;  // float2 [wave][row of its tile], then column sums
    static constexpr size_t off_nu = off_red + 4 * ROWS * sizeof(float2);
    static constexpr size_t off_gam = off_nu + (PRIOR ? (KEYS + kPriorMaxHalo) * sizeof(float) : 0);
    static constexpr size_t off_misc = off_gam + (PRIOR ? KEYS * sizeof(float) : 0);
    static constexpr size_t bytes = off_misc + 16 * sizeof(float);
    static_assert(KEYS * sizeof(float) <= 4 * ROWS * sizeof(float2) || NT == 1, "column sums of the second tile");
    static_assert(off_red / NT % 16 == 0, "a tile's rows are read and written 16 bytes at a time");
};

// STEPS: 256-key steps of a workgroup's range, all of whose exponentials are held: NB * STEPS <= 4.
// NT = 2: two tiles of rows, eight waves; waves w and w + 4 take the same keys, one tile each.
template <int D, int NB, int NT, int STEPS, int PRIOR>
__global__ __launch_bounds__(256 * NT, 2) void window_hold_kernel(ScoreGeom g, int nparts, Exchange x, u32x4 *stats,
                                                                  u32x4 *maxima, float *scores) {
    using S = TileSmem<D, NB>;
    using H = HoldSmem<D, NB, NT, STEPS * kWgKeys, PRIOR != 0>;
    static_assert(NB * STEPS <= 4 && (NT == 1 || STEPS == 1), "exponentials in registers");
    constexpr int THREADS = 256 * NT, WAVES = 4 * NT, VM = NT == 2 ? 1 : kMB;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wave = uniform((int)threadIdx.x >> 6), tile = NT == 2 ? wave >> 2 : 0, kw = wave & 3;
    __bf16 *sQ = (__bf16 *)(smem + tile * S::stride);
    float *sLam = (float *)(smem + tile * S::stride + S::q_bytes);
    int *sPos = (int *)(sLam + S::ROWS);
    float *sL = (float *)(sPos + S::ROWS);
    int *sBlk = (int *)(sL + S::ROWS);
    float2 *sRed = (float2 *)(smem + H::off_red);
    float *sCol = (float *)sRed;
    float *sNu = (float *)(smem + H::off_nu), *sGam = (float *)(smem + H::off_gam);
    float *sMax = (float *)(smem + H::off_misc);
    int *sMissing = (int *)sMax + 8;

    const int own = (int)blockIdx.x % nparts, z = (int)blockIdx.x / nparts;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const RowMap rm{g.n, g.r, g.R, nullptr};
    const __bf16 *kbase = (const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1];
    const __bf16 *vbase = (const __bf16 *)g.v + b * g.vs[0] + h * g.vs[1];

    Count count;
    const Words rows(stats + (int64_t)z * nparts * (H::ROWS / 2), x.tag), priors(maxima + (int64_t)z * nparts * WAVES, x.tag);
    f32x16 acc[STEPS][NB][kMB];
    float ref[STEPS][NB];
    int pos[NB], bmin[NB];
    int key_begin, key_end;
    for (int part = own;;) {
        // (the loop nearly always runs once; through an opaque move, what depends on the thread is
        // formed in it and not kept in registers across it)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, ht = tid & 255;
        if (part == 0 && tid == THREADS - 1) count.look(x, z);
        key_begin = part * STEPS * kWgKeys;
        key_end = min(g.n, key_begin + STEPS * kWgKeys);
        auto kb_of = [&](int st) { return key_begin + st * kWgKeys + kw * kWaveKeys; };
        bf16x8 a[kMB][D / 16], w[kMB][D / 16];
        auto load_values = [&](int st) {
            load_rows<D, PRIOR == kValuesOnce, VM>(vbase, g.vs[2], kb_of(st) + (NT == 2 ? tile * 32 : 0), key_end, lane, w);
        };
        PriorHalo<D> halo;
        {
            QTileRegs<D, NB> qt;
            q_tile_request<D, NB>(g, b, h, tile * H::TROWS, ht, qt);
            const float lam_req = q_tile_scale<D, NB>(g, rm, tile * H::TROWS, ht);
            __builtin_amdgcn_sched_barrier(0);  // the keys are requested last
            load_a<D>(kbase, g.ks[2], kb_of(0), key_end, lane, a);
            if (PRIOR) {
                load_values(0);
                halo.request(g, vbase, key_begin, key_end, tid);
            }
            q_tile_meta<D, NB>(g, rm, tile * H::TROWS, ht, lam_req, sLam, sPos, sBlk);
            q_tile_commit<D, NB>(qt, ht, sQ);
        }
        __syncthreads();
        float m[NB], s[NB], lam[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            lam[nb] = sLam[nb * 32 + (lane & 31)];
            pos[nb] = sPos[nb * 32 + (lane & 31)];
            if (pos[nb] < 0) lam[nb] = kLeastScale;  // (no row)
            bmin[nb] = uniform(sBlk[NB + nb]);
            m[nb] = -INFINITY;
            s[nb] = 0.f;
        }
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const int kb = kb_of(st);
            if constexpr (PRIOR) {  // (first: the value rows' registers are then free for the products)
                int row;
                const float nu = loaded_row_norm<D, VM>(w, lane, row);
                row += kb + (NT == 2 ? tile * 32 : 0);
                if (row < key_end) sNu[row - max(0, key_begin - (g.pool - 1) / 2)] = nu;
                __builtin_amdgcn_sched_barrier(0);
                if (st + 1 < STEPS) load_values(st + 1);
            }
            // (keys at or past n, in the last range, lie behind every row's position)
            if (st == STEPS - 1 && part == 0 && tid == THREADS - 1) count.start(x, z);
            bf16x8 qf = query_fragment<D, NB>(sQ, 0, 0, lane);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                mma_block_stream<D, NB>(a, sQ, nb, nb + 1 < NB ? nb + 1 : 0, lane, qf, acc[st][nb]);
                if (nb == NB - 1 && st + 1 < STEPS) load_a<D>(kbase, g.ks[2], kb_of(st + 1), key_end, lane, a);
                const bool masked = kb + kWaveKeys - 1 > bmin[nb];
                float scale = lam[nb];  // (of this block: hiding may put it into the products)
                if (masked) hide_unseen(acc[st][nb], pos[nb] - acc_key(kb, 0, 0, lane), scale);
                stats_weights(acc[st][nb], scale, m[nb], s[nb], ref[st][nb]);
            }
        }
        // fold the half-waves (same query row, other keys), then the waves
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float m2, s2;
            from_other_half(m[nb], s[nb], m2, s2);
            merge_stats(m[nb], s[nb], m2, s2);
            if (lane < 32) sRed[wave * H::TROWS + nb * 32 + lane] = make_float2(m[nb], s[nb]);
        }
        if (PRIOR) {
            const float hn = halo.norm();
            if (halo.valid && tid % PriorHalo<D>::CPR == 0)
                sNu[halo.pos - max(0, key_begin - (g.pool - 1) / 2)] = hn;
        }
        if (part == 0 && wave == WAVES - 1) count.started(x);
        __syncthreads();
        if (tid < H::ROWS) {
            float M = -INFINITY, sum = 0.f;
            const float2 *src = sRed + (NT == 2 ? tid / H::TROWS * 4 * H::TROWS : 0) + tid % H::TROWS;
#pragma unroll
            for (int wv = 0; wv < 4; ++wv) merge_stats(M, sum, src[wv * H::TROWS].x, src[wv * H::TROWS].y);
            put_rows(rows, part * (H::ROWS / 2), tid, M + log2f(sum));
        }
        if (PRIOR) {
            const float gm = wave_max(pool_norms(g, key_begin, key_end, sNu, sGam, tid, THREADS));
            if (lane == 0) priors.put(part * WAVES + wave, gm, 0.f);
        }
        __syncthreads();
        int missing = merge_parts<H::TROWS, 4>(rows, tile * (H::TROWS / 2), H::ROWS / 2, nparts, own, x.looks,
                                               sRed + wave * H::TROWS, kw, lane);
        if (PRIOR) {
            float gm;
            missing = min(missing, largest_of<WAVES>(priors, nparts, own, x.looks, tid, THREADS, gm));
            if (lane == 0) sMax[wave] = gm;
        }
        missing = least_missing(missing);
        if (lane == 0) sMissing[wave] = missing;
        count.arrived(x);
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < WAVES; ++wv) missing = min(missing, sMissing[wv]);
        missing = uniform(missing);
        if (missing == INT32_MAX && part == own) break;
        // somebody is not there: done here (and no more waiting); in the end the own part again, whose
        // exponentials the accumulators have to hold
        part = missing != INT32_MAX ? missing ^ own : own;
        x.looks = 0;
        __syncthreads();
    }
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == THREADS - 1) count.arrive(x, z);
    if (tid < H::ROWS) {
        float M = -INFINITY, sum = 0.f;
        const int t = tid / H::TROWS, row = tid % H::TROWS;
        const float2 *src = sRed + t * 4 * H::TROWS + row;
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) merge_stats(M, sum, src[wv * H::TROWS].x, src[wv * H::TROWS].y);
        // (in the scales' place: reciprocal sums; rows past the last one add nothing)
        float *meta = (float *)(smem + t * S::stride + S::q_bytes) + row;
        meta[0] = tid < g.R ? 1.f / sum : 0.f;
        meta[2 * S::ROWS] = tid < g.R ? M : INFINITY;
    }
    __syncthreads();
    float ginv = 1.f;
    if (PRIOR) {
        float gm = sMax[0];
#pragma unroll
        for (int wv = 1; wv < WAVES; ++wv) gm = fmaxf(gm, sMax[wv]);
        ginv = prior_inverse(gm);
    }
    // a block's weights -> probabilities
    float f[STEPS][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const float M = sL[nb * 32 + (lane & 31)], rs = sLam[nb * 32 + (lane & 31)];
#pragma unroll
        for (int st = 0; st < STEPS; ++st) f[st][nb] = fast_exp2(ref[st][nb] - M) * rs;
    }
    const int my_v = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 +
                     ((lane >> 1) & 1);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int kb = key_begin + st * kWgKeys + kw * kWaveKeys;
        f32x16 col[kMB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const bool masked = kb + kWaveKeys - 1 > bmin[nb], none = !(f[st][nb] < INFINITY);
            if (__builtin_expect(masked && __builtin_amdgcn_ballot_w64(none) != 0, 0))
                weights_without_factor(acc[st][nb], pos[nb] - acc_key(kb, 0, 0, lane), none, f[st][nb]);
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    col[mb][v] = nb ? fmaf(acc[st][nb][mb][v], f[st][nb], col[mb][v]) : acc[st][nb][mb][v] * f[st][nb];
        }
        float tot[kMB];
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) tot[mb] = fold16_over32(col[mb], lane);
        if constexpr (NT == 2) {  // the second tile's sums meet the first's (sRed has been read)
            if (tile == 1 && (lane & 1) == 0) {
#pragma unroll
                for (int mb = 0; mb < kMB; ++mb) sCol[acc_key(kb, mb, my_v, lane) - key_begin] = tot[mb];
            }
            __syncthreads();
            if (tile == 1) break;
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb) tot[mb] += sCol[acc_key(kb, mb, my_v, lane) - key_begin];
        }
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) {
            const int j = acc_key(kb, mb, my_v, lane);
            if ((lane & 1) == 0 && j < key_end)
                scores[(int64_t)z * g.n + j] = PRIOR ? tot[mb] * prior_factor(sGam[j - key_begin], ginv) : tot[mb];
        }
    }
    if (leave(x, z, nparts, count, tid == THREADS - 1, sMissing + 1)) {
        Words::take_away(stats + (int64_t)z * nparts * (H::ROWS / 2), nparts * (H::ROWS / 2), tid, THREADS);
        if (PRIOR) Words::take_away(maxima + (int64_t)z * nparts * WAVES, nparts * WAVES, tid, THREADS);
    }
}

// ---- the logits formed twice --------------------------------------------------------------------
// window_stream_kernel: more rows than whose exponentials a wave can hold, or longer ranges.  A workgroup of
// eight waves owns a CU and a range of keys; the first sweep over the range leaves the rows' statistics, the
// second, from the last step to the first, starts on keys that are in the caches still and sums columns.
// NT = 1: one tile of up to 256 rows, the waves take 64 keys each.  NT = 2: two tiles, of up to 512 rows;
// waves w and w + 4 take the same 64 keys, one tile each, and add their column sums in LDS.
template <int D, int NB, int NT>
struct StreamSmem {
    static constexpr int TROWS = NB * 32, ROWS = NT * TROWS, KW = 8 / NT, STEP = KW * kWaveKeys;
    static constexpr size_t off_red = NT * TileSmem<D, NB>::stride;  // float2 [8][TROWS], then norms, then column sums
    static constexpr size_t red_bytes = 8 * TROWS * sizeof(float2) > (kPriorPiece + kPriorMaxHalo) * sizeof(float)
                                            ? 8 * TROWS * sizeof(float2)
                                            : (kPriorPiece + kPriorMaxHalo) * sizeof(float);
    static constexpr size_t off_misc = (off_red + red_bytes + 15) / 16 * 16;
    static constexpr size_t off_nu = off_misc + 16 * sizeof(float);
    // ranges of up to KEYS keys keep their norms and prior in LDS, longer ones the norms in the workspace and the prior in the scores
    static constexpr size_t room = 160 * 1024 - off_nu - kPriorMaxHalo * sizeof(float);
    static constexpr int KEYS = room >= 2048 * 8 ? 2048 : (int)(room / 8) / 256 * 256;
    static constexpr size_t off_gam = off_nu + (KEYS ? (KEYS + kPriorMaxHalo) * sizeof(float) : 0);
    static constexpr size_t bytes = off_gam + KEYS * sizeof(float);
    static_assert(2 * 4 * kWaveKeys * sizeof(float) <= red_bytes, "column sums of two steps");
    static_assert(off_red / NT % 16 == 0, "a tile's rows are read and written 16 bytes at a time");
    static_assert(bytes <= 160 * 1024, "LDS of a CU");
};

template <int D, int NB, int NT, int PRIOR>
__global__ __launch_bounds__(512, 2) void window_stream_kernel(ScoreGeom g, int nparts, int part_keys, Exchange x,
                                                               u32x4 *stats, u32x4 *maxima, float *nu_g, float *scores) {
    using S = TileSmem<D, NB>;
    using W = StreamSmem<D, NB, NT>;
    // with two tiles a wave takes 32 of the 64 value rows it shares
    constexpr int VM = NT == 2 ? 1 : kMB;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wave = uniform((int)threadIdx.x >> 6), half = wave >> 2;
    const int tile = NT == 2 ? half : 0, kw = NT == 2 ? wave & 3 : wave;
    __bf16 *sQ = (__bf16 *)(smem + tile * S::stride);
    float *sLam = (float *)(smem + tile * S::stride + S::q_bytes);
    int *sPos = (int *)(sLam + S::ROWS);
    float *sL = (float *)(sPos + S::ROWS);
    int *sBlk = (int *)(sL + S::ROWS);
    float2 *sRed = (float2 *)(smem + W::off_red);
    float *sCol = (float *)sRed, *sNu = (float *)sRed;
    float *sMax = (float *)(smem + W::off_misc);
    int *sMissing = (int *)sMax + 8;
    float *sN = (float *)(smem + W::off_nu), *sGam = (float *)(smem + W::off_gam);
    const bool in_lds = W::KEYS && part_keys <= W::KEYS;

    const int own = (int)blockIdx.x % nparts, z = (int)blockIdx.x / nparts;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const RowMap rm{g.n, g.r, g.R, nullptr};
    const __bf16 *kbase = (const __bf16 *)g.k + b * g.ks[0] + h * g.ks[1];
    const __bf16 *vbase = (const __bf16 *)g.v + b * g.vs[0] + h * g.vs[1];
    const int tile_min = rm.min_pos(tile * W::TROWS, (tile + 1) * W::TROWS);

    Count count;
    const Words rows(stats + (int64_t)z * nparts * (W::ROWS / 2), x.tag), priors(maxima + (int64_t)z * nparts * 8, x.tag);
    bf16x8 a0[kMB][D / 16], a1[kMB][D / 16];  // the next key block loads while one multiplies
    int key_begin, key_end, nsteps;
    auto kb_of = [&](int i) { return i >= 0 && i < nsteps ? key_begin + i * W::STEP + kw * kWaveKeys : key_end; };
    auto set_range = [&](int part) {
        key_begin = part * part_keys;
        key_end = min(g.n, key_begin + part_keys);
        nsteps = (key_end - key_begin + W::STEP - 1) / W::STEP;
    };
    auto load_values = [&](int kb, int lane, bf16x8 (&w)[kMB][D / 16]) {
        if (NT == 2) load_a<D, VM>(vbase, g.vs[2], kb + tile * 32, key_end, lane, w);
        else load_rows<D, PRIOR == kValuesOnce>(vbase, g.vs[2], kb, key_end, lane, w);
        if (VM == 1) {  // (never read; an array that is only half written stays in memory)
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) w[1][ks] = bf16x8{};
        }
    };
    // the query rows and their scales to LDS, the keys of step `first` into a0 (and its value rows into a1)
    auto set_up = [&](int tid, int first) {
        constexpr int NBL = NB * NT / 2;  // row blocks that 256 threads load
        const int ht = tid & 255;
        QTileRegs<D, NBL> qt;
        q_tile_request<D, NBL>(g, b, h, half * NBL * 32, ht, qt);
        const int mt = NT == 2 ? ht : tid;
        const float lam_req = q_tile_scale<D, NB>(g, rm, tile * W::TROWS, mt);
        __builtin_amdgcn_sched_barrier(0);  // the keys are requested last
        load_a<D>(kbase, g.ks[2], kb_of(first), key_end, tid & 63, a0);
        if (PRIOR) load_values(kb_of(first), tid & 63, a1);
        q_tile_meta<D, NB>(g, rm, tile * W::TROWS, mt, lam_req, sLam, sPos, sBlk);
        q_tile_commit<D, NBL>(qt, ht, NT == 2 ? sQ : sQ + half * NBL * 32 * S::LD);
    };
    // norms of the wave's value rows of the step at kb, and where they go
    auto store_norms = [&](const bf16x8 (&w)[kMB][D / 16], int kb, int lane) {
        int row;
        float nu;
        if constexpr (NT == 2) {
            float x[kMB];
            fragment_row_norms<D, VM>(w, x);
            nu = x[0];
            row = lane < 32 ? kb + tile * 32 + lane : key_end;
        } else {
            nu = loaded_row_norm<D>(w, lane, row);
            row += kb;
        }
        if (row >= key_end) return;
        if (in_lds) sN[row - max(0, key_begin - (g.pool - 1) / 2)] = nu;
        else nu_g[(int64_t)z * g.n + row] = nu;
    };
    // One step of a sweep: blocks(a, kb, from, to) on the keys in `a` while `nx` receives those of kb_next
    // (unconditionally: past the range, clamped rows that are never used).  With VALUES the step's
    // value rows pass through `nx` as well: those of the first step came with its keys, so the next
    // keys have the whole step to travel; the last step has no next keys, and its value rows the whole
    // step; in between, value rows travel under the first half and keys under the second.
    auto sweep_step = [&](auto values, auto &&blocks, const bf16x8 (&a)[kMB][D / 16], bf16x8 (&nx)[kMB][D / 16], int kb,
                          int kb_next, bool first, bool last) {
        // (through an opaque move: addresses are formed in each step, not kept and spilled)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        if constexpr (!decltype(values)::value) {
            load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            blocks(a, kb, 0, NB);
        } else {
            constexpr int NB1 = NB / 4;  // (the first keys are there before the first value rows)
            if (!first) load_values(kb, lane, nx);
            __builtin_amdgcn_sched_barrier(0);
            blocks(a, kb, 0, NB1);
            __builtin_amdgcn_sched_barrier(0);
            if (first) {
                store_norms(nx, kb, lane);
                __builtin_amdgcn_sched_barrier(0);
                load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            }
            __builtin_amdgcn_sched_barrier(0);
            blocks(a, kb, NB1, NB / 2);
            __builtin_amdgcn_sched_barrier(0);
            if (!first && !last) {
                store_norms(nx, kb, lane);
                __builtin_amdgcn_sched_barrier(0);
                load_a<D>(kbase, g.ks[2], kb_next, key_end, lane, nx);
            }
            __builtin_amdgcn_sched_barrier(0);
            blocks(a, kb, NB / 2, NB);
            __builtin_amdgcn_sched_barrier(0);
            if (!first && last) store_norms(nx, kb, lane);
        }
    };
    // the column sums of the range, the last step first, its keys in a0 already
    auto second_sweep = [&](float ginv) {
        const int lane = threadIdx.x & 63;
        // (one base for what a lane reads per block: scale, position, normaliser)
        int at = lane & 31;
        asm volatile("" : "+v"(at));
        const float *meta = sLam + at;
        auto step = [&](const bf16x8 (&a)[kMB][D / 16], bf16x8 (&nx)[kMB][D / 16], int i) {
            const int kb = kb_of(i);
            int ln = threadIdx.x & 63;
            asm volatile("" : "+v"(ln));
            const int my_v = ((ln >> 4) & 1) * 8 + ((ln >> 3) & 1) * 4 + ((ln >> 2) & 1) * 2 + ((ln >> 1) & 1);
            float gam[kMB];
            if (PRIOR && !in_lds) {  // (in the scores' places, which nobody else writes or reads)
#pragma unroll
                for (int mb = 0; mb < kMB; ++mb)
                    gam[mb] = scores[(int64_t)z * g.n + min(acc_key(kb, mb, my_v, ln), key_end - 1)];
            }
            f32x16 col[kMB];
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) col[mb][v] = 0.f;
            auto blocks = [&](const bf16x8 (&ak)[kMB][D / 16], int kbb, int nb0, int nb1) {
                if (kbb >= key_end) return;  // (a wave past the range's ragged end)
                if (kbb + kWaveKeys - 1 <= tile_min) {
                    // all rows of the tile see all 64 keys: no masks, no skipped blocks
                    bf16x8 qf = query_fragment<D, NB>(sQ, nb0, 0, lane);
#pragma unroll
                    for (int nb = nb0; nb < nb1; ++nb) {
                        f32x16 acc[kMB];
                        // (scale and normaliser of the lane's row from LDS in each block: the registers are needed)
                        const float lam = meta[nb * 32], L = meta[2 * S::ROWS + nb * 32];
                        mma_block_stream<D, NB>(ak, sQ, nb, nb + 1 < nb1 ? nb + 1 : nb0, lane, qf, acc);
                        colsum_update<false>(acc, lam, L, 0, kbb, lane, col);
                    }
                    return;
                }
#pragma unroll
                for (int nb = nb0; nb < nb1; ++nb) {
                    if (uniform(sBlk[nb]) < kbb) continue;
                    f32x16 acc[kMB];
                    mma_block<D, NB>(ak, sQ, nb, lane, acc);
                    const float lam = meta[nb * 32], L = meta[2 * S::ROWS + nb * 32];
                    if (kbb + kWaveKeys - 1 > uniform(sBlk[NB + nb]))
                        colsum_update<true>(acc, lam, L, ((const int *)meta)[S::ROWS + nb * 32], kbb, lane, col);
                    else
                        colsum_update<false>(acc, lam, L, 0, kbb, lane, col);
                }
            };
            sweep_step(std::false_type{}, blocks, a, nx, kb, kb_of(i - 1), i == nsteps - 1, i == 0);
            float tot[kMB];
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb) tot[mb] = fold16_over32(col[mb], ln);
            if constexpr (NT == 2) {
                // the second tile's sums meet the first's (two steps' places: one barrier a step)
                float *sc = sCol + (i & 1) * 4 * kWaveKeys + kw * kWaveKeys;
                if (tile == 1 && (ln & 1) == 0) {
#pragma unroll
                    for (int mb = 0; mb < kMB; ++mb) sc[acc_key(0, mb, my_v, ln)] = tot[mb];
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (tile == 0) {
#pragma unroll
                    for (int mb = 0; mb < kMB; ++mb) tot[mb] += sc[acc_key(0, mb, my_v, ln)];
                }
            }
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb) {
                const int j = acc_key(kb, mb, my_v, ln);
                if ((ln & 1) || tile || j >= key_end) continue;
                const float gm = PRIOR ? (in_lds ? sGam[j - key_begin] : gam[mb]) : 1.f;
                scores[(int64_t)z * g.n + j] = PRIOR ? tot[mb] * prior_factor(gm, ginv) : tot[mb];
            }
        };
        for (int i = nsteps - 1; i >= 0; i -= 2) {
            step(a0, a1, i);
            if (i == 0) break;
            step(a1, a0, i - 1);
        }
    };
    // the prior of the range from its norms (kept: of the own one); the wave's largest gamma
    auto pool_range = [&](const PriorHalo<D> &halo, int tid, bool kept) {
        float gm;
        if (in_lds) {
            const float hn = halo.norm();
            if (halo.valid && tid % PriorHalo<D>::CPR == 0) sN[halo.pos - max(0, key_begin - (g.pool - 1) / 2)] = hn;
            __syncthreads();
            gm = pool_norms(g, key_begin, key_end, sN, sGam, tid, 512);
        } else {
            __syncthreads();  // (the statistics' LDS becomes the norms')
            gm = pool_norms_of_range<D, 512>(g, z, key_begin, key_end, nu_g, halo, sNu, tid, [&](int j, float gam) {
                if (kept) scores[(int64_t)z * g.n + j] = gam;  // (another's range may have its scores already)
            });
        }
        return wave_max(gm);
    };
    auto largest = [&]() {
        return fmaxf(fmaxf(fmaxf(sMax[0], sMax[1]), fmaxf(sMax[2], sMax[3])),
                     fmaxf(fmaxf(sMax[4], sMax[5]), fmaxf(sMax[6], sMax[7])));
    };
    for (int part = own;;) {
        // (through an opaque move, what depends on the thread is formed in the loop and not kept in
        // registers across it; it nearly always runs once)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        if (part == 0 && tid == 511) count.look(x, z);
        set_range(part);
        set_up(tid, 0);
        __syncthreads();
        int at = lane & 31;
        asm volatile("" : "+v"(at));
        const float *meta = sLam + at;
        float m[NB], s[NB], u = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            m[nb] = -INFINITY;
            s[nb] = 0.f;
        }
        auto blocks = [&](const bf16x8 (&a)[kMB][D / 16], int kb, int nb0, int nb1) {
            if (kb >= key_end) return;  // (a wave past the range's ragged end)
            if (kb + kWaveKeys - 1 <= tile_min) {
                bf16x8 qf = query_fragment<D, NB>(sQ, nb0, 0, lane);
#pragma unroll
                for (int nb = nb0; nb < nb1; ++nb) {
                    f32x16 acc[kMB];
                    const float lam = meta[nb * 32];
                    mma_block_stream<D, NB>(a, sQ, nb, nb + 1 < nb1 ? nb + 1 : nb0, lane, qf, acc);
                    stats_update<false, false>(acc, lam, 0, kb, lane, m[nb], s[nb], u);
                }
                return;
            }
#pragma unroll
            for (int nb = nb0; nb < nb1; ++nb) {
                if (uniform(sBlk[nb]) < kb) continue;  // nothing of this block sees these keys
                f32x16 acc[kMB];
                mma_block<D, NB>(a, sQ, nb, lane, acc);
                const float lam = meta[nb * 32];
                if (kb + kWaveKeys - 1 > uniform(sBlk[NB + nb]))
                    stats_update<true, false>(acc, lam, ((const int *)meta)[S::ROWS + nb * 32], kb, lane, m[nb], s[nb], u);
                else
                    stats_update<false, false>(acc, lam, 0, kb, lane, m[nb], s[nb], u);
            }
        };
        for (int i = 0; i < nsteps; i += 2) {
            sweep_step(std::bool_constant<PRIOR != 0>{}, blocks, a0, a1, kb_of(i), kb_of(i + 1), i == 0, i + 1 == nsteps);
            if (i + 1 >= nsteps) break;
            sweep_step(std::bool_constant<PRIOR != 0>{}, blocks, a1, a0, kb_of(i + 1), kb_of(i + 2), false, i + 2 == nsteps);
        }
        if (part == 0 && tid == 511) count.start(x, z);
        PriorHalo<D> halo;
        if (PRIOR) halo.request(g, vbase, key_begin, key_end, tid);  // travels while the statistics are reduced
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float m2, s2;
            from_other_half(m[nb], s[nb], m2, s2);
            merge_stats(m[nb], s[nb], m2, s2);
            if (lane < 32) sRed[wave * W::TROWS + nb * 32 + lane] = make_float2(m[nb], s[nb]);
        }
        if (part == 0 && wave == 7) count.started(x);
        __syncthreads();
        if (tid < W::ROWS) {
            float M = -INFINITY, sum = 0.f;
            const float2 *src = sRed + (NT == 2 ? tid / W::TROWS * 4 * W::TROWS : 0) + tid % W::TROWS;
#pragma unroll
            for (int wv = 0; wv < W::KW; ++wv) merge_stats(M, sum, src[wv * W::TROWS].x, src[wv * W::TROWS].y);
            put_rows(rows, part * (W::ROWS / 2), tid, M + log2f(sum));
        }
        if (PRIOR) {
            const float gm = pool_range(halo, tid, part == own);
            if (lane == 0) priors.put(part * 8 + wave, gm, 0.f);
        }
        __syncthreads();
        int missing = merge_parts<W::TROWS, W::KW>(rows, tile * (W::TROWS / 2), W::ROWS / 2, nparts, own, x.looks,
                                               sRed + wave * W::TROWS, kw, lane);
        if (PRIOR) {
            float gm;
            missing = min(missing, largest_of<8>(priors, nparts, own, x.looks, tid, 512, gm));
            if (lane == 0) sMax[wave] = gm;
        }
        missing = least_missing(missing);
        if (lane == 0) sMissing[wave] = missing;
        count.arrived(x);
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < 8; ++wv) missing = min(missing, sMissing[wv]);
        missing = uniform(missing);
        if (missing == INT32_MAX && part == own) break;
        // somebody is not there: done here (and no more waiting); in the end the own part again, whose
        // prior the LDS has to hold
        part = missing != INT32_MAX ? missing ^ own : own;
        x.looks = 0;
        __syncthreads();
    }
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == 511) count.arrive(x, z);
    load_a<D>(kbase, g.ks[2], kb_of(nsteps - 1), key_end, lane, a0);
    if (tid < W::ROWS) {
        float M = -INFINITY, sum = 0.f;
        const int t = tid / W::TROWS, row = tid % W::TROWS;
        const float2 *src = sRed + (NT == 2 ? t * 4 * W::TROWS : 0) + row;
#pragma unroll
        for (int wv = 0; wv < W::KW; ++wv) merge_stats(M, sum, src[wv * W::TROWS].x, src[wv * W::TROWS].y);
        // (rows past the last one add nothing)
        ((float *)(smem + t * S::stride + S::q_bytes) + 2 * S::ROWS)[row] = tid < g.R ? M + log2f(sum) : INFINITY;
    }
    __syncthreads();
    second_sweep(PRIOR ? prior_inverse(largest()) : 1.f);
    if (leave(x, z, nparts, count, tid == 511, sMissing + 1)) {
        Words::take_away(stats + (int64_t)z * nparts * (W::ROWS / 2), nparts * (W::ROWS / 2), tid, 512);
        if (PRIOR) Words::take_away(maxima + (int64_t)z * nparts * 8, nparts * 8, tid, 512);
    }
}

// ---------------------------------------------------------------- launch --
template <int D, int NB, int NT, int STEPS, int PRIOR>
static hipError_t launch_hold(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, char *w, float *scores,
                              hipStream_t st) {
    using H = HoldSmem<D, NB, NT, STEPS * kWgKeys, PRIOR != 0>;
    const auto kernel = window_hold_kernel<D, NB, NT, STEPS, PRIOR>;
    if (H::bytes > 64 * 1024) {
        static DeviceOnce once;
        const hipError_t e = device_once(once, [kernel] {
            return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)H::bytes);
        });
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(pl.Z * pl.win_parts)), dim3(256 * NT), H::bytes, st, g, pl.win_parts, x,
                       (u32x4 *)(w + pl.off_wstats), (u32x4 *)(w + pl.off_wmax), scores);
    return hipGetLastError();
}

template <int D, int NB, int NT, int PRIOR>
static hipError_t launch_stream(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, char *w, float *scores,
                                hipStream_t st) {
    using W = StreamSmem<D, NB, NT>;
    const auto kernel = window_stream_kernel<D, NB, NT, PRIOR>;
    static DeviceOnce once;
    const hipError_t e = device_once(once, [kernel] {
        return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)W::bytes);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(pl.Z * pl.win_parts)), dim3(512), W::bytes, st, g, pl.win_parts,
                       pl.win_keys, x, (u32x4 *)(w + pl.off_wstats), (u32x4 *)(w + pl.off_wmax),
                       (float *)(w + pl.off_wnu), scores);
    return hipGetLastError();
}

template <int D, int PRIOR>
static hipError_t launch_d(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, char *w, float *scores,
                           hipStream_t st) {
    const int steps = pl.win_keys / kWgKeys;
#define AHA_HOLD(NB, NT, STEPS)                                                                 \
    if (pl.win_hold && pl.win_nb == NB && pl.win_tiles == NT && steps == STEPS) \
        return launch_hold<D, NB, NT, STEPS, PRIOR>(g, pl, x, w, scores, st);
#define AHA_STREAM(NB, NT)                                            \
    if (!pl.win_hold && pl.win_nb == NB && pl.win_tiles == NT) \
        return launch_stream<D, NB, NT, NT == 2 && PRIOR ? kValuesCached : PRIOR>(g, pl, x, w, scores, st);
    AHA_HOLD(1, 1, 4) AHA_HOLD(1, 1, 1) AHA_HOLD(1, 1, 2) AHA_HOLD(2, 1, 1) AHA_HOLD(2, 1, 2) AHA_HOLD(3, 1, 1)
    AHA_HOLD(4, 1, 1) AHA_HOLD(3, 2, 1) AHA_HOLD(4, 2, 1)
    if constexpr (D == 64) { AHA_STREAM(4, 1) AHA_STREAM(8, 1) }  // (d = 128: held, or two launches; score_share.hip)
    AHA_STREAM(6, 1) AHA_STREAM(6, 2)
#undef AHA_HOLD
#undef AHA_STREAM
    return hipErrorInvalidValue;
}

int stream_keys_in_lds(int d, int nb, int tiles) {
    if (d == 128) return tiles == 2 ? StreamSmem<128, 6, 2>::KEYS : StreamSmem<128, 6, 1>::KEYS;
    if (tiles == 2) return StreamSmem<64, 6, 2>::KEYS;
    return nb == 4 ? StreamSmem<64, 4, 1>::KEYS : nb == 6 ? StreamSmem<64, 6, 1>::KEYS : StreamSmem<64, 8, 1>::KEYS;
}

hipError_t launch_score_window(const ScoreGeom &g, const PrefillPlan &pl, void *ws, const ExchangeCall &call,
                               float *scores, hipStream_t st) {
    char *w = (char *)ws;
    const Exchange x{(uint64_t *)(w + pl.off_wwords), call.tag, call.looks, call.replayed};
    auto launch = [&](auto prior) {
        constexpr int PRIOR = decltype(prior)::value;
        return g.d == 64 ? launch_d<64, PRIOR>(g, pl, x, w, scores, st) : launch_d<128, PRIOR>(g, pl, x, w, scores, st);
    };
    if (!g.value_prior) return launch(std::integral_constant<int, kNoValues>{});
    return g.v_once ? launch(std::integral_constant<int, kValuesOnce>{}) : launch(std::integral_constant<int, kValuesCached>{});
}

}  // namespace aha
