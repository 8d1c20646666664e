// C ABI of the AhaKV eviction path: argument checks, workspace layout and
// kernel launches.  Every check runs on the host before anything is
// enqueued, so the error paths need no GPU.
#include <stdarg.h>
#include <stdio.h>

#include <algorithm>
#include <atomic>
#include <chrono>

#include "aha_host.h"

namespace aha {

static thread_local char g_err[512] = "";
static thread_local hipEvent_t g_stage_ev[4] = {nullptr, nullptr, nullptr, nullptr};
static thread_local bool g_stage_on = false;

static hipError_t stage(int i, hipStream_t st) {
    return g_stage_on ? hipEventRecord(g_stage_ev[i], st) : hipSuccess;
}

// Looks at the other workgroups' parts before a workgroup does missing ones itself, at most: 1.4 us each
// (fewer: patience).
constexpr int32_t kLooks = 4000;

static int32_t fail(int32_t code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int esize(int dtype) { return dtype == AHA_BF16 ? 2 : 4; }

// Checks shared by all entry points.
static int32_t check_common(const aha_params *p) {
    if (!p) return fail(AHA_ERR_INVALID_ARG, "params is null");
    if (p->batch < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1)
        return fail(AHA_ERR_INVALID_ARG, "batch, n_q_heads and n_kv_heads must be >= 1");
    if (p->n_q_heads % p->n_kv_heads != 0)
        return fail(AHA_ERR_INVALID_ARG, "n_q_heads (%d) is not a multiple of n_kv_heads (%d)",
                    p->n_q_heads, p->n_kv_heads);
    if ((int64_t)p->batch * p->n_kv_heads > 65535)  // a grid's y dimension in several launches
        return fail(AHA_ERR_UNSUPPORTED, "batch * n_kv_heads (%lld) exceeds 65535",
                    (long long)p->batch * p->n_kv_heads);
    if (p->dtype != AHA_F32 && p->dtype != AHA_BF16)
        return fail(AHA_ERR_INVALID_ARG, "dtype %d is neither AHA_F32 nor AHA_BF16", p->dtype);
    if (p->head_dim != 64 && p->head_dim != 128)
        return fail(AHA_ERR_UNSUPPORTED, "head_dim %d: only 64 and 128 are built", p->head_dim);
    if (p->budget < 1) return fail(AHA_ERR_INVALID_ARG, "budget must be >= 1");
    if (p->budget > 1 << 30) return fail(AHA_ERR_UNSUPPORTED, "budget beyond 2^30");
    if (p->recent < 0 || p->recent > p->budget)
        return fail(AHA_ERR_INVALID_ARG, "recent (%d) must lie in [0, budget=%d]", p->recent,
                    p->budget);
    if (p->scale_mode != AHA_SCALE_FIXED && p->scale_mode != AHA_SCALE_ADAPTIVE)
        return fail(AHA_ERR_INVALID_ARG, "scale_mode %d is unknown", p->scale_mode);
    if (p->scale_mode == AHA_SCALE_FIXED && !(p->fixed_scale >= 0.f))
        return fail(AHA_ERR_INVALID_ARG, "fixed_scale must be >= 0");
    if (p->sink < 0 || (int64_t)p->sink + p->recent > p->budget)
        return fail(AHA_ERR_INVALID_ARG, "sink (%d) must be >= 0 and sink + recent (%d) <= budget (%d)",
                    p->sink, p->recent, p->budget);
    if (p->decode_value_prior != 0 && p->decode_value_prior != 1)
        return fail(AHA_ERR_INVALID_ARG, "decode_value_prior must be 0 or 1");
    if (p->reserved != 0) return fail(AHA_ERR_INVALID_ARG, "reserved must be 0");
    return AHA_OK;
}

static int32_t check_stride(const char *name, const int64_t s[3], int dtype, int d) {
    const int a = 16 / esize(dtype);
    for (int t = 0; t < 3; ++t)
        if (s[t] < 0 || s[t] % a != 0)
            return fail(AHA_ERR_INVALID_ARG, "%s_stride[%d]=%lld must be a non-negative multiple of %d elements",
                        name, t, (long long)s[t], a);
    if (s[2] < d)
        return fail(AHA_ERR_INVALID_ARG, "%s_stride[2]=%lld is smaller than head_dim", name,
                    (long long)s[2]);
    return AHA_OK;
}

static int32_t check_prefill(const aha_params *p, bool need_strides) {
    int32_t rc = check_common(p);
    if (rc) return rc;
    if (p->seq_len < 1) return fail(AHA_ERR_INVALID_ARG, "seq_len must be >= 1");
    if (p->seq_len > 1 << 30) return fail(AHA_ERR_UNSUPPORTED, "seq_len beyond 2^30");
    if (p->budget > p->seq_len)
        return fail(AHA_ERR_INVALID_ARG, "budget (%d) exceeds seq_len (%d)", p->budget, p->seq_len);
    if (p->window < 1 || p->window > p->seq_len)
        return fail(AHA_ERR_INVALID_ARG, "window (%d) must lie in [1, seq_len=%d]", p->window,
                    p->seq_len);
    if (p->value_prior != 0 && p->value_prior != 1)
        return fail(AHA_ERR_INVALID_ARG, "value_prior must be 0 or 1");
    if (p->value_prior && (p->pool_kernel < 1 || p->pool_kernel > 255 || p->pool_kernel % 2 == 0))
        return fail(AHA_ERR_INVALID_ARG, "pool_kernel (%d) must be odd and in [1, 255]",
                    p->pool_kernel);
    if ((int64_t)(p->n_q_heads / p->n_kv_heads) * p->window > (int64_t)1 << 30)
        return fail(AHA_ERR_UNSUPPORTED, "group * window is too large");
    if (p->score_pool < 0 || p->score_pool > 255 || (p->score_pool > 1 && p->score_pool % 2 == 0))
        return fail(AHA_ERR_INVALID_ARG, "score_pool (%d) must be 0 or odd and in [1, 255]",
                    p->score_pool);
    if (need_strides) {
        if ((rc = check_stride("q", p->q_stride, p->dtype, p->head_dim))) return rc;
        if ((rc = check_stride("k", p->k_stride, p->dtype, p->head_dim))) return rc;
        if ((rc = check_stride("v", p->v_stride, p->dtype, p->head_dim))) return rc;
    }
    return AHA_OK;
}

// Compaction reads K, V, the scores and the index list: only what those need is checked.
static int32_t check_compact(const aha_params *p) {
    int32_t rc = check_common(p);
    if (rc) return rc;
    if (p->seq_len < 1) return fail(AHA_ERR_INVALID_ARG, "seq_len must be >= 1");
    if (p->seq_len > 1 << 30) return fail(AHA_ERR_UNSUPPORTED, "seq_len beyond 2^30");
    if (p->budget > p->seq_len)
        return fail(AHA_ERR_INVALID_ARG, "budget (%d) exceeds seq_len (%d)", p->budget, p->seq_len);
    if ((rc = check_stride("k", p->k_stride, p->dtype, p->head_dim))) return rc;
    return check_stride("v", p->v_stride, p->dtype, p->head_dim);
}

static int32_t check_ptr(const char *name, const void *ptr, size_t align) {
    if (!ptr) return fail(AHA_ERR_INVALID_ARG, "%s is null", name);
    if ((uintptr_t)ptr % align != 0)
        return fail(AHA_ERR_INVALID_ARG, "%s is not %zu-byte aligned", name, align);
    return AHA_OK;
}

static ScoreGeom make_geom(const aha_params *p, const void *q, const void *k, const void *v) {
    ScoreGeom g{};
    g.q = q; g.k = k; g.v = v; g.rows = nullptr;
    for (int t = 0; t < 3; ++t) { g.qs[t] = p->q_stride[t]; g.ks[t] = p->k_stride[t]; g.vs[t] = p->v_stride[t]; }
    g.batch = p->batch; g.Hq = p->n_q_heads; g.Hkv = p->n_kv_heads; g.G = g.Hq / g.Hkv;
    g.d = p->head_dim; g.n = p->seq_len; g.r = p->window; g.R = g.G * g.r;
    g.budget = p->budget; g.scale_mode = p->scale_mode; g.fixed_scale = p->fixed_scale;
    g.lambda_floor = p->lambda_floor; g.value_prior = p->value_prior; g.pool = p->pool_kernel;
    g.dtype = p->dtype;
    return g;
}

// Key ranges of a problem for workgroups of which the chip holds `resident` at once: in rounds of the whole
// chip, the number of ranges with the shortest sum over the rounds of a range's steps (of `step` keys) and
// its set-up and exchange, about as long as a step.  Ranges have at most `most_keys`, a multiple of `step`.
// `whole`: a round counts the problems it holds whole; those that begin at its end keep their workgroups waiting for
// the next one (given normalisers, 8 heads x 1048576 keys x 256 rows 1117 us in ranges of 6656 keys, 158 to a problem, 875 in
// 256 of 4096; 420 shapes 1.009 times as fast on average, none slower).  The two sweeps' ranges are the same either way.
static void best_ranges(int64_t Z, int64_t n, int64_t step, int64_t resident, int64_t most_keys, bool whole, int64_t &parts,
                        int64_t &keys) {
    const int64_t all = (n + step - 1) / step;
    int64_t best = INT64_MAX;
    const int64_t least = (n + most_keys - 1) / most_keys;
    parts = least;
    for (int64_t c = least; c <= all && c <= 256; ++c) {
        const int64_t held = c < resident ? resident / c : 1;  // whole problems
        const int64_t rounds = whole ? (Z + held - 1) / held : (Z * c + resident - 1) / resident;
        const int64_t sum = rounds * ((all + c - 1) / c + 1);
        if (sum < best) best = sum, parts = c;
    }
    keys = (all + parts - 1) / parts * step;
    parts = (n + keys - 1) / keys;
}

// Workgroups of which the chip holds two per CU at once.  A problem never has more ranges than that: those that
// run would wait for those that cannot start (8 x 300000 x 64 rows, 586 ranges: 56 ms).
constexpr int64_t kHeldAtOnce = 512;
constexpr int64_t kSweptSteps = 800;  // steps of 256 keys in all from which 65 to 128 rows, d = 64, are swept twice
// Exponentials held in several rounds of the whole chip, nb blocks of rows: up to which number of ranges that is the faster
// one.  The workgroups of a problem that begins at the end of a round wait for the next one, and every range reads
// all ranges' statistics, so it costs more the more ranges there are and the more problems share them (`shared`); two launches
// leave their own last round nearly empty unless their workgroups are just the chip's 512 (`even`).  us otherwise (two launches; d = 64 and
// more than 64 rows the two sweeps), held, over 1450 shapes of 3 to 500 ranges, 2 to 296 heads:
//  - up to 32 rows: 1.5 times as fast on average (hardly more than one round is not taken, but in ranges of two steps, d = 128 with a
//    prior, up to 256 of them, at any number of rounds: 33 x 18 62.5, 38.0; 5 x 202 85.3, 68.7; 8 x 256 139, 109; 64 x 256 1172, 836; 3 x
//    330 72, 73; 16 x 400 447, 463);
//  - d = 128, 33 to 64 rows: up to 256: 16 x 101 72.2, 58.3; 8 x 256 131, 113; 64 x 192 871, 727; more than that where uneven, or for two
//    heads: 24 x 280 1.23 times as fast; even 16 x 320 0.91;
//  - d = 128, 65 to 128 rows: 80 x 9 55.6, 32.3; uneven 37 x 145 261, 214; 21 x 150 150, 130, without a prior 48 x 115 1.02 times as
//    fast, 24 x 145 0.92; few heads in more: 6 x 180 70.9, 56.2, 5 x 256 1.10; 12 x 230 0.89; even 16 x 100 55.3, 52.2; 8 x 160 62.8, 56.3; 16
//    x 150 65.5, 71.0; 64 x 64 138, 136 (not taken); 32 x 150 174, 206;
//  - d = 64, 33 to 64 rows: uneven with a prior 15 x 140 92.7, 83.1, 27 x 180 1.03 times as fast, without 27 x 130 0.89, 9 x 145 1.09, 48
//    x 160 1.07; even 8 x 140 51.9, 49.2; 8 x 173 57.3, 60.5; 64 x 64 138, 133; without a prior 8 x 100 30.7, 25.2; 64 x 32 48.4, 46.2;
//    128 x 32 93.5, 99.1;
//  - d = 64, 65 to 128 rows: where the sweeps would not be taken either, 28 x 20 36.6, 21.1; 15 x 51 37.6, 25.3; 4 x 190 36.6, 33.4; 2 x
//    260 1.35 times as fast, x 390 0.86; 13 x 74 28.7, 36.2 (sweeps, held).
// Of 900 of them in two launches or held this takes 1.007 times the faster one's time on average.
static bool held_in_rounds(const aha_params *p, const PrefillPlan &pl, int nb, int per, int64_t parts, int64_t steps) {
    const bool even = (int64_t)pl.Z * pl.nchunks <= 512, prior = p->value_prior;
    const int64_t shared = parts * (pl.Z + 6);
    if (nb == 1) return per == 2 || (parts <= 128 && pl.Z * parts >= 600);
    if (p->head_dim == 128 && nb == 2) return parts <= (even && pl.Z > 2 ? 256 : kHeldAtOnce);
    if (p->head_dim == 128 && even) return parts <= 256 && (shared <= 2432 || (prior && parts <= 48));
    if (p->head_dim == 128) return parts <= 256 && (shared <= 2900 || parts <= (prior ? 170 : 100));
    if (nb > 2) return pl.Z * steps < kSweptSteps && shared <= 2100;
    if (even) return shared <= (prior ? 2112 : 1600) || (parts <= 64 && (prior || pl.Z * parts <= 2048));
    return shared <= 2400 || parts <= (prior ? 180 : pl.Z < 32 ? 122 : 160);
}

// Windowed bf16 scores in one launch.  Its layout starts where the one of two launches does, but may be longer: a
// call whose workspace does not hold it takes two launches.  Where, and which kernel, follows from the times of the
// score stage both ways over 400 shapes (1 to 512 rows, 1 to 256 KV heads, 400 to 65536 keys, d = 64 and 128), 1.30
// times as fast as two launches on average.  us in two launches, in one:
//  - up to 128 rows, exponentials held, where the ranges fit the chip at once (two workgroups per CU): 32 heads x
//    4113 keys x 32 rows 33.6, 25.6; 16 x 4823 x 63 26.2, 19.2; 2 x 631 x 63 (d = 64) 13.7, 10.0; 96 and 128 rows in up to
//    512 ranges: 1 x 131072 x 128 53.8, 39.5, 6 x 19416 x 96 32.6, 22.4, 1 x 25600 x 128 20.1, 12.6 (88 shapes 1.44 times as fast on
//    average, 1.18 at least).
//    In several rounds the exchange is waited for in each (held_in_rounds).
//  - 65 to 128 rows, d = 64, longer problems, swept twice: 6 x 46683 x 126 52.7, 36.3 (d = 128, bound by its
//    bytes: 8 x 29221 x 128 48.3, 48.9, not taken).
//  - 129 to 256 rows, held by eight waves where one workgroup per CU covers the problem (in several rounds 62 shapes take 1.4 times as long; 16 x 1117 x 152
//    22.9, 17.1; 32 x 1502 x 256 32.8, 20.4), else swept twice (24 x 32929 x 160 163, 126; 6 x 29092 x
//    256 68.5, 47.7; held in 32 x 1502 x 256 the sweeps' 37.4 become 22.2).
//  - 257 to 512 rows, two tiles, swept twice (64 x 940 x 315 46.7, 30.4, d = 64 35.3, 22.2; 8 x 9057 x 504 56.3, 42.6, d = 64
//    42.5, 37.6; 64 x 65536 x 512, d = 64 881, 877).
// Over 160 shapes of 129 to 512 rows, 700 to 65536 keys, 1 to 64 heads (two launches of several tiles: score_full.hip's) one
// launch is the slower one in three: 8 x 17721 x 224 without a prior 36.7, 38.1; 8 x 2567 x 384 31.3, 33.4; 1 x 1219 x 384, d =
// 64, 24.0, 25.0.
// Full tiles that are swept twice, waves that share the keys (win_share): us with the keys in each wave's registers,
// shared, d = 128: 8 heads x 24576 x 256 55.7, 48.0; 32 x 3000 x 256 38.4, 31.3; 8 x 12000 x 400 51.3, 42.5; 2 x
// 50000 x 512 52.3, 41.7; 64 x 700 x 512 38.8, 28.0; 2 x 30000 x 256 25.2, 25.2; 64 x 40000 x 256 457, 457; d = 64: 8 x
// 12000 x 512 39.5, 38.2; 64 x 6000 x 512 91.7, 79.8.  Not taken: d = 64, 8 x 24576 x 256 41.2, 41.7, x 224 39.9, 41.5
// (half the products per byte of LDS); tiles of 192 rows in places for 256, d = 128, 8 x 24576 x 160 45.8, 46.7.
static void plan_window(const aha_params *p, PrefillPlan &pl) {
    pl.win_nb = 0;
    const int64_t R = (int64_t)(p->n_q_heads / p->n_kv_heads) * p->window;
    if (p->dtype != AHA_BF16 || R > 512 || (p->value_prior && p->pool_kernel > 17)) return;
    const int blocks = (int)((R + 31) / 32);
    const int64_t steps = (p->seq_len + kP2Keys - 1) / kP2Keys;
    int64_t parts = 0, keys = 0;
    int nb = 0, tiles = 1;
    bool hold = false;
    if (blocks <= 4) {
        // the shortest ranges of which two per CU cover the problem, else the longest that can be held
        nb = blocks;
        int per = 1;
        // (four steps beside value rows take more registers than there are, d = 128: us of four and two, 16 heads x 25716 keys x 16
        // rows 59.2, 49.0; 173 x 2481 x 32 79.3, 50.0; 22 shapes 1.33 times as fast on average, without a prior 0.97; but longer problems,
        // in one round or in two of two steps: 3 x 168740 x 32 68.7, 73.2; 1 x 500000 71.0, two launches 91.7)
        const int most = nb == 2 || (p->head_dim == 128 && p->value_prior && (steps + 1) / 2 <= 256) ? 2 : 4;
        while (2 * per * nb <= 4 && 2 * per <= most && pl.Z * ((steps + per - 1) / per) > kHeldAtOnce) per *= 2;
        parts = (steps + per - 1) / per;
        keys = per * kP2Keys;
        hold = pl.Z * parts <= kHeldAtOnce || held_in_rounds(p, pl, nb, per, parts, steps);
        if (!hold && (blocks < 3 || p->head_dim != 64 || pl.Z * steps < kSweptSteps)) return;
        if (!hold) nb = 4;
    } else if (blocks <= 8) {
        hold = pl.Z * steps <= 256;
        nb = hold ? (blocks + 1) / 2 : (blocks + 1) / 2 * 2;
        tiles = hold ? 2 : 1;
        parts = steps;
        keys = kP2Keys;
    } else {
        tiles = 2;
        nb = blocks <= 12 ? 6 : 8;
    }
    if (!hold) best_ranges(pl.Z, p->seq_len, 512 / tiles, 256, INT64_MAX / 2, false, parts, keys);
    if (pl.Z * parts > 1 << 30 || parts >= 1 << 19) return;
    pl.win_nb = nb;
    pl.win_tiles = tiles;
    pl.win_hold = hold;
    pl.win_share = !hold && nb == 8 && (p->head_dim == 128 || tiles == 2);
    pl.win_parts = (int)parts;
    pl.win_keys = (int)keys;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes, 256); return at; };
    pl.off_wstats = take(8 * (size_t)pl.Z * parts * tiles * nb * 32);  // (words of 16 bytes: two values and the tag)
    // (a word per wave, or per range where the waves share the keys)
    if (p->value_prior) pl.off_wmax = take(16 * (pl.win_share ? 1 : hold ? 4 * tiles : 8) * (size_t)pl.Z * parts);
    pl.off_wwords = take(kExchangeBytes * (size_t)pl.Z);
    if (!hold && p->value_prior &&
        keys > (pl.win_share ? share_keys_in_lds(p->head_dim, tiles) : stream_keys_in_lds(p->head_dim, nb, tiles)))
        pl.off_wnu = take(sizeof(float) * (size_t)pl.Z * p->seq_len);
    pl.win_bytes = off;
}

// Windowed bf16 scores from given normalisers in one launch (score_given.hip), likewise: one query
// tile, and a prior whose pooling halo a workgroup holds.  Against two launches 1.15 times as fast on average
// over 110 shapes (1 to 256 rows, 2 to 128 KV heads, 250 to 61000 keys), us in two, in one: 8 heads x 32768 keys x
// 256 rows 46.3, 39.7; 128 x 16384 x 64 198, 172; 32 x 4096 x 64 19.7, 19.1; 2 x 512 x 32 8.3, 7.2.  Not taken
// where it was the slower one: few heads in many ranges of a step or two, where the exchange is most of the time (8 x
// 6172 x 32, d = 64 9.5, 10.4; 4 x 60798 x 32 27.2, 29.5; 4 x 31485 x 128 21.6, 22.5), eight blocks of rows in
// steps of 512 keys for at most half of the CUs (8 x 3600 x 256 18.5, 19.9, 4 x 12000, d = 64 13.7, 15.4; not 8 x
// 12000 23.9, 22.3), and without a prior,
// of which a second launch would have to be saved, many steps of the largest tile (32 x 31856 x 256 86.3, 90.1, d = 64, 32 x 59762
// 104, 115; but 192 rows, which two launches pad to 256: 32 x 31856 97.8, 77.4, d = 64 64.5, 52.6).
static void plan_given(const aha_params *p, PrefillPlan &pl) {
    pl.given_nb = 0;
    const int64_t R = (int64_t)(p->n_q_heads / p->n_kv_heads) * p->window;
    if (p->dtype != AHA_BF16 || R > 256 || (p->value_prior && p->pool_kernel > 17)) return;
    const int blocks = (int)((R + 31) / 32);
    const int nb = blocks <= 2 ? blocks : (blocks + 1) / 2 * 2, resident = nb <= 4 ? 512 : 256;
    int64_t parts, keys;
    best_ranges(pl.Z, p->seq_len, nb <= 4 ? 256 : 512, resident, p->value_prior ? given_keys(p->head_dim, nb) : INT64_MAX / 2,
                p->value_prior, parts, keys);
    if (pl.Z * parts > 1 << 30 || parts > resident) return;  // (all of a problem's workgroups have to run at once)
    if (p->value_prior ? nb <= 4 && pl.Z <= 8 && parts > (nb <= 2 ? 24 : 50) : nb == 8 && (int64_t)pl.Z * p->seq_len > 1 << 19) return;
    if (p->value_prior && blocks == 8 && pl.Z * (((int64_t)p->seq_len + 511) / 512) <= 128) return;
    pl.given_nb = nb;
    pl.given_parts = (int)parts;
    pl.given_keys = (int)keys;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes, 256); return at; };
    if (p->value_prior) {
        pl.off_gmax = take(16 * (size_t)pl.Z * parts);
        pl.off_gwords = take(kExchangeBytes * (size_t)pl.Z);
    }
    pl.given_bytes = off;
}

// fp32 scores in one launch (score_hold_f32.hip), where its workgroups are on the chip at once.  Score stage, us in two launches, in one
// (88 shapes of 8 to 192 rows, 1 to 96 heads, 200 to 5000 keys: 1.25 times as fast on average):
//  - more than 32 rows: in ranges of 32 keys, up to 64 of them (4 heads x 1070 keys x 64 rows, d = 64 14.9, 10.5; 8 x 4
//    x 32 of 315, d = 64 17.4, 11.9; 1 x 1896 x 128, d = 64 17.5, 16.4, in ranges of 128 keys 19.5), else of 128 (2 x 4131 x 128, d = 64
//    23.4, 21.6, of 32 keys 25.7; 8 x 3048 x 64, d = 128 37.8, 20.2; 32 x 358 x 119 27.6, 26.4);
//  - up to 32 rows: in ranges of 128 keys (8 x 1224 x 8, d = 64 11.5, 10.8; 4 x 2968 x 32, d = 64 20.3, 11.1; 2 x 512 x 32 10.1, 10.3).
// Two launches give each row a workgroup, one launch each 128 keys all rows: with few rows, fewer of them than CUs and short prompts
// two take less time, unless on the matrix core (of 1725 shapes 584 such ones 1.11 times as long in one launch, the others 0.79; 8 x
// 1541 x 24, d = 128, 63 wide, matrix core, 0.7): 8 x 329 x 8, d = 64 9.1, 10.5; 4 x 500 x 16 9.5, 10.4; 1 x 300 x 8 9.0, 9.9; d = 128 with a
// prior 4 x 700 x 32 13.3, 13.9; pool widths above 17 (each range squares the halo's rows) 2 x 842 x 32, d = 64, 63 wide 1.05 times
// as long, 4 x 1273 x 8 1.13.
// But up to pool widths of 17, unless d = 128 with a prior, the host's launch is longer than the difference: us of the step with selection and
// compaction, 8 x 329 x 8 17.4, 16.9, 1 x 300 x 8 17.3, 15.6; in a captured graph 14.9, 16.9 and 14.3, 15.7.  So there
// captured calls take two launches.  (What is left of the difference in graphs comes from the words that a captured call takes
// away, exchange.h: 0.7 us.)
static void plan_hold_f32(const aha_params *p, PrefillPlan &pl) {
    pl.hold32_parts = 0;
    const int64_t R = (int64_t)(p->n_q_heads / p->n_kv_heads) * p->window, blocks = (R + 31) / 32;
    if (p->dtype != AHA_F32 || blocks > kHoldF32Blocks) return;
    const bool d64 = p->head_dim == 64, prior = p->value_prior, wide = prior && p->pool_kernel > 17;
    // below how many keys of few problems and rows two launches take less time
    int64_t least = d64 ? (prior ? 1500 - 35 * R : 0) : prior ? std::max<int64_t>(1000, 2000 - 35 * R) : 1350 - 35 * R;
    if (wide) least = 8 * std::max<int64_t>(least, 800) / 5;
    const bool few = pl.Z * R < (d64 || R > 8 ? 256 : 300) && ((int64_t)pl.Z * p->seq_len < 14000 || (R < 4 && prior));
    const bool longer = !pl.f32_mfma && ((few && p->seq_len < least && R <= (prior && (!d64 || wide) ? 64 : 32)) ||
                                         (!d64 && prior && blocks == 1 && (double)pl.Z * R * p->seq_len < 6e4));
    if (longer && (wide || (!d64 && prior))) return;
    pl.hold32_eager = longer;
    int64_t parts, keys = blocks == 1 ? 128 : 32;
    for (;; keys = 128) {
        parts = ((int64_t)p->seq_len + keys - 1) / keys;
        // workgroups that the chip holds at once
        const int64_t resident = hold_f32_lds(p->head_dim, (int)blocks, (int)keys) + kHoldF32Static <= 80 * 1024 ? 512 : 256;
        if (pl.Z * parts <= resident && (keys == 128 || parts <= 64)) break;
        if (keys == 128) return;
    }
    pl.hold32_keys = (int)keys;
    pl.hold32_parts = (int)parts;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes, 256); return at; };
    pl.off_h32stats = take(16 * (size_t)pl.Z * parts * R);
    pl.off_h32max = take(16 * (size_t)pl.Z * parts);
    pl.off_h32words = take(kExchangeBytes * (size_t)pl.Z);
    pl.hold32_bytes = off;
}

// Several query tiles (score_full.hip).
// Places of a query head: whole waves', unless the tiles become many more (their statistics use the room behind, which only
// the row statistics' output needs, too).  A further tile costs its products with all keys, whole waves save masks for the
// share r / n of them; where the chip holds all workgroups at once it costs nothing.  us with the rows' places in their order,
// and so: 16 x 8 heads x 263 of 4208 rows, d = 64, 9 tiles or 10, 77, 95 (not taken); 16 x 3 x 400 of 12822, 5 or 6, 158, 213
// (not taken), of 1941, d = 64, 40.4, 36.9; 1 x 3 x 1450 of 5800, d = 64, 17 or 18, 35.1, 30.8; 32 x 3 x 899 of 1168, 11 or 12,
// 87.8, 76.1; 4 x 4 x 4891 of 9782, d = 64, 77 either way, 345, 264.  (No more workgroups than a launch takes, 2^32 threads.)
// Parts of a pair's keys: as many as the chip holds at once, down to one or two steps each in the column sums, rather two
// where a CU gets two of them (32 x 7 heads x 160 rows 28.3 us, 31.0 with one); the row statistics leave a value per row and
// part, so no more of them than the workspace has chunks.  us in nchunks parts, and so: given normalisers, few pairs, parts of
// a step of 256 keys: 1 x 2 heads x 300 of 2676 rows, d = 64 15.7, 10.4, 2 x 1020 of 4080 21.4, 14.4; both kernels, 520 and
// more workgroups for 512 places: 8 x 2 x 1237 of 3711 67.8, 52.1, 8 x 2867 of 5734 90.6, 72.9.  Not taken: two parts for
// three, 4 x 7 x 4395, d = 64 138, 150, 8 x 3 x 4654 of 6050 264, 279.
static void plan_full(const aha_params *p, PrefillPlan &pl) {
    const int64_t G = p->n_q_heads / p->n_kv_heads, wave_rows = pl.NB * 8;
    pl.full_pr = p->window;
    pl.full_tiles = pl.n_qtiles;
    pl.full_parts = pl.full_sum_parts = pl.nchunks;
    if (pl.n_qtiles == 1) return;
    const int64_t padded = (p->window + wave_rows - 1) / wave_rows * wave_rows, tiles = (G * padded + pl.qtile - 1) / pl.qtile;
    const int64_t more = tiles - pl.n_qtiles, wgs = (tiles + 1) / 2 * pl.Z * pl.nchunks;
    if (4 * more <= pl.n_qtiles && (wgs <= 512 || (wgs < 1 << 24 && 5 * more * p->seq_len <= 2 * (int64_t)pl.n_qtiles * p->window))) {
        pl.full_pr = (int)padded;
        pl.full_tiles = (int)tiles;
    }
    const int64_t pairs = (int64_t)((pl.full_tiles + 1) / 2) * pl.Z, steps = (p->seq_len + kFullKeys - 1) / kFullKeys;
    const int64_t held = std::min(512 / pairs, std::max(2 * steps / 3, std::min(steps, 256 / pairs)));  // parts
    if (held >= pl.nchunks || (held >= 3 && steps >= 2 * held)) pl.full_sum_parts = (int)held;
    pl.full_parts = std::min(pl.nchunks, pl.full_sum_parts);
}

// Workspace layout of aha_prefill_scores.
static PrefillPlan plan_prefill(const aha_params *p) {
    PrefillPlan pl{};
    const int G = p->n_q_heads / p->n_kv_heads;
    const int64_t R = (int64_t)G * p->window;
    const int n = p->seq_len;
    pl.Z = p->batch * p->n_kv_heads;
    pl.n_vtiles = (n + kVTileRows - 1) / kVTileRows;
    if (p->dtype == AHA_BF16) {
        const int blocks = (int)((R + 31) / 32);
        pl.NB = blocks >= 8 ? 8 : blocks > 2 ? 4 : blocks;  // 1, 2, 4, 8
        if (blocks == 3) pl.NB = 4;
        pl.qtile = pl.NB * 32;
        pl.n_qtiles = (int)((R + pl.qtile - 1) / pl.qtile);
        // Work units: query tiles are paired (first with last, ...) so that in full
        // accumulation every pair sees about the same number of keys, and the key steps of
        // a pair are cut into `nchunks` parts so that about 512 workgroups (two per CU) exist.
        const int64_t npairs = (pl.n_qtiles + 1) / 2;
        const int64_t units = (int64_t)pl.Z * npairs;
        const int target_wgs = 512;
        int64_t want = (target_wgs + units - 1) / units;
        const int64_t steps = (n + kP2Keys - 1) / kP2Keys;          // 256-key steps of a full tile
        const int64_t pair_steps = pl.n_qtiles > 1 ? steps + 1 : steps;
        if (want > pair_steps) want = pair_steps;
        if (want < 1) want = 1;
        pl.nchunks = (int)want;
        pl.chunk_keys = (int)(((steps + want - 1) / want) * kP2Keys);
        // windowed pass 2 (one tile) walks over the same key ranges, several steps per workgroup
        pl.p2_keys = pl.chunk_keys;
        plan_full(p, pl);
    } else {
        pl.NB = 0;
        pl.qtile = 1;
        pl.n_qtiles = 1;
        pl.chunk_keys = n;
        pl.nchunks = 1;
        pl.p2_keys = kP2Keys;
        // The matrix core from this many (row, key) pairs on, unless its blocks of 32 rows would be
        // mostly empty; otherwise the vector ALU's smaller pieces of work are done sooner.  Both
        // passes, us on the vector ALU and the matrix core, d = 64: 131 K pairs (8 heads x 64 rows x 256
        // keys) 13.4, 13.7, 205 K (400 keys) 14.6, 14.5, 410 K (128 rows x 400) 21.3, 14.8, 1.1 M (128 x
        // 1100) 30.0, 19.7; 16 rows: 64 heads x 1100 keys 30.9, 33.9; 4 rows: 64 x 2000 25.3, 44.4.
        pl.f32_mfma = R >= 24 && (double)pl.Z * R * n >= 2e5;
        if (pl.f32_mfma) {
            const int64_t units = pl.Z * ((R + 31) / 32), steps = (n + 127) / 128;
            int64_t want = (512 + units - 1) / units;
            if (want > steps) want = steps;
            if (want > 16) want = 16;  // (every pass-2 wave folds them)
            pl.nchunks = (int)want;
        }
    }
    size_t off = 0;
    pl.off_rowL = off;  // fp32 path: log-sum-exp of every observed row
    const size_t rows = p->dtype == AHA_BF16 ? (size_t)pl.n_qtiles * pl.qtile : (size_t)R;
    if (p->dtype != AHA_BF16) off = align_up(off + sizeof(float) * (size_t)pl.Z * rows, 256);
    pl.off_partial = off;
    if (p->dtype == AHA_BF16)
        off = align_up(off + sizeof(float) * (size_t)pl.Z * rows * pl.nchunks, 256);
    else if (pl.f32_mfma)
        off = align_up(off + 2 * sizeof(float) * (size_t)pl.Z * ((R + 31) / 32 * 32) * pl.nchunks, 256);
    pl.off_partial_mean = off;  // aha_prefill_row_stats: per-chunk mean scaled logit
    if (p->dtype == AHA_BF16)
        off = align_up(off + sizeof(float) * (size_t)pl.Z * rows * pl.nchunks, 256);
    pl.off_gamma = off;
    off = align_up(off + sizeof(float) * (size_t)pl.Z * n, 256);
    pl.off_gblockmax = off;  // per-range maxima of the value prior: per tile, or per key chunk
    const size_t n_maxima = (size_t)(pl.n_vtiles > pl.nchunks ? pl.n_vtiles : pl.nchunks);
    off = align_up(off + sizeof(float) * (size_t)pl.Z * n_maxima, 256);
    // windowed bf16 scores: pass 1 forms the value prior itself (the pooling halo it gathers
    // at a range's ends is bounded: pool widths up to 17)
    pl.can_fold = p->dtype == AHA_BF16 && pl.n_qtiles == 1 && pl.NB <= 4 && p->pool_kernel <= 17;
    pl.bytes = off;
    plan_window(p, pl);
    plan_given(p, pl);
    plan_hold_f32(p, pl);
    return pl;
}

// Attention output of the observed rows: workgroups over (group of 32-row blocks, key range,
// problem); the key ranges' partials go through the workspace.
// bf16 has two forms: pairs of row blocks (steps of 128 keys, two workgroups per CU, about 512 in
// all) and, for d = 128 and five or more blocks, eight blocks that share their keys (steps of 64
// keys, one workgroup per CU).  Either runs in rounds of the whole chip, so its time goes with
// rounds * (steps of a range + set-up), and each further range costs the merge a little.  The set-ups
// (four steps and two and a half), the merge's share (a twentieth of a step) and the weight of a step (1 and 0.9) were
// fitted to both forms' times over 1 to 256 KV heads, 300 to 48000 keys and 5 to 32 blocks (570
// shapes): taking the form with the smaller sum is 1.149 times as fast as the first form throughout
// (the better of both, known beforehand, 1.159) and more than 3 % slower in 26 of them, 14 % at worst.
// us of first and second form, 8 blocks: 1 head x 48000 keys 28.5, 41.3 (64 workgroups), 8 x 16000
// 38.5, 37.7, 48 x 16000 203, 130; 5 blocks: 24 x 1000 29.6, 21.9.
// d = 64 always takes the first form: with half the products per byte read from LDS the second was
// 3 % slower on average over 586 such shapes, 40 % at worst.
static WindowAttnPlan plan_window_attn(const aha_params *p) {
    WindowAttnPlan pl{};
    const int64_t R = (int64_t)(p->n_q_heads / p->n_kv_heads) * p->window;
    const int64_t Z = (int64_t)p->batch * p->n_kv_heads;
    pl.n_blocks = (int)((R + 31) / 32);
    pl.nparts = 1;
    pl.nq = pl.n_blocks >= 2 ? 2 : 1;  // row blocks per workgroup
    if (p->dtype != AHA_BF16) return pl;  // fp32: one workgroup per row, no partials
    constexpr int64_t kMaxParts = 64;
    const int64_t groups = (pl.n_blocks + pl.nq - 1) / pl.nq, steps = (p->seq_len + 127) / 128;
    int64_t parts = (512 + Z * groups - 1) / (Z * groups);
    if (parts > steps) parts = steps;
    if (parts > kMaxParts) parts = kMaxParts;
    pl.nparts = (int)parts;
    if (p->head_dim == 128 && pl.n_blocks >= 5) {
        // (in twentieths of a step; two workgroups per CU: half a round per 256)
        int64_t best = 10 * ((Z * groups * parts + 255) / 256) * ((steps + parts - 1) / parts + 4) + parts;
        const int64_t wide_groups = (pl.n_blocks + 7) / 8, wide_steps = (p->seq_len + 63) / 64;
        for (int64_t n = 1; n <= kMaxParts && n <= wide_steps; ++n) {
            const int64_t sum = 9 * ((Z * wide_groups * n + 255) / 256) * (2 * ((wide_steps + n - 1) / n) + 5) + n;
            if (sum < best) { best = sum; pl.nparts = (int)n; pl.wide = true; }
        }
    }
    const size_t rows = (size_t)Z * pl.nparts * pl.n_blocks * 32;
    pl.off_ms = align_up(sizeof(float) * rows * p->head_dim, 256);
    pl.bytes = align_up(pl.off_ms + 2 * sizeof(float) * rows, 256);
    return pl;
}

// Whether a step with fewer than 128 (batch, KV head) problems gives every head to one workgroup
// all the same.  The split path streams the heads' caches with the whole chip but pays a second
// launch and the partials' round trip; one workgroup streams a head at the rate of its CU, which
// falls with the group (dots and weighted sums in the vector ALU).  So a single launch wins up to a
// size of the head, counted as its keys and values and 64 bytes of other work per slot, and the
// fewer ways a head would be split, the larger that size.  The table holds, in thousands of these
// bytes, where the two cross: steps of 2 to 127 heads with 100 to 8000 slots, d = 64 and 128, were timed
// both ways (us in one launch against split; fp32, d = 128, G = 1: 8 heads x 300 slots 9.4 and
// 10.2, 80 x 1000 21.0 and 23.3, 80 x 3000 56.1 and 50.9, 112 x 8000 203 and 188; bf16, d = 128,
// G = 4: 32 x 257 12.7 and 10.7, d = 64 9.85 and 9.81; 96 x 257 12.9 and 12.5, 112 x 801 21.6 and 18.6).
// Wider groups always split (bf16, d = 128, G = 8: 8 x 100 17.8 and 11.9, 112 x 257 18.9 and 14.1).
// Exactly 128 heads in groups of four: 128 x 257 13.0 and 13.1, d = 64 x 801 14.4 and 14.4, d = 128 x 801
// 20.9 and 19.1.
// `room`: the workspace holds the split.  Without it the steps of four query heads that were served in one launch and
// without a workspace while the split was the slower one (112 x 1000 25.0 and 26.0 us) still are.
static bool decode_one_launch(int dtype, int Z, int G, int d, int live, bool room) {
    if (G > 4) return false;
    const int ways = (256 + Z - 1) / Z;  // workgroups per head if split
    constexpr int kAny = INT32_MAX;
    static const int limit[2][4][4] = {   // G = 1 .. 4
        {{330, 290, 220, 200},            // fp32: seven and more ways,
         {870, 450, 410, 290},            // five and six,
         {1300, 1160, 870, 410},          // four,
         {2350, kAny, 3300, 1700}},       // three (86 heads and more)
        {{330, 224, 120, 96},             // bf16
         {480, 400, 170, 96},
         {1200, 800, 320, 96},
         {2350, kAny, 2350, 325}}};
    if (Z >= kDecodeSplitHeads) return G < 4 || (int64_t)live * (2 * d * esize(dtype) + 64) <= 250 * 1000;
    const int row = ways >= 7 ? 0 : ways >= 5 ? 1 : ways == 4 ? 2 : 3;
    const int64_t size = (int64_t)live * (2 * d * esize(dtype) + 64);
    const int most = !room && dtype == AHA_BF16 && G == 4 && row == 3 ? 580 : limit[dtype == AHA_BF16][row][G - 1];
    return size <= (int64_t)most * 1000;
}

// The most heads whose slots the matrix-core split stage divides.  Four or six splits of 128 heads fill the three
// slots of every CU; five of 129 do not, while one workgroup per head keeps more than half of the chip busy.
// With d = 128 and six and more query heads the split is the faster one all the same up to 144 heads (100 to
// 3100 slots: 1.11 times as fast on average, 3 % slower at worst).  us in one launch, split, d = 128: G = 8, 144
// heads x 300 slots 19.0, 16.4, x 801 24.8, 25.1, x 1200 32.9, 30.0, 160 x 801 25.3, 26.0, 192 x 1537 41.1, 43.6;
// G = 4, 128 x 801 22.1, 20.8, 129 x 801 22.4, 23.9; d = 64, G = 5, 128 x 801 14.7, 14.8, 129 x 801 15.1, 16.5.
static int most_split_heads(int G, int d) { return d == 128 && G >= 6 ? 144 : kDecodeSplitHeads; }

// Decode: split a head's slots over workgroups when there are too few heads to fill the GPU.
// A split workgroup keeps group * (slots of its range) dots and 4 * group * head_dim partial
// outputs in LDS; the number of splits is raised until that fits kDecodeSplitLds (the limit
// a launch may ask for without an attribute), and `fits` says whether kMaxDecodeSplit
// splits were enough.
//
// The matrix-core split stage (bf16, G >= 4) is resident three times per CU, so more splits than
// one workgroup per CU may pay, also for 128 heads and some more (most_split_heads); what matters is that the chip is
// evenly filled.  Its time goes with the slots per CU (64 of them, d = 128, weigh as much as a wave's block of 32
// slots) and the blocks of a wave one after the other; a further split costs the merge a twelfth of a
// block.  us of the step at the former count and at this rule's, d = 128, G = 8: 96 heads x 1537 slots 32.7
// (3 splits), 26.3 (5); 48 x 3073 33.7, 27.5; 128 x 1537 38.3 (one launch), 33.0 (4); over 156 shapes
// 1.064 times as fast on average.  `limit`: bytes of workspace there are; without room for the plan's
// the former count (and 128 heads in one launch).
static DecodePlan plan_decode(const aha_params *p, size_t limit = SIZE_MAX) {
    DecodePlan pl{};
    const int Z = p->batch * p->n_kv_heads, G = p->n_q_heads / p->n_kv_heads;
    const int live = p->budget + 1;
    // one workgroup per head: dots and output probabilities of all live slots in LDS
    const bool mfma = p->dtype == AHA_BF16 && G >= kDecodeMfmaGroup;
    const bool mfma_v = p->dtype == AHA_BF16 && G >= kDecodeMfmaValuesGroup;
    const size_t w_floats = decode_w_floats(G, live, p->head_dim, mfma, mfma_v);
    const size_t q_tile = mfma ? kDecodeQTileBytes(p->head_dim) : 0;
    const bool one_fits = (w_floats + (size_t)G * live) * 4 + q_tile <= kDecodeSingleLds;
    pl.fits = true;
    int nsplit = 1;
    if (Z < kDecodeSplitHeads) {
        nsplit = (256 + Z - 1) / Z;
        const int max_by_size = (live + 63) / 64;  // at least 64 slots per workgroup
        if (nsplit > max_by_size) nsplit = max_by_size;
        if (nsplit > kMaxDecodeSplit) nsplit = kMaxDecodeSplit;
        if (nsplit > 1) {
            const int64_t room = (int64_t)kDecodeSplitLds / 4 - 4 * (int64_t)G * p->head_dim;
            const int64_t max_sps = room / G;  // slots per split whose dots fit beside the outputs
            const int64_t need = max_sps > 0 ? (live + max_sps - 1) / max_sps : kMaxDecodeSplit + 1;
            if (need > nsplit) nsplit = need > kMaxDecodeSplit ? kMaxDecodeSplit : (int)need;
            if (need > kMaxDecodeSplit) pl.fits = false;
        }
    }
    pl.sps = (live + nsplit - 1) / nsplit;
    pl.nsplit = (live + pl.sps - 1) / pl.sps;
    // with `stats` floats behind every partial output; value prior inside the loop: the live slots'
    // value norms and their maximum per head
    const size_t norms = p->decode_value_prior ? sizeof(float) * ((size_t)Z * live + Z) : 0;
    auto layout = [&](int stats) {
        pl.off_part = pl.nsplit > 1 ? align_up(sizeof(float) * (size_t)Z * G * live, 256) : 0;
        const size_t partials = sizeof(float) * (size_t)Z * pl.nsplit * G * (p->head_dim + stats);
        pl.off_nu = pl.nsplit > 1 ? align_up(pl.off_part + partials, 256) : 0;
        return align_up(pl.off_nu + norms, 256);
    };
    pl.static_bytes = layout(2);
    pl.bytes = layout(kPartStats);
    bool room = pl.bytes <= limit;
    if (p->dtype == AHA_BF16 && G >= kDecodeSplitMfmaGroup && pl.fits &&
        (Z < kDecodeSplitHeads ? pl.nsplit > 1 : Z <= most_split_heads(G, p->head_dim) && one_fits)) {
        auto cost = [&](int sps, int ns) {
            const int64_t per_cu = ((int64_t)Z * ns + 255) / 256;
            return per_cu * sps * p->head_dim / (128. * 64.) + ((sps + 31) / 32 + 3) / 4 + 0.08 * ns;
        };
        const DecodePlan former = pl;
        double best = pl.nsplit > 1 ? 0.9 * cost(pl.sps, pl.nsplit) : 1e30;  // (left only for a clear gain)
        for (int n = 2; n <= kMaxDecodeSplit && Z * n <= 768 && n <= (live + 31) / 32; ++n) {
            const int sps = (live + n - 1) / n, ns = (live + sps - 1) / sps;
            if (ns > 1 && cost(sps, ns) < best) {
                best = cost(sps, ns);
                pl.sps = sps;
                pl.nsplit = ns;
            }
        }
        pl.bytes = layout(kPartStats);
        room = pl.bytes <= limit;
        if (!room) pl = former;
    }
    if (pl.nsplit > 1 && !(one_fits && pl.fits && decode_one_launch(p->dtype, Z, G, p->head_dim, live, room)))
        return pl;
    if (pl.nsplit <= 1 && !one_fits) pl.fits = false;
    pl.nsplit = 1;
    pl.sps = live;
    pl.bytes = layout(kPartStats);
    return pl;
}

static int32_t check_ws(const void *ws, size_t have, size_t need) {
    if (need == 0) return AHA_OK;
    if (!ws) return fail(AHA_ERR_WORKSPACE, "workspace is null (%zu bytes needed)", need);
    if ((uintptr_t)ws % 256 != 0) return fail(AHA_ERR_WORKSPACE, "workspace is not 256-byte aligned");
    if (have < need)
        return fail(AHA_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", have, need);
    return AHA_OK;
}

static int32_t hip_result(hipError_t e, const char *what) {
    if (e == hipSuccess) return AHA_OK;
    return fail(AHA_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace aha

using namespace aha;

extern "C" {

// Selection: the pooled scores, when the scores are smoothed first.
static size_t topk_ws_bytes(const aha_params *p) {
    if (p->score_pool <= 1) return 0;
    return align_up(sizeof(float) * (size_t)p->batch * p->n_kv_heads * p->seq_len, 256);
}

int32_t aha_workspace_bytes(const aha_params *p, size_t *out_bytes) {
    if (!out_bytes) return fail(AHA_ERR_INVALID_ARG, "out_bytes is null");
    if (p && p->seq_len == 0) {  // a caller of aha_decode_step only
        const int32_t rc = check_common(p);
        if (rc) return rc;
        *out_bytes = plan_decode(p).bytes;
        return AHA_OK;
    }
    int32_t rc = check_prefill(p, false);
    if (rc) return rc;
    const PrefillPlan pl = plan_prefill(p);
    *out_bytes = std::max({pl.bytes, pl.win_bytes, pl.given_bytes, pl.hold32_bytes, plan_decode(p).bytes, topk_ws_bytes(p)});
    return AHA_OK;
}

// Shared by aha_prefill_scores (lse == nullptr), aha_prefill_scores_lse and
// aha_prefill_scores_rows (rows != nullptr).

// A number that no other call of this process uses, for the exchanges inside a launch: the upper 44
// bits of a counter that starts anywhere, never zero.
static uint64_t next_tag() {
    static std::atomic<uint64_t> next{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() *
                                      0x9E3779B97F4A7C15u};
    for (;;) {
        const uint64_t t = next.fetch_add(1, std::memory_order_relaxed) << 20;
        if (t) return t;
    }
}
static thread_local int32_t g_looks = kLooks;

// `unknown`: for a stream that does not say.
static bool captured(hipStream_t st, bool unknown) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(st, &status);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess ? status != hipStreamCaptureStatusNone : unknown;
}
__global__ __launch_bounds__(256) void no_words_kernel(uint4 *words, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) words[i] = make_uint4(0u, 0u, 0u, 0u);
}
// A call of Z problems and `workgroups` in all, of which the chip holds `resident` at once, that exchanges words in the workspace's first
// `bytes`.  Captured calls are replayed with the same tag, and no word may outlive a replay.  A problem's last workgroup takes its
// words away, which it finds out by a count that all wait for at their end, and does alone: a launch that does it in front is shorter
// from some 6000 words on and in several rounds of the chip.  us of the score stage eager, replayed either way: 2 x 512 x 32, d = 64 8.5, 8.9,
// 10.5; 32 x 4096 x 64 18.9, 19.9, 21.1; 4 x 19793 x 224, d = 64, 5000 words 27.6, 30.3, 30.3; 1 x 131072 x 64 26.8, 32.1, 29.0; 1 x 60757 x
// 448, d = 64, 30000 words 37.7, 48.1, 40.2; 5 x 107065 x 48, d = 64, two rounds 37.8, 45.4, 40.4; 128 x 16384 x 64 203, 209, 207.
static hipError_t exchange_call(hipStream_t st, int looks, int64_t Z, int64_t workgroups, int64_t resident, void *workspace, size_t bytes,
                                ExchangeCall &call) {
    call = {0, looks, false};
    if (bytes == 0) return hipSuccess;  // (nothing to exchange)
    call.tag = next_tag();
    call.replayed = captured(st, true);
    const int64_t words = (int64_t)(bytes / 16);
    if (!call.replayed || (workgroups <= resident && words <= 6000 * Z)) return hipSuccess;
    call.replayed = false;
    hipLaunchKernelGGL(no_words_kernel, dim3((unsigned)std::min<int64_t>((words + 1023) / 1024, 512)), dim3(256), 0, st, (uint4 *)workspace, words);
    return hipGetLastError();
}

// Looks of a call of `workgroups` in all, of which the chip holds `resident` at once and each multiplies nb blocks of
// 32 rows with each of `steps` key blocks per wave for its part.  All of them at once: a few times what a part takes (set-up
// and exchange 15 us; a step its loads, 15 us with the whole chip loading, or its products, 2.5 us a
// block).  In several rounds some are waited for until a round ends.
static int patience(int64_t workgroups, int64_t resident, int64_t steps, int64_t nb) {
    const int64_t looks = (30 + steps * (20 + 10 * nb)) * (workgroups <= resident ? 1 : 8);
    return (int)(looks < g_looks ? looks : g_looks);
}
static int window_patience(const PrefillPlan &pl) {
    const bool wide = !pl.win_hold && pl.win_tiles == 1;  // 512 keys to a step
    return patience((int64_t)pl.Z * pl.win_parts, pl.win_hold && pl.win_tiles == 1 ? kHeldAtOnce : 256,
                    pl.win_keys / (wide ? 512 : 256), pl.win_nb);
}
static int given_patience(const PrefillPlan &pl) {
    const bool wide = pl.given_nb > 4;
    return patience((int64_t)pl.Z * pl.given_parts, wide ? 256 : 512, pl.given_keys / (wide ? 512 : 256), pl.given_nb);
}

// Whether the one-launch scores read the value rows past the caches, given the bytes of K and V.  Kept
// there they serve the gather of the retained rows, as long as the last-level cache (256 MB) has room for
// them; read past it they are faster.  us, through the caches and past them: 32 heads x 4096 keys (67 MB), the
// whole step 29.9, 31.0; 48 x 6846 (84 MB), scores 56.1, 47.5; 8 x 32768 (134 MB), step 89.9, 85.8; 128 x 16384
// (1.07 GB), step 347, 340.  With given normalisers the attention has just read them: 8 x 32768, step 118.7, 121.4.
static bool values_once(int64_t bytes, bool after_attention) {
    return bytes > (after_attention ? 200 * 1000 * 1000 : 80 * 1000 * 1000);
}

static int32_t prefill_scores_impl(const aha_params *p, const void *q, const void *k,
                                   const void *v, const float *lse, bool with_lse,
                                   const int32_t *rows, float *scores, void *workspace,
                                   size_t workspace_bytes, void *stream) {
    int32_t rc = check_prefill(p, true);
    if (rc) return rc;
    if ((rc = check_ptr("q", q, 16)) || (rc = check_ptr("k", k, 16)) ||
        (rc = check_ptr("scores", scores, 4)))
        return rc;
    if (with_lse && (rc = check_ptr("lse", lse, 4))) return rc;
    if (p->value_prior && (rc = check_ptr("v", v, 16))) return rc;
    const PrefillPlan pl = plan_prefill(p);
    if ((rc = check_ws(workspace, workspace_bytes, pl.bytes))) return rc;
    // the bf16 score launches are one-dimensional over all their workgroups
    const int64_t score_wgs = (int64_t)pl.Z * ((pl.n_qtiles + 1) / 2) * pl.nchunks;
    if (score_wgs > (int64_t)1 << 30)
        return fail(AHA_ERR_UNSUPPORTED, "problem exceeds the launch grid limits");
    // chosen accumulator rows: the bf16 kernels keep them in one query tile
    if (rows && p->dtype == AHA_BF16 && pl.n_qtiles != 1)
        return fail(AHA_ERR_UNSUPPORTED,
                    "chosen accumulator rows: group * window (%d) must not exceed 256 for bf16",
                    (p->n_q_heads / p->n_kv_heads) * p->window);
    ScoreGeom g = make_geom(p, q, k, v);
    g.rows = rows;
    g.v_once = values_once((int64_t)4 * pl.Z * g.n * g.d, with_lse);
    hipStream_t st = (hipStream_t)stream;
    if ((rc = hip_result(stage(0, st), "stage event"))) return rc;
    if (with_lse ? pl.given_nb && workspace_bytes >= pl.given_bytes
                 : pl.win_nb && !rows && workspace_bytes >= pl.win_bytes) {
        ExchangeCall call;
        const hipError_t e = with_lse ? exchange_call(st, given_patience(pl), pl.Z, (int64_t)pl.Z * pl.given_parts, pl.given_nb <= 4 ? 512 : 256,
                                                      workspace, pl.off_gwords, call)
                                      : exchange_call(st, window_patience(pl), pl.Z, (int64_t)pl.Z * pl.win_parts,
                                                      pl.win_hold && pl.win_tiles == 1 ? kHeldAtOnce : 256, workspace, pl.off_wwords, call);
        if ((rc = hip_result(e, "windowed score kernel")) || (rc = hip_result(stage(1, st), "stage event")) ||
            (rc = hip_result(with_lse ? launch_score_given(g, pl, workspace, call, lse, scores, st)
                                      : pl.win_share ? launch_score_share(g, pl, workspace, call, scores, st)
                                                     : launch_score_window(g, pl, workspace, call, scores, st),
                             "windowed score kernel")) ||
            (rc = hip_result(stage(2, st), "stage event")))
            return rc;
        return hip_result(stage(3, st), "stage event");
    }
    if (pl.hold32_parts && !with_lse && !rows && workspace_bytes >= pl.hold32_bytes && !(pl.hold32_eager && captured(st, false))) {
        const int looks = patience((int64_t)pl.Z * pl.hold32_parts, 256, 1, 2 * ((g.R + 31) / 32));
        ExchangeCall call;
        const hipError_t e = exchange_call(st, looks, pl.Z, 1, 1, workspace, pl.off_h32words, call);  // (all at once)
        if ((rc = hip_result(e, "windowed score kernel")) || (rc = hip_result(stage(1, st), "stage event")) ||
            (rc = hip_result(launch_score_hold_f32(g, pl, workspace, call, scores, st), "windowed score kernel")) ||
            (rc = hip_result(stage(2, st), "stage event")))
            return rc;
        return hip_result(stage(3, st), "stage event");
    }
    // the windowed bf16 scores and the fp32 scores form the value prior inside their
    // row-statistics launch
    const bool fold_prior = p->value_prior && !with_lse && (p->dtype == AHA_F32 || (pl.can_fold && !rows));
    if ((rc = hip_result(launch_value_prior(g, pl, workspace, scores, lse,
                                            p->value_prior && !fold_prior, st),
                         "value-prior kernel")))
        return rc;
    if ((rc = hip_result(stage(1, st), "stage event"))) return rc;
    hipEvent_t mid = g_stage_on ? g_stage_ev[2] : nullptr;
    if (p->dtype == AHA_BF16 && pl.n_qtiles > 1)
        rc = hip_result(launch_score_full(g, pl, workspace, scores, st, mid, with_lse), "bf16 score kernels");
    else if (p->dtype == AHA_BF16)
        rc = hip_result(launch_score_bf16(g, pl, workspace, scores, st, mid, with_lse, fold_prior),
                        "bf16 score kernels");
    else
        rc = hip_result(launch_score_f32(g, pl, workspace, scores, st, mid, with_lse),
                        "fp32 score kernels");
    if (rc) return rc;
    return hip_result(stage(3, st), "stage event");
}

int32_t aha_prefill_scores(const aha_params *p, const void *q, const void *k, const void *v,
                           float *scores, void *workspace, size_t workspace_bytes, void *stream) {
    return prefill_scores_impl(p, q, k, v, nullptr, false, nullptr, scores, workspace,
                               workspace_bytes, stream);
}

int32_t aha_prefill_scores_rows(const aha_params *p, const void *q, const void *k, const void *v,
                                const int32_t *rows, float *scores, void *workspace,
                                size_t workspace_bytes, void *stream) {
    const int32_t rc = check_ptr("rows", rows, 4);
    if (rc) return rc;
    return prefill_scores_impl(p, q, k, v, nullptr, false, rows, scores, workspace,
                               workspace_bytes, stream);
}

int32_t aha_prefill_scores_lse(const aha_params *p, const void *q, const void *k, const void *v,
                               const float *lse, float *scores, void *workspace,
                               size_t workspace_bytes, void *stream) {
    return prefill_scores_impl(p, q, k, v, lse, true, nullptr, scores, workspace, workspace_bytes,
                               stream);
}

int32_t aha_window_attention_workspace_bytes(const aha_params *p, size_t *out_bytes) {
    if (!out_bytes) return fail(AHA_ERR_INVALID_ARG, "out_bytes is null");
    const int32_t rc = check_prefill(p, false);
    if (rc) return rc;
    *out_bytes = plan_window_attn(p).bytes;
    return AHA_OK;
}

int32_t aha_prefill_window_attention(const aha_params *p, const void *q, const void *k,
                                     const void *v, void *out, float *lse, void *workspace,
                                     size_t workspace_bytes, void *stream) {
    int32_t rc = check_prefill(p, true);
    if (rc) return rc;
    if ((rc = check_ptr("q", q, 16)) || (rc = check_ptr("k", k, 16)) || (rc = check_ptr("v", v, 16)) ||
        (rc = check_ptr("out", out, 16)))
        return rc;
    if (lse && (rc = check_ptr("lse", lse, 4))) return rc;
    const WindowAttnPlan pl = plan_window_attn(p);
    if ((rc = check_ws(workspace, workspace_bytes, pl.bytes))) return rc;
    const int64_t Z = (int64_t)p->batch * p->n_kv_heads;
    const int64_t wgs = p->dtype == AHA_BF16 ? (Z * pl.nparts + 7) / 8 * 8 * pl.n_blocks
                                             : (int64_t)pl.n_blocks * 32;
    if (wgs > (int64_t)1 << 30 || (int64_t)pl.n_blocks * 32 > (int64_t)1 << 30)
        return fail(AHA_ERR_UNSUPPORTED, "problem exceeds the launch grid limits");
    const ScoreGeom g = make_geom(p, q, k, v);
    return hip_result(launch_window_attention(g, pl, workspace, out, lse, (hipStream_t)stream),
                      "window attention kernels");
}

int32_t aha_prefill_row_stats(const aha_params *p, const void *q, const void *k, float *lse,
                              float *entropy, void *workspace, size_t workspace_bytes,
                              void *stream) {
    int32_t rc = check_prefill(p, false);
    if (rc) return rc;
    if ((rc = check_stride("q", p->q_stride, p->dtype, p->head_dim)) ||
        (rc = check_stride("k", p->k_stride, p->dtype, p->head_dim)))
        return rc;
    if ((rc = check_ptr("q", q, 16)) || (rc = check_ptr("k", k, 16))) return rc;
    if (!lse && !entropy) return fail(AHA_ERR_INVALID_ARG, "lse and entropy are both null");
    if ((lse && (rc = check_ptr("lse", lse, 4))) || (entropy && (rc = check_ptr("entropy", entropy, 4))))
        return rc;
    const PrefillPlan pl = plan_prefill(p);
    if ((rc = check_ws(workspace, workspace_bytes, pl.bytes))) return rc;
    const int64_t score_wgs = (int64_t)pl.Z * ((pl.n_qtiles + 1) / 2) * pl.nchunks;
    if (score_wgs > (int64_t)1 << 30)
        return fail(AHA_ERR_UNSUPPORTED, "problem exceeds the launch grid limits");
    const ScoreGeom g = make_geom(p, q, k, nullptr);
    if (p->dtype == AHA_BF16)
        return hip_result(launch_row_stats_bf16(g, pl, workspace, lse, entropy, (hipStream_t)stream),
                          "bf16 row-statistics kernels");
    return hip_result(launch_row_stats_f32(g, pl, workspace, lse, entropy, (hipStream_t)stream),
                      "fp32 row-statistics kernel");
}

int32_t aha_select_topk(const aha_params *p, const float *scores, int32_t *idx, void *workspace,
                        size_t workspace_bytes, void *stream) {
    int32_t rc = check_prefill(p, false);
    if (rc) return rc;
    if ((rc = check_ptr("scores", scores, 4)) || (rc = check_ptr("idx", idx, 4))) return rc;
    const int pool = p->score_pool > 1 ? p->score_pool : 1;
    if (pool > 1 && (rc = check_ws(workspace, workspace_bytes, topk_ws_bytes(p)))) return rc;
    return hip_result(launch_topk(scores, p->batch * p->n_kv_heads, p->seq_len, p->budget,
                                  p->recent, p->sink, pool, (float *)workspace, idx,
                                  (hipStream_t)stream),
                      "top-k kernels");
}

int32_t aha_compact_kv(const aha_params *p, const void *k, const void *v, const float *scores,
                       const int32_t *idx, void *k_cache, void *v_cache, float *scores_c,
                       int32_t *pos_c, int32_t *free_slot, int32_t cache_slots, void *stream) {
    int32_t rc = check_compact(p);
    if (rc) return rc;
    if ((rc = check_ptr("k", k, 16)) || (rc = check_ptr("v", v, 16)) ||
        (rc = check_ptr("scores", scores, 4)) || (rc = check_ptr("idx", idx, 4)) ||
        (rc = check_ptr("k_cache", k_cache, 16)) || (rc = check_ptr("v_cache", v_cache, 16)) ||
        (rc = check_ptr("scores_c", scores_c, 4)) || (rc = check_ptr("pos_c", pos_c, 4)) ||
        (rc = check_ptr("free_slot", free_slot, 4)))
        return rc;
    if (cache_slots < p->budget + 1)
        return fail(AHA_ERR_INVALID_ARG, "cache_slots (%d) must be >= budget + 1 (%d)", cache_slots,
                    p->budget + 1);
    const ScoreGeom g = make_geom(p, nullptr, k, v);
    return hip_result(launch_compact(g, scores, idx, p->budget, cache_slots, p->dtype, k_cache,
                                     v_cache, scores_c, pos_c, free_slot, (hipStream_t)stream),
                      "compaction kernel");
}

// Bytes of the built-in scratch of aha_decode_step_static (below).
constexpr size_t kScratchBytes = (size_t)4 << 20;  // of static_bytes
// A partial output has kPartStats statistics, two more floats than are counted; the count holds
// fewer than 4 MiB / (4 * 66) of them (at least 64 channels and two statistics each).
constexpr size_t kScratchMargin = kScratchBytes / (4 * 66) * 4 * (kPartStats - 2) + 256;

// Host checks shared by aha_decode_step and its variant without a workspace argument
// (`scratch_limit` > 0: the scratch is the library's own and that many bytes long; the
// workspace arguments are then not looked at).  Nothing here touches the HIP runtime.
static int32_t decode_step_check(const aha_params *p, const void *q_new, const void *k_new,
                                 const void *v_new, void *k_cache, void *v_cache, float *scores_c,
                                 int32_t *pos_c, int32_t *free_slot, int32_t cache_slots,
                                 int32_t logical_pos, void *out, const void *workspace,
                                 size_t workspace_bytes, size_t scratch_limit, DecodePlan *plan) {
    int32_t rc = check_common(p);
    if (rc) return rc;
    if ((rc = check_ptr("q_new", q_new, 16)) || (rc = check_ptr("k_new", k_new, 16)) ||
        (rc = check_ptr("v_new", v_new, 16)) || (rc = check_ptr("k_cache", k_cache, 16)) ||
        (rc = check_ptr("v_cache", v_cache, 16)) || (rc = check_ptr("scores_c", scores_c, 4)) ||
        (rc = check_ptr("pos_c", pos_c, 4)) || (rc = check_ptr("free_slot", free_slot, 4)) ||
        (rc = check_ptr("out", out, 16)))
        return rc;
    if (cache_slots < p->budget + 1)
        return fail(AHA_ERR_INVALID_ARG, "cache_slots (%d) must be >= budget + 1 (%d)", cache_slots,
                    p->budget + 1);
    if (logical_pos < p->budget + 1)
        return fail(AHA_ERR_INVALID_ARG, "logical_pos (%d) must be >= budget + 1 (%d)", logical_pos,
                    p->budget + 1);
    const int G = p->n_q_heads / p->n_kv_heads;
    if (G > 8)
        return fail(AHA_ERR_UNSUPPORTED, "decode is built for query groups of up to 8 heads, not %d", G);
    // (a workspace that cannot be used counts as none: steps that need none do not look at it)
    const bool usable = workspace && (uintptr_t)workspace % 256 == 0;
    *plan = plan_decode(p, scratch_limit ? kScratchBytes + kScratchMargin : usable ? workspace_bytes : 0);
    if (!plan->fits)
        return fail(AHA_ERR_UNSUPPORTED,
                    "decode keeps group * (budget + 1) dots in LDS; %d * %d does not fit (%d splits)",
                    G, p->budget + 1, plan->nsplit);
    if (scratch_limit) {
        // (the same shapes are refused whichever path serves them)
        if (plan->static_bytes > scratch_limit)
            return fail(AHA_ERR_UNSUPPORTED,
                        "split over workgroups this shape's scratch counts %zu bytes, the built-in buffer "
                        "is for %zu: use aha_decode_step with a workspace", plan->static_bytes, scratch_limit);
        return AHA_OK;
    }
    return check_ws(workspace, workspace_bytes, plan->bytes);
}

static int32_t decode_step_launch(const aha_params *p, const DecodePlan &dpl, const void *q_new,
                                  const void *k_new, const void *v_new, void *k_cache,
                                  void *v_cache, float *scores_c, int32_t *pos_c,
                                  int32_t *free_slot, int32_t cache_slots, int32_t logical_pos,
                                  void *out, void *workspace, void *stream) {
    DecodeGeom g{};
    g.q = q_new; g.k_new = k_new; g.v_new = v_new; g.kc = k_cache; g.vc = v_cache; g.out = out;
    g.fc = scores_c; g.pos = pos_c; g.free_slot = free_slot;
    g.batch = p->batch; g.Hq = p->n_q_heads; g.Hkv = p->n_kv_heads; g.G = g.Hq / g.Hkv;
    g.d = p->head_dim;
    g.budget = p->budget; g.recent = p->recent; g.slots = cache_slots; g.logical_pos = logical_pos;
    g.scale_mode = p->scale_mode; g.fixed_scale = p->fixed_scale; g.lambda_floor = p->lambda_floor;
    g.sink = p->sink; g.value_prior = p->decode_value_prior;
    return hip_result(launch_decode(g, dpl, workspace, p->dtype, (hipStream_t)stream),
                      "decode kernel");
}

int32_t aha_decode_step(const aha_params *p, const void *q_new, const void *k_new,
                        const void *v_new, void *k_cache, void *v_cache, float *scores_c,
                        int32_t *pos_c, int32_t *free_slot, int32_t cache_slots,
                        int32_t logical_pos, void *out, void *workspace, size_t workspace_bytes,
                        void *stream) {
    DecodePlan dpl{};
    const int32_t rc = decode_step_check(p, q_new, k_new, v_new, k_cache, v_cache, scores_c, pos_c,
                                         free_slot, cache_slots, logical_pos, out, workspace,
                                         workspace_bytes, 0, &dpl);
    if (rc) return rc;
    return decode_step_launch(p, dpl, q_new, k_new, v_new, k_cache, v_cache, scores_c, pos_c,
                              free_slot, cache_slots, logical_pos, out, workspace, stream);
}

// ---- generation step without a workspace argument ----
// Scratch of the split decode path (raw dots and the splits' partial outputs) for callers
// that can neither allocate nor carry a workspace.  The array's name is only a host-side
// stand-in: its device address is asked for once per device (each GPU holds its own copy
// at its own address) and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[kScratchBytes + kScratchMargin];
static void *g_scratch_ptr[kMaxDevices];
static DeviceOnce g_scratch_once;

int32_t aha_decode_step_static(const aha_params *p, const void *q_new, const void *k_new,
                               const void *v_new, void *k_cache, void *v_cache, float *scores_c,
                               int32_t *pos_c, int32_t *free_slot, int32_t cache_slots,
                               int32_t logical_pos, void *out, void *stream) {
    DecodePlan dpl{};
    const int32_t rc = decode_step_check(p, q_new, k_new, v_new, k_cache, v_cache, scores_c, pos_c,
                                         free_slot, cache_slots, logical_pos, out, nullptr, 0,
                                         kScratchBytes, &dpl);
    if (rc) return rc;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_result(e, "hipGetDevice");
    e = device_once(g_scratch_once, [dev] {
        void *ptr = nullptr;
        const hipError_t es = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        g_scratch_ptr[dev] = es == hipSuccess ? ptr : nullptr;
        return es;
    });
    if (e != hipSuccess) return hip_result(e, "address of the built-in scratch buffer");
    // every value the kernels read from the scratch is written earlier in the same call:
    // nothing has to start from zero
    return decode_step_launch(p, dpl, q_new, k_new, v_new, k_cache, v_cache, scores_c, pos_c,
                              free_slot, cache_slots, logical_pos, out, g_scratch_ptr[dev], stream);
}

int32_t aha_exchange_looks(int32_t looks) {
    if (looks < 0) return fail(AHA_ERR_INVALID_ARG, "looks must be >= 0");
    g_looks = looks;
    return AHA_OK;
}

int32_t aha_profile_events(void *const *events, int32_t count) {
    if (count == 0 && !events) {
        g_stage_on = false;
        return AHA_OK;
    }
    if (count != 4 || !events) return fail(AHA_ERR_INVALID_ARG, "events must be NULL/0 or 4 handles");
    for (int i = 0; i < 4; ++i) {
        if (!events[i]) return fail(AHA_ERR_INVALID_ARG, "events[%d] is null", i);
        g_stage_ev[i] = (hipEvent_t)events[i];
    }
    g_stage_on = true;
    return AHA_OK;
}

const char *aha_last_error(void) { return g_err; }

const char *aha_version(void) { return "aha-gfx950 0.1"; }

}  // extern "C"
