// Selection (Alg. 1: recent set, TopK, union): per (batch, KV head) the
// budget - recent highest scores among the non-recent tokens, ties to the
// lower position, written as ascending token positions followed by the recent
// positions.
//
// One workgroup per problem.  Each wave owns a contiguous range of token positions and walks
// it 64 positions at a time, lane = position: the loads coalesce whatever a row's alignment,
// and a comparison over a step is one 64-bit mask on the scalar unit - counted with s_bcnt1,
// turned into output slots with v_mbcnt - so that nothing per key is kept but the key itself
// (the scores turned into order-preserving 32-bit keys, in registers).  The last selected
// element is found by
//   1. the key range [kmin, kmax] of the problem (one block reduction);
//   2. ONE histogram of BINS bins that are linear in key - kmin over exactly that range, so the
//      keys spread over the bins whatever their exponents (few same-address LDS atomics), and
//      a block-wide suffix scan that finds the bin holding the threshold;
//   3. an exact rank among the (typically few dozen) keys of that bin, kept in LDS; if the bin
//      is crowded (many equal or nearly equal scores) the low bits are resolved by 8-bit radix
//      rounds instead.
// Keys above that bin are selected for certain; the ones inside are decided by (key, position)
// against the last selected element, so the ascending output needs one count per wave and no
// further scan.  Of sequences with more than 32 keys per thread the rest is re-read from memory
// in every pass.
//
// Bound by the latency of its chain (launch, first loads, six barriers) and, from 8K tokens on,
// by the one CU that works on a problem.  In-kernel stamps at 8 x 32768 scores (us): loads 1.9, range 1.2, histogram 2.2 (the LDS
// atomics' rate), scan 1.0, candidates 1.9, rank 0.8, output 1.9; a vector instruction per key costs 0.2.  The masks of the
// candidates' pass are kept on the scalar unit, so that the output compares again only in steps with keys in the threshold
// bin (back to back 8 x 32768 13.4 -> 12.5 us).  From 12
// steps on scores that are not negative skip most of the conversion, from 24 on waves of whole steps skip the padding's
// instructions and four steps share a branch: 8 x 12000 7.41 -> 7.12, 8 x 16384 8.57 -> 8.21, 8 x 20000 10.7 -> 9.8, 8 x 32768 13.3 ->
// 12.2, 8 x 65536 34.2 -> 32.2 (with negative ones among them 8.49, 8.58; 9.93, 9.99; 12.7, 13.0; 16.8, 16.4; 38.3, 36.4).  Against lanes that own consecutive positions (scattered
// loads, per-lane bit masks, a second scan), back to back: 2 x 512 scores 5.9 -> 3.4 us,
// 32 x 4096 6.6 -> 4.8, 12 x 5003 9.0 -> 5.4, 8 x 16384 10.0 -> 8.4, 128 x 16384 11.2 -> 9.5,
// 8 x 32768 16.1 -> 13.2, 8 x 65536 34.8 -> 31.8, 8 x 120000 290 -> 67.
#include "aha_dev.h"
#include "aha_host.h"

namespace aha {

constexpr int kCandMax = 1024;   // keys of the threshold bin ranked directly

// Order-preserving key, never 0: that is the padding key, and the counts that address the output
// add up only if every real position has another one (the NaN of all ones would be 0).
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return max((u & 0x80000000u) ? ~u : (u | 0x80000000u), 1u);
}

template <int WAVES, int BINS>
struct TopkSmem {
    int hist[BINS];
    unsigned long long cand[kCandMax];  // key << 32 | ~position: descending = selection order
    uint32_t red[2][WAVES];
    int wsum[WAVES];   // histogram counts per wave
    int wcnt[WAVES];   // selected elements per wave
    int bin, need, nbin, ncand;
    uint32_t T;        // key and position of the last selected element
    int posT;
};

// Inclusive prefix sum over the wave in the vector ALU: within the rows of 16 lanes, then the
// last lane of a row added to the next row, then the last lane of the first half to the second.
__device__ __forceinline__ int wave_prefix_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15, rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31, rows 2 and 3
    return x;
}

// `first` plus the number of lanes below this one whose bit is set
__device__ __forceinline__ int mask_rank(unsigned long long m, int first) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, first));
}

// Block-wide: given per-thread counts `loc` of consecutive, ascending key ranges (thread
// t covers lower keys than thread t+1), the number of keys in the ranges above this thread's.
template <int WAVES>
__device__ __forceinline__ int suffix_above(int loc, int lane, int wave, int *wsum) {
    const int incl = wave_prefix_sum(loc);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    if (lane == 0) wsum[wave] = total;
    __syncthreads();
    int above = total - incl;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) above += w > wave ? wsum[w] : 0;
    return above;
}

// A wave owns 64 * ipt positions; the keys of its first ITEMS steps live in registers, one per
// lane and step.  LONG: there are more steps, whose scores are re-read in every pass.
// `sink`: positions below it are retained without being ranked (their keys are the padding
// key 0, which lies below every real key and is never counted), like the `recent` last ones.
template <int WAVES, int ITEMS, int BINS, bool LONG>
__global__ __launch_bounds__(WAVES * 64) void topk_kernel(const float *__restrict__ scores, int n,
                                                          int budget, int recent, int sink,
                                                          int32_t *__restrict__ idx) {
    constexpr int THREADS = WAVES * 64, BPT = BINS / THREADS;
    static_assert(BPT % 4 == 0 && THREADS >= 256, "a thread owns whole 16-byte groups of bins");
    __shared__ __attribute__((aligned(16))) TopkSmem<WAVES, BINS> sm;

    const int z = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *sc = scores + (int64_t)z * n;
    int32_t *out = idx + (int64_t)z * budget + sink;  // the ranked part starts behind the sinks
    const int n_cand = n - recent;
    const int k = budget - recent - sink;

    const int ipt = LONG ? (n_cand + THREADS - 1) / THREADS : ITEMS;
    const int base = wave * 64 * ipt;  // the wave's first position
    // (LONG: batches of eight steps may reach behind the wave's last one)
    const bool whole = base >= sink && base + 64 * ipt <= n_cand && (!LONG || (ipt - ITEMS) % 8 == 0);
    // keys of N steps from step t0 on: all requested (clamped to the row) before the first is
    // used, and only then turned into keys, so that no step waits for another one's round trip
    auto load = [&](auto &u, int t0) {
        constexpr int N = sizeof(u) / sizeof(u[0]);
        const float *row = sc + base;
        const int last = n - 1 - base;  // (negative for a wave behind the row's end)
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const int off = (t0 + t) * 64 + lane;
            u[t] = __float_as_uint(row[whole ? off : min(off, last)]);
        }
        // (scores are rarely negative: then a key is the value with its sign bit set, one instruction instead of four)
        uint32_t any = 0;
#pragma unroll
        for (int t = 0; t < N; ++t) any |= u[t];
        if (N >= 12 && __builtin_amdgcn_ballot_w64((int)any < 0) == 0) {
#pragma unroll
            for (int t = 0; t < N; ++t) u[t] |= 0x80000000u;
        } else {
#pragma unroll
            for (int t = 0; t < N; ++t) u[t] = order_key(__uint_as_float(u[t]));
        }
        if (!whole) {
#pragma unroll
            for (int t = 0; t < N; ++t) {
                const int j = base + (t0 + t) * 64 + lane;
                u[t] = ((j >= sink) & (j < n_cand) & (t0 + t < ipt)) ? u[t] : 0u;
            }
        }
    };
    uint32_t key[ITEMS];
    if (k > 0) load(key, 0);
    for (int t = tid; t < BINS; t += THREADS) sm.hist[t] = 0;
    if (tid == 0) sm.ncand = 0;
    for (int t = tid; t < sink; t += THREADS) out[t - sink] = t;
    for (int t = tid; t < recent; t += THREADS) out[k + t] = n_cand + t;
    if (k == 0) return;
    // every step of the wave in position order: f(keys of the 64 lanes, step)
    auto for_steps = [&](auto f) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) f(key[t], t);
        if (LONG) {
            for (int t0 = ITEMS; t0 < ipt; t0 += 8) {  // (eight requests in flight; past the last: padding)
                uint32_t u[8];
                load(u, t0);
#pragma unroll
                for (int t = 0; t < 8; ++t) f(u[t], t0 + t);
            }
        }
    };
    auto ballot = [](bool p) { return (unsigned long long)__builtin_amdgcn_ballot_w64(p); };

    // 1. range of the keys (padding: 0 - 1 wraps to the top and never is the minimum)
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    if (!LONG && ITEMS >= 24 && whole) {  // (no padding; with 16 steps the path costs more than it saves: 8 x 16384 8.21, 8.29 with it)
        for_steps([&](uint32_t u, int) { kmin = min(kmin, u); kmax = max(kmax, u); });
        kmin -= 1u;
    } else {
        for_steps([&](uint32_t u, int) { kmin = min(kmin, u - 1u); kmax = max(kmax, u); });
    }
    kmin = reduce_lanes<1, 64>(kmin, OpMinU{});
    kmax = reduce_lanes<1, 64>(kmax, OpMaxU{});
    if (lane == 0) { sm.red[0][wave] = kmin; sm.red[1][wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { kmin = min(kmin, sm.red[0][w]); kmax = max(kmax, sm.red[1][w]); }
    kmin += 1u;

    // 2. one histogram, linear in key - kmin, over the occupied range only
    const uint32_t range = kmax - kmin;
    constexpr int kBinBits = 31 - __builtin_clz(BINS);
    const int sh = range ? max(0, 32 - __clz(range) - kBinBits) : 0;  // (range >> sh) < BINS
    if (!LONG && ITEMS >= 24 && whole) {
        for_steps([&](uint32_t u, int) { atomicAdd(&sm.hist[(u - kmin) >> sh], 1); });
    } else {
        for_steps([&](uint32_t u, int) {
            if (u >= kmin) atomicAdd(&sm.hist[(u - kmin) >> sh], 1);  // (padding keys are not counted)
        });
    }
    __syncthreads();
    {
        int cb[BPT], loc = 0;
#pragma unroll
        for (int t = 0; t < BPT; ++t) {
            cb[t] = sm.hist[BPT * tid + t];
            loc += cb[t];
        }
        int above = suffix_above<WAVES>(loc, lane, wave, sm.wsum);
        if (above < k && k <= above + loc) {
#pragma unroll
            for (int t = BPT - 1; t >= 0; --t) {
                if (above < k && k <= above + cb[t]) {
                    sm.bin = BPT * tid + t;
                    sm.need = k - above;
                    sm.nbin = cb[t];  // keys in the threshold bin
                }
                above += cb[t];
            }
        }
    }
    __syncthreads();
    const uint32_t bin = (uint32_t)__builtin_amdgcn_readfirstlane(sm.bin);
    int need = __builtin_amdgcn_readfirstlane(sm.need);
    const int nbin = __builtin_amdgcn_readfirstlane(sm.nbin);

    // the last selected element (T, posT): selected are the keys above T, and those equal to T
    // at positions up to posT
    const uint32_t lo = kmin + (bin << sh), span = (1u << sh) - 1u;
    const uint32_t hi = span > ~lo ? ~0u : lo + span;
    uint32_t T = lo;
    int posT = n;
    auto selected = [&](uint32_t u, int t) {
        return (u > T) | ((u == T) & (base + t * 64 + lane <= posT));
    };
    auto count_selected = [&] {
        int c = 0;
        for_steps([&](uint32_t u, int t) { c += __popcll(ballot(selected(u, t))); });
        if (lane == 0) sm.wcnt[wave] = c;
    };
    const bool ranked = nbin <= kCandMax;  // (uniform)
    // of a ranked bin: per step the lanes whose keys are above it, per group of steps whether any are inside
    constexpr bool KEPT = !LONG;
    constexpr int GROUP = KEPT && ITEMS >= 24 ? 4 : 1;  // steps that share a branch: few have keys inside (16 steps: 8 x 16384 8.05, 8.38 with four)
    unsigned long long over[KEPT ? ITEMS : 1];
    uint32_t inside = 0;
    static_assert(!KEPT || ITEMS <= 32, "a bit per step");
    if (ranked) {
        // 3a. exact rank among the keys of the threshold bin
        int above = 0;  // keys of this wave above the bin
        auto collect = [&](unsigned long long in, bool cand, uint32_t u, int t) {
            int slot = 0;
            if (lane == 0) slot = atomicAdd(&sm.ncand, __popcll(in));
            slot = __builtin_amdgcn_readfirstlane(slot);
            if (cand) sm.cand[mask_rank(in, slot)] = ((unsigned long long)u << 32) | (uint32_t)(~(base + t * 64 + lane));
        };
        if constexpr (GROUP > 1) {
#pragma unroll
            for (int t0 = 0; t0 < ITEMS; t0 += GROUP) {
                unsigned long long in[GROUP], any = 0;
#pragma unroll
                for (int i = 0; i < GROUP; ++i) {
                    over[t0 + i] = ballot(key[t0 + i] > hi);
                    in[i] = ballot(key[t0 + i] >= lo) & ~over[t0 + i];
                    above += __popcll(over[t0 + i]);
                    any |= in[i];
                }
                if (any) {
                    inside |= 1u << (t0 / GROUP);
#pragma unroll
                    for (int i = 0; i < GROUP; ++i)
                        if (in[i]) collect(in[i], __builtin_amdgcn_inverse_ballot_w64(in[i]), key[t0 + i], t0 + i);
                }
            }
        } else {
            for_steps([&](uint32_t u, int t) {
                if constexpr (LONG) {
                    const unsigned long long gts = ballot(u > hi), in = ballot(u >= lo) & ~gts;
                    above += __popcll(gts);
                    if (in) collect(in, __builtin_amdgcn_inverse_ballot_w64(in), u, t);
                } else {
                    const bool gt = u > hi, cand = (u >= lo) & !gt;
                    over[t] = ballot(gt);
                    above += __popcll(over[t]);
                    const unsigned long long in = ballot(cand);
                    if (in) {
                        inside |= 1u << t;
                        collect(in, cand, u, t);
                    }
                }
            });
        }
        if (lane == 0) sm.wcnt[wave] = above;
        __syncthreads();
        for (int i = tid; i < nbin; i += THREADS) {
            const unsigned long long mine = sm.cand[i];
            int rank = 0;  // number of candidates selected before this one
            int u = 0;
            for (; u + 4 <= nbin; u += 4)
                rank += (sm.cand[u] > mine) + (sm.cand[u + 1] > mine) + (sm.cand[u + 2] > mine) +
                        (sm.cand[u + 3] > mine);
            for (; u < nbin; ++u) rank += sm.cand[u] > mine;
            const int j = (int)~(uint32_t)mine;
            if (rank < need) atomicAdd(&sm.wcnt[j / (64 * ipt)], 1);
            if (rank == need - 1) {
                sm.T = (uint32_t)(mine >> 32);
                sm.posT = j;
            }
        }
        __syncthreads();
        T = sm.T;
        posT = sm.posT;
    } else {
        // 3b. crowded bin: 8-bit radix rounds over the low `sh` bits of key - kmin
        uint32_t prefix = bin << sh;
        for (int shift = ((sh + 7) / 8 - 1) * 8; shift >= 0; shift -= 8) {
            __syncthreads();
            if (tid < 256) sm.hist[tid] = 0;
            __syncthreads();
            const uint32_t hi_mask = 0xffffffffu << min(shift + 8, 31);  // sh <= 24: never 32
            for_steps([&](uint32_t u, int) {
                const uint32_t rel = u - kmin;
                if (u != 0u && (rel >> sh) == bin && (rel & hi_mask) == (prefix & hi_mask))
                    atomicAdd(&sm.hist[(rel >> shift) & 255u], 1);
            });
            __syncthreads();
            const int c = tid < 256 ? sm.hist[tid] : 0;
            const int ab = suffix_above<WAVES>(c, lane, wave, sm.wsum);  // threads >= 256 hold 0
            if (tid < 256 && ab < need && need <= ab + c) { sm.bin = tid; sm.need = need - ab; }
            __syncthreads();
            prefix |= (uint32_t)sm.bin << shift;
            need = sm.need;
        }
        T = kmin + prefix;
        // the position of the need-th key that equals T
        int eq = 0;
        for_steps([&](uint32_t u, int) { eq += __popcll(ballot(u == T)); });
        __syncthreads();
        if (lane == 0) sm.wsum[wave] = eq;
        __syncthreads();
        int before = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) before += w < wave ? sm.wsum[w] : 0;
        if (before < need && need <= before + eq) {
            for_steps([&](uint32_t u, int t) {
                const unsigned long long m = ballot(u == T);
                if (((m >> lane) & 1) && mask_rank(m, before) == need - 1)
                    sm.posT = base + t * 64 + lane;
                before += __popcll(m);
            });
        }
        __syncthreads();
        posT = sm.posT;
        count_selected();
        __syncthreads();
    }
    T = (uint32_t)__builtin_amdgcn_readfirstlane((int)T);
    posT = __builtin_amdgcn_readfirstlane(posT);

    // ascending output: the wave's first slot, then step by step
    int o = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) o += w < wave ? sm.wcnt[w] : 0;
    auto put = [&](unsigned long long m, bool sel, int t) {
        if (sel) out[mask_rank(m, o)] = base + t * 64 + lane;
        o += __popcll(m);
    };
    if constexpr (KEPT) {
        if (ranked) {  // (the comparisons have been made, but for keys in the bin)
            if constexpr (GROUP > 1) {
#pragma unroll
                for (int t0 = 0; t0 < ITEMS; t0 += GROUP) {
                    if (inside & (1u << (t0 / GROUP))) {
#pragma unroll
                        for (int t = t0; t < t0 + GROUP; ++t) over[t] = ballot(selected(key[t], t));
                    }
#pragma unroll
                    for (int t = t0; t < t0 + GROUP; ++t) put(over[t], __builtin_amdgcn_inverse_ballot_w64(over[t]), t);
                }
            } else {
                for_steps([&](uint32_t u, int t) {
                    unsigned long long m = over[t];
                    if (inside & (1u << t)) m = ballot(selected(u, t));
                    put(m, __builtin_amdgcn_inverse_ballot_w64(m), t);
                });
            }
            return;
        }
    }
    for_steps([&](uint32_t u, int t) {
        const bool sel = selected(u, t);
        put(ballot(sel), sel, t);
    });
}

template <int WAVES, int ITEMS, int BINS, bool LONG = false>
static void launch_items(const float *scores, int Z, int n, int budget, int recent, int sink,
                         int32_t *idx, hipStream_t st) {
    static_assert(sizeof(TopkSmem<WAVES, BINS>) <= 64 * 1024, "top-k LDS must fit the static limit");
    hipLaunchKernelGGL((topk_kernel<WAVES, ITEMS, BINS, LONG>), dim3(Z), dim3(WAVES * 64), 0, st, scores, n,
                       budget, recent, sink, idx);
}

// Scores smoothed over tokens before the selection (caption of the method's overview
// figure): average pool of odd width, stride 1, mean over the taps inside the sequence.
// The pooled value decides which tokens are kept, so it is formed exactly as stated - the
// taps added left to right in fp32, then one division - and not by a running sum.
__global__ __launch_bounds__(256) void pool_scores_kernel(const float *__restrict__ scores, int n,
                                                          int half, float *__restrict__ pooled) {
    const int z = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const float *s = scores + (int64_t)z * n;
    const int lo = max(0, j - half), hi = min(n - 1, j + half);
    float acc = 0.f;
    for (int t = lo; t <= hi; ++t) acc = __fadd_rn(acc, s[t]);
    pooled[(int64_t)z * n + j] = __fdiv_rn(acc, (float)(hi - lo + 1));
}

hipError_t launch_topk(const float *scores, int Z, int n, int budget, int recent, int sink,
                       int pool, float *pooled, int32_t *idx, hipStream_t st) {
    if (pool > 1) {
        hipLaunchKernelGGL(pool_scores_kernel, dim3((n + 255) / 256, Z), dim3(256), 0, st, scores, n,
                           (pool - 1) / 2, pooled);
        scores = pooled;
    }
    const int n_cand = n - recent;
    auto steps = [&](int waves) { return (n_cand + waves * 64 - 1) / (waves * 64); };
    // Four waves up to 2048 candidates (32 x 2000: 6.3 -> 4.7 us; barriers and scans of 16 waves
    // cost more than the keys), then 16; as many keys per thread as the row needs, since a step of
    // padding costs what a step of keys does (12 x 5003 with eight steps instead of six: 6.3 us
    // instead of 5.4).  More than 32 registers of keys per thread spill.
#define AHA_TOPK(W, I, B) \
    if (steps(W) <= I) { launch_items<W, I, B>(scores, Z, n, budget, recent, sink, idx, st); return hipGetLastError(); }
    AHA_TOPK(4, 2, 2048) AHA_TOPK(4, 4, 2048) AHA_TOPK(4, 8, 2048)
    AHA_TOPK(16, 4, 8192) AHA_TOPK(16, 6, 8192) AHA_TOPK(16, 8, 8192) AHA_TOPK(16, 12, 8192)
    AHA_TOPK(16, 16, 8192) AHA_TOPK(16, 24, 8192) AHA_TOPK(16, 32, 8192)
#undef AHA_TOPK
    launch_items<16, 32, 8192, true>(scores, Z, n, budget, recent, sink, idx, st);
    return hipGetLastError();
}

}  // namespace aha
