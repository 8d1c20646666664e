// Exchange between the workgroups of one problem inside one launch: every workgroup leaves its
// part of a result in the workspace, and uses the others' parts once all of them are there.
//
// No cache is written back or invalidated for it (a device-scope release does that for the whole
// L2 of an XCD, microseconds per workgroup): what is exchanged is stored and loaded with agent-scope
// accesses, which go past the caches that are not shared, and it carries a TAG beside the values (Words),
// so a reader looks at the data itself, nothing waits for stores to arrive, and there is one trip to memory each way.  With
// announcements behind the data, which a wave looked at before all fetched the data, it was three.  us of the step before and after:
// 12 heads x 5003 keys x 120 rows 23.5 -> 21.2, 32 x 4096 x 64 31.6 -> 31.1, 128 x 16384 x 64 338 -> 336, 8 x 16384 x 512 65.6 ->
// 63.2, 8 x 32768 x 256 79.5 -> 77.0.
// Taken back: the priors' maxima looked for together with the row statistics (32 x 4096 0.9 slower: they come later), or
// requested before these are merged (0.3 slower).
//
// The tag is a 64-bit number that no other call of the process uses, so the workspace needs no clearing launch
// (3 us) in front: whatever it holds on entry is not this tag.  A captured graph replays a call with
// its tag, and other work may have written to any part of the workspace since, so nothing that lies there can tell two replays
// apart: no word may outlive a replay.  The workgroup that is the last of its problem to have seen all parts takes
// the words away, or, where these are many, a launch in front does (exchange_call in aha_api.hip); only captured calls do that (the host
// asks the stream).  The last workgroup is found by a counter that starts itself: its upper bits are the call's number, and
// an arrival that finds other bits there sets them.  us of the score stage, eager and replayed: 32 x 4096 x 64 20.4, 21.1; 8 x 16384 x
// 512 46.2, 47.4.  (Words told apart by a number in the workspace that each call moved on cost a load per workgroup instead, 20.3
// and 46.8 either way, and were taken for the next replay's once other work had put that number back.  Each workgroup its own part's
// words, told by a second count at its end: 1 x 60757 x 448 48.1 -> 42.6, 40.2 with the launch, but 1 x 131072 x 64 32.1 -> 38.0.)
//
// Nobody depends on workgroups that may not be running: after `looks` looks at the others' parts a
// workgroup does missing parts itself and leaves them too (a part's result is the same bits whoever
// forms it).  The workgroups that have waited in vain share what is missing, so together they are done in
// about the time that the missing ones would have taken, and `looks` is a few times that (patience in
// aha_api.hip): beside other work that keeps half of a problem's workgroups out, waiting costs about
// as much as the work.
#pragma once

#include "aha_dev.h"
#include "aha_host.h"

namespace aha {

struct Exchange {
    uint64_t *counts;  // [problem][kExchangeBytes / 8], a count for each
    uint64_t tag;      // of this call; the low kCountBits are zero, the rest is not
    int looks;         // at the others' parts before missing ones are done here
    bool replayed;     // the call is captured, and nothing takes its words away in front
    __device__ __forceinline__ uint64_t *count(int z) const { return counts + (int64_t)z * (kExchangeBytes / 8); }
};
constexpr int kCountBits = 20;  // parts of a problem: fewer than 2^20

template <class T>
__device__ __forceinline__ void put(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T get(const T *p) {
    return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a part leaves goes as words of 16 bytes that carry the tag beside two floats: {value, lo, value, hi}, stored and loaded in
// one piece (each half proves its own float if they ever were not: either of lo and hi differs between any two of 2^32
// consecutive calls).
struct Words {
    __amdgpu_buffer_rsrc_t at;
    uint32_t lo, hi;  // both zero for no call
    // (a problem's words lie within 2^31 bytes)
    __device__ __forceinline__ Words(void *base, uint64_t tag)
        : at(__builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000)), lo((uint32_t)(tag >> kCountBits)),
          hi((uint32_t)(tag >> (kCountBits + 32)) + lo * 0x9E3779B1u) {}
    static constexpr int kAgent = 16;  // (sc1: past the caches that are not shared)
    __device__ __forceinline__ void put(int word, float a, float b) const {
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(a), lo, __float_as_uint(b), hi}, at, word * 16, 0, kAgent);
    }
    __device__ __forceinline__ u32x4 get(int word) const {
        return __builtin_amdgcn_raw_buffer_load_b128(at, word * 16, 0, kAgent);
    }
    // The first `words` of them at `base` are none any more, by all threads of a workgroup.  (Through the caches: that has to have
    // arrived at the launch's end only.  Eight stores to a branch, past the last word dropped: one CU does it.)
    static __device__ __forceinline__ void take_away(void *base, int words, int tid, int threads) {
        const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(base, 0, words * 16, 0x00027000);
        for (int i = tid; i < words; i += 8 * threads)
#pragma unroll
            for (int t = 0; t < 8; ++t)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, to, (i + t * threads) * 16, 0, 0);
    }
    __device__ __forceinline__ bool there(u32x4 w) const { return w.y == lo && w.w == hi; }
};

// The words `load(t)` of N parts `part(t)` (nparts and more: none, and what it loads is not used), all requested before the
// first is looked at; what is not there is asked for again, up to `looks` times.  The least (part ^ own) of a lane's missing
// parts, INT32_MAX if there is none: of several parts the one nearest to the workgroup's own by exclusive or, so
// that each begins with another one.
template <int N, class Part, class Load>
__device__ __forceinline__ int look_for(const Words &x, int nparts, int own, int looks, u32x4 (&w)[N], Part &&part, Load &&load) {
#pragma unroll
    for (int t = 0; t < N; ++t) w[t] = load(t);
    for (int look = 0;; ++look) {
        int missing = INT32_MAX;
#pragma unroll
        for (int t = 0; t < N; ++t)
            if (part(t) < nparts && !x.there(w[t])) missing = min(missing, part(t) ^ own);
        if (__builtin_amdgcn_ballot_w64(missing != INT32_MAX) == 0 || look >= looks) return missing;
        __builtin_amdgcn_s_sleep(4);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < N; ++t)
            if (__builtin_amdgcn_ballot_w64(part(t) < nparts && !x.there(w[t])) != 0) w[t] = load(t);
    }
}
// The least over the wave, for the workgroup's decision.
__device__ __forceinline__ int least_missing(int missing) {
    return __builtin_amdgcn_ballot_w64(missing != INT32_MAX) == 0 ? INT32_MAX : reduce_lanes<1, 64>(missing, OpMinI{});
}

// The largest of EACH values (none below 0) per part, one to a word, over all parts, by `threads` threads; the wave's
// largest, and what is missing, as look_for().
template <int EACH>
__device__ __forceinline__ int largest_of(const Words &x, int nparts, int own, int looks, int tid, int threads, float &largest) {
    const int words = EACH * nparts;
    int missing = INT32_MAX;
    largest = 0.f;
    for (int p0 = tid; p0 - (tid & 63) < words; p0 += 2 * threads) {
        u32x4 w[2];
        auto at = [&](int t) { return p0 + t * threads; };
        missing = look_for(x, nparts, own, looks, w, [&](int t) { return at(t) < words ? at(t) / EACH : INT32_MAX; },
                           [&](int t) { return x.get(min(at(t), words - 1)); });
        if (__builtin_amdgcn_ballot_w64(missing != INT32_MAX) != 0) break;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (at(t) < words) largest = fmaxf(largest, __uint_as_float(w[t].x));
    }
    largest = wave_max(largest);
    return missing;
}

// The count of a problem's workgroups that have seen all parts, so that the last one can take the words away.
// Whoever does part 0 sets it to the tag (unless somebody else has) before leaving that part's words:
// nobody counts himself before.  One thread of the workgroup: `look` early, `start` some time
// before, `started` (its wave) in front of the barrier before the first word.  Calls that are not replayed count nothing.
struct Count {
    uint64_t found;
    __device__ __forceinline__ void look(const Exchange &x, int z) {
        if (x.replayed) found = get(x.count(z));
    }
    __device__ __forceinline__ void start(const Exchange &x, int z) {
        if (x.replayed && (found ^ x.tag) >> kCountBits)
            (void)__hip_atomic_compare_exchange_strong(x.count(z), &found, x.tag, __ATOMIC_RELAXED,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void started(const Exchange &x) { arrived(x); }
    // The wave's words have arrived: in front of a barrier between the last word and `arrive`.  (Else one of this workgroup's could
    // come behind the taking away, where another has done its part, too.)
    static __device__ __forceinline__ void arrived(const Exchange &x) {
        if (x.replayed) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    // once per workgroup, when all its waves have seen all parts
    __device__ __forceinline__ void arrive(const Exchange &x, int z) {
        if (x.replayed) found = __hip_atomic_fetch_add(x.count(z), (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};
// At the end of the workgroup's work, by all its threads; `counted`: the one that arrived; `flag`: in LDS, used by nobody since a
// barrier.  Whether it is the last of its problem, which takes the words away.
__device__ __forceinline__ bool leave(const Exchange &x, int z, int nparts, const Count &c, bool counted, int *flag) {
    if (!x.replayed) return false;
    if (counted) *flag = c.found == x.tag + (uint64_t)(nparts - 1);
    __syncthreads();
    if (*flag != 0 && counted) put(x.count(z), (uint64_t)0);
    return *flag != 0;
}

// Row statistics.
// The pair held by lane ^ 32.
__device__ __forceinline__ void from_other_half(float M, float s, float &M2, float &s2) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(M), __float_as_uint(M), false, false);
    const auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    const bool hi = threadIdx.x & 32;  // the swap leaves (low half's, high half's) in both
    M2 = __uint_as_float(hi ? a[0] : a[1]);
    s2 = __uint_as_float(hi ? c[0] : c[1]);
}

// (max, sum of exp2(value - max)) of (M, s) and (M2, s2)
__device__ __forceinline__ void merge_stats(float &M, float &s, float M2, float s2) {
    const float mn = fmaxf(M, M2), ref = mn == -INFINITY ? 0.f : mn;
    s = s * fast_exp2(M - ref) + s2 * fast_exp2(M2 - ref);
    M = mn;
}

// The pair held by lane ^ 16.
__device__ __forceinline__ void from_other_row(float M, float s, float &M2, float &s2) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(M), __float_as_uint(M), false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    const bool odd = threadIdx.x & 16;
    M2 = __uint_as_float(odd ? a[0] : a[1]);
    s2 = __uint_as_float(odd ? c[0] : c[1]);
}

// A row's value (log2-sum-exp2 of a range) of threads 0 .. ROWS - 1, two rows to a word; `first`: the part's first word.
__device__ __forceinline__ void put_rows(const Words &x, int first, int tid, float value) {
    const float other = from_lane_xor<1>(value);
    if ((tid & 1) == 0) x.put(first + (tid >> 1), value, other);
}

// A wave's share of merging the ranges' values of a problem's ROWS rows: parts wave + WAVES * i, lanes
// over pairs of rows (and parts, for fewer than 128 rows), several loads in flight; its (max, sum) pairs into
// `first` (its entry of row 0).  `word0`: of part 0; `ld`: words between parts.  What is missing, as look_for().
template <int ROWS, int WAVES>
__device__ __forceinline__ int merge_parts(const Words &x, int word0, int ld, int nparts, int own, int looks, float2 *first,
                                           int wave, int lane) {
    constexpr int WORDS = ROWS / 2, LW = WORDS <= 16 ? 16 : WORDS <= 32 ? 32 : 64, SUBS = 64 / LW;
    constexpr int WPL = (WORDS + 63) / 64, BATCH = WPL == 1 ? 8 : 4;  // words of a lane and part; parts in flight
    const int sub = lane / LW, at = min(lane % LW, WORDS - 1);
    float M[WPL][2], s[WPL][2];
#pragma unroll
    for (int r = 0; r < WPL; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) M[r][c] = -INFINITY, s[r][c] = 0.f;
    for (int i0 = 0; wave + WAVES * i0 * SUBS < nparts; i0 += BATCH) {
        u32x4 e[WPL * BATCH];
        auto part = [&](int t) { return wave + WAVES * ((i0 + t / WPL) * SUBS + sub); };
        const int missing = look_for(x, nparts, own, looks, e, part, [&](int t) {
            return x.get(word0 + min(part(t), nparts - 1) * ld + (t % WPL ? min(64 + at, WORDS - 1) : at));
        });
        if (__builtin_amdgcn_ballot_w64(missing != INT32_MAX) != 0) return missing;
#pragma unroll
        for (int r = 0; r < WPL; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float v[BATCH], bm = -INFINITY, bs = 0.f;
#pragma unroll
                for (int t = 0; t < BATCH; ++t) {
                    v[t] = part(t * WPL) < nparts ? __uint_as_float(c ? e[t * WPL + r].z : e[t * WPL + r].x) : -INFINITY;
                    bm = fmaxf(bm, v[t]);
                }
                const float ref = bm == -INFINITY ? 0.f : bm;
#pragma unroll
                for (int t = 0; t < BATCH; ++t) bs += fast_exp2(v[t] - ref);
                merge_stats(M[r][c], s[r][c], bm, bs);
            }
    }
#pragma unroll
    for (int r = 0; r < WPL; ++r) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float M2, s2;
            if constexpr (SUBS >= 2) {
                from_other_half(M[r][c], s[r][c], M2, s2);
                merge_stats(M[r][c], s[r][c], M2, s2);
            }
            if constexpr (SUBS == 4) {
                from_other_row(M[r][c], s[r][c], M2, s2);
                merge_stats(M[r][c], s[r][c], M2, s2);
            }
        }
        const int word = lane % LW + 64 * r;
        if (sub == 0 && word < WORDS) *(f32x4 *)(first + 2 * word) = f32x4{M[r][0], s[r][0], M[r][1], s[r][1]};
    }
    return INT32_MAX;
}

}  // namespace aha
