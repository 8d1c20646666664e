// Exchange between the workgroups of one problem inside one launch: every workgroup leaves its
// part of a result in the workspace, announces it, and uses the others' parts once all of them
// are announced.
//
// No cache is written back or invalidated for it (a device-scope release does that for the whole
// L2 of an XCD, microseconds per workgroup): what is exchanged is stored and loaded with relaxed
// agent-scope accesses, which go past the caches that are not shared, and an announcement is
// stored once the wave's counter of outstanding accesses says that its data has arrived
// (announce).  512 workgroups, 16 to 64 to a problem: 1.5 to 3 us from the first store to the last
// load.
//
// An announcement is the call's TAG, a 64-bit number that no other call of the process uses, so
// the workspace needs no clearing launch (3 us) in front: whatever it holds on entry is not this
// tag.  A captured graph replays a call with its tag, so the workgroup that is the last of its problem to have
// seen all announcements clears them.  It is found by a counter that starts itself: its upper
// bits are the tag's, and an arrival that finds other bits there sets them.
//
// Nobody depends on workgroups that may not be running: after `looks` looks at the announcements a
// workgroup does missing parts itself and announces them too (a part's result is the same bits whoever
// forms it).  The workgroups that have waited in vain share what is missing, so together they are done in
// about the time that the missing ones would have taken, and `looks` is a few times that (patience in
// aha_api.hip): beside other work that keeps half of a problem's workgroups out, waiting costs about
// as much as the work.
#pragma once

#include "aha_dev.h"

namespace aha {

struct Exchange {
    uint64_t *tags;    // [problem][part], or [problem][part][2] (announce_value)
    uint64_t *counts;  // [problem]
    uint64_t tag;      // of this call; the low kCountBits are zero, the rest is not
    int looks;         // at the announcements before missing parts are done here
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

// Every thread's put()s so far belong to part `part` of problem z: wait until they have arrived,
// then announce the part.  Called by the whole workgroup; one barrier.
__device__ __forceinline__ void announce(const Exchange &x, int z, int nparts, int part, int tid) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) put(x.tags + (int64_t)z * nparts + part, x.tag);
}

// A part of problem z that has not been announced after x.looks looks, nparts if there is none.  Of several the one
// nearest to the workgroup's own by exclusive or, so that each begins with another one.  Called by one wave of workgroup `own` (more of them would get in the way of the data's loads);
// every lane gets the result.
__device__ __forceinline__ int first_missing(const Exchange &x, int z, int nparts, int own, int lane) {
    const uint64_t *t = x.tags + (int64_t)z * nparts;
    int missing;
    for (int look = 0;; ++look) {
        missing = INT32_MAX;
        for (int p = lane; p < nparts; p += kWave)
            if (get(t + p) != x.tag) missing = min(missing, p ^ own);
        if (__builtin_amdgcn_ballot_w64(missing != INT32_MAX) == 0) return nparts;
        if (look >= x.looks) break;
        __builtin_amdgcn_s_sleep(4);
    }
    return reduce_lanes<1, 64>(missing, OpMinI{}) ^ own;
}

// Where all that a part leaves is one float, the announcement carries it: two words per part, the tag with
// one half of the value in its low bits each, both of which a reader has to find.  One trip to memory
// each way instead of two, and nothing to wait for in between.
__device__ __forceinline__ void announce_value(const Exchange &x, int z, int nparts, int part, float value, int tid) {
    if (tid >= 2) return;
    const uint32_t bits = __float_as_uint(value);
    put(x.tags + ((int64_t)z * nparts + part) * 2 + tid, x.tag | (tid ? bits >> 16 : bits & 0xffffu));
}
// first_missing() of such parts; the largest value (none is below 0) if there is none missing.  Two parts per
// lane at a time, and only by lanes that still miss one: waiting workgroups then stay out of the way
// of those that announce.
__device__ __forceinline__ int largest_value(const Exchange &x, int z, int nparts, int own, int lane, float &largest) {
    const uint64_t *t = x.tags + (int64_t)z * nparts * 2;
    largest = 0.f;
    for (int p0 = 0; p0 < nparts; p0 += 2 * kWave) {
        int missing = p0 + lane;  // of this lane's parts
        for (int look = 0;; ++look) {
            if (missing < nparts) {
                const int p1 = min(p0 + kWave + lane, nparts - 1);
                const uint64_t lo0 = get(t + 2 * (p0 + lane)), hi0 = get(t + 2 * (p0 + lane) + 1);
                const uint64_t lo1 = get(t + 2 * p1), hi1 = get(t + 2 * p1 + 1);
                const bool there0 = ((lo0 ^ x.tag) | (hi0 ^ x.tag)) >> kCountBits == 0;
                const bool there1 = ((lo1 ^ x.tag) | (hi1 ^ x.tag)) >> kCountBits == 0;
                if (there0 && there1) {
                    const float a = __uint_as_float((uint32_t)(lo0 & 0xffffu) | (uint32_t)(hi0 & 0xffffu) << 16);
                    const float b = __uint_as_float((uint32_t)(lo1 & 0xffffu) | (uint32_t)(hi1 & 0xffffu) << 16);
                    largest = fmaxf(largest, fmaxf(a, b));
                }
                missing = there0 ? (there1 ? nparts : p1) : p0 + lane;
            }
            if (__builtin_amdgcn_ballot_w64(missing < nparts) == 0) break;
            if (look >= x.looks)
                return reduce_lanes<1, 64>(missing < nparts ? missing ^ own : INT32_MAX, OpMinI{}) ^ own;
            __builtin_amdgcn_s_sleep(4);
        }
    }
    largest = wave_max(largest);
    return nparts;
}

// The count of a problem's workgroups that have seen all announcements, so that the last one can clear
// them.  Whoever does part 0 sets it to the tag (unless somebody else has) before announcing that part:
// nobody counts himself before.  One thread of the workgroup: `look` early, `start` some time
// before announce(), which waits for it.
struct Count {
    uint64_t found;
    __device__ __forceinline__ void look(const Exchange &x, int z) { found = get(x.counts + z); }
    __device__ __forceinline__ void start(const Exchange &x, int z) {
        if ((found ^ x.tag) >> kCountBits)
            (void)__hip_atomic_compare_exchange_strong(x.counts + z, &found, x.tag, __ATOMIC_RELAXED,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // once per workgroup, when it has seen all announcements
    __device__ __forceinline__ void arrive(const Exchange &x, int z) {
        found = __hip_atomic_fetch_add(x.counts + z, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};
// By the whole wave of the thread that arrived (its last lane), at the end of the workgroup's work.  WORDS: of
// an announcement.
template <int WORDS = 1>
__device__ __forceinline__ void leave(const Exchange &x, int z, int nparts, const Count &c, int lane) {
    if (__builtin_amdgcn_ballot_w64(lane == kWave - 1 && c.found == x.tag + (uint64_t)(nparts - 1)) == 0) return;
    for (int p = lane; p < WORDS * nparts; p += kWave) put(x.tags + (int64_t)z * nparts * WORDS + p, (uint64_t)0);
    if (lane == 0) put(x.counts + z, (uint64_t)0);
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

// A wave's share of merging the ranges' values of a problem's ROWS rows: parts wave + WAVES * i, lanes
// over rows (and parts, for fewer than 64 rows), several loads in flight; its (max, sum) pairs into
// red[wave][row] (`first`: its entry of row 0).  `ld`: floats between parts.
template <int ROWS, int WAVES>
__device__ __forceinline__ void merge_parts(const float *src, int ld, int nparts, float2 *first, int wave, int lane) {
    constexpr int RW = ROWS < 64 ? ROWS : 64, SUBS = 64 / RW, RPL = (ROWS + 63) / 64;
    constexpr int BATCH = RPL == 1 ? 8 : 4;  // loads of a row in flight
    const int sub = lane / RW;
    const float *p0 = src + lane % RW;
    float M[RPL], s[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) M[r] = -INFINITY, s[r] = 0.f;
    for (int i0 = 0; wave + WAVES * i0 * SUBS < nparts; i0 += BATCH) {
        float e[RPL][BATCH];
#pragma unroll
        for (int h = 0; h < BATCH; h += 4) {
            if (wave + WAVES * (i0 + h) * SUBS >= nparts) break;  // uniform
#pragma unroll
            for (int t = h; t < h + 4; ++t)
#pragma unroll
                for (int r = 0; r < RPL; ++r)
                    e[r][t] = get(p0 + (int64_t)min(wave + WAVES * ((i0 + t) * SUBS + sub), nparts - 1) * ld +
                                  (ROWS % 64 && r ? min(64, ROWS - 1 - lane % RW) : 64 * r));
        }
#pragma unroll
        for (int h = 0; h < BATCH; h += 4) {
            if (wave + WAVES * (i0 + h) * SUBS >= nparts) break;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                float bm = -INFINITY, bs = 0.f;
#pragma unroll
                for (int t = h; t < h + 4; ++t) {
                    if (wave + WAVES * ((i0 + t) * SUBS + sub) >= nparts) e[r][t] = -INFINITY;
                    bm = fmaxf(bm, e[r][t]);
                }
                const float ref = bm == -INFINITY ? 0.f : bm;
#pragma unroll
                for (int t = h; t < h + 4; ++t) bs += fast_exp2(e[r][t] - ref);
                merge_stats(M[r], s[r], bm, bs);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        if constexpr (SUBS == 2) {
            float M2, s2;
            from_other_half(M[r], s[r], M2, s2);
            merge_stats(M[r], s[r], M2, s2);
        }
        const int row = lane % RW + 64 * r;
        if (sub == 0 && row < ROWS) first[row] = make_float2(M[r], s[r]);
    }
}

}  // namespace aha
