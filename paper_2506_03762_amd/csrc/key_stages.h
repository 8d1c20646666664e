// Keys shared through LDS: what the kernels have in common whose waves own query rows, as fragments in registers, and take the
// keys from stages of LDS that hold a step's key rows for all of them (score_full.hip, score_share.hip).
#pragma once

#include "score_block.h"

namespace aha {

// The query rows of a KV head as the tiles count them: `pr` places per query head, of which the last pr - r are empty.  With pr a
// multiple of a wave's rows no wave has the end of one head and the start of the next, whose keys would be masked in every
// step and hold the other waves up (4 x 7 heads x 5000 rows 376 us, so 263; tiles in LDS 291); with pr = r the rows follow each other.
struct PlaceMap {
    static constexpr const int32_t *rows = nullptr;
    int n, r, G, pr;
    __device__ __forceinline__ bool valid(int at) const { return at < G * pr && at % pr < r; }
    __device__ __forceinline__ int pos(int at) const { return valid(at) ? n - r + at % pr : -1; }
    // largest / smallest position of the places [lo, hi)
    __device__ __forceinline__ int max_pos(int lo, int hi) const {
        hi = min(hi, G * pr);
        if (lo >= hi) return -1;
        if (lo / pr != (hi - 1) / pr) return n - 1;
        return lo % pr < r ? n - r + min(r - 1, (hi - 1) % pr) : -1;
    }
    __device__ __forceinline__ int min_pos(int lo, int hi) const {
        hi = min(hi, G * pr);
        if (lo >= hi) return n;
        if (lo / pr != (hi - 1) / pr) return n - r;
        return lo % pr < r ? n - r + lo % pr : n;
    }
};

// The wave's share of a step's key rows -> a stage of LDS, without passing registers: instruction j covers the RPI rows of
// group wave + WAVES j of a step of KEYS, lane -> row lane / CPR, position lane % CPR.  The loads are assembly and the waits for them by
// hand: the compiler would wait for everything behind each.
template <int D, int KEYS, int WAVES>
struct KeyRequest {
    using R = KeyRows<D>;
    static constexpr int NI = KEYS / R::RPI / WAVES;
    const __bf16 *kbase;
    int64_t tstride;
    int n, lane, wave, chunk;
    uint32_t lane_off, lds0;
    bool far;  // the token stride does not fit the 32-bit lane offset
    __device__ __forceinline__ KeyRequest(const __bf16 *kbase_, int64_t tstride_, int n_, int lane_, int wave_, const char *stages)
        : kbase(kbase_), tstride(tstride_), n(n_), lane(lane_), wave(wave_) {
        chunk = (lane % R::CPR) ^ R::swizzle(lane / R::CPR);  // (RPI rows: a multiple of the swizzle's period)
        lane_off = (uint32_t)((lane / R::CPR) * tstride * 2) + (uint32_t)(chunk * 16);
        lds0 = uniform((int)((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)stages + wave * R::group));
        far = tstride * 2 * R::RPI >= ((int64_t)1 << 31);
    }
    __device__ __forceinline__ void operator()(int kb, int st) const {
        const uint32_t dst = lds0 + st * R::bytes(KEYS);
        if (kb + KEYS <= n && !far) {
            const __bf16 *row0 = kbase + (int64_t)(kb + wave * R::RPI) * tstride;
#pragma unroll
            for (int j = 0; j < NI; ++j)
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                             :
                             : "v"(lane_off), "s"(row0 + (int64_t)(WAVES * R::RPI * j) * tstride), "s"(dst + j * WAVES * R::group)
                             : "memory");
            return;
        }
        const int r = wave * R::RPI + lane / R::CPR;
#pragma unroll
        for (int j = 0; j < NI; ++j) {  // rows past the sequence re-read its last one: masked
            const __bf16 *src = kbase + (int64_t)min(kb + r + WAVES * R::RPI * j, n - 1) * tstride + chunk * 8;
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                         :
                         : "v"(src), "s"(dst + j * WAVES * R::group)
                         : "memory");
        }
    }
};

// A wave's query rows: fragments of the rows at rho0 + 32 q + lane % 32 (empty places read a head's last row).
template <int D, int NQ>
__device__ __forceinline__ void load_rows_of_wave(const ScoreGeom &g, const PlaceMap &rm, int b, int h, int rho0, int lane,
                                                  bf16x8 (&qf)[NQ][D / 16]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int at = min(rho0 + 32 * q + (lane & 31), g.G * rm.pr - 1), gi = at / rm.pr, ii = min(at - gi * rm.pr, g.r - 1);
        const __bf16 *p = (const __bf16 *)g.q + b * g.qs[0] + (int64_t)(h * g.G + gi) * g.qs[1] +
                          (int64_t)(g.n - g.r + ii) * g.qs[2] + (lane >> 5) * 8;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[q][ks] = *(const bf16x8 *)(p + ks * 16);
    }
}

// The products `acc` of 32 keys (fragments kf) and 32 query rows (qf); with LAST, the last rows for these keys, the key
// fragments are replaced by those of the block at `next`.  In between 16 elements' vector work in D / 16 portions,
// `work(portion)`, whose instructions stay where they are written.  KEYS_M: keys on M, else on N.
template <int D, bool KEYS_M, bool LAST, class Work>
__device__ __forceinline__ void pipelined(const bf16x8 (&qf)[D / 16], bf16x8 (&kf)[D / 16], const char *next, int place,
                                          f32x16 &acc, Work work) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        acc = KEYS_M ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], ks ? acc : zero, 0, 0, 0)
                     : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], kf[ks], ks ? acc : zero, 0, 0, 0);
        if (LAST) kf[ks] = key_fragment(next, place, ks);
        __builtin_amdgcn_sched_barrier(0);
        work(ks);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// (the compiler moves what is only needed later behind the next barrier otherwise, out of the products' shadow)
__device__ __forceinline__ void keep_here(float &x) { asm volatile("" : "+v"(x)); }

// s_waitcnt vmcnt(N) alone; everything in LDS done.
template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// M + log2 s.  The logarithm is taken of s's mantissa: that of a sum of hundreds, relative to a reference of the first keys, is
// rounded down at its own size (with it the normalisers were 1.0e-7 too small on average, 4e-8 with waves that share a
// range's keys, whose sums are smaller).  The mantissa lies around 1, so that a single value, s = 1, stays as it is: from 0.5
// on, M + 1 - 1, given normalisers around 0.69 made the scores 5.0e-8 to 5.8e-8 wrong (rms) instead of 3.5e-8.
__device__ __forceinline__ float log2_sum(float M, float s) {
    const float m = __builtin_amdgcn_frexp_mantf(s);
    const bool low = m < 0.70710678f;
    return (M + (float)(__builtin_amdgcn_frexp_expf(s) - (low ? 1 : 0))) + log2f(low ? 2.f * m : m);
}

// Exact update of a row's (m, s) with 32 keys.
template <bool MASK>
__device__ __forceinline__ void exact_stats(const f32x16 &acc, float lam, int pos, int kb, int lane, float &m, float &s) {
    float amax = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) amax = fmaxf(amax, MASK && acc_key(kb, 0, v, lane) > pos ? -INFINITY : acc[v]);
    const float mn = fmaxf(m, amax == -INFINITY ? -INFINITY : amax * lam);
    const float mref = mn == -INFINITY ? 0.f : mn;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float e = fast_exp2(fmaf(acc[v], lam, -mref));
        sum[v & 3] += MASK && acc_key(kb, 0, v, lane) > pos ? 0.f : e;
    }
    s = s * fast_exp2(m - mref) + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
    m = mn;
}

}  // namespace aha
