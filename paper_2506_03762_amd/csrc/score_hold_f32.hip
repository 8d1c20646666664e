// fp32 eviction scores (Sec. 4.1 - 4.3; Alg. 1 Prefill) of smaller problems in ONE launch.
//
// A workgroup owns a range of a (batch, KV head) problem's keys: 128, 32 to a wave, or, where workgroups are few and a wave would
// have several blocks of 32 rows one after the other, 32 keys whose row blocks are dealt to its four waves.  A block
// of 32 rows leaves its exponentials, relative to the largest product that a lane sees, in LDS, and
// per row their (maximum, sum) pair; the workgroups exchange the pairs and their largest priors
// (exchange.h), and a factor per row turns the exponentials into probabilities.  One exponential per row and key, and the
// keys are read once, where two launches (score_f32.hip) form both twice; what is exchanged is
// not rounded to a log-sum-exp of some tens.
//
// Bound by latency.  Stamps at 2 heads x 512 keys x 32 rows, d = 64 (us): rows, keys and values in LDS 2.5, 32 products 1, 16
// exponentials and the row's sum 0.8, prior 0.6, exchange 2, probabilities and sums 1.  us of the score stage in two launches and
// here: 4 heads x 2968 keys x 32 rows, d = 64 18.7, 9.6; 8 x 3048 x 64, d = 128 37.8, 20.2; 16 x 1335 x 128 50.2, 27.6; 4
// x 2 x 64 rows of 216 (ranges of 32 keys) 21.7, 14.2; 2 x 512 x 32, d = 64 as long, but a launch less to enqueue.
#include "exchange.h"
#include "f32_tile.h"
#include "value_tile.h"

namespace aha {

// (m, s): maximum and sum relative to it
__device__ __forceinline__ void merge_pair(float &m, float &s, float m2, float s2) {
    const float M = fmaxf(m, m2), ref = M == -INFINITY ? 0.f : M;
    s = s * exp2f(m - ref) + s2 * exp2f(m2 - ref);
    m = M;
}

// Static LDS. KW: waves over the keys, of four; the others over the row blocks
template <int KW>
struct HoldF32Smem {
    static constexpr int KEYS = KW * 32, ROWS = kHoldF32Blocks * 32;
    float2 row[KW][ROWS], mrg[256];
    float ref[kHoldF32Blocks][KW * 64], lam[ROWS], M[ROWS], inv[ROWS];
    float nu[KEYS + 256], gam[KEYS], max[4], all[4], acc[4 / KW][KEYS];
    int missing[4];
};
static_assert(sizeof(HoldF32Smem<1>) <= kHoldF32Static && sizeof(HoldF32Smem<4>) <= kHoldF32Static, "what the plan reckons with");

template <int D, int KW>
__global__ __launch_bounds__(256, 2) void f32_hold_kernel(ScoreGeom g, int nparts, Exchange x, u32x4 *stats, u32x4 *maxima,
                                                          float *scores) {
    constexpr int RW = 4 / KW, KEYS = KW * 32, GT = KW * 64, QB = 32 * f32_ld(D);
    extern __shared__ __attribute__((aligned(16))) float dyn[];  // a query block per RW; weights [block][key wave][element][lane]
    __shared__ HoldF32Smem<KW> sm;
    const int nblocks = (g.R + 31) / 32, rp = nblocks * 32;
    float *sw = dyn + RW * QB;

    const int wave = uniform((int)threadIdx.x >> 6), kw = wave % KW, rw = wave / KW;
    float *sq = dyn + rw * QB;
    const int own = (int)blockIdx.x % nparts, z = (int)blockIdx.x / nparts;
    const int b = z / g.Hkv, h = z % g.Hkv;
    const RowMap rm{g.n, g.r, g.R, nullptr};
    const float *kbase = (const float *)g.k + b * g.ks[0] + h * g.ks[1];
    const char *vbase = (const char *)((const float *)g.v + b * g.vs[0] + h * g.vs[1]);
    const int half = (g.pool - 1) / 2;

    Count count;
    const Words rows(stats + (int64_t)z * nparts * g.R, x.tag), priors(maxima + (int64_t)z * nparts, x.tag);
    int kbeg;
    for (int part = own;;) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        kbeg = part * KEYS;
        const int kb = kbeg + kw * 32, gt = tid % GT;
        if (part == 0 && tid == 255) count.look(x, z);
        F32QueryBlock<D, GT> qb;
        qb.request(g, rm, b, h, rw * 32, gt);
        f32x4 a[D / 8];
        f32_load_keys<D>(kbase, g.ks[2], kb, g.n - 1, lane, a);
        if (tid < rp)  // (while the loads travel)
            sm.lam[tid] = row_scale_log2(g.scale_mode, g.fixed_scale, g.lambda_floor, max(rm.pos(tid), 0) + 1, g.budget, g.d);
        if (g.value_prior)
            value_norms_to_lds<4>(vbase, g.vs[2], D, max(0, kbeg - half), min(g.n, kbeg + KEYS + half), sm.nu, tid);
        if (part == 0 && tid == 255) count.start(x, z);
        qb.commit(gt, sq);
        __syncthreads();
        for (int nb0 = 0;;) {
            const int nb = nb0 + rw;  // (past the last block: nothing is left of it)
            const int pos = rm.pos(nb * 32 + (lane & 31));  // -1 past the last row
            const float lam = sm.lam[min(nb * 32, rp - 32) + (lane & 31)];
            f32x16 t = f32_block_dots<D>(a, sq + (lane & 31) * f32_ld(D) + 4 * (lane >> 5));
            float mx = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (acc_key(kb, 0, v, lane) <= pos) mx = fmaxf(mx, t[v]);
            float m = mx == -INFINITY ? -INFINITY : mx * lam;
            const float mref = m == -INFINITY ? 0.f : m;
            if (nb < nblocks) {
                float *w = sw + ((nb * KW + kw) * 16) * 64 + lane;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    t[v] = acc_key(kb, 0, v, lane) <= pos ? exp2f(fmaf(t[v], lam, -mref)) : 0.f;
                    w[v * 64] = t[v];
                }
                sm.ref[nb][gt] = m;
#pragma unroll
                for (int o = 8; o; o >>= 1)
#pragma unroll
                    for (int v = 0; v < o; ++v) t[v] += t[v + o];
                float s = t[0];
                merge_pair(m, s, __shfl_xor(m, 32), __shfl_xor(s, 32));
                if (lane < 32) sm.row[kw][nb * 32 + lane] = make_float2(m, s);
            }
            nb0 += RW;
            if (nb0 >= nblocks) break;
            qb.request(g, rm, b, h, (nb0 + rw) * 32, gt);
            __syncthreads();
            qb.commit(gt, sq);
            __syncthreads();
        }
        if (g.value_prior) {
            float gam = 0.f;
            const int j = kbeg + tid;
            if (tid < KEYS && j < g.n) {
                const int lo = max(0, kbeg - half), first = max(0, j - half), last = min(g.n - 1, j + half);
                float s = 0.f;
                for (int t = first; t <= last; ++t) s += sm.nu[t - lo];
                gam = s / (float)(last - first + 1);
                sm.gam[tid] = gam;
            }
            gam = wave_max(gam);
            if (lane == 0) sm.max[wave] = gam;
        }
        if (part == 0 && wave == 3) count.started(x);
        __syncthreads();
        if (g.value_prior && tid == 255) priors.put(part, fmaxf(fmaxf(sm.max[0], sm.max[1]), fmaxf(sm.max[2], sm.max[3])), 0.f);
        if (tid < g.R) {
            float m = sm.row[0][tid].x, s = sm.row[0][tid].y;
#pragma unroll
            for (int wv = 1; wv < KW; ++wv) merge_pair(m, s, sm.row[wv][tid].x, sm.row[wv][tid].y);
            rows.put(part * g.R + tid, m, s);
        }
        // the rows' pairs over all parts: a thread takes a row of every subs-th part; the priors of up to 256 parts travel with them
        const int subs = 256 / rp, row = tid % rp, sub = tid / rp;
        u32x4 prior = priors.get(min(tid, nparts - 1));
        const bool active = row < g.R && sub < subs;
        float m = -INFINITY, s = 0.f;
        int missing = INT32_MAX;
        for (int p0 = 0; p0 < nparts; p0 += 4 * subs) {
            u32x4 w[4];
            auto at = [&](int t) { return active ? p0 + sub + t * subs : INT32_MAX; };
            missing = look_for(rows, nparts, own, x.looks, w, at,
                               [&](int t) { return rows.get(min(p0 + sub + t * subs, nparts - 1) * g.R + min(row, g.R - 1)); });
            if (__builtin_amdgcn_ballot_w64(missing != INT32_MAX) != 0) break;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (at(t) < nparts) merge_pair(m, s, __uint_as_float(w[t].x), __uint_as_float(w[t].z));
        }
        sm.mrg[tid] = make_float2(m, s);
        if (g.value_prior && __builtin_amdgcn_ballot_w64(missing != INT32_MAX) == 0) {
            float gm;
            if (nparts <= 256 && __builtin_amdgcn_ballot_w64(tid < nparts && !priors.there(prior)) == 0)
                gm = wave_max(tid < nparts ? __uint_as_float(prior.x) : 0.f);
            else
                missing = largest_of<1>(priors, nparts, own, x.looks, tid, 256, gm);
            if (lane == 0) sm.all[wave] = gm;
        }
        missing = least_missing(missing);
        if (lane == 0) sm.missing[wave] = missing;
        count.arrived(x);
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) missing = min(missing, sm.missing[wv]);
        missing = uniform(missing);
        if (missing == INT32_MAX && part == own) break;
        // somebody is not there: done here (and no more waiting); in the end the own part again, whose weights LDS has to hold
        part = missing != INT32_MAX ? missing ^ own : own;
        x.looks = 0;
        __syncthreads();
    }
    const int tid = threadIdx.x, lane = tid & 63, kb = kbeg + kw * 32;
    if (tid == 255) count.arrive(x, z);
    if (tid < rp) {
        float m = -INFINITY, s = 0.f;
        for (int sub = 0; sub < min(256 / rp, nparts); ++sub) merge_pair(m, s, sm.mrg[sub * rp + tid].x, sm.mrg[sub * rp + tid].y);
        sm.M[tid] = m;
        sm.inv[tid] = 1.f / s;
    }
    __syncthreads();
    f32x16 col;
#pragma unroll
    for (int v = 0; v < 16; ++v) col[v] = 0.f;
    for (int nb = rw; nb < nblocks; nb += RW) {
        const int row = nb * 32 + (lane & 31), pos = rm.pos(row);
        const float f = exp2f(sm.ref[nb][tid % GT] - sm.M[row]) * sm.inv[row];
        const float *w = sw + ((nb * KW + kw) * 16) * 64 + lane;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = w[v * 64] * f;
            col[v] += acc_key(kb, 0, v, lane) <= pos ? p : 0.f;  // (a row that is not finite: nothing for keys it does not see)
        }
    }
    const float tot = fold16_over32(col, lane);
    const int my_v = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
    if ((lane & 1) == 0) sm.acc[rw][acc_key(kw * 32, 0, my_v, lane)] = tot;
    __syncthreads();
    const int j = kbeg + tid;
    if (tid < KEYS && j < g.n) {
        float out = RW == 1 ? sm.acc[0][tid] : (sm.acc[0][tid] + sm.acc[RW > 1 ? 1 : 0][tid]) + (sm.acc[RW > 2 ? 2 : 0][tid] + sm.acc[RW > 2 ? 3 : 0][tid]);
        if (g.value_prior) {
            const float gm = fmaxf(fmaxf(sm.all[0], sm.all[1]), fmaxf(sm.all[2], sm.all[3]));
            out = gm > 0.f ? out * (sm.gam[tid] / gm) : out;  // all-zero values: no prior
        }
        scores[(int64_t)z * g.n + j] = out;
    }
    if (leave(x, z, nparts, count, tid == 255, &sm.missing[1])) {
        Words::take_away(stats + (int64_t)z * nparts * g.R, nparts * g.R, tid, 256);
        if (g.value_prior) Words::take_away(maxima + (int64_t)z * nparts, nparts, tid, 256);
    }
}

template <int D, int KW>
static hipError_t launch_t(const ScoreGeom &g, const PrefillPlan &pl, const Exchange &x, char *w, float *scores, hipStream_t st) {
    const size_t bytes = hold_f32_lds(D, (g.R + 31) / 32, KW * 32);
    static DeviceOnce once;
    const hipError_t e = device_once(once, [] {
        return hipFuncSetAttribute((const void *)f32_hold_kernel<D, KW>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)hold_f32_lds(D, kHoldF32Blocks, KW * 32));
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((f32_hold_kernel<D, KW>), dim3((unsigned)(pl.Z * pl.hold32_parts)), dim3(256), bytes, st, g, pl.hold32_parts, x,
                       (u32x4 *)(w + pl.off_h32stats), (u32x4 *)(w + pl.off_h32max), scores);
    return hipGetLastError();
}

hipError_t launch_score_hold_f32(const ScoreGeom &g, const PrefillPlan &pl, void *ws, const ExchangeCall &call, float *scores,
                                 hipStream_t st) {
    char *w = (char *)ws;
    const Exchange x{(uint64_t *)(w + pl.off_h32words), call.tag, call.looks, call.replayed};
    if (pl.hold32_keys == 32) return g.d == 64 ? launch_t<64, 1>(g, pl, x, w, scores, st) : launch_t<128, 1>(g, pl, x, w, scores, st);
    return g.d == 64 ? launch_t<64, 4>(g, pl, x, w, scores, st) : launch_t<128, 4>(g, pl, x, w, scores, st);
}

}  // namespace aha
