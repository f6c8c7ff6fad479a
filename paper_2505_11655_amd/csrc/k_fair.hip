// Fair draws from weighted samples: the last step of an ILE run (extrinsic
// samples drawn fairly from the weighted Monte Carlo samples) and of the
// posterior construction.  k independent draws with replacement; index i has
// probability q_i / sum q with q_i = floor(exp(lw_i - max lw) 2^40) (0 for
// non-finite lw).  Integer masses give exact prefix sums, so every draw's
// index is independent of the order of accumulation:
//   1. k_fair_max: each block's max lw (order-preserving integer keys);
//   2. k_fair_sums: masses summed by granules of 64 samples (one wave load),
//      the inclusive prefix of the granules inside each block's run of tiles,
//      and the run's total;
//   3. k_fair_pick: draw j with Philox counter (j lo, j hi, round, 16 * 5),
//      r = w0 2^32 + w1, target = floor(r * total / 2^64); the index is the
//      first i whose cumulative mass exceeds target: a search over the runs
//      (scanned in LDS by every block), then over the run's granules, then
//      through the granule's 64 samples, whose masses are formed again.
//      With total = 0 the index is -1.
// What bounds it: the two reads of lw.  Only one prefix per 64 samples is
// written (0.125 B per sample, where a prefix per sample costs 8 B), and the
// exponential is taken only where the mass is not certainly zero.
// Measured, FP32, 2^26 samples to 2^20 draws: max 49 us (5.5 TB/s; 173 us with
// one load in flight per lane and an atomic per wave), sums 47 us (597 us for
// tile sums plus a prefix per sample), pick 43 us (32 us from a prefix per
// sample, plus a 31 us scan kernel); the call 812 -> 159 us.
#include "ile_internal.h"

namespace ile {

namespace {

constexpr int kFairThreads = 256;
constexpr int kFairGran = 64;                              // samples per granule: one wave load
constexpr int kFairLoads = 16;                             // loads in flight per lane
constexpr int kFairTile = kFairThreads * kFairLoads;       // samples per tile
constexpr int kFairTileGran = kFairTile / kFairGran;       // 64: one granule per lane of a wave
constexpr int kFairRuns = 2048;                            // most runs (blocks of k_fair_sums): 8 per CU
constexpr int kFairMaxBlocks = 1024;                       // most blocks of k_fair_max: 4 per CU
constexpr uint32_t kFairAttempt = 5;
static_assert(kFairTileGran == 64, "the granules of a tile are scanned by one wave");

// Scratch: [0] max key, [1 .. 1 + kFairMaxBlocks) the blocks' max keys,
// [.. + kFairRuns) the runs' totals, then the granule prefixes.
constexpr int kFairTotals = 1 + kFairMaxBlocks;
constexpr int kFairHead = kFairTotals + kFairRuns;

struct FairPlan {
    int64_t ntiles, per;   // tiles, and tiles per run
    int runs, mblocks;
};
FairPlan fair_plan(int64_t n) {
    FairPlan p;
    p.ntiles = (n + kFairTile - 1) / kFairTile;
    p.per = (p.ntiles + kFairRuns - 1) / kFairRuns;
    p.runs = (int)((p.ntiles + p.per - 1) / p.per);
    p.mblocks = (int)(p.ntiles < kFairMaxBlocks ? p.ntiles : kFairMaxBlocks);
    return p;
}

// One tile's samples, kFairLoads per thread, the lanes of a wave on
// consecutive samples (no alignment is asked of lw); -inf past the end.
template <class TO, class F>
__device__ __forceinline__ void fair_tile(const TO *__restrict__ lw, int64_t base, int64_t n, int wv, int lane, F &&f) {
    TO x[kFairLoads];
    const int64_t i0 = base + (int64_t)wv * (kFairLoads * kFairGran) + lane;
    if (base + kFairTile <= n) {
#pragma unroll
        for (int j = 0; j < kFairLoads; j++) x[j] = lw[i0 + j * kFairGran];
    } else {
#pragma unroll
        for (int j = 0; j < kFairLoads; j++) x[j] = i0 + j * kFairGran < n ? lw[i0 + j * kFairGran] : (TO)-INFINITY;
    }
#pragma unroll
    for (int j = 0; j < kFairLoads; j++) f(j, x[j]);
}

template <class TO>
__global__ void __launch_bounds__(kFairThreads) k_fair_max(const TO *__restrict__ lw, int64_t n,
                                                           unsigned long long *__restrict__ scratch) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    TO m = (TO)-INFINITY;
    for (int64_t base = (int64_t)blockIdx.x * kFairTile; base < n; base += (int64_t)gridDim.x * kFairTile)
        fair_tile(lw, base, n, wv, lane, [&](int, TO v) { m = (v < (TO)INFINITY && v > m) ? v : m; });
    unsigned long long km = m > (TO)-INFINITY ? ord_key(m) : 0ull;   // 0: no finite sample
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long k2 = __shfl_xor(km, o);
        km = k2 > km ? k2 : km;
    }
    __shared__ unsigned long long sm[kFairThreads / 64];
    if (lane == 0) sm[wv] = km;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kFairThreads / 64; i++) km = sm[i] > km ? sm[i] : km;
        scratch[1 + blockIdx.x] = km;
    }
}

// The mass of a sample (0 for a non-finite one).
template <class TO>
__device__ __forceinline__ unsigned long long fmass(TO v, double vmax) {
    return v < (TO)INFINITY ? mass_fx((double)v, vmax) : 0ull;
}

// A run of `per` tiles per block.  The waves sum the granules of a tile while
// the first wave scans the previous tile's (two LDS rows).
template <class TO>
__global__ void __launch_bounds__(kFairThreads)
    k_fair_sums(const TO *__restrict__ lw, int64_t n, int64_t ntiles, int64_t per, int mblocks,
                unsigned long long *__restrict__ scratch) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __shared__ unsigned long long sk[kFairThreads / 64], sg[2][kFairTileGran];
    // the blocks' max keys, reduced by every block
    unsigned long long km = 0;
    for (int i = threadIdx.x; i < mblocks; i += kFairThreads) {
        const unsigned long long k2 = scratch[1 + i];
        km = k2 > km ? k2 : km;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long k2 = __shfl_xor(km, o);
        km = k2 > km ? k2 : km;
    }
    if (lane == 0) sk[wv] = km;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kFairThreads / 64; i++) km = sk[i] > km ? sk[i] : km;
    if (blockIdx.x == 0 && threadIdx.x == 0) scratch[0] = km;
    const double vmax = km ? ord_value(km, sizeof(TO) * 8) : 0.0;
    unsigned long long *pre = scratch + kFairHead;
    const int64_t t0 = (int64_t)blockIdx.x * per, t1 = t0 + per < ntiles ? t0 + per : ntiles;
    unsigned long long carry = 0;   // first wave: the run's mass so far
    int buf = 0;
    for (int64_t t = t0; t < t1; t++) {
        unsigned long long mine = 0;
        fair_tile(lw, t * kFairTile, n, wv, lane, [&](int j, TO v) {
            unsigned long long q = km ? fmass(v, vmax) : 0ull;
            if (__ballot(q != 0)) {   // most granules of a peaked run hold no mass
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
            }
            mine = lane == j ? q : mine;
        });
        if (lane < kFairLoads) sg[buf][wv * kFairLoads + lane] = mine;
        __syncthreads();
        if (wv == 0) {
            unsigned long long s = sg[buf][lane];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long a = __shfl_up(s, o);
                s += lane >= o ? a : 0ull;
            }
            s += carry;
            pre[t * kFairTileGran + lane] = s;
            carry = __shfl(s, 63);
        }
        buf ^= 1;
    }
    if (threadIdx.x == 0) scratch[kFairTotals + blockIdx.x] = carry;
}

template <class TO, class TT>
__global__ void __launch_bounds__(kFairThreads)
    k_fair_pick(const TO *__restrict__ lw, int64_t n, int64_t ntiles, int64_t per, int runs,
                const unsigned long long *__restrict__ scratch, uint64_t seed, uint32_t round, int64_t k,
                int64_t *__restrict__ idx, const TT *__restrict__ theta, int64_t ld, TT *__restrict__ theta_out,
                int64_t ld_out) {
    // inclusive prefix of the runs' totals: kRt consecutive runs per thread
    constexpr int kRt = kFairRuns / kFairThreads;
    __shared__ unsigned long long run[kFairRuns], sw[kFairThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    unsigned long long v[kRt], s = 0;
#pragma unroll
    for (int i = 0; i < kRt; i++) {
        const int r = threadIdx.x * kRt + i;
        v[i] = r < runs ? scratch[kFairTotals + r] : 0ull;
        s += v[i];
    }
    unsigned long long inc = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long a = __shfl_up(inc, o);
        inc += lane >= o ? a : 0ull;
    }
    if (lane == 63) sw[wv] = inc;
    __syncthreads();
    unsigned long long off = inc - s;
    for (int i = 0; i < wv; i++) off += sw[i];
#pragma unroll
    for (int i = 0; i < kRt; i++) {
        off += v[i];
        run[threadIdx.x * kRt + i] = off;
    }
    __syncthreads();
    const unsigned long long total = run[kFairRuns - 1], km = scratch[0];
    const double vmax = km ? ord_value(km, sizeof(TO) * 8) : 0.0;
    const unsigned long long *pre = scratch + kFairHead;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    for (int64_t j = (int64_t)blockIdx.x * kFairThreads + threadIdx.x; j < k; j += (int64_t)gridDim.x * kFairThreads) {
        int64_t pick = -1;
        if (total > 0) {
            const U4 w = philox4x32_10(U4{(uint32_t)j, (uint32_t)((uint64_t)j >> 32), round, 16u * kFairAttempt}, k0,
                                       k1);
            const unsigned long long r = ((unsigned long long)w.x << 32) | w.y;
            unsigned long long target = __umul64hi(r, total);
            // the run, then the granule of the run, that holds the target
            int lo = 0, hi = runs - 1;
            while (lo < hi) {
                const int mid = (lo + hi) / 2;
                if (run[mid] > target)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            target -= lo > 0 ? run[lo - 1] : 0ull;
            const int64_t g0 = (int64_t)lo * per * kFairTileGran;
            int64_t gl = g0, gh = ((lo + 1) * per < ntiles ? (lo + 1) * per : ntiles) * kFairTileGran - 1;
            while (gl < gh) {
                const int64_t mid = gl + (gh - gl) / 2;
                if (pre[mid] > target)
                    gh = mid;
                else
                    gl = mid + 1;
            }
            target -= gl > g0 ? pre[gl - 1] : 0ull;
            // first sample of the granule whose cumulative mass exceeds the target
            const int64_t b = gl * kFairGran, e = b + kFairGran < n ? b + kFairGran : n;
            unsigned long long cum = 0;
            pick = e - 1;
            for (int64_t i = b; i < e; i++) {
                cum += fmass(lw[i], vmax);
                if (cum > target) {
                    pick = i;
                    break;
                }
            }
        }
        if (idx) idx[j] = pick;
        if (theta_out) {
#pragma unroll
            for (int c = 0; c < 7; c++) theta_out[c * ld_out + j] = pick >= 0 ? theta[c * ld + pick] : (TT)NAN;
        }
    }
}

template <class TO, class TT>
hipError_t fair_t(const TO *lw, int64_t n, uint64_t seed, uint32_t round, int64_t k, int64_t *idx, const TT *theta,
                  int64_t ld, TT *theta_out, int64_t ld_out, unsigned long long *scratch, hipStream_t st) {
    const FairPlan p = fair_plan(n);
    hipLaunchKernelGGL(k_fair_max<TO>, dim3(p.mblocks), dim3(kFairThreads), 0, st, lw, n, scratch);
    hipLaunchKernelGGL(k_fair_sums<TO>, dim3(p.runs), dim3(kFairThreads), 0, st, lw, n, p.ntiles, p.per, p.mblocks,
                       scratch);
    int64_t gk = (k + kFairThreads - 1) / kFairThreads;
    gk = gk > 2048 ? 2048 : gk;
    hipLaunchKernelGGL((k_fair_pick<TO, TT>), dim3((unsigned)gk), dim3(kFairThreads), 0, st, lw, n, p.ntiles, p.per,
                       p.runs, scratch, seed, round, k, idx, theta, ld, theta_out, ld_out);
    return hipGetLastError();
}

}  // namespace

size_t fair_scratch_bytes(int64_t n) {
    return ((size_t)kFairHead + (size_t)fair_plan(n).ntiles * kFairTileGran) * sizeof(unsigned long long);
}

hipError_t launch_fair_draw(int policy, const void *lw, int64_t n, uint64_t seed, uint32_t round, int64_t k,
                            int64_t *idx, const void *theta, int64_t ld, void *theta_out, int64_t ld_out,
                            void *scratch, hipStream_t st) {
    if (n <= 0 || k <= 0) return hipSuccess;
    unsigned long long *sc = (unsigned long long *)scratch;
    if (policy == kFP32)
        return fair_t<float, float>((const float *)lw, n, seed, round, k, idx, (const float *)theta, ld,
                                    (float *)theta_out, ld_out, sc, st);
    if (policy == kFP64)
        return fair_t<double, double>((const double *)lw, n, seed, round, k, idx, (const double *)theta, ld,
                                      (double *)theta_out, ld_out, sc, st);
    return fair_t<double, float>((const double *)lw, n, seed, round, k, idx, (const float *)theta, ld,
                                 (float *)theta_out, ld_out, sc, st);
}

}  // namespace ile
