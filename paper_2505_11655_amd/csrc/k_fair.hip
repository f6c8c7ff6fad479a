// Fair draws from weighted samples: the last step of an ILE run (extrinsic
// samples drawn fairly from the weighted Monte Carlo samples) and of the
// posterior construction.  k independent draws with replacement; index i has
// probability q_i / sum q with q_i = floor(exp(lw_i - max lw) 2^40) (0 for
// non-finite lw).  Integer masses give exact prefix sums, so every draw's
// index is independent of the order of accumulation:
//   1. k_fair_max: each block's max lw (order-preserving integer keys);
//   2. k_fair_sums: the inclusive prefix of the masses inside each block's run
//      of tiles, by samples or by granules of 64 samples (one wave load), and
//      the run's total;
//   3. k_fair_pick: draw j with Philox counter (j lo, j hi, round, 16 * 5),
//      r = w0 2^32 + w1, target = floor(r * total / 2^64); the index is the
//      first i whose cumulative mass exceeds target: a search over the runs
//      (scanned in LDS by every block), then over the run's samples, or over
//      its granules and through the granule's 64 samples, whose masses are
//      formed again.  With total = 0 the index is -1.
// What bounds it: the two reads of lw.  By granules only 0.125 B per sample is
// written, where a prefix per sample costs 8 B, but a draw costs up to 64
// exponentials one after the other.  So by samples where the call is latency, up
// to 1.5 x 2^20 samples, and above with more than a draw per 16 samples.  By
// samples against by granules, FP32, us per call: weights of an event, to 4,096
// draws, 2^12 samples 16, 17; 2^16 15, 23; 2^20 17, 24; 2^21 18, 18; FP64, 2^22 29, 22;
// 2^18 draws 33, 28.  Weights spread so that every sample has mass: 100 samples to
// 1,000 draws 12, 28; 2^20 to 2^20 74, 181; 2^22 to 2^18 51, 75, to 2^20 109, 210; 2^26
// to 2^20 528, 504, to 2^22 1190, 1233.
// Measured, FP32, 2^26 samples to 2^20 draws: max 49 us (5.5 TB/s; 173 us with
// one load in flight per lane and an atomic per wave), sums 47 us (597 us for
// tile sums plus a prefix per sample in two passes), pick 43 us (32 us from a
// prefix per sample, plus a 31 us scan kernel); the call 812 -> 159 us.
#include <type_traits>

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
constexpr int64_t kFairAllSamples = 3 << 19;               // a prefix per sample up to so many samples,
constexpr int64_t kFairAllDraws = 16;                      // or with more than a draw per so many
static_assert(kFairTileGran == 64, "the granules of a tile are scanned by one wave");

// Scratch: [0] max key, [1 .. 1 + kFairMaxBlocks) the blocks' max keys,
// [.. + kFairRuns) the runs' totals, then the prefixes.
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

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ unsigned long long wave_scan(unsigned long long s, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long a = __shfl_up(s, o);
        s += lane >= o ? a : 0ull;
    }
    return s;
}

// A run of `per` tiles per block.  Granules: the waves sum the granules of a
// tile while the first wave scans the previous tile's (two LDS rows).  Samples
// (ALL): the waves scan their granules, and each adds the prefix of the tile's
// granules.
template <class TO, bool ALL>
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
    unsigned long long carry = 0;   // the run's mass so far (granules: in the first wave)
    int buf = 0;
    for (int64_t t = t0; t < t1; t++) {
        unsigned long long mine = 0, inc[ALL ? kFairLoads : 1];
        fair_tile(lw, t * kFairTile, n, wv, lane, [&](int j, TO v) {
            unsigned long long q = km ? fmass(v, vmax) : 0ull;
            if (__ballot(q != 0)) {   // most granules of a peaked run hold no mass
                if constexpr (ALL) {
                    q = wave_scan(q, lane);
                } else {
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
                }
            }
            if constexpr (ALL) {
                inc[j] = q;
                q = __shfl(q, 63);
            }
            mine = lane == j ? q : mine;
        });
        if (lane < kFairLoads) sg[buf][wv * kFairLoads + lane] = mine;
        __syncthreads();
        if constexpr (ALL) {
            const unsigned long long g = sg[buf][lane], s = wave_scan(g, lane) + carry;
            const int64_t i0 = t * kFairTile + (int64_t)wv * kFairTile / (kFairThreads / 64) + lane;
#pragma unroll
            for (int j = 0; j < kFairLoads; j++) {
                const unsigned long long c = inc[j] + __shfl(s - g, wv * kFairLoads + j);
                if (i0 + j * kFairGran < n) pre[i0 + j * kFairGran] = c;
            }
            carry = __shfl(s, 63);
        } else if (wv == 0) {
            const unsigned long long s = wave_scan(sg[buf][lane], lane) + carry;
            pre[t * kFairTileGran + lane] = s;
            carry = __shfl(s, 63);
        }
        buf ^= 1;
    }
    if (threadIdx.x == 0) scratch[kFairTotals + blockIdx.x] = carry;
}

template <class TO, class TT, bool ALL>
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
    const unsigned long long inc = wave_scan(s, lane);
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
            // the run, then the granule (or the sample) of the run, that holds the target
            int lo = 0, hi = runs - 1;
            while (lo < hi) {
                const int mid = (lo + hi) / 2;
                if (run[mid] > target)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            target -= lo > 0 ? run[lo - 1] : 0ull;
            constexpr int kPer = ALL ? kFairTile : kFairTileGran;   // prefixes per tile
            const int64_t g0 = (int64_t)lo * per * kPer;
            int64_t gl = g0, gh = ((lo + 1) * per < ntiles ? (lo + 1) * per : ntiles) * kPer - 1;
            if (ALL) gh = gh < n ? gh : n - 1;
            while (gl < gh) {
                const int64_t mid = gl + (gh - gl) / 2;
                if (pre[mid] > target)
                    gh = mid;
                else
                    gl = mid + 1;
            }
            if constexpr (ALL) {
                pick = gl;
            } else {
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
                  int64_t ld, TT *theta_out, int64_t ld_out, bool all, unsigned long long *scratch, hipStream_t st) {
    const FairPlan p = fair_plan(n);
    const dim3 block(kFairThreads);
    hipLaunchKernelGGL(k_fair_max<TO>, dim3(p.mblocks), block, 0, st, lw, n, scratch);
    int64_t gk = (k + kFairThreads - 1) / kFairThreads;
    gk = gk > 4096 ? 4096 : gk;
    auto go = [&](auto A_) {
        constexpr bool ALL = decltype(A_)::value;
        hipLaunchKernelGGL((k_fair_sums<TO, ALL>), dim3(p.runs), block, 0, st, lw, n, p.ntiles, p.per, p.mblocks, scratch);
        hipLaunchKernelGGL((k_fair_pick<TO, TT, ALL>), dim3((unsigned)gk), block, 0, st, lw, n, p.ntiles, p.per, p.runs,
                           scratch, seed, round, k, idx, theta, ld, theta_out, ld_out);
    };
    if (all)
        go(std::true_type{});
    else
        go(std::false_type{});
    return hipGetLastError();
}

}  // namespace

bool fair_all(int64_t n, int64_t k) { return n <= kFairAllSamples || k > n / kFairAllDraws; }

size_t fair_scratch_bytes(int64_t n, bool all) {
    const int64_t prefixes = all ? n : fair_plan(n).ntiles * kFairTileGran;
    return ((size_t)kFairHead + (size_t)prefixes) * sizeof(unsigned long long);
}

hipError_t launch_fair_draw(int policy, const void *lw, int64_t n, uint64_t seed, uint32_t round, int64_t k,
                            int64_t *idx, const void *theta, int64_t ld, void *theta_out, int64_t ld_out, bool all,
                            void *scratch, hipStream_t st) {
    if (n <= 0 || k <= 0) return hipSuccess;
    unsigned long long *sc = (unsigned long long *)scratch;
    if (policy == kFP32)
        return fair_t<float, float>((const float *)lw, n, seed, round, k, idx, (const float *)theta, ld,
                                    (float *)theta_out, ld_out, all, sc, st);
    if (policy == kFP64)
        return fair_t<double, double>((const double *)lw, n, seed, round, k, idx, (const double *)theta, ld,
                                      (double *)theta_out, ld_out, all, sc, st);
    return fair_t<double, float>((const double *)lw, n, seed, round, k, idx, (const float *)theta, ld,
                                 (float *)theta_out, ld_out, all, sc, st);
}

}  // namespace ile
