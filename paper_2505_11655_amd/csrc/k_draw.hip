// Counter-based extrinsic draws for eq. (lnL:MonteCarlo): theta ~ p_s, with
// p_s the prior or the mixture proposal (1-eps) sum_j pi_j N_j/Z_j + eps p.
//
// Counter layout (key = seed words; each block gives four words):
//   sample i, round r, attempt a, block b:  (i lo, i hi, r, 16 a + b).
// Prior draw: 7 uniforms from blocks 0..3 of attempt 0 (words 2c, 2c+1),
// mapped by inverse CDFs.  Mixture draw: the selector is the first uniform of
// block 0 (attempt 0); the prior fallback and the non-mixture columns use
// blocks 1..4 of attempt 0; attempt a = 1..64 of a component draws z from
// four Box-Muller pairs of blocks 1..4 of attempt a (never the words of the
// prior draw, so the fallback is independent of the rejections) and accepts
// x = mu + L z if every bounded column is inside its interval and every
// periodic offset lies in (-P/2, P/2]; after 64 rejected attempts the prior
// draw is kept.  The density of the draw is therefore
//   p_s(x) = [eps + (1-eps) sum_j pi_j r_j] p(x)
//          + (1-eps) sum_j pi_j (1 - r_j) N_j(x) p_rest(x) / Z_j,
// r_j = (1 - Z_j)^64 the chance that all attempts fail, p_rest the prior of
// the columns outside the mixture (pi_j normalised).
//
// Two instantiations per sample type: prior-only launches (no mixture code,
// so the kernel stays small and occupancy high) and launches where some job
// carries a mixture.  A mixture spans its job's sampled columns, all seven or
// (distance integrated) all but the distance, so columns, bounds and periods
// are compile-time constants of D = 7 or 6 and every per-sample array stays in
// registers.
#include "ile_sincos.h"
#include <type_traits>

#include "ile_internal.h"

namespace ile {

namespace {

constexpr int kDrawThreads = 256;
constexpr int kMaxAttempts = 64;
constexpr double kPi = 3.14159265358979323846;

__device__ __forceinline__ void words(uint64_t seed, uint64_t i, uint32_t r, uint32_t a, int b0, int nb,
                                      uint32_t *w) {
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int b = 0; b < nb; b++) {
        U4 o = philox4x32_10(U4{(uint32_t)i, (uint32_t)(i >> 32), r, a * 16u + (uint32_t)(b0 + b)}, k0, k1);
        w[4 * b + 0] = o.x;
        w[4 * b + 1] = o.y;
        w[4 * b + 2] = o.z;
        w[4 * b + 3] = o.w;
    }
}

// Theta column, support and period of mixture dimension a.
constexpr int mix_col(int D, int a) { return D == 6 && a >= 3 ? a + 1 : a; }
constexpr double mix_period(int D, int a) {
    const int c = mix_col(D, a);
    return (c == 0 || c == 5) ? 2 * kPi : (c == 6 ? kPi : 0.0);
}
__device__ __forceinline__ void bounds(const PriorDev &pr, int col, double &lo, double &hi) {
    switch (col) {
    case 1: lo = -0.5 * kPi; hi = 0.5 * kPi; break;
    case 2: lo = -pr.t_window; hi = pr.t_window; break;
    case 3: lo = pr.d_min; hi = pr.d_max; break;
    default: lo = -1.0; hi = 1.0; break;   // cos iota; the other columns are periodic
    }
}

__device__ __forceinline__ void prior_from_words(const PriorDev &pr, const uint32_t *w, double th[7]) {
    double u[7];
#pragma unroll
    for (int c = 0; c < 7; c++) u[c] = u53(w[2 * c], w[2 * c + 1]);
    prior_map(pr, u, th);
}

// The parts of ln prior that do not depend on the sample: -ln(2 t_w) and
// 3 / (D_max^3 - D_min^3).
struct LnPrior {
    double t, d3;
};
__device__ __forceinline__ LnPrior ln_prior_consts(const PriorDev &pr) {
    const double a3 = pr.d_min * pr.d_min * pr.d_min, b3 = pr.d_max * pr.d_max * pr.d_max;
    return LnPrior{-log(2.0 * pr.t_window), 3.0 / (b3 - a3)};
}
constexpr double kLn2Pi = 1.8378770664093454836, kLnPi = 1.1447298858494001741, kLn2 = 0.69314718055994530942;

typedef __attribute__((address_space(4))) const GmmDev cgmm;
// A mixture's address, the same in every lane, in scalar registers.
__device__ __forceinline__ cgmm *uniform_gmm(const GmmDev *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (cgmm *)(((uint64_t)hi << 32) | lo);
}

// Running log-sum-exp: m the running maximum, s the sum of e^{t - m}.
// FAST: the exponential of the (FP64) difference taken in FP32, for sums
// whose terms need only FP32 relative accuracy.
template <bool FAST = false>
__device__ __forceinline__ void lse_add(double &m, double &s, double t) {
    if (!(t > -INFINITY)) return;
    // one exponential for both orders; below kLseSkip it is under half an ulp
    // of the sum (which is at least 1) and is not evaluated
    constexpr double kLseSkip = -37.5;
    const double d = -fabs(t - m);
    const double e = d > kLseSkip ? (FAST ? (double)__expf((float)d) : exp(d)) : 0.0;
    if (t > m) {
        s = s * e + 1.0;
        m = t;
    } else {
        s += e;
    }
}

// A sample's mixture coordinates (phase shear applied) and ln of the prior of
// the mixture columns (the other columns' prior cancels in ln p_s - ln p).
template <int D>
__device__ __forceinline__ void mix_coords(int shear, const LnPrior &lp, const double th[7], double xm[7],
                                           double &lpm) {
#pragma unroll
    for (int a = 0; a < D; a++) xm[a] = th[mix_col(D, a)];
    if (shear) xm[D - 1] = shear_phase(th[6], th[5], shear);
    // the columns' terms in their order
    lpm = -kLn2Pi;
    double sd, cd;
    sincos_rad(th[1], &sd, &cd);   // no large-argument path (its registers and scratch cost half the occupancy)
    lpm += log(0.5 * cd);
    lpm += lp.t;
    if (D == 7) lpm += log(th[3] * th[3] * lp.d3);
    lpm += -kLn2;
    lpm += -kLn2Pi;
    lpm += -kLnPi;
}
// t_k = ln p_s(x_k) - ln p(x_k) for NS samples of one mixture (the density of
// a mixture draw above):
//   t = ln[ sum_j e^{lnc_j} N_j(x) / p_mix(x) + e^{ln_fb} ],
// by a running log-sum-exp.  The mixture is read through the scalar cache
// (the component loop is uniform) and applied row by row to every sample; a
// periodic offset is wrapped as u - P rint(u / P) (the floor form's value
// except at exactly half a period, where both images are equally far).
template <int NS, int D, bool FAST = false>
__device__ __forceinline__ void mix_log_ratio(cgmm &g_, const double (&xm)[NS][7], const double (&lpm)[NS],
                                              double (&t)[NS]) {
    constexpr double c0 = -0.5 * D * kLn2Pi;
    double mm[NS], ss[NS];
#pragma unroll
    for (int k = 0; k < NS; k++) {
        mm[k] = -INFINITY;
        ss[k] = 0.0;
        lse_add(mm[k], ss[k], g_.ln_fb);
    }
    const int nc = g_.n_comp;
#pragma unroll 1
    for (int j = 0; j < nc; j++) {
        // the mixture looks redefined per component, so that its constants are
        // read here instead of being held in (and spilled from) scalar registers
        cgmm *gp = &g_;
        asm volatile("" : "+s"(gp));
        cgmm &g = *gp;
        if (g.lnc[j] == -INFINITY) continue;
        const double cj = g.lnc[j] - g.logdet_half[j] + c0;
        double df[NS][D], qf[NS];
#pragma unroll
        for (int a = 0; a < D; a++) {
            const double mu = g.mean[j][a];
            constexpr auto P = [](int q) { return mix_period(D, q); };
#pragma unroll
            for (int k = 0; k < NS; k++) {
                const double u = xm[k][a] - mu;
                df[k][a] = P(a) > 0.0 ? u - P(a) * rint(u * (1.0 / P(a))) : u;
            }
        }
#pragma unroll
        for (int k = 0; k < NS; k++) qf[k] = 0.0;
#pragma unroll
        for (int a = 0; a < D; a++) {
            double y[NS];
#pragma unroll
            for (int k = 0; k < NS; k++) y[k] = 0.0;
#pragma unroll
            for (int b = 0; b <= a; b++) {
                const double lab = g.Linv[j][a][b];
#pragma unroll
                for (int k = 0; k < NS; k++) y[k] = fma(lab, df[k][b], y[k]);
            }
#pragma unroll
            for (int k = 0; k < NS; k++) qf[k] = fma(y[k], y[k], qf[k]);
        }
#pragma unroll
        for (int k = 0; k < NS; k++) lse_add<FAST>(mm[k], ss[k], cj - 0.5 * qf[k] - lpm[k]);
    }
#pragma unroll
    for (int k = 0; k < NS; k++) t[k] = mm[k] > -INFINITY ? mm[k] + log(ss[k]) : -INFINITY;
}

// One candidate of a component with mean mu[D] and factor L (packed rows):
// Box-Muller pairs from words w[0 ..), x in the mixture's coordinates; false
// when a bounded column leaves its interval or a periodic offset its half
// period.
template <int D, class M, class F>
__device__ __forceinline__ bool gmm_candidate(const PriorDev &pr, const M &mu, const F &L, const uint32_t *w,
                                              double (&x)[D]) {
    constexpr int NP = (D + 1) / 2;
    double z[2 * NP];
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const double u1 = u53(w[4 * p], w[4 * p + 1]), u2 = u53(w[4 * p + 2], w[4 * p + 3]);
        const double r = sqrt(-2.0 * log(u1));
        double s, c;
        sincos_rad(2 * kPi * u2, &s, &c);   // FP64 reduction + series (no large-argument path)
        z[2 * p] = r * c;
        z[2 * p + 1] = r * s;
    }
    bool in = true;
#pragma unroll
    for (int a = 0; a < D; a++) {
        double off = 0.0;
#pragma unroll
        for (int b = 0; b <= a; b++) off += L(a, b) * z[b];
        double v = mu(a) + off;
        constexpr auto P = [](int q) { return mix_period(D, q); };
        if (P(a) > 0.0) {
            in = in && off > -0.5 * P(a) && off <= 0.5 * P(a);
            v = v - P(a) * floor(v * (1.0 / P(a)));
        } else {
            double lo, hi;
            bounds(pr, mix_col(D, a), lo, hi);
            in = in && v >= lo && v <= hi;
        }
        x[a] = v;
    }
    return in;
}
// Philox blocks of one candidate: one per Box-Muller pair (the words of a
// fourth pair are not used with six columns).
template <int D>
constexpr int cand_blocks() { return (D + 1) / 2; }

// Most samples of a tile of mixture draws, and the tile's working set in LDS:
// the mixture (cumulative weights, means, packed factors) and the samples
// still to be drawn.
constexpr int kMixTile = 2048;
struct MixLds {
    double cum[kMaxComp], mean[kMaxComp][7], L[kMaxComp][28];
    int last;                       // last component with weight, -1: none
    int n[3];                       // entries of the queues and of the prior list
    uint32_t q[2][kMixTile];        // sample | attempt << 11 | component << 18
    uint32_t prior[kMixTile];       // samples that take the prior draw
};
static_assert(kMixTile <= 1 << 11 && kMaxAttempts < 1 << 7, "queue entry fields");

// Mixture draws of one tile: theta, then ln p - ln p_s.  Every sample makes its
// selection and first attempt; what is rejected goes through queues in LDS
// (attempt by attempt, the queue spread over the whole block again), and so
// do the samples that take the prior draw (defensive fraction, 64 rejected
// attempts), so that neither the rare retries nor the prior's inverse CDFs are
// paid for by every wave.  The order in a queue does not enter a sample's
// value.  Bounded by FP64 issue and the scalar reads of the mixture: 2^20 draws
// of 8 components, 7 columns 96 us (182 us when every wave carried the
// retries, the prior map and the library cosine, with 1,900 spilled scalars);
// 2^16 draws, 6 columns 28 us (124 us on 32 CUs).
template <class TT, int D>
__device__ __forceinline__ void draw_mix_tile(const DrawJob &J, int64_t begin, int n, MixLds &S) {
    TT *__restrict__ th_out = (TT *)J.theta + begin;
    TT *__restrict__ lr_out = J.lnpmps ? (TT *)J.lnpmps + begin : nullptr;
    const int64_t ld = J.ld, first = J.first + begin;
    cgmm &g = *uniform_gmm(J.gmm);
    const int nc = g.n_comp, shear = g.shear;
    const double eps = g.eps_def;
    const PriorDev pr = J.pr;
    const LnPrior lp = ln_prior_consts(pr);
    __syncthreads();   // the previous tile is done with
    for (int t = threadIdx.x; t < nc * 28; t += kDrawThreads) {
        const int j = t / 28, k = t % 28;
        int a = 0;
        while ((a + 1) * (a + 2) / 2 <= k) a++;
        S.L[j][k] = J.gmm->L[j][a][k - a * (a + 1) / 2];
        if (k < 7) S.mean[j][k] = J.gmm->mean[j][k];
    }
    if (threadIdx.x == 0) {
        // selection: the first component with weight whose cumulative share exceeds v
        double tot = 0.0, acc = 0.0;
        for (int j = 0; j < nc; j++) tot += g.w[j];
        int last = -1;
        for (int j = 0; j < nc; j++) {
            if (g.w[j] > 0.0) {
                acc += g.w[j] / tot;
                last = j;
            }
            S.cum[j] = g.w[j] > 0.0 ? acc : -INFINITY;
        }
        S.last = last;
        S.n[0] = S.n[1] = S.n[2] = 0;
    }
    __syncthreads();
    // phase 0: every sample's selection and first attempt; 1: queue rounds (at
    // most kMaxAttempts - 1); 2: prior draws
    int phase = 0, cur = 0, m = n;
    for (;;) {
#pragma unroll 1
        for (int e = threadIdx.x; e < m; e += kDrawThreads) {
            int s = e, a = 1, j = -1;
            double th[7];
            bool got = false;
            if (phase == 0) {
                uint32_t w[4];
                words(J.seed, (uint64_t)(first + s), J.round, 0, 0, 1, w);
                const double usel = u53(w[0], w[1]);
                if (usel >= eps) {
                    const double v = (usel - eps) / (1.0 - eps);
                    j = S.last;
                    for (int k = nc - 1; k >= 0; k--) j = v < S.cum[k] ? k : j;
                }
            } else if (phase == 1) {
                const uint32_t it = S.q[cur][e];
                s = (int)(it & 2047u);
                a = (int)((it >> 11) & 127u);
                j = (int)(it >> 18);
            } else {
                s = (int)S.prior[e];
                uint32_t w[16];
                words(J.seed, (uint64_t)(first + s), J.round, 0, 1, 4, w);
                prior_from_words(pr, w, th);
                got = true;
            }
            if (j >= 0) {
                uint32_t w[4 * cand_blocks<D>()];
                words(J.seed, (uint64_t)(first + s), J.round, (uint32_t)a, 1, cand_blocks<D>(), w);
                double x[D];
                got = gmm_candidate<D>(
                    pr, [&](int k) { return S.mean[j][k]; },
                    [&](int r, int c) { return S.L[j][r * (r + 1) / 2 + c]; }, w, x);
                th[3] = pr.d_ref;   // D = 6: the distance is not sampled
#pragma unroll
                for (int k = 0; k < D; k++) th[mix_col(D, k)] = x[k];
                // accepted in the mixture's coordinates: back to psi
                if (shear) th[6] = shear_phase(th[6], th[5], -shear);
            }
            if (got) {
                double xm[1][7], lpm[1], t[1];
                mix_coords<D>(shear, lp, th, xm[0], lpm[0]);
                mix_log_ratio<1, D>(g, xm, lpm, t);
#pragma unroll
                for (int c = 0; c < 7; c++) th_out[c * ld + s] = (TT)th[c];
                if (lr_out) lr_out[s] = (TT)(-t[0]);
            } else if (j >= 0 && a < kMaxAttempts) {
                const int q = phase == 0 ? 0 : cur ^ 1;
                S.q[q][atomicAdd(&S.n[q], 1)] = (uint32_t)s | (uint32_t)(a + 1) << 11 | (uint32_t)j << 18;
            } else {
                S.prior[atomicAdd(&S.n[2], 1)] = (uint32_t)s;
            }
        }
        if (phase == 2) break;
        __syncthreads();
        if (phase == 1) {
            if (threadIdx.x == 0) S.n[cur] = 0;
            cur ^= 1;
        }
        m = S.n[cur];
        phase = m > 0 ? 1 : 2;
        if (phase == 2) m = S.n[2];
        __syncthreads();   // the counts are read before the next round adds to them
    }
}

template <class TT>
__device__ __forceinline__ void draw_prior_tile(const DrawJob &J, int64_t begin, int64_t end) {
    TT *__restrict__ th_out = (TT *)J.theta;
    TT *__restrict__ lr_out = (TT *)J.lnpmps;
    for (int64_t s = begin + threadIdx.x; s < end; s += kDrawThreads) {
        const uint64_t idx = (uint64_t)(J.first + s);
        double th[7];
        uint32_t w[16];
        words(J.seed, idx, J.round, 0, 0, 4, w);
        prior_from_words(J.pr, w, th);
#pragma unroll
        for (int c = 0; c < 7; c++) th_out[c * J.ld + s] = (TT)th[c];
        if (lr_out) lr_out[s] = (TT)0;
    }
}

template <class TT, bool MIX>
__global__ void __launch_bounds__(kDrawThreads, MIX ? 4 : 1)
    k_draw(const DrawJob *__restrict__ jobs, const Tile *__restrict__ tiles, const DrawJob single, int64_t tile) {
    DrawJob J = single;
    int64_t begin = (int64_t)blockIdx.x * tile, end = begin + tile < single.n ? begin + tile : single.n;
    if (jobs != nullptr) {
        const Tile tl = tiles[blockIdx.x];
        J = jobs[tl.job];
        begin = tl.begin;
        end = tl.end;
    }
    if constexpr (MIX) {
        if (J.gmm != nullptr) {
            __shared__ MixLds S;
            const int nd = J.gmm->n_dim;
            for (; begin < end; begin += kMixTile) {
                const int n = end - begin < kMixTile ? (int)(end - begin) : kMixTile;
                if (nd == 6)
                    draw_mix_tile<TT, 6>(J, begin, n, S);
                else
                    draw_mix_tile<TT, 7>(J, begin, n, S);
            }
            return;
        }
    }
    draw_prior_tile<TT>(J, begin, end);
}

template <class TT>
void launch_draw_t(bool mix, const DrawJob *d_jobs, const Tile *d_tiles, int n_tiles, const DrawJob &single,
                   int64_t tile, hipStream_t st) {
    if (mix)
        hipLaunchKernelGGL((k_draw<TT, true>), dim3(n_tiles), dim3(kDrawThreads), 0, st, d_jobs, d_tiles, single,
                           tile);
    else
        hipLaunchKernelGGL((k_draw<TT, false>), dim3(n_tiles), dim3(kDrawThreads), 0, st, d_jobs, d_tiles, single,
                           tile);
}

// Mixture pool update (see PoolJob).  A block takes kPoolTileSamples samples
// of one job, kPoolSpt per thread held in registers in the mixture's
// coordinates; each proposal q adds t_q = ln p_s,q(x) - ln p(x) (mix_log_ratio)
// to every sample's running log-sum over proposals.
constexpr int kPoolSpt = 2;
static_assert(kPoolTileSamples == (int64_t)kPoolSpt * kDrawThreads, "pool tile = samples per thread x block");


template <class TT, class TO, class TL>
__global__ void __launch_bounds__(kDrawThreads)
    k_pool_mix(const PoolJob *__restrict__ jobs, const int n_jobs) {
    // this block's job: the last whose first block is at or before it
    int jb = 0;
    for (int q = 1; q < n_jobs; q++)
        if (jobs[q].tile_begin <= (int64_t)blockIdx.x) jb = q;
    const PoolJob &J = jobs[jb];
    const int64_t begin = ((int64_t)blockIdx.x - J.tile_begin) * kPoolTileSamples;
    const int64_t end = min(begin + kPoolTileSamples, (int64_t)(J.round + 1) * J.n_round);
    const TT *__restrict__ th = (const TT *)J.theta;
    const TO *__restrict__ L = (const TO *)J.lnL;
    TL *__restrict__ lw = (TL *)J.lw;
    const int r = J.round;
    const int64_t first_new = (int64_t)r * J.n_round;
    const double ln_rounds = log((double)(r + 1));
    cgmm *hist = uniform_gmm(J.hist);
    double x[kPoolSpt][7], m[kPoolSpt], sum[kPoolSpt];
    int q0[kPoolSpt];
#pragma unroll
    for (int k = 0; k < kPoolSpt; k++) {
        const int64_t i = begin + threadIdx.x + (int64_t)k * kDrawThreads;
#pragma unroll
        for (int c = 0; c < 7; c++) x[k][c] = i < end ? (double)th[c * J.ld + i] : 0.0;
        const bool fresh = i >= first_new;
        m[k] = (fresh || i >= end) ? 0.0 : J.lmix[i];   // the prior's term, e^0, is in every sum
        sum[k] = 1.0;
        q0[k] = i >= end ? r + 1 : (fresh ? 1 : r);
    }
    const int qlo = end > first_new ? 1 : r;
    // the FP32 policy's pooled weights need FP32 relative accuracy only
    constexpr bool kFast = sizeof(TO) == 4;
    // the mixture columns and the shear are the same for every proposal of the job
    auto proposals = [&](auto D_) {
        constexpr int D = decltype(D_)::value;
        double xm[kPoolSpt][7], lpm[kPoolSpt];
        const LnPrior lp = ln_prior_consts(J.pr);
#pragma unroll
        for (int k = 0; k < kPoolSpt; k++) mix_coords<D>(hist[r].shear, lp, x[k], xm[k], lpm[k]);
        for (int q = qlo; q <= r; q++) {
            double t[kPoolSpt];
            mix_log_ratio<kPoolSpt, D, kFast>(hist[q], xm, lpm, t);
#pragma unroll
            for (int k = 0; k < kPoolSpt; k++)
                if (q >= q0[k]) lse_add<kFast>(m[k], sum[k], t[k]);
        }
    };
    if (r > 0) {
        if (hist[r].n_dim == 6)
            proposals(std::integral_constant<int, 6>{});
        else
            proposals(std::integral_constant<int, 7>{});
    }
#pragma unroll
    for (int k = 0; k < kPoolSpt; k++) {
        const int64_t i = begin + threadIdx.x + (int64_t)k * kDrawThreads;
        if (i >= end) continue;
        const double lm = m[k] + log(sum[k]);
        J.lmix[i] = lm;
        lw[i] = (TL)((double)L[i] - lm + ln_rounds);
    }
}

}  // namespace

hipError_t launch_pool_mix(int policy, const PoolJob *d_jobs, int n_jobs, int64_t n_tiles, hipStream_t st) {
    if (n_tiles <= 0 || n_jobs <= 0) return hipSuccess;
    if (n_tiles > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)n_tiles), block(kDrawThreads);
    if (policy == kFP64)
        hipLaunchKernelGGL((k_pool_mix<double, double, double>), grid, block, 0, st, d_jobs, n_jobs);
    else if (policy == kFP32)
        hipLaunchKernelGGL((k_pool_mix<float, float, float>), grid, block, 0, st, d_jobs, n_jobs);
    else
        hipLaunchKernelGGL((k_pool_mix<float, double, double>), grid, block, 0, st, d_jobs, n_jobs);
    return hipGetLastError();
}

hipError_t launch_draw(int policy, const DrawJob *d_jobs, const Tile *d_tiles, int n_tiles, const DrawJob &single,
                       int64_t tile, bool mix, hipStream_t st) {
    if (n_tiles <= 0) return hipSuccess;
    if (policy == kFP64)
        launch_draw_t<double>(mix, d_jobs, d_tiles, n_tiles, single, tile, st);
    else
        launch_draw_t<float>(mix, d_jobs, d_tiles, n_tiles, single, tile, st);
    return hipGetLastError();
}

// ------------------------------------------------------------------ in-support mass
// Z_j of each job's mixture: the fraction of z_draws candidates of component j
// (Philox counter (i, 0x5A000000 + j, round, block)) that fall in the support.
// The factor kernel that precedes it on the stream has cleared the counters.
namespace {

constexpr int kZThreads = 256;
constexpr int kZBlocks = 64;

template <int D>
__device__ __forceinline__ uint32_t inbox_count(const EmJob &J, int j) {
    cgmm &g = *uniform_gmm(J.gmm);   // the component is uniform: its constants come through the scalar cache
    const uint32_t k0 = (uint32_t)J.z_seed, k1 = (uint32_t)(J.z_seed >> 32);
    const PriorDev pr = J.pr;
    uint32_t acc = 0;
#pragma unroll 1
    for (int64_t i = (int64_t)blockIdx.x * kZThreads + threadIdx.x; i < J.z_draws; i += (int64_t)gridDim.x * kZThreads) {
        uint32_t w[4 * cand_blocks<D>()];
#pragma unroll
        for (int b = 0; b < cand_blocks<D>(); b++) {
            U4 o = philox4x32_10(U4{(uint32_t)i, 0x5A000000u + (uint32_t)j, J.z_round, (uint32_t)b}, k0, k1);
            w[4 * b] = o.x; w[4 * b + 1] = o.y; w[4 * b + 2] = o.z; w[4 * b + 3] = o.w;
        }
        double x[D];
        acc += gmm_candidate<D>(
                   pr, [&](int k) { return g.mean[j][k]; }, [&](int r, int c) { return g.L[j][r][c]; }, w, x)
                   ? 1u
                   : 0u;
    }
    return acc;
}
__global__ void __launch_bounds__(kZThreads) k_gmm_inbox(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const int j = blockIdx.y;
    if (j >= J.gmm->n_comp) return;
    uint32_t acc = J.gmm->n_dim == 6 ? inbox_count<6>(J, j) : inbox_count<7>(J, j);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    __shared__ uint32_t sacc[kZThreads / 64];
    if ((threadIdx.x & 63) == 0) sacc[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kZThreads / 64; w++) acc += sacc[w];
        atomicAdd(&J.zcount[j], acc);
    }
}

// ln Z_j and the constants of the draw density, one lane per component: r_j =
// (1 - Z_j)^64, pi_j normalised; the sums over components in their order.
__global__ void k_gmm_setz(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    GmmDev *g = J.gmm;
    const int j = threadIdx.x, nc = g->n_comp;
    const double wj = j < nc ? g->w[j] : 0.0;
    double lnz = 0.0;
    if (j < nc) {
        const double c = (double)J.zcount[j];
        lnz = log((c > 0 ? c : 0.5) / (double)J.z_draws);
        g->lnZ[j] = lnz;
    }
    double tot = 0.0;
    for (int q = 0; q < nc; q++) {
        const double w = __shfl(wj, q, 64);
        tot += w > 0.0 ? w : 0.0;
    }
    const double eps = g->eps_def;
    const bool on = j < nc && wj > 0.0 && tot > 0.0;
    double term = 0.0;
    if (on) {
        const double pi = wj / tot, z = exp(lnz);
        const double lr = (double)kMaxAttempts * log1p(-(z < 1.0 ? z : 1.0));   // ln r_j
        term = (1.0 - eps) * pi * exp(lr);
        // ln(1 - r_j), accurate on both sides of r_j = 1/2
        const double l1mr = lr > -0.69314718055994531 ? log(-expm1(lr)) : log1p(-exp(lr));
        g->lnc[j] = log1p(-eps) + log(pi) + l1mr - lnz;
    } else if (j < kMaxComp) {
        g->lnc[j] = -INFINITY;
    }
    const unsigned long long mask = __ballot(on);
    double fb = eps;
    for (int q = 0; q < nc; q++) {
        const double t = __shfl(term, q, 64);
        if ((mask >> q) & 1) fb += t;
    }
    if (j == 0) g->ln_fb = fb > 0.0 ? log(fb) : -INFINITY;
}

}  // namespace

hipError_t launch_gmm_mass(const EmJob *d_jobs, int n_jobs, hipStream_t st) {
    if (n_jobs <= 0) return hipSuccess;
    if (n_jobs > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gmm_inbox, dim3(kZBlocks, kMaxComp, n_jobs), dim3(kZThreads), 0, st, d_jobs);
    hipLaunchKernelGGL(k_gmm_setz, dim3(1, 1, n_jobs), dim3(64), 0, st, d_jobs);
    return hipGetLastError();
}

}  // namespace ile
