// Gaussian-mixture sampling prior (paper: GMM sampling priors for a chosen
// subset of dimensions, refit from weighted samples).  All steps run on the
// device in FP64 with deterministic fixed-order reductions:
//
//   factor : Cholesky L_j of Sigma_j, L_j^{-1}, sum ln diag(L_j), ln pi_j;
//   weights: w_i = e^{beta (lw_i - max lw)}, beta the tempering exponent;
//   init   : means at the n_comp highest-weight distinct samples (among the
//            2 n_comp highest), common covariance = weighted second moment of
//            the differences (wrapped for periodic columns) about the best
//            sample minus the outer product of their mean, plus the floor;
//   EM     : responsibilities from the untruncated components
//            pi_j N(wrap(x - mu_j); Sigma_j); means from the wrapped offsets
//            about the current mu_j; covariances centred on the new offsets;
//            Sigma_j += 1e-8 diag(range^2).  A component with no weight keeps
//            its mean and covariance.
//
// Every kernel serves a batch of jobs (blockIdx.z = job): the refits of all
// jobs of a serving pass are one launch per stage.  Per-sample stages tile
// each job's samples (em_layout: at most 256 tiles, a function of the job's n
// alone, so that a job's result does not depend on its batch); per-job stages
// are one block each, with one wave per mixture component.
// A refit of one job of 2^16 samples is latency: with 8,192 samples per tile
// it ran on eight CUs (moments 28 us, tempering 102 us against 14), the component
// update summed and factored in one thread per component (35 us against 10.5),
// and the responsibilities made a round trip through memory; the whole refit
// of that size with its installation and draw took 1057 us against 467.
#include <type_traits>

#include "ile_internal.h"

#include <algorithm>

namespace ile {

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kEmThreads = 256;
constexpr int kEmMaxTiles = 256;
constexpr int kTopK = 2 * kMaxComp;
constexpr int kBetaGrid = 48;   // beta_k = 2^(-k/4)
constexpr int kBetaChunk = 16;   // grid values per block reduction
constexpr int kMom = 36;        // W, 7 first and 28 second moments

// Work buffer of one job (doubles): scalars, then the per-tile partials of
// each stage.  Tiles of whole blocks of samples, one per CU from 2^16 samples
// up: the smallest tile that keeps the count at kEmMaxTiles.
constexpr int kWMax = 0, kWCount = 1, kWBeta = 2, kWPart = 64;
struct EmLayout {
    int64_t tile, nblk;
    size_t stat, init, beta, max, top, total;
};
__host__ __device__ inline EmLayout em_layout(int64_t n) {
    EmLayout L;
    const int64_t blocks = (n + kEmThreads - 1) / kEmThreads;
    L.tile = (blocks + kEmMaxTiles - 1) / kEmMaxTiles * kEmThreads;
    L.nblk = (n + L.tile - 1) / L.tile;
    L.stat = kWPart;
    L.init = L.stat + (size_t)kMaxComp * L.nblk * kMom;
    L.beta = L.init + (size_t)L.nblk * kMom;
    L.max = L.beta + (size_t)L.nblk * 2 * kBetaGrid;
    L.top = L.max + (size_t)L.nblk * 2;
    L.total = L.top + (size_t)L.nblk * 2 * kTopK;
    return L;
}

__device__ __forceinline__ double col_period(int col) {
    return (col == 0 || col == 5) ? 2 * kPi : (col == 6 ? kPi : 0.0);
}
__device__ __forceinline__ double col_range(const PriorDev &pr, int col) {
    switch (col) {
    case 0: return 2 * kPi;
    case 1: return kPi;
    case 2: return 2 * pr.t_window;
    case 3: return pr.d_max - pr.d_min;
    case 4: return 2.0;
    case 5: return 2 * kPi;
    default: return kPi;
    }
}
// wrapped difference in (-P/2, P/2]: d - P floor(d/P), folded; for |d| < P
// (both ends inside one period) the same value without the division
__device__ __forceinline__ double wrapd(double d, double P) {
    if (P <= 0.0) return d;
    double r;
    if (d >= 0.0 && d < P)
        r = d;
    else if (d < 0.0 && d >= -P)
        r = d + P;
    else
        r = d - P * floor(d / P);
    return r > 0.5 * P ? r - P : r;
}

template <class TT>
__device__ __forceinline__ double load_col(const TT *th, int64_t ld, int col, int64_t i) {
    return (double)th[col * ld + i];
}

// Column col of sample i in the mixture's coordinates (phase shear of column 6).
template <class TT>
__device__ __forceinline__ double load_mix(const TT *th, int64_t ld, int col, int64_t i, int shear) {
    const double v = (double)th[col * ld + i];
    if (col != 6 || shear == 0) return v;
    return shear_phase(v, (double)th[5 * ld + i], shear);
}

__device__ __forceinline__ bool finite_d(double v) { return v > -INFINITY && v < INFINITY; }

__device__ __forceinline__ double sample_weight(double lwv, double mlw, double beta) {
    return finite_d(lwv) ? exp(beta * (lwv - mlw)) : 0.0;
}

// Sums of NV values over the group of 2 OFF consecutive lanes that a lane
// belongs to, each lane keeping part of them: at every step the lanes of a
// pair split what is left (half the values travel, where a butterfly over
// every value moves them all at each step).  Afterwards v[0 .. lim) of a lane
// are the sums of values base .. base + lim - 1 (association fixed by the lane
// numbers; lanes that share a value hold the same sum).
template <int NV, int OFF>
__device__ __forceinline__ void lane_sums(double *v, int lane, int &base, int &lim) {
    if constexpr (OFF > 0) {
        if constexpr (NV == 1) {
            v[0] += __shfl_xor(v[0], OFF, 64);
            lane_sums<1, OFF / 2>(v, lane, base, lim);
        } else {
            constexpr int H = (NV + 1) / 2;
            const bool up = (lane & OFF) != 0;
#pragma unroll
            for (int i = 0; i < H; i++) {
                const double lo = v[i], hi = i + H < NV ? v[i + H] : 0.0;
                v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, OFF, 64);
            }
            base += up ? H : 0;
            lim = up ? lim - H : (lim < H ? lim : H);
            lane_sums<H, OFF / 2>(v, lane, base, lim);
        }
    }
}
template <int NV>
constexpr int lane_left(int off) {
    int n = NV;
    for (; off > 0; off /= 2) n = (n + 1) / 2;
    return n;
}

// Block sum of NV doubles per thread into out[0], out[stride], ..: within each
// wave (lane_sums), then the waves in order.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double *out, int64_t stride) {
    __shared__ double red[kEmThreads / 64][NV];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int base = 0, lim = NV;
    lane_sums<NV, 32>(v, lane, base, lim);
#pragma unroll
    for (int t = 0; t < lane_left<NV>(32); t++)
        if (t < lim) red[w][base + t] = v[t];
    __syncthreads();
    for (int c = threadIdx.x; c < NV; c += blockDim.x) {
        double s = red[0][c];
        for (int q = 1; q < kEmThreads / 64; q++) s += red[q][c];
        out[c * stride] = s;
    }
    __syncthreads();
}

// Cholesky factor L of component j's covariance, L^{-1}, sum ln diag(L) and
// ln pi_j by one wave: lane r < d holds row r of the covariance (lower part)
// and of L; then lane c holds column c of the inverse.
__device__ void wave_factor(GmmDev &g, int j, int lane, int d, const double (&cov)[7]) {
    double L[7], Li[7];
    bool ok = true;
#pragma unroll
    for (int c = 0; c < 7; c++) L[c] = 0.0;
#pragma unroll
    for (int c = 0; c < 7; c++) {
        if (c >= d) break;
        // every lane r >= c: t = cov[r][c] - sum_k L[r][k] L[c][k]
        double t = cov[c];
#pragma unroll
        for (int k = 0; k < c; k++) t -= L[k] * __shfl(L[k], c, 64);
        double s = __shfl(t, c, 64);
        if (!(s > 0.0)) {
            ok = false;
            s = 1e-300;
        }
        const double dg = sqrt(s);
        L[c] = lane == c ? dg : (lane > c && lane < d ? t / dg : 0.0);
    }
#pragma unroll
    for (int r = 0; r < 7; r++) {
        if (r >= d) {
            Li[r] = 0.0;
            continue;
        }
        double t = (r == lane) ? 1.0 : 0.0;
#pragma unroll
        for (int k = 0; k < r; k++) t -= __shfl(L[k], r, 64) * Li[k];
        const double dg = __shfl(L[r], r, 64);
        Li[r] = (r < lane || lane >= d) ? 0.0 : t / dg;
    }
    double own = 1.0;
#pragma unroll
    for (int c = 0; c < 7; c++) own = (c == lane && c < d) ? L[c] : own;
    const double lg = log(own);
    double ld = 0.0;
    for (int c = 0; c < d; c++) ld += __shfl(lg, c, 64);
    if (lane < 7) {
#pragma unroll
        for (int b = 0; b < 7; b++) {
            g.L[j][lane][b] = lane < d ? L[b] : 0.0;
            g.Linv[j][b][lane] = Li[b];
        }
    }
    if (lane == 0) {
        g.logdet_half[j] = ld;
        g.logw[j] = (g.w[j] > 0.0) ? log(g.w[j]) : -INFINITY;
        if (!ok) g.valid = 0;
    }
}

// Sums over the tiles of NV consecutive values of a [value][tile] partial array
// by one wave: a lane takes every 64th tile (every load in flight at once),
// then lane_sums.  Into out[0 .. NV) (LDS).
template <int NV>
__device__ __forceinline__ void tile_sums(const double *p, int64_t nblk, int lane, double *out) {
    static_assert(kEmMaxTiles <= 256, "four tiles per lane");
    double v[NV];
#pragma unroll
    for (int c = 0; c < NV; c++) {
        double t[4];
#pragma unroll
        for (int q = 0; q < 4; q++) t[q] = lane + 64 * q < nblk ? p[c * nblk + lane + 64 * q] : 0.0;
        v[c] = (t[0] + t[1]) + (t[2] + t[3]);
    }
    int base = 0, lim = NV;
    lane_sums<NV, 32>(v, lane, base, lim);
#pragma unroll
    for (int t = 0; t < lane_left<NV>(32); t++)
        if (t < lim) out[base + t] = v[t];
}
// A component's 36 moments, twelve at a time (96 registers in flight).
__device__ __forceinline__ void moment_sums(const double *p, int64_t nblk, int lane, double *out) {
#pragma unroll 1
    for (int c = 0; c < kMom; c += 12) tile_sums<12>(p + (size_t)c * nblk, nblk, lane, out + c);
}

// ------------------------------------------------------------- weights
// Block maximum and sum of one pair per thread (every thread gets them).
__device__ __forceinline__ void block_max_sum(double &m, double &c) {
    __shared__ double sm[kEmThreads / 64], sc[kEmThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        m = fmax(m, __shfl_xor(m, off, 64));
        c += __shfl_xor(c, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = m;
        sc[threadIdx.x >> 6] = c;
    }
    __syncthreads();
    m = sm[0];
    c = sc[0];
    for (int w = 1; w < kEmThreads / 64; w++) {
        m = fmax(m, sm[w]);
        c += sc[w];
    }
}

// per tile: max of the finite lw and their count
template <class TL>
__global__ void __launch_bounds__(kEmThreads) k_em_scan(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const EmLayout Lo = em_layout(J.n);
    if (blockIdx.x >= Lo.nblk) return;
    const TL *__restrict__ lw = (const TL *)J.lw;
    const int64_t b0 = (int64_t)blockIdx.x * Lo.tile, b1 = min(b0 + Lo.tile, J.n);
    double m = -INFINITY, c = 0.0;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += kEmThreads) {
        const double v = (double)lw[i];
        if (finite_d(v)) {
            m = fmax(m, v);
            c += 1.0;
        }
    }
    block_max_sum(m, c);
    if (threadIdx.x == 0) {
        J.work[Lo.max + 2 * blockIdx.x] = m;
        J.work[Lo.max + 2 * blockIdx.x + 1] = c;
    }
}

// Every block reduces the tiles' maxima and counts (the first one stores
// them).  Tempering exponent: the largest beta_k = 2^(-k/4) whose tempered
// weights have (sum w^beta)^2 / sum w^(2 beta) >= frac * (finite samples).
// Per tile: the 48 pairs (sum w^beta_k, sum w^(2 beta_k)).
template <class TL>
__global__ void __launch_bounds__(kEmThreads) k_em_beta(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const EmLayout Lo = em_layout(J.n);
    const bool temper = J.temper > 0.0;
    if (blockIdx.x >= Lo.nblk || (!temper && blockIdx.x > 0)) return;
    static_assert(kEmMaxTiles <= kEmThreads, "one tile's maximum per thread");
    double mlw = -INFINITY, cnt = 0.0;
    if (threadIdx.x < Lo.nblk) {
        mlw = J.work[Lo.max + 2 * threadIdx.x];
        cnt = J.work[Lo.max + 2 * threadIdx.x + 1];
    }
    block_max_sum(mlw, cnt);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        J.work[kWMax] = mlw;
        J.work[kWCount] = cnt;
        J.work[kWBeta] = 1.0;
    }
    if (!temper) return;
    const TL *__restrict__ lw = (const TL *)J.lw;
    const int64_t b0 = (int64_t)blockIdx.x * Lo.tile, b1 = min(b0 + Lo.tile, J.n);
    double *out = J.work + Lo.beta + blockIdx.x;
    for (int c0 = 0; c0 < kBetaGrid; c0 += kBetaChunk) {
        double acc[2 * kBetaChunk], bk[kBetaChunk];
#pragma unroll
        for (int q = 0; q < kBetaChunk; q++) {
            bk[q] = exp2(-(double)(c0 + q) / 4.0);
            acc[2 * q] = 0.0;
            acc[2 * q + 1] = 0.0;
        }
        for (int64_t i = b0 + threadIdx.x; i < b1; i += kEmThreads) {
            const double v = (double)lw[i];
            const double x = finite_d(v) ? v - mlw : -INFINITY;
#pragma unroll
            for (int q = 0; q < kBetaChunk; q++) {
                const double e = exp(bk[q] * x);
                acc[2 * q] += e;
                acc[2 * q + 1] += e * e;
            }
        }
        block_sum<2 * kBetaChunk>(acc, out + (size_t)2 * c0 * Lo.nblk, Lo.nblk);
    }
}

__global__ void __launch_bounds__(256) k_em_beta_final(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    if (!(J.temper > 0.0)) return;
    const EmLayout Lo = em_layout(J.n);
    __shared__ double s[2 * kBetaGrid];
    constexpr int kPer = 2 * kBetaGrid / 4;   // values per wave
    const int wv = threadIdx.x >> 6;
    tile_sums<kPer>(J.work + Lo.beta + (size_t)wv * kPer * Lo.nblk, Lo.nblk, threadIdx.x & 63, s + wv * kPer);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const double target = J.temper * J.work[kWCount];
    const int k = threadIdx.x < kBetaGrid ? threadIdx.x : kBetaGrid - 1;
    const double s1 = s[2 * k], s2 = s[2 * k + 1];
    const unsigned long long hit = __ballot(s1 * s1 / s2 >= target) & ((1ull << kBetaGrid) - 1);
    const int first = hit ? __ffsll((long long)hit) - 1 : kBetaGrid - 1;
    if (threadIdx.x == 0) J.work[kWBeta] = exp2(-(double)first / 4.0);
}

// ---------------------------------------------------------------- first fit
struct Cand {
    double v;
    int64_t i;
};
__device__ __forceinline__ bool better(const Cand &a, const Cand &b) {
    return a.v > b.v || (a.v == b.v && a.i < b.i);
}
// The block's best candidate (every thread gets it).
__device__ __forceinline__ Cand block_best(Cand c, Cand *sh) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const Cand o{__shfl_xor(c.v, off, 64), (int64_t)__shfl_xor((long long)c.i, off, 64)};
        c = better(o, c) ? o : c;
    }
    __syncthreads();   // the previous round's reads are done
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
    __syncthreads();
    c = sh[0];
    for (int w = 1; w < kEmThreads / 64; w++) c = better(sh[w], c) ? sh[w] : c;
    return c;
}
// candidates of a first fit: the 2 n_comp highest-weight samples
__device__ __forceinline__ int top_count(const EmJob &J) { return 2 * J.n_comp < kTopK ? 2 * J.n_comp : kTopK; }

// per tile: the highest finite lw (ties: lower index first), one round per
// candidate: the best sample that comes after the previous round's
template <class TL>
__global__ void __launch_bounds__(kEmThreads) k_em_top(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const EmLayout Lo = em_layout(J.n);
    if (!J.first || blockIdx.x >= Lo.nblk) return;
    const TL *__restrict__ lw = (const TL *)J.lw;
    __shared__ Cand sh[kEmThreads / 64];
    const int64_t b0 = (int64_t)blockIdx.x * Lo.tile, b1 = min(b0 + Lo.tile, J.n);
    double *o = J.work + Lo.top + (size_t)blockIdx.x * 2 * kTopK;
    const int nk = top_count(J);
    Cand prev{INFINITY, -1};
    for (int k = 0; k < nk; k++) {
        Cand best{-INFINITY, INT64_MAX};
        if (prev.v > -INFINITY) {
            for (int64_t i = b0 + threadIdx.x; i < b1; i += kEmThreads) {
                const Cand c{(double)lw[i], i};
                if (finite_d(c.v) && better(prev, c) && better(c, best)) best = c;
            }
            best = block_best(best, sh);
        }
        if (threadIdx.x == 0) {
            o[2 * k] = best.v;
            o[2 * k + 1] = (double)best.i;
        }
        prev = best;
    }
}

// merge the tiles' sorted lists (one per thread, its head advanced when it
// wins a round); reset the mixture and place the means at the highest-weight
// distinct samples
template <class TT>
__global__ void __launch_bounds__(kEmThreads) k_em_top_final(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    if (!J.first) return;
    GmmDev *g = J.gmm;
    {   // zero the whole state
        double *p = (double *)g;
        const size_t nd = sizeof(GmmDev) / sizeof(double);
        for (size_t k = threadIdx.x; k < nd; k += blockDim.x) p[k] = 0.0;
    }
    const EmLayout Lo = em_layout(J.n);
    const TT *th = (const TT *)J.theta;
    const int d = J.n_dim, nc = J.n_comp, nk = top_count(J);
    __shared__ Cand sh[kEmThreads / 64], cur[kTopK];
    __shared__ double sx[kTopK][7];
    const double *o = J.work + Lo.top + (size_t)threadIdx.x * 2 * kTopK;
    int pos = 0;
    for (int k = 0; k < nk; k++) {
        Cand c{-INFINITY, INT64_MAX};
        if (threadIdx.x < Lo.nblk && pos < nk && o[2 * pos] > -INFINITY) c = Cand{o[2 * pos], (int64_t)o[2 * pos + 1]};
        const Cand b = block_best(c, sh);
        if (b.v > -INFINITY && b.i == c.i) pos++;
        if (threadIdx.x == 0) cur[k] = b;
    }
    __syncthreads();
    // phase shear from the inclination of the best sample: face-on
    // (cos iota >= 1/2, where the m = +2 end of each multiplet dominates) the
    // ridge runs along psi + phi_c, face-off along psi - phi_c; in between
    // there is no single ridge and the phases stay as they are
    int shear = 0;
    if (J.shear_auto && cur[0].v > -INFINITY) {
        const double ci = load_col(th, J.ld, 4, cur[0].i);
        shear = ci >= 0.5 ? 1 : (ci <= -0.5 ? -1 : 0);
    }
    if ((int)threadIdx.x < 8 * nk) {
        const int k = threadIdx.x >> 3, a = threadIdx.x & 7;
        if (a < d && cur[k].v > -INFINITY) sx[k][a] = load_mix(th, J.ld, J.dims[a], cur[k].i, shear);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    g->n_dim = d;
    for (int a = 0; a < 7; a++) g->dims[a] = a < d ? J.dims[a] : 0;
    g->eps_def = J.eps_def;
    g->valid = 1;
    g->shear = shear;
    // the distinct candidates in their order
    int got = 0, from[kMaxComp];
    for (int k = 0; k < nk && got < nc; k++) {
        if (!(cur[k].v > -INFINITY)) break;
        bool dup = false;
        for (int q = 0; q < got && !dup; q++) {
            bool same = true;
            for (int a = 0; a < d; a++) same = same && (sx[k][a] == sx[from[q]][a]);
            dup = same;
        }
        if (!dup) from[got++] = k;
    }
    // no finite weight: the first mean stays as it is
    for (int q = 0; q < nc && got > 0; q++)
        for (int a = 0; a < d; a++) g->mean[q][a] = sx[from[q < got ? q : got - 1]][a];
    g->n_comp = nc;
}

// first fit: weighted moments of the differences about the best sample
template <class TT, class TL>
__global__ void __launch_bounds__(kEmThreads) k_em_init(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const EmLayout Lo = em_layout(J.n);
    if (!J.first || blockIdx.x >= Lo.nblk) return;
    const TT *__restrict__ th = (const TT *)J.theta;
    const TL *__restrict__ lw = (const TL *)J.lw;
    const GmmDev *g = J.gmm;
    const int d = g->n_dim;
    const double mlw = J.work[kWMax], beta = J.work[kWBeta];
    double acc[kMom];
    for (int c = 0; c < kMom; c++) acc[c] = 0.0;
    const int64_t b0 = (int64_t)blockIdx.x * Lo.tile, b1 = min(b0 + Lo.tile, J.n);
    for (int64_t i = b0 + threadIdx.x; i < b1; i += kEmThreads) {
        const double w = sample_weight((double)lw[i], mlw, beta);
        double x[7];
#pragma unroll
        for (int a = 0; a < 7; a++) {
            x[a] = 0.0;
            if (a < d) {
                const int col = g->dims[a];
                x[a] = wrapd(load_mix(th, J.ld, col, i, g->shear) - g->mean[0][a], col_period(col));
            }
        }
        acc[0] += w;
        int k = 1;
#pragma unroll
        for (int a = 0; a < 7; a++) acc[k++] += w * x[a];
#pragma unroll
        for (int a = 0; a < 7; a++)
#pragma unroll
            for (int b = 0; b <= a; b++) acc[k++] += w * x[a] * x[b];
    }
    block_sum<kMom>(acc, J.work + Lo.init + blockIdx.x, Lo.nblk);
}

// One wave per component: covariance rows from the moments s[36] (LDS),
// centred on the mean offsets, plus the floor; the lane's row (lane < d).
__device__ __forceinline__ void wave_cov(const double *s, const PriorDev &pr, const GmmDev &g, int lane, int d,
                                         double (&row)[7], double &m) {
    const double W = s[0];
    m = lane < d ? s[1 + lane] / W : 0.0;
    const int r = lane < 7 ? lane : 0;
#pragma unroll
    for (int b = 0; b < 7; b++) {
        const double mb = __shfl(m, b, 64);
        const int hi = r > b ? r : b, lo = r > b ? b : r;
        double v = (lane < d && b < d) ? s[8 + hi * (hi + 1) / 2 + lo] / W - (r >= b ? m * mb : mb * m) : 0.0;
        if (b == lane && lane < d) {
            const double rg = col_range(pr, g.dims[lane]);
            v += 1e-8 * rg * rg;
        }
        row[b] = v;
    }
}

// The common first covariance, in every component, and its factors.
__global__ void __launch_bounds__(64 * kMaxComp) k_em_init_final(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    if (!J.first) return;
    const EmLayout Lo = em_layout(J.n);
    GmmDev *g = J.gmm;
    const int lane = threadIdx.x & 63, j = threadIdx.x >> 6;
    __shared__ double s[kMom];
    if (j == 0) moment_sums(J.work + Lo.init, Lo.nblk, lane, s);
    __syncthreads();
    const int d = g->n_dim;
    if (j >= g->n_comp) return;
    double row[7], m;
    wave_cov(s, J.pr, *g, lane, d, row, m);
    if (lane < 7)
        for (int b = 0; b < 7; b++) g->cov[j][lane][b] = row[b];
    if (lane == 0) g->w[j] = 1.0 / g->n_comp;
    __threadfence_block();
    wave_factor(*g, j, lane, d, row);
}

__global__ void __launch_bounds__(64 * kMaxComp) k_gmm_factor(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    GmmDev *g = J.gmm;
    const int lane = threadIdx.x & 63, j = threadIdx.x >> 6;
    if (threadIdx.x == 0) g->valid = 1;
    if (threadIdx.x < kMaxComp) J.zcount[threadIdx.x] = 0u;   // for the mass estimate that follows
    __syncthreads();
    if (j >= g->n_comp) return;
    double row[7];
#pragma unroll
    for (int b = 0; b < 7; b++) row[b] = lane < 7 ? g->cov[j][lane][b] : 0.0;
    wave_factor(*g, j, lane, g->n_dim, row);
}

// ------------------------------------------------------------------ EM
// E step and the tile's moments in one pass.  A block takes its tile 256
// samples at a time; they sit in LDS, and 256 / NC consecutive threads serve
// one component (NC: the component count rounded up to 4, 8 or 16):
//   ln pi_j N_j(x_i) of its samples, the component's mean and inverse factor in
//     registers;
//   then one thread per sample turns the column of LDS into responsibilities
//     times weights, R_ij = w_i pi_j N_j(x_i) / sum_k pi_k N_k(x_i);
//   then W_j and the first and second moments of the offsets wrap(x - mu_j),
//     36 sums per thread (the covariance centred on the mean offset m_j is
//     S2/W - m_j m_j^T, the same quantity as the centred two-pass sum).
// The responsibilities never leave the CU.  Latency and FP64 issue bound it:
// 2^16 samples, 8 components, 6 dimensions: 11.7 us, where responsibilities
// through memory and moments of 8,192-sample tiles took 13.8 + 28.4 us.
// A mixture spans its job's sampled columns, all seven (D = 7) or all but the
// distance (D = 6): columns and periods are compile-time constants.
constexpr int mix_col(int D, int a) { return D == 6 && a >= 3 ? a + 1 : a; }
constexpr double mix_period(int D, int a) {
    const int c = mix_col(D, a);
    return (c == 0 || c == 5) ? 2 * kPi : (c == 6 ? kPi : 0.0);
}
// wrapd by rounding to the nearest period (the same value but for the last
// bit, and at exactly half a period, where both images are equally far)
__device__ __forceinline__ double wrapn(double d, double P, double iP) { return d - P * rint(d * iP); }

struct EmShared {
    double x[7][kEmThreads];
    double w[kEmThreads];
    double r[kMaxComp][kEmThreads];
};

template <class TT, class TL, int D, int NC>
__device__ __forceinline__ void em_pass(const EmJob &J, const EmLayout &Lo, EmShared &S) {
    constexpr int LP = kEmThreads / NC;              // threads per component
    static_assert(LP <= 64 && NC <= kMaxComp, "whole components per wave");
    const TT *__restrict__ th = (const TT *)J.theta;
    const TL *__restrict__ lw = (const TL *)J.lw;
    const GmmDev *g = J.gmm;
    const int nc = g->n_comp;
    const int tid = threadIdx.x, lane = tid & 63, j = tid / LP, l = tid % LP;
    const bool comp = j < nc;
    double mu[D], li[D * (D + 1) / 2];
#pragma unroll
    for (int a = 0; a < D; a++) {
        mu[a] = comp ? g->mean[j][a] : 0.0;
#pragma unroll
        for (int b = 0; b <= a; b++) li[a * (a + 1) / 2 + b] = comp ? g->Linv[j][a][b] : 0.0;
    }
    auto off = [&](int a, double v) {   // wrapped offset from the component's mean
        const double u = v - mu[a], P = mix_period(D, a);
        return P > 0.0 ? wrapn(u, P, 1.0 / P) : u;
    };
    const double cj = (comp && g->logw[j] != -INFINITY) ? g->logw[j] - g->logdet_half[j] - 0.5 * D * log(2 * kPi)
                                                         : -INFINITY;
    const int shear = g->shear;
    const double mlw = J.work[kWMax], beta = J.work[kWBeta];
    double acc[kMom];
#pragma unroll
    for (int c = 0; c < kMom; c++) acc[c] = 0.0;
    const int64_t b0 = (int64_t)blockIdx.x * Lo.tile, b1 = min(b0 + Lo.tile, J.n);
    for (int64_t c0 = b0; c0 < b1; c0 += kEmThreads) {
        __syncthreads();   // the previous samples are done with
        {
            const int64_t i = c0 + tid < b1 ? c0 + tid : b1 - 1;
            double x[D];
#pragma unroll
            for (int a = 0; a < D; a++) x[a] = load_col(th, J.ld, mix_col(D, a), i);
            const double lwv = (double)lw[i];
            if (shear) x[D - 1] = shear_phase(x[D - 1], x[D - 2], shear);   // psi by phi_c
#pragma unroll
            for (int a = 0; a < D; a++) S.x[a][tid] = x[a];
            S.w[tid] = c0 + tid < b1 ? sample_weight(lwv, mlw, beta) : 0.0;
        }
        __syncthreads();
        if (comp) {
#pragma unroll 1
            for (int s = l; s < kEmThreads; s += LP) {
                double df[D], q = 0.0;
#pragma unroll
                for (int a = 0; a < D; a++) df[a] = off(a, S.x[a][s]);
#pragma unroll
                for (int a = 0; a < D; a++) {
                    double y = 0.0;
#pragma unroll
                    for (int b = 0; b <= a; b++) y += li[a * (a + 1) / 2 + b] * df[b];
                    q += y * y;
                }
                S.r[j][s] = cj == -INFINITY ? -INFINITY : cj - 0.5 * q;
            }
        }
        __syncthreads();
        {
            double m = -INFINITY, sum = 0.0;
            for (int k = 0; k < nc; k++) m = fmax(m, S.r[k][tid]);
            for (int k = 0; k < nc; k++) {
                const double v = S.r[k][tid];
                const double e = (v == -INFINITY) ? 0.0 : exp(v - m);
                S.r[k][tid] = e;
                sum += e;
            }
            // a sample past the tile has no weight (its x is the last one's)
            const double scale = (m > -INFINITY && c0 + tid < b1) ? S.w[tid] / sum : 0.0;
            for (int k = 0; k < nc; k++) S.r[k][tid] *= scale;
        }
        __syncthreads();
        if (comp) {
#pragma unroll 1
            for (int s = l; s < kEmThreads; s += LP) {
                const double r = S.r[j][s];
                double x[D];
#pragma unroll
                for (int a = 0; a < D; a++) x[a] = off(a, S.x[a][s]);
                acc[0] += r;
                // the moments of an absent dimension stay 0
#pragma unroll
                for (int a = 0; a < D; a++) {
                    const double rx = r * x[a];
                    acc[1 + a] += rx;
#pragma unroll
                    for (int b = 0; b <= a; b++) acc[8 + a * (a + 1) / 2 + b] += rx * x[b];
                }
            }
        }
    }
    // a component's threads are lanes of one wave
    int base = 0, lim = kMom;
    lane_sums<kMom, LP / 2>(acc, lane, base, lim);
    if (comp) {
        double *o = J.work + Lo.stat + (size_t)j * Lo.nblk * kMom + blockIdx.x;   // [component][moment][tile]
#pragma unroll
        for (int t = 0; t < lane_left<kMom>(LP / 2); t++)
            if (t < lim) o[(base + t) * Lo.nblk] = acc[t];
    }
}

template <class TT, class TL>
__global__ void __launch_bounds__(kEmThreads) k_em_pass(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const EmLayout Lo = em_layout(J.n);
    if (blockIdx.x >= Lo.nblk) return;
    __shared__ EmShared S;
    const int nc = J.gmm->n_comp;
    if (blockIdx.x == 0 && threadIdx.x == 0) J.gmm->valid = 1;   // the update clears it if a factor fails
    auto go = [&](auto D_) {
        constexpr int D = decltype(D_)::value;
        if (nc <= 4)
            em_pass<TT, TL, D, 4>(J, Lo, S);
        else if (nc <= 8)
            em_pass<TT, TL, D, 8>(J, Lo, S);
        else
            em_pass<TT, TL, D, 16>(J, Lo, S);
    };
    if (J.gmm->n_dim == 6)
        go(std::integral_constant<int, 6>{});
    else
        go(std::integral_constant<int, 7>{});
}

// M-step: weights, means (old mean + offset, wrapped into the period),
// covariances + floor, then the factorisation.  One block per component: its
// tiles' moments (74 KB at 256 tiles) are what it waits for, and one block
// for all of a job's components was bound by one CU's read rate (24 us
// against 10.5; 35 us with one thread per component).  Four waves sum nine moments each and four components'
// weights; the first goes on alone.
__global__ void __launch_bounds__(256) k_em_update(const EmJob *__restrict__ jobs) {
    const EmJob &J = jobs[blockIdx.z];
    const EmLayout Lo = em_layout(J.n);
    GmmDev *g = J.gmm;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, j = blockIdx.x;
    const int nc = g->n_comp, d = g->n_dim;
    if (j >= nc) return;
    __shared__ double s[kMom], W[kMaxComp];
    const double *st = J.work + Lo.stat;
    constexpr int kPer = kMom / 4;
    tile_sums<kPer>(st + ((size_t)j * kMom + wv * kPer) * Lo.nblk, Lo.nblk, lane, s + wv * kPer);
    for (int q = wv; q < nc; q += 4) tile_sums<1>(st + (size_t)q * kMom * Lo.nblk, Lo.nblk, lane, W + q);
    if (j == 0 && threadIdx.x < kMaxComp) J.zcount[threadIdx.x] = 0u;   // for the mass estimate after the last iteration
    __syncthreads();
    if (wv != 0) return;
    double tot = 0.0;
    for (int q = 0; q < nc; q++) tot += W[q];
    const double Wj = s[0];
    if (lane == 0) g->w[j] = Wj / tot;
    double row[7], m = 0.0;
    if (Wj > 0.0) {
        wave_cov(s, J.pr, *g, lane, d, row, m);
        if (lane < 7)
            for (int b = 0; b < 7; b++) g->cov[j][lane][b] = row[b];
        if (lane < d) {
            double mu = g->mean[j][lane] + m;
            const double P = col_period(g->dims[lane]);
            if (P > 0.0) mu = mu - P * floor(mu / P);
            g->mean[j][lane] = mu;
        }
    } else {
#pragma unroll
        for (int b = 0; b < 7; b++) row[b] = lane < 7 ? g->cov[j][lane][b] : 0.0;
    }
    __threadfence_block();
    wave_factor(*g, j, lane, d, row);
}

template <class TT, class TL>
void launch_em_t(const EmJob *d_jobs, int n_jobs, int64_t nblk_max, bool any_first, int n_iter, hipStream_t st) {
    const dim3 jz(1, 1, n_jobs), tiles(nblk_max, 1, n_jobs);
    hipLaunchKernelGGL((k_em_scan<TL>), tiles, dim3(kEmThreads), 0, st, d_jobs);
    hipLaunchKernelGGL((k_em_beta<TL>), tiles, dim3(kEmThreads), 0, st, d_jobs);
    hipLaunchKernelGGL(k_em_beta_final, jz, dim3(256), 0, st, d_jobs);
    if (any_first) {
        hipLaunchKernelGGL((k_em_top<TL>), tiles, dim3(kEmThreads), 0, st, d_jobs);
        hipLaunchKernelGGL((k_em_top_final<TT>), jz, dim3(kEmThreads), 0, st, d_jobs);
        hipLaunchKernelGGL((k_em_init<TT, TL>), tiles, dim3(kEmThreads), 0, st, d_jobs);
        hipLaunchKernelGGL(k_em_init_final, jz, dim3(64 * kMaxComp), 0, st, d_jobs);
    }
    for (int it = 0; it < n_iter; it++) {
        hipLaunchKernelGGL((k_em_pass<TT, TL>), tiles, dim3(kEmThreads), 0, st, d_jobs);
        hipLaunchKernelGGL(k_em_update, dim3(kMaxComp, 1, n_jobs), dim3(256), 0, st, d_jobs);
    }
}

}  // namespace

size_t em_work_bytes(int64_t n) { return em_layout(n).total * sizeof(double); }

hipError_t launch_gmm_factor(const EmJob *d_jobs, int n_jobs, hipStream_t st) {
    if (n_jobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gmm_factor, dim3(1, 1, n_jobs), dim3(64 * kMaxComp), 0, st, d_jobs);
    return hipGetLastError();
}

hipError_t launch_em_batch(int policy, const EmJob *d_jobs, const EmJob *h_jobs, int n_jobs, int n_iter,
                           hipStream_t st) {
    if (n_jobs <= 0) return hipSuccess;
    if (n_jobs > 65535) return hipErrorInvalidValue;
    int64_t nblk_max = 1;
    bool any_first = false;
    for (int k = 0; k < n_jobs; k++) {
        if (h_jobs[k].n < 1) return hipErrorInvalidValue;
        nblk_max = std::max<int64_t>(nblk_max, em_layout(h_jobs[k].n).nblk);
        any_first = any_first || h_jobs[k].first;
    }
    if (policy == kFP64)
        launch_em_t<double, double>(d_jobs, n_jobs, nblk_max, any_first, n_iter, st);
    else if (policy == kFP32)
        launch_em_t<float, float>(d_jobs, n_jobs, nblk_max, any_first, n_iter, st);
    else
        launch_em_t<float, double>(d_jobs, n_jobs, nblk_max, any_first, n_iter, st);
    return hipGetLastError();
}

}  // namespace ile
