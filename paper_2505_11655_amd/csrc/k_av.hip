// Adaptive volume integration (Section "Adaptive volume integration") on the
// GPU: the sampler is uniform over a set of active hypercubes of a grid of nb
// bins per sampled column, in the unit cube of the prior's CDF coordinates u
// (theta = inverse-CDF map of u), so ln p - ln p_s = ln V with V the active
// volume.  After a round of n samples with log-weights lw:
//   1. threshold: the largest lw value v such that the samples at or above v
//      hold at least min(ceil(p_thr * total), total) of the fixed-point masses
//      q_i = floor(exp(lw_i - max lw) 2^40) and number at least
//      min(n_min_live, n_finite).  Found by two radix selects (one on the
//      enclosed mass, one on the count) over order-preserving integer keys of
//      lw, eight bits per pass; integer sums make it independent of the order
//      of accumulation.
//   2. refinement, eq. (nbins_V): nb' = ceil((1/dV)^(1/d)) with
//      dV = V n_min / (n sqrt(n_min)), clamped to [1, max_bins].
//   3. the new active cells: the cells of the nb' grid holding a sample at or
//      above the threshold, each listed once, in order of its first such
//      sample (an open-addressing set keeps each cell's lowest sample index;
//      a block-count scan compacts the first samples in index order).
// A sample's u is regenerated from its Philox counter and the grid it was
// drawn from, so the update needs no stored coordinates.
//
// Counter layout (the prior draw's): sample i of round r uses blocks 0..3 of
// attempt 0, ctr = (i lo, i hi, r, b); column c takes u53(w[2c], w[2c+1]) and
// the cell is floor(u53(w14, w15) n_cells) (at most n_cells - 1), so the
// one-cell grid draws exactly the prior.
#include <algorithm>

#include "ile_internal.h"

namespace ile {

namespace {

constexpr int kAvThreads = 256;
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;
constexpr unsigned long long kEmpty = ~0ull;

__device__ __forceinline__ void av_words(uint64_t seed, uint64_t i, uint32_t r, uint32_t *w) {
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int b = 0; b < 4; b++) {
        const U4 o = philox4x32_10(U4{(uint32_t)i, (uint32_t)(i >> 32), r, (uint32_t)b}, k0, k1);
        w[4 * b + 0] = o.x;
        w[4 * b + 1] = o.y;
        w[4 * b + 2] = o.z;
        w[4 * b + 3] = o.w;
    }
}

// Unit-cube coordinates of one sample drawn from the grid (nb, n_cells, cells).
__device__ __forceinline__ void av_unit(const AvDev &S, const uint16_t *cells, const uint32_t *w, double u[7]) {
    const double sel = floor(u53(w[14], w[15]) * (double)S.n_cells);
    int64_t j = (int64_t)sel;
    if (j > S.n_cells - 1) j = S.n_cells - 1;
    const uint16_t *cj = cells + j * 8;
    const double nbd = (double)S.nb;
#pragma unroll
    for (int c = 0; c < 7; c++) {
        const double U = u53(w[2 * c], w[2 * c + 1]);
        const int k = S.kcol[c];
        u[c] = k >= 0 ? ((double)cj[k] + U) / nbd : U;
    }
}

__device__ __forceinline__ const uint16_t *cur_cells(const AvBufs &b, const AvDev &S) {
    return S.cur ? b.cells[1] : b.cells[0];
}

__device__ __forceinline__ unsigned long long mix64(unsigned long long x) {
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}

__global__ void k_av_reset(AvBufs b, int d, int d0, int d1, int d2, int d3, int d4, int d5, int d6) {
    if (threadIdx.x != 0) return;
    AvDev &S = *b.st;
    const int dims[7] = {d0, d1, d2, d3, d4, d5, d6};
    S.d = d;
    for (int c = 0; c < 7; c++) S.kcol[c] = -1;
    for (int k = 0; k < 7; k++) {
        S.dims[k] = k < d ? dims[k] : -1;
        if (k < d) S.kcol[dims[k]] = k;
    }
    S.nb = 1;
    S.nb_next = 1;
    S.cur = 0;
    S.valid = 0;
    S.n_cells = 1;
    S.n_cells_next = 1;
    S.ln_vol = 0.0;
    S.thr = -INFINITY;
    S.n_min = 0;
    S.n_live = 0;
    S.vol_mc = 0.0;
    for (int k = 0; k < 8; k++) b.cells[0][k] = 0;
}

// Samples of job blockIdx.z: each block strides over its job's samples.
#define AV_JOB const AvJob &J = jobs[blockIdx.z]
#define AV_SAMPLES(s) \
    for (int64_t s = (int64_t)blockIdx.x * kAvThreads + threadIdx.x; s < J.n; s += (int64_t)gridDim.x * kAvThreads)

template <class TT>
__global__ void __launch_bounds__(kAvThreads) k_av_draw(const AvJob *__restrict__ jobs) {
    AV_JOB;
    const AvDev &S = *J.b.st;
    const uint16_t *cells = cur_cells(J.b, S);
    const double lnv = S.ln_vol;
    TT *th_out = (TT *)J.theta;
    TT *lr_out = (TT *)J.lnpmps;
    AV_SAMPLES(s) {
        uint32_t w[16];
        av_words(J.seed, (uint64_t)(J.first + s), J.round, w);
        double u[7], th[7];
        av_unit(S, cells, w, u);
        prior_map(J.pr, u, th);
#pragma unroll
        for (int c = 0; c < 7; c++) th_out[c * J.ld + s] = (TT)th[c];
        if (lr_out) lr_out[s] = (TT)lnv;
    }
}

// The set of one update uses its first `used` slots (a power of two >= 2n).
__device__ __forceinline__ uint64_t av_set_mask(const AvJob &J) {
    uint64_t used = 1024;
    while (used < (uint64_t)2 * (uint64_t)J.n) used <<= 1;
    return (used - 1 < J.b.hmask ? used : J.b.hmask + 1) - 1;
}

// The state of an update, its histogram and the part of the cell set that its
// samples can use.
__global__ void __launch_bounds__(kAvThreads) k_av_begin(const AvJob *__restrict__ jobs) {
    AV_JOB;
    AvDev &S = *J.b.st;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            S.key_max = 0;
            S.n_fin = 0;
            S.total = 0;
            for (int c = 0; c < 2; c++) {
                S.prefix[c] = 0;
                S.above_cnt[c] = 0;
                S.above_mass[c] = 0;
                S.target[c] = 0;
                S.last_cnt[c] = 0;
            }
            S.valid = 0;
            S.thr = -INFINITY;
            S.n_min = 0;
            S.n_live = J.n;
            S.vol_mc = 0.0;
        }
        for (int i = threadIdx.x; i < 2 * 256 * 2; i += blockDim.x) J.b.hist[i] = 0;
    }
    const uint64_t used = av_set_mask(J) + 1;
    for (uint64_t i = (uint64_t)blockIdx.x * kAvThreads + threadIdx.x; i < used; i += (uint64_t)gridDim.x * kAvThreads) {
        J.b.hkey[i] = kEmpty;
        J.b.hidx[i] = kNoSlot;
    }
}

template <class TO>
__global__ void __launch_bounds__(kAvThreads) k_av_max(const AvJob *__restrict__ jobs) {
    AV_JOB;
    const TO *lw = (const TO *)J.lw;
    unsigned long long km = 0, cnt = 0;
    AV_SAMPLES(s) {
        const TO v = lw[s];
        if (isfinite(v)) {
            const unsigned long long k = ord_key(v);
            km = k > km ? k : km;
            cnt += 1;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long k2 = __shfl_xor(km, o);
        km = k2 > km ? k2 : km;
        cnt += __shfl_xor(cnt, o);
    }
    __shared__ unsigned long long smk[kAvThreads / 64], smc[kAvThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        smk[wv] = km;
        smc[wv] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kAvThreads / 64; i++) {
            km = smk[i] > km ? smk[i] : km;
            cnt += smc[i];
        }
        if (cnt) {
            atomicMax(&J.b.st->key_max, km);
            atomicAdd(&J.b.st->n_fin, cnt);
        }
    }
}

// One radix-select pass: digit (key >> shift) & 255 of every finite sample
// whose higher digits match the chain's prefix; chain 0 counts and sums the
// fixed-point masses, chain 1 counts.  Bound by latency: the samples' LDS atomics
// on few buckets and the chain of four (FP64 eight) passes, so few samples per
// thread.  The digits are a launch of their own: a last block that picks them
// needs every wave of every block to write its L2 back before it reports
// (2^16 samples, an update and two draws: FP32 98 us against 91, FP64 137, 122;
// 2^20: 244, 202 and 325, 245).
template <class TO>
__global__ void __launch_bounds__(kAvThreads) k_av_hist(const AvJob *__restrict__ jobs, int shift) {
    AV_JOB;
    AvDev &S = *J.b.st;
    if (S.n_fin == 0 || (int64_t)blockIdx.x * kAvThreads >= J.n) return;
    __shared__ unsigned long long h[2 * 256 * 2];
    for (int i = threadIdx.x; i < 2 * 256 * 2; i += kAvThreads) h[i] = 0;
    __syncthreads();
    constexpr int nbits = sizeof(TO) * 8;
    const bool top = shift + 8 == nbits;
    const unsigned long long p0 = top ? 0 : (S.prefix[0] >> (shift + 8));
    const unsigned long long p1 = top ? 0 : (S.prefix[1] >> (shift + 8));
    const double vmax = ord_value(S.key_max, nbits);
    const TO *lw = (const TO *)J.lw;
    AV_SAMPLES(s) {
        const TO v = lw[s];
        if (!isfinite(v)) continue;
        const unsigned long long k = ord_key(v);
        const unsigned long long hi = top ? 0 : (k >> (shift + 8));
        const int dg = (int)((k >> shift) & 255u);
        if (hi == p0) {
            atomicAdd(&h[(0 * 256 + dg) * 2 + 0], 1ull);
            atomicAdd(&h[(0 * 256 + dg) * 2 + 1], mass_fx((double)v, vmax));
        }
        if (hi == p1) atomicAdd(&h[(1 * 256 + dg) * 2 + 0], 1ull);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * 256 * 2; i += kAvThreads)
        if (h[i]) atomicAdd(&J.b.hist[i], h[i]);
}

// Inclusive sums over the block's 256 threads of a and b.
__device__ __forceinline__ void block_scan2(unsigned long long &a, unsigned long long &b) {
    __shared__ unsigned long long wa[kAvThreads / 64], wb[kAvThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long x = __shfl_up(a, o), y = __shfl_up(b, o);
        if (lane >= o) {
            a += x;
            b += y;
        }
    }
    __syncthreads();
    if (lane == 63) {
        wa[wv] = a;
        wb[wv] = b;
    }
    __syncthreads();
    for (int i = 0; i < wv; i++) {
        a += wa[i];
        b += wb[i];
    }
}

// Each chain's digit: thread t holds bucket d = 255 - t; sums from the top
// bucket down give the enclosed count and mass at and above each bucket, and
// the chosen digit is the highest bucket where the chain's target is reached.
// After the last pass: the threshold, n_min and eq. (nbins_V).
template <class TO>
__global__ void __launch_bounds__(kAvThreads) k_av_pick(const AvJob *__restrict__ jobs, int shift) {
    AV_JOB;
    constexpr int nbits = sizeof(TO) * 8;
    AvDev &S = *J.b.st;
    if (S.n_fin == 0) return;
    unsigned long long *H = J.b.hist;
    const int t = threadIdx.x, d = 255 - t;
    __shared__ unsigned long long sh_prefix[2], sh_count[2], sh_total;
    unsigned long long cc[2], mm[2], suf_c[2], suf_m[2];
#pragma unroll
    for (int c = 0; c < 2; c++) {
        cc[c] = H[(c * 256 + d) * 2 + 0];
        mm[c] = H[(c * 256 + d) * 2 + 1];
    }
#pragma unroll
    for (int c = 0; c < 2; c++) {
        suf_c[c] = cc[c];
        suf_m[c] = mm[c];
        block_scan2(suf_c[c], suf_m[c]);
    }
    unsigned long long target0 = S.target[0], target1 = S.target[1];
    if (shift + 8 == nbits) {
        if (t == 255) sh_total = suf_m[0];
        __syncthreads();
        const unsigned long long tot = sh_total, nfin = S.n_fin;
        const unsigned long long tm = (unsigned long long)ceil(J.p_thr * (double)tot);
        target0 = tm < tot ? tm : tot;
        target1 = (unsigned long long)J.n_min_live < nfin ? (unsigned long long)J.n_min_live : nfin;
        if (t == 0) {
            S.total = tot;
            S.target[0] = target0;
            S.target[1] = target1;
            S.valid = 1;
        }
    }
    // the first thread (highest bucket) that reaches the target, found as such:
    // the masses wrap at 2^64 (more than 2^24 samples at the maximum), and a
    // lower bucket can then reach the target again behind one that does not
    __shared__ unsigned long long sh_hit[2][kAvThreads / 64];
    unsigned long long above_c[2], above_m[2], prefix[2];
#pragma unroll
    for (int c = 0; c < 2; c++) {
        above_c[c] = S.above_cnt[c];
        above_m[c] = S.above_mass[c];
        prefix[c] = S.prefix[c];
        const bool hit = c == 0 ? above_m[0] + suf_m[0] >= target0 : above_c[1] + suf_c[1] >= target1;
        const unsigned long long mask = __ballot(hit);
        if ((t & 63) == 0) sh_hit[c][t >> 6] = mask;
    }
    __syncthreads();   // (and every thread has read the chains' state)
#pragma unroll
    for (int c = 0; c < 2; c++) {
        int first = kAvThreads;
#pragma unroll
        for (int w = kAvThreads / 64 - 1; w >= 0; w--)
            if (sh_hit[c][w]) first = 64 * w + __ffsll((long long)sh_hit[c][w]) - 1;
        if (t == first) {
            const unsigned long long p = prefix[c] | ((unsigned long long)d << shift);
            S.last_cnt[c] = cc[c];
            S.above_cnt[c] = above_c[c] + suf_c[c] - cc[c];
            S.above_mass[c] = above_m[c] + suf_m[c] - mm[c];
            S.prefix[c] = p;
            sh_prefix[c] = p;
            sh_count[c] = above_c[c] + suf_c[c];
        }
    }
    __syncthreads();
    if (t == 0 && shift == 0) {
        const int c = sh_prefix[0] <= sh_prefix[1] ? 0 : 1;
        const int64_t n_min = (int64_t)sh_count[c];
        const double ln_vol = S.ln_vol;
        S.thr_key = sh_prefix[c];
        S.n_min = n_min;
        S.thr = ord_value(sh_prefix[c], nbits);
        S.vol_mc = exp(ln_vol) * (double)n_min / (double)J.n;
        const double ln_dv = ln_vol + 0.5 * log((double)n_min) - log((double)J.n);
        const double x = exp(-ln_dv / (double)S.d);
        double nbd = ceil(x - 1e-9);
        nbd = nbd < 1.0 ? 1.0 : (nbd > (double)J.max_bins ? (double)J.max_bins : nbd);
        S.nb_next = (int)nbd;
    }
    for (int i = t; i < 2 * 256 * 2; i += 256) H[i] = 0;
}

// Cells (of the refined grid) of the samples at or above the threshold, into
// the set; each slot keeps the lowest sample index that reached it.
template <class TO>
__global__ void __launch_bounds__(kAvThreads) k_av_insert(const AvJob *__restrict__ jobs) {
    AV_JOB;
    const AvDev &S = *J.b.st;
    if (!S.valid) return;
    const unsigned long long thr = S.thr_key;
    const unsigned long long nb2 = (unsigned long long)S.nb_next;
    const double nb2d = (double)S.nb_next;
    const uint16_t *cells = cur_cells(J.b, S);
    const uint64_t mask = av_set_mask(J);
    const TO *lw = (const TO *)J.lw;
    AV_SAMPLES(s) {
        const TO v = lw[s];
        uint32_t sl = kNoSlot;
        if (isfinite(v) && ord_key(v) >= thr) {
            uint32_t w[16];
            av_words(J.seed, (uint64_t)(J.first + s), J.round, w);
            double u[7];
            av_unit(S, cells, w, u);
            unsigned long long id = 0;
#pragma unroll
            for (int c = 6; c >= 0; c--) {
                if (S.kcol[c] >= 0) {
                    double f = floor(u[c] * nb2d);
                    f = f > nb2d - 1.0 ? nb2d - 1.0 : f;
                    id = id * nb2 + (unsigned long long)f;
                }
            }
            uint64_t h = mix64(id) & mask;
            for (uint64_t probe = 0; probe <= mask; probe++) {
                const unsigned long long prev = atomicCAS(&J.b.hkey[h], kEmpty, id);
                if (prev == kEmpty || prev == id) {
                    atomicMin(&J.b.hidx[h], (uint32_t)s);
                    sl = (uint32_t)h;
                    break;
                }
                h = (h + 1) & mask;
            }
        }
        J.b.slot[s] = sl;
    }
}

// The sample is the first (lowest index) of its cell.
__device__ __forceinline__ bool av_first(const AvJob &J, int64_t s) {
    if (s >= J.n) return false;
    const uint32_t sl = J.b.slot[s];
    return sl != kNoSlot && J.b.hidx[sl] == (uint32_t)s;
}

// The compaction works by spans of whole 256-sample rows: one row up to 2^20
// samples, and at most 4096 spans.
__device__ __forceinline__ int64_t av_span(int64_t n) {
    return (n + (int64_t)kAvThreads * 4096 - 1) / ((int64_t)kAvThreads * 4096) * kAvThreads;
}

// First samples of every span, a wave at a span.
__global__ void __launch_bounds__(kAvThreads) k_av_count(const AvJob *__restrict__ jobs) {
    AV_JOB;
    const AvDev &S = *J.b.st;
    constexpr int kWaves = kAvThreads / 64;
    const int64_t span = av_span(J.n);
    const int nblk = (int)((J.n + span - 1) / span);
    if (!S.valid || (int)blockIdx.x * kWaves >= nblk) return;
    for (int sp = (int)blockIdx.x * kWaves + (int)(threadIdx.x >> 6); sp < nblk; sp += (int)gridDim.x * kWaves) {
        int cnt = 0;
        const int64_t s1 = (sp + 1) * span;
        for (int64_t s = sp * span + (threadIdx.x & 63); s < s1; s += 256) {
            const bool f0 = av_first(J, s), f1 = av_first(J, s + 64), f2 = av_first(J, s + 128),
                       f3 = av_first(J, s + 192);
            cnt += __popcll(__ballot(f0)) + __popcll(__ballot(f1)) + __popcll(__ballot(f2)) + __popcll(__ballot(f3));
        }
        if ((threadIdx.x & 63) == 0) J.b.bcnt[sp] = (uint32_t)cnt;
    }
}

// The spans' counts into offsets (in place), which gives the new number of
// cells, and the new grid made the current one.
__global__ void __launch_bounds__(kAvThreads) k_av_scan(const AvJob *__restrict__ jobs) {
    AV_JOB;
    AvDev &S = *J.b.st;
    if (!S.valid) return;
    const int64_t span = av_span(J.n);
    const int nblk = (int)((J.n + span - 1) / span);
    const int per = (nblk + kAvThreads - 1) / kAvThreads;   // at most 16
    const int lo = threadIdx.x * per;
    uint32_t c[16];
    unsigned long long sum = 0, none = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        c[i] = i < per && lo + i < nblk ? J.b.bcnt[lo + i] : 0u;
        sum += c[i];
    }
    unsigned long long run = sum;
    block_scan2(run, none);
    if (threadIdx.x == kAvThreads - 1) {
        S.cur ^= 1;
        S.nb = S.nb_next;
        S.n_cells_next = (int64_t)run;
        S.n_cells = (int64_t)run;
        S.ln_vol = log((double)run) - S.d * log((double)S.nb);
    }
    run -= sum;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        if (i < per && lo + i < nblk) J.b.bcnt[lo + i] = (uint32_t)run;
        run += c[i];
    }
}

__global__ void __launch_bounds__(kAvThreads) k_av_compact(const AvJob *__restrict__ jobs) {
    AV_JOB;
    const AvDev &S = *J.b.st;
    const int64_t span = av_span(J.n), s0 = (int64_t)blockIdx.x * span;
    if (!S.valid || s0 >= J.n) return;
    uint16_t *cells = S.cur ? J.b.cells[1] : J.b.cells[0];
    const uint64_t nb2 = (uint64_t)S.nb;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __shared__ int wc[2][kAvThreads / 64];
    int64_t base = (int64_t)J.b.bcnt[blockIdx.x];
    int row = 0;
    for (int64_t sr = s0; sr < s0 + span && sr < J.n; sr += kAvThreads, row ^= 1) {
        const int64_t s = sr + threadIdx.x;
        const bool f = av_first(J, s);
        const unsigned long long m = __ballot(f);
        if (lane == 0) wc[row][wv] = __popcll(m);
        __syncthreads();
        int64_t pos = base + __popcll(m & ((1ull << lane) - 1ull));
        for (int i = 0; i < kAvThreads / 64; i++) {
            if (i < wv) pos += wc[row][i];
            base += wc[row][i];
        }
        if (!f) continue;
        uint64_t id = J.b.hkey[J.b.slot[s]];
        uint16_t *out = cells + pos * 8;
        for (int k = 0; k < 8; k++) {
            if (k < S.d) {
                out[k] = (uint16_t)(id % nb2);
                id /= nb2;
            } else {
                out[k] = 0;
            }
        }
    }
}

// Blocks per job: samples per thread from `least` (few samples, every kernel is
// a chain of latency: 2^16 samples draw in 4.7 us and insert in 6.8 with one per
// thread, 9.2 and 15 with four) to `most`, which a launch reaches as it fills
// the chip, with `fill` blocks (the blocks' merges and shared state then cost
// more than the chains: 100 jobs served, 2^16 samples a round, 106 ms with up to
// sixteen, 129 with the least; the maximum of 2^20 samples 11.5 us in 256 blocks,
// 16 in 512).
int grid_for(int64_t n, int n_jobs, int least, int most, int fill) {
    const int64_t want = n * n_jobs / ((int64_t)kAvThreads * fill);
    const int64_t per = std::max<int64_t>(least, std::min<int64_t>(most, want));
    const int64_t g = (n + kAvThreads * per - 1) / (kAvThreads * per);
    return (int)(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

template <class TO>
hipError_t av_update_t(const AvJob *d, int n_jobs, int64_t nmax, hipStream_t st) {
    constexpr int nbits = sizeof(TO) * 8;
    const unsigned nz = (unsigned)n_jobs;
    const dim3 threads(kAvThreads), one(1, 1, nz);
    uint64_t used = 1024;
    while (used < (uint64_t)2 * (uint64_t)nmax) used <<= 1;
    hipLaunchKernelGGL(k_av_begin, dim3(grid_for((int64_t)used, n_jobs, 4, 4, 512), 1, nz), threads, 0, st, d);
    const dim3 g(grid_for(nmax, n_jobs, 4, 16, 256), 1, nz);
    hipLaunchKernelGGL(k_av_max<TO>, g, threads, 0, st, d);
    for (int shift = nbits - 8; shift >= 0; shift -= 8) {
        hipLaunchKernelGGL(k_av_hist<TO>, g, threads, 0, st, d, shift);
        hipLaunchKernelGGL(k_av_pick<TO>, one, threads, 0, st, d, shift);
    }
    hipLaunchKernelGGL(k_av_insert<TO>, dim3(grid_for(nmax, n_jobs, 1, 4, 512), 1, nz), threads, 0, st, d);
    const int nblk = (int)std::min<int64_t>((nmax + kAvThreads - 1) / kAvThreads, 4096);
    hipLaunchKernelGGL(k_av_count, dim3((nblk + 3) / 4, 1, nz), threads, 0, st, d);
    hipLaunchKernelGGL(k_av_scan, one, threads, 0, st, d);
    hipLaunchKernelGGL(k_av_compact, dim3(nblk, 1, nz), threads, 0, st, d);
    return hipGetLastError();
}

int64_t max_n(const AvJob *h, int n_jobs) {
    int64_t m = 0;
    for (int k = 0; k < n_jobs; k++) m = h[k].n > m ? h[k].n : m;
    return m;
}

}  // namespace

hipError_t launch_av_reset(const AvBufs &b, int d, const int *dims, hipStream_t st) {
    int dd[7] = {-1, -1, -1, -1, -1, -1, -1};
    for (int k = 0; k < d && k < 7; k++) dd[k] = dims[k];
    hipLaunchKernelGGL(k_av_reset, dim3(1), dim3(64), 0, st, b, d, dd[0], dd[1], dd[2], dd[3], dd[4], dd[5], dd[6]);
    return hipGetLastError();
}

hipError_t launch_av_draw(int policy, const AvJob *d_jobs, const AvJob *h_jobs, int n_jobs, hipStream_t st) {
    const int64_t nmax = max_n(h_jobs, n_jobs);
    if (n_jobs <= 0 || nmax <= 0) return hipSuccess;
    const dim3 grid(grid_for(nmax, n_jobs, 1, 4, 512), 1, (unsigned)n_jobs);
    if (policy == kFP64)
        hipLaunchKernelGGL(k_av_draw<double>, grid, dim3(kAvThreads), 0, st, d_jobs);
    else
        hipLaunchKernelGGL(k_av_draw<float>, grid, dim3(kAvThreads), 0, st, d_jobs);
    return hipGetLastError();
}

hipError_t launch_av_update(int policy, const AvJob *d_jobs, const AvJob *h_jobs, int n_jobs, hipStream_t st) {
    const int64_t nmax = max_n(h_jobs, n_jobs);
    if (n_jobs <= 0 || nmax <= 0) return hipSuccess;
    if (policy == kFP32) return av_update_t<float>(d_jobs, n_jobs, nmax, st);
    return av_update_t<double>(d_jobs, n_jobs, nmax, st);
}

}  // namespace ile
