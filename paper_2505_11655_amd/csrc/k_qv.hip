// Inner products of eq. (QUV) from the modes and the data on the GPU (the
// precompute behind every likelihood: Q time series over the narrow window,
// and the mode-mode matrices U and V), in FP64, for several intrinsic points
// sharing one data set:
//   Q[p][k][a][i] = 2 df sum_f e^{2 pi i f tau_i} conj(h_pa(f)) d_k(f) w_k(f),
//   U[p][k][a][b] = 2 df sum_f conj(h_pa(f)) h_pb(f) w_k(f),
//   V[p][k][a][b] = 2 df sum_f h_pa(-f) h_pb(f) w_k(f),
// over the band f_lo <= |f| <= f_hi of the two-sided grid f_m = m' df (m' the
// signed FFT-order index), tau_i = (i - win_half) / (n df).
// Q is a dense complex product [window times] x [band] . [band] x [(p, k, a)]:
// X = 2 df conj(h) d w is formed once per band bin and column, the phases come
// from a table e^{2 pi i r / n} at r = (m' j) mod n (exact integer phase), and
// the product runs on the FP64 matrix cores (16 x 16 x 4 steps, the operands
// held in registers so that each LDS or memory read feeds several matrix
// steps) over a slice of the band; slices are summed in order by a second
// kernel (deterministic).  U and V use the symmetries U_ba = conj(U_ab),
// V_ba = V_ab: only a <= b is summed (one block per pair, fixed-order tree
// reduction).
// The decimated route splits the DFT behind Q once (the first step of a
// decimation-in-frequency FFT, Section "Reduce duplication of inner products"
// weighs FFTs against the direct sum): with n = R N2, m = m2 + N2 a (m the
// unsigned grid index, 0 <= m2 < N2, 0 <= a < R) and j = i - win_half =
// R p + q (0 <= q < R),
//   e^{2 pi i m j / n} = e^{2 pi i m2 p / N2} e^{2 pi i m2 q / n} e^{2 pi i a q / R},
// so Q(j) = sum_m2 e^{2 pi i m2 p / N2} Y_q(m2) with the radix-R partial sums
// Y_q(m2) = e^{2 pi i m2 q / n} sum_a X(m2 + N2 a) (X zero off the band).
// Y is formed by a streaming kernel, and the remaining sum is the direct
// route's matrix-core product over N2 bins, R columns per column and only
// the decimated times p of the window (at most 64: one time tile).  Every
// factor is a table value at an exact integer index.
#include <type_traits>

#include "ile_internal.h"
#include "k_qv.h"

namespace ile {

namespace {

constexpr int kQvThreads = 256;
constexpr int kQvTT = 64;     // window times per block tile (direct route)
constexpr int kQvNS = 4;      // 16-column tiles per wave
// columns per block tile: two waves across a 64-time tile, four across a
// 32-time tile
constexpr int qv_tc(int tt) { return tt == 64 ? 32 * kQvNS : 64 * kQvNS; }
constexpr int kQvTC = qv_tc(kQvTT);
constexpr int kQvKB = 32;     // band bins per LDS stage of phases

__global__ void k_qv_twiddle(double2 *__restrict__ tw, int64_t n) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        double s, c;
        sincospi(2.0 * (double)r / (double)n, &s, &c);
        tw[r] = make_double2(c, s);
    }
}

// X[b][col] = 2 df conj(h_pa(f_b)) d_k(f_b) w_k(f_b), col = (p * nd + k) * na + a.
// One column per thread (its (p, k, a) decoded once), kQvXRun consecutive
// bins per block row: the writes are coalesced along the columns, and each
// cache line of a mode row serves several bins.
constexpr int kQvXRun = 16;
__global__ void __launch_bounds__(kQvThreads)
    k_qv_x(const double2 *__restrict__ hlm, const double2 *__restrict__ data, const double *__restrict__ inv_psd,
           const int64_t *__restrict__ band, int64_t n_band, int64_t n, int na, int nd, int np, double df,
           double2 *__restrict__ X) {
    const int64_t cols = (int64_t)np * nd * na;
    const int64_t col = (int64_t)blockIdx.x * kQvThreads + threadIdx.x;
    if (col >= cols) return;
    const int a = (int)(col % na);
    const int k = (int)((col / na) % nd);
    const int64_t p = col / ((int64_t)na * nd);
    const double2 *h = hlm + (p * na + a) * n;
    const double2 *dk = data + (int64_t)k * n;
    const double *wk = inv_psd ? inv_psd + (int64_t)k * n : nullptr;
    for (int64_t b0 = (int64_t)blockIdx.y * kQvXRun; b0 < n_band; b0 += (int64_t)gridDim.y * kQvXRun) {
        const int64_t b1 = b0 + kQvXRun < n_band ? b0 + kQvXRun : n_band;
        for (int64_t b = b0; b < b1; b++) {
            const int64_t m = band[b];
            const double2 hv = h[m];
            const double2 d = dk[m];
            const double w = 2.0 * df * (wk ? wk[m] : 1.0);
            // conj(h) d
            const double re = hv.x * d.x + hv.y * d.y, im = hv.x * d.y - hv.y * d.x;
            X[b * cols + col] = make_double2(re * w, im * w);
        }
    }
}

// Partial Q of one (time tile, column tile, band slice) on the FP64 matrix
// cores.  A block of four waves covers TT = 64 window times x 128 columns (two
// waves along the times, two along the columns) or TT = 32 times x 256
// columns (four waves along the columns); each wave a 32 x 64 sub-tile as
// 2 x 4 tiles of 16 x 16 (kQvNS = 4 column tiles),
// with the real and the imaginary part of every tile in its own accumulator.
// One step of v_mfma_f64_16x16x4f64 takes four band bins: lane l holds the A
// element (time l % 16, bin l / 16) and the B element (bin l / 16, column
// l % 16), and its four results are times l / 16 + 4 r (r = 0..3) of column
// l % 16.  Each complex product is four real ones, Re += Er Xr - Ei Xi,
// Im += Er Xi + Ei Xr.
// The phases of a stage of 32 bins x TT times sit in LDS (the column waves of
// a time range share them), double-buffered: every thread reads its TT / 8
// phases of the next stage (one bin, TT / 8 consecutive times: one 64-bit
// remainder, then r += m' mod n per time) from the table during the
// stage's first matrix step, after that step's X reads (the memory counter
// retires in order, so waiting for X then never waits for the table), and
// writes them to LDS after the stage's last step.  X is read by each wave
// straight from memory (no other wave of the block uses it), one step ahead.
// Blocks are numbered so that the time tiles of one column tile run on one
// XCD and share its L2.
typedef double qv_d4 __attribute__((ext_vector_type(4)));

template <int TT>
__global__ void __launch_bounds__(kQvThreads)
    k_qv_q(const double2 *__restrict__ X, const double2 *__restrict__ tw, const int64_t *__restrict__ msig,
           int64_t n_band, int64_t n, int64_t cols, int n_time, int win_half, int64_t slice, int n_tt, int n_tc,
           double2 *__restrict__ part) {
    static_assert(TT == 64 || TT == 32, "time tile of 64 or 32");
    constexpr int TC = qv_tc(TT);
    constexpr int PT = TT / 8;   // phases per thread and stage
    __shared__ double2 sE[2][kQvKB][TT];
    const int64_t nb = gridDim.x;
    const int64_t h = blockIdx.x;
    const int64_t lid = nb % 8 == 0 ? (h % 8) * (nb / 8) + h / 8 : h;
    const int tt = (int)(lid % n_tt);
    const int tc = (int)((lid / n_tt) % n_tc);
    const int64_t z = lid / ((int64_t)n_tt * n_tc);
    const int64_t b_lo = z * slice;
    const int64_t b_hi = b_lo + slice < n_band ? b_lo + slice : n_band;
    const int t0 = tt * TT;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    // the wave's first time within the tile and first column
    const int wt = TT == 64 ? 32 * (wv & 1) : 0;
    const int64_t cw = (int64_t)tc * TC + 16 * kQvNS * (TT == 64 ? (wv >> 1) : wv);
    // this thread's share of a phase stage: bin gb, times gt .. gt + PT - 1
    const int gb = threadIdx.x >> 3, gt = (threadIdx.x & 7) * PT;
    static_assert(kQvThreads * PT == kQvKB * TT, "PT phases per thread and stage");
    // m' of the thread's bin in the stage at bb (the bin itself when msig is
    // null); a bin past the slice gets m' = 0 and a zero phase (its X, read
    // at a clamped index, is then multiplied by 0)
    auto bin_m = [&](int64_t bb, double &f) -> int64_t {
        const int64_t b = bb + gb;
        f = b < b_hi ? 1.0 : 0.0;
        return b < b_hi ? (msig ? msig[b] : b) : 0;
    };
    // The thread's PT phases for bin m', r = m' (t - win_half) mod n,
    // then r += m' mod n per time (r stays in [0, n)).  Rows past the window
    // need no mask: they are never stored.
    auto phase_get = [&](int64_t m, double f, double2 (&pv)[PT]) {
        int64_t r = (m * (int64_t)(t0 + gt - win_half)) % n;
        r = r < 0 ? r + n : r;
        int64_t step = m % n;
        step = step < 0 ? step + n : step;
#pragma unroll
        for (int q = 0; q < PT; q++) {
            const double2 w = tw[r];
            pv[q] = make_double2(w.x * f, w.y * f);
            r += step;
            r = r >= n ? r - n : r;
        }
    };
    qv_d4 accR[2][kQvNS], accI[2][kQvNS];
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int s = 0; s < kQvNS; s++) {
            accR[r][s] = qv_d4{0.0, 0.0, 0.0, 0.0};
            accI[r][s] = qv_d4{0.0, 0.0, 0.0, 0.0};
        }
    // X of one step of four bins: the lane's bin b4 + lk, its columns.
    // Indices past the slice or the columns are clamped to a valid element
    // (unconditional loads): such a bin has a zero phase, such a column is
    // never stored.
    auto load_x = [&](int64_t b4, double2 (&x)[kQvNS]) {
        const int64_t b = b4 + lk;
        const int64_t bc = b < b_hi ? b : b_hi - 1;
#pragma unroll
        for (int s = 0; s < kQvNS; s++) {
            const int64_t c = cw + 16 * s + li;
            const double2 w = X[bc * cols + (c < cols ? c : cols - 1)];
            x[s] = make_double2(w.x, w.y);
        }
    };
    {
        double2 pv[PT];
        double f;
        const int64_t m = bin_m(b_lo, f);
        phase_get(m, f, pv);
#pragma unroll
        for (int q = 0; q < PT; q++) sE[0][gb][gt + q] = pv[q];
    }
    double f_next;
    int64_t m_next = bin_m(b_lo + kQvKB, f_next);   // read one stage before it is used
    double2 xc[kQvNS];
    load_x(b_lo, xc);
    __syncthreads();
    int buf = 0;
    for (int64_t bb = b_lo; bb < b_hi; bb += kQvKB) {
        const int nk = b_hi - bb < kQvKB ? (int)(b_hi - bb) : kQvKB;
        const bool more = bb + kQvKB < b_hi;
        double2 pv[PT];
        for (int ks = 0; ks < nk; ks += 4) {
            // the next step's X is in flight while this step's products run
            double2 xn[kQvNS];
            load_x(bb + ks + 4, xn);
            // the next stage's phases: read during the first step, written
            // after the last
            if (more && ks == 0) {
                phase_get(m_next, f_next, pv);
                m_next = bin_m(bb + 2 * kQvKB, f_next);
            }
            double2 e[2];
#pragma unroll
            for (int r = 0; r < 2; r++) e[r] = sE[buf][ks + lk][wt + 16 * r + li];
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const double ni = -e[r].y;
#pragma unroll
                for (int s = 0; s < kQvNS; s++) {
                    accR[r][s] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[r].x, xc[s].x, accR[r][s], 0, 0, 0);
                    accR[r][s] = __builtin_amdgcn_mfma_f64_16x16x4f64(ni, xc[s].y, accR[r][s], 0, 0, 0);
                    accI[r][s] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[r].x, xc[s].y, accI[r][s], 0, 0, 0);
                    accI[r][s] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[r].y, xc[s].x, accI[r][s], 0, 0, 0);
                }
            }
#pragma unroll
            for (int s = 0; s < kQvNS; s++) xc[s] = xn[s];
        }
        if (more) {
#pragma unroll
            for (int q = 0; q < PT; q++) sE[buf ^ 1][gb][gt + q] = pv[q];
        }
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int s = 0; s < kQvNS; s++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int t = t0 + wt + 16 * r + lk + 4 * q;
                const int64_t c = cw + 16 * s + li;
                if (t < n_time && c < cols)
                    part[(z * cols + c) * n_time + t] = make_double2(accR[r][s][q], accI[r][s][q]);
            }
}

// Q[col][t] = sum over slices in order.
__global__ void k_qv_reduce(const double2 *__restrict__ part, int n_slices, int64_t cols, int n_time,
                            double2 *__restrict__ Q) {
    const int64_t total = cols * n_time;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        double re = 0.0, im = 0.0;
        for (int s = 0; s < n_slices; s++) {
            const double2 v = part[(int64_t)s * total + e];
            re += v.x;
            im += v.y;
        }
        Q[e] = make_double2(re, im);
    }
}

// Stage one of the decimated route: Y[m2][col R + q] for every column and
// m2 in [0, N2), from the R aliases m2 + N2 a (X = 2 df conj(h) d w on the
// band's bins, 0 elsewhere).  A block covers kDecM consecutive m2 (the lanes
// of a wave, so that every read of a mode row, the data and the weight is
// one contiguous run) by kDecC columns (one per wave).  The outputs of each
// (m2, column) go through LDS, at most eight q at a time (two passes for
// R = 16, which keeps the block's LDS near 33 KB), and the tile's rows are
// written out from there in runs of whole cache lines.
constexpr int kDecM = 64;
constexpr int kDecC = kQvThreads / 64;

// In place, v[q] <- sum_a v[a] e^{2 pi i a q / R} (R a power of two): radix-2
// decimation in time over the bit-reversed inputs, log2 R passes of R / 2
// butterflies, wr[r] = e^{2 pi i r / R}; a butterfly with twiddle 1 skips its
// product.
template <int R>
__device__ __forceinline__ void dft_radix2(double2 (&v)[R], const double2 (&wr)[R]) {
    constexpr int LG = R == 2 ? 1 : R == 4 ? 2 : R == 8 ? 3 : 4;
    static_assert((1 << LG) == R, "R in {2, 4, 8, 16}");
#pragma unroll
    for (int a = 0; a < R; a++) {
        int b = 0;
#pragma unroll
        for (int k = 0; k < LG; k++) b |= ((a >> k) & 1) << (LG - 1 - k);
        if (a < b) {
            const double2 t = v[a];
            v[a] = v[b];
            v[b] = t;
        }
    }
#pragma unroll
    for (int len = 2; len <= R; len <<= 1) {
        const int half = len / 2, step = R / len;
#pragma unroll
        for (int st = 0; st < R; st += len)
#pragma unroll
            for (int j = 0; j < half; j++) {
                const double2 u = v[st + j], x = v[st + j + half];
                double2 t = x;
                if (j != 0) {
                    const double2 w = wr[j * step];
                    t = make_double2(x.x * w.x - x.y * w.y, x.x * w.y + x.y * w.x);
                }
                v[st + j] = make_double2(u.x + t.x, u.y + t.y);
                v[st + j + half] = make_double2(u.x - t.x, u.y - t.y);
            }
    }
}
template <int R>
__global__ void __launch_bounds__(kQvThreads)
    k_qv_dec1(const double2 *__restrict__ hlm, const double2 *__restrict__ data, const double *__restrict__ inv_psd,
              const double2 *__restrict__ tw, int64_t n, int na, int nd, int np, double df, double f_lo, double f_hi,
              int64_t n_mt, double2 *__restrict__ Y) {
    constexpr int QC = R < 8 ? R : 8;       // q per LDS pass
    constexpr int RW = kDecC * QC + 1;      // LDS row (one element of padding)
    __shared__ double2 sY[kDecM * RW];
    const int64_t cols = (int64_t)np * nd * na;
    const int64_t n2 = n / R;
    // blocks numbered so that consecutive tiles run on one XCD: the columns
    // of one mode row for the other detectors (na columns apart) then find
    // its lines in that XCD's L2
    const int64_t nbk = gridDim.x, hb = blockIdx.x;
    const int64_t lid = nbk % 8 == 0 ? (hb % 8) * (nbk / 8) + hb / 8 : hb;
    const int64_t mt = lid % n_mt, ct = lid / n_mt;
    const int64_t m2_0 = mt * kDecM, col0 = ct * kDecC;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t m2 = m2_0 + lane, col = col0 + wv;
    const bool live = m2 < n2 && col < cols;
    double2 yq[R];
    if (live) {
        const int a = (int)(col % na);
        const int k = (int)((col / na) % nd);
        const int64_t p = col / ((int64_t)na * nd);
        const double2 *h = hlm + (p * na + a) * n;
        const double2 *dk = data + (int64_t)k * n;
        const double *wk = inv_psd ? inv_psd + (int64_t)k * n : nullptr;
        // every alias's reads are issued before any is used; the band test is
        // the host's (|m' df| in [f_lo, f_hi], m' the signed index), and a
        // mode value off the band is not read
        double2 hv[R], dv[R];
        double wpsd[R];
        bool inb[R];
#pragma unroll
        for (int al = 0; al < R; al++) {
            const int64_t m = m2 + n2 * al;
            const int64_t ms = m < (n + 1) / 2 ? m : m - n;
            const double af = fabs((double)ms * df);
            inb[al] = af >= f_lo && af <= f_hi;
            hv[al] = make_double2(0.0, 0.0);
            if (inb[al]) hv[al] = h[m];
            dv[al] = dk[m];
            wpsd[al] = wk ? wk[m] : 1.0;
        }
        double2 x[R];
#pragma unroll
        for (int al = 0; al < R; al++) {
            const double w = inb[al] ? 2.0 * df * wpsd[al] : 0.0;
            const double2 hh = hv[al], d = dv[al];
            x[al] = make_double2((hh.x * d.x + hh.y * d.y) * w, (hh.x * d.y - hh.y * d.x) * w);
        }
        double2 wr[R];   // e^{2 pi i r / R}
#pragma unroll
        for (int r = 0; r < R; r++) wr[r] = tw[(int64_t)r * n2];
        dft_radix2<R>(x, wr);
#pragma unroll
        for (int q = 0; q < R; q++) {
            const double2 t = tw[m2 * q];   // e^{2 pi i m2 q / n}, m2 q < n
            yq[q] = make_double2(x[q].x * t.x - x[q].y * t.y, x[q].x * t.y + x[q].y * t.x);
        }
    }
    const int64_t ncol = cols - col0 < kDecC ? cols - col0 : kDecC;
#pragma unroll
    for (int h = 0; h < R / QC; h++) {
        if (h > 0) __syncthreads();   // the previous pass's reads are done
        if (live) {
#pragma unroll
            for (int q = 0; q < QC; q++) sY[lane * RW + wv * QC + q] = yq[h * QC + q];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < kDecM * kDecC * QC; e += kQvThreads) {
            const int row = e / (kDecC * QC), c = e % (kDecC * QC);
            const int cl = c / QC, q = h * QC + c % QC;
            if (m2_0 + row < n2 && cl < ncol)
                Y[(m2_0 + row) * cols * R + (col0 + cl) * R + q] = sY[row * RW + c];
        }
    }
}

// Q[col][i] of the decimated route: the slice partials of decimated column
// col R + q at decimated time p - p_lo, j = i - win_half = R p + q, summed
// in slice order.
__global__ void k_qv_dec_reduce(const double2 *__restrict__ part, int n_slices, int64_t cols, int radix, int n_t2,
                                int n_time, int win_half, int p_lo, double2 *__restrict__ Q) {
    const int64_t total = cols * n_time;
    const int64_t stride = cols * radix * n_t2;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t col = e / n_time;
        const int j = (int)(e % n_time) - win_half;
        const int pd = j >= 0 ? j / radix : -((-j + radix - 1) / radix);
        const int q = j - pd * radix;
        const int64_t src = (col * radix + q) * n_t2 + (pd - p_lo);
        double re = 0.0, im = 0.0;
        for (int s = 0; s < n_slices; s++) {
            const double2 v = part[(int64_t)s * stride + src];
            re += v.x;
            im += v.y;
        }
        Q[e] = make_double2(re, im);
    }
}

// U and V: a block per (point, band slice, detector group of up to kUvDet,
// pair group of up to kQvThreads pairs a <= b).  The band is symmetric in f, so
// a slice is a run of bins m >= 0 and each bin stands for f and -f: the block
// stages chunks of its slice in LDS, h_a(f) and h_a(-f) of every mode and
// w_k(f), w_k(-f) of its detectors, and every staged value serves both
//   U: w(f) conj(h_a(f)) h_b(f) + w(-f) conj(h_a(-f)) h_b(-f),
//   V: w(f) h_a(-f) h_b(f) + w(-f) h_a(f) h_b(-f)
// (a bin that is its own mirror, m = 0 or n / 2, has w(-f) = 0 here), which
// halves the reads of the modes against a pass over both signs.  The rows of
// the chunk are one element longer than it, so that the lanes of a wave, on
// different rows at one bin, fall on different banks.  Each thread
// accumulates a strip of up to three pairs (a, b), (a, b + 1), (a, b + 2) for
// all the group's detectors over every G-th bin of a chunk (G bin lanes per
// strip): 11 LDS reads for three pairs where one pair alone takes 7.  The
// lanes are summed in lane order, and the slices in slice order by
// k_qv_uv_sum (with one slice the block writes U and V itself).
// Deterministic for a given launch shape.  Bounded by the vector unit and the
// LDS reads together.
// Measured, 256 points x 9 modes x 3 detectors x 8,034 band bins: 0.17 ms;
// 0.32 ms with one pair per thread and a pass over both signs.
constexpr int kUvDet = 4;
constexpr int kUvChunk = 128;  // most bins per LDS chunk (a power of two, fewer for many modes)
constexpr int kUvStrip = 3;    // pairs per thread
__host__ __device__ inline int uv_strips(int na) {
    int q = 0;
    for (int a = 0; a < na; a++) q += (na - a + kUvStrip - 1) / kUvStrip;
    return q;
}

__device__ __forceinline__ void uv_pair(int q, int na, int &a, int &b) {
    a = 0;
    while (q >= na - a) {
        q -= na - a;
        a++;
    }
    b = a + q;
}

__device__ __forceinline__ void uv_store(double2 *U, double2 *V, int64_t base, int na, int a, int b, double f,
                                         const double (&s)[4]) {
    const double ui = a == b ? 0.0 : f * s[1];   // the diagonal <h_a|h_a> is real
    U[base + a * na + b] = make_double2(f * s[0], ui);
    U[base + b * na + a] = make_double2(f * s[0], -ui);
    V[base + a * na + b] = make_double2(f * s[2], f * s[3]);
    V[base + b * na + a] = make_double2(f * s[2], f * s[3]);
}

template <int ND>
__global__ void __launch_bounds__(kQvThreads)
    k_qv_uv(const double2 *__restrict__ hlm, const double *__restrict__ inv_psd, int64_t m_lo, int64_t n_half,
            int64_t n, int na, int nd, double df, int64_t slice, int n_sl, int lcb, int n_dg, int n_strip,
            double *__restrict__ partial, double2 *__restrict__ U, double2 *__restrict__ V) {
    extern __shared__ double uv_lds[];
    const int npair = na * (na + 1) / 2;
    const int64_t p = blockIdx.x;
    const int sl = blockIdx.y;
    const int dg = (int)(blockIdx.z % n_dg), sg = (int)(blockIdx.z / n_dg);
    const int k0 = dg * kUvDet;
    const int nk = nd - k0 < ND ? nd - k0 : ND;
    const int strip0 = sg * kQvThreads;
    const int ns_here = n_strip - strip0 < kQvThreads ? n_strip - strip0 : kQvThreads;
    const int G = kQvThreads / ns_here;
    const int tid = threadIdx.x;
    const bool active = tid < ns_here * G;
    const int ls = active ? tid / G : 0, g = tid % G;   // consecutive lanes on consecutive bins of one row
    const int cb = 1 << lcb, row = cb + 1;
    // the strip's row a and first column b, and the pairs it holds
    int a = 0, q = strip0 + ls;
    while (q >= (na - a + kUvStrip - 1) / kUvStrip) {
        q -= (na - a + kUvStrip - 1) / kUvStrip;
        a++;
    }
    const int b = a + kUvStrip * q;
    const int nb = na - b < kUvStrip ? na - b : kUvStrip;
    double2 *sH = (double2 *)uv_lds;            // [na][row]  h_a(f)
    double2 *sM = sH + (size_t)na * row;        // [na][row]  h_a(-f)
    double2 *sW = sM + (size_t)na * row;        // [ND][row]  w_k(f), w_k(-f)
    double acc[kUvStrip][ND][4];
#pragma unroll
    for (int t = 0; t < kUvStrip; t++)
#pragma unroll
        for (int kk = 0; kk < ND; kk++)
#pragma unroll
            for (int c = 0; c < 4; c++) acc[t][kk][c] = 0.0;
    const int64_t e_lo = (int64_t)sl * slice;
    const int64_t e_hi = e_lo + slice < n_half ? e_lo + slice : n_half;
    const double2 *hp = hlm + p * na * n;
    for (int64_t eb = e_lo; eb < e_hi; eb += cb) {
        const int ncb = e_hi - eb < cb ? (int)(e_hi - eb) : cb;
        __syncthreads();
        if (lcb >= 6) {
            // straight to LDS, 64 bins of one row per wave instruction, all in
            // flight at once (a bin past the chunk loads its first bin, unused)
            const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), per = 1 << (lcb - 6);
            for (int e = wv; e < 2 * na * per; e += kQvThreads / 64) {
                const int c = 64 * (e & (per - 1)) + lane, r = e >> (lcb - 6), am = r >> 1;
                const int64_t m = m_lo + eb + (c < ncb ? c : 0);
                const double2 *src = hp + (int64_t)am * n + ((r & 1) && m > 0 ? n - m : m);
                double2 *dst = ((r & 1) ? sM : sH) + am * row + 64 * (e & (per - 1));
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                                 (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
            }
        } else {
            for (int e = tid; e < na << lcb; e += kQvThreads) {
                const int am = e >> lcb, c = e & (cb - 1);
                const int64_t m = m_lo + eb + (c < ncb ? c : 0);
                sH[am * row + c] = hp[(int64_t)am * n + m];
                sM[am * row + c] = hp[(int64_t)am * n + (m > 0 ? n - m : 0)];
            }
        }
        for (int e = tid; e < nk << lcb; e += kQvThreads) {
            const int kk = e >> lcb, c = e & (cb - 1);
            const int64_t m = m_lo + eb + (c < ncb ? c : 0);
            const bool own = m == 0 || 2 * m == n;
            const double *w = inv_psd ? inv_psd + (int64_t)(k0 + kk) * n : nullptr;
            sW[kk * row + c] = make_double2(w ? w[m] : 1.0, own ? 0.0 : (w ? w[n - m] : 1.0));
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's loads have reached LDS
        __syncthreads();
        if (active) {
            for (int c = g; c < ncb; c += G) {
                const double2 x = sH[a * row + c], z = sM[a * row + c];   // f, -f
                double2 w[ND];
#pragma unroll
                for (int kk = 0; kk < ND; kk++)
                    if (kk < nk) w[kk] = sW[kk * row + c];
#pragma unroll
                for (int s = 0; s < kUvStrip; s++) {
                    if (s >= nb) break;
                    const double2 y = sH[(b + s) * row + c], t = sM[(b + s) * row + c];
                    const double p0 = x.x * y.x + x.y * y.y, p1 = x.x * y.y - x.y * y.x;   // conj(h_a) h_b at f
                    const double p2 = z.x * y.x - z.y * y.y, p3 = z.x * y.y + z.y * y.x;   // h_a(-f) h_b(f)
                    const double q0 = z.x * t.x + z.y * t.y, q1 = z.x * t.y - z.y * t.x;   // the same, f -> -f
                    const double q2 = x.x * t.x - x.y * t.y, q3 = x.x * t.y + x.y * t.x;
#pragma unroll
                    for (int kk = 0; kk < ND; kk++) {
                        if (kk < nk) {
                            acc[s][kk][0] = fma(w[kk].y, q0, fma(w[kk].x, p0, acc[s][kk][0]));
                            acc[s][kk][1] = fma(w[kk].y, q1, fma(w[kk].x, p1, acc[s][kk][1]));
                            acc[s][kk][2] = fma(w[kk].y, q2, fma(w[kk].x, p2, acc[s][kk][2]));
                            acc[s][kk][3] = fma(w[kk].y, q3, fma(w[kk].x, p3, acc[s][kk][3]));
                        }
                    }
                }
            }
        }
    }
    // bin lanes summed in lane order, one pair of the strips at a time
    double *red = uv_lds;   // [kQvThreads][ND * 4]
#pragma unroll
    for (int s = 0; s < kUvStrip; s++) {
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < ND; kk++)
#pragma unroll
            for (int c = 0; c < 4; c++) red[tid * ND * 4 + kk * 4 + c] = acc[s][kk][c];
        __syncthreads();
        if (!active || g != 0 || s >= nb) continue;
        for (int kk = 0; kk < nk; kk++) {
            double t[4] = {0.0, 0.0, 0.0, 0.0};
            for (int gg = 0; gg < G; gg++)
#pragma unroll
                for (int c = 0; c < 4; c++) t[c] += red[(ls * G + gg) * ND * 4 + kk * 4 + c];
            const int64_t pk = p * nd + k0 + kk;
            if (n_sl == 1) {
                uv_store(U, V, pk * na * na, na, a, b + s, 2.0 * df, t);
            } else {
                const int pair = a * na - a * (a - 1) / 2 + (b + s - a);
                double *o = partial + ((pk * npair + pair) * n_sl + sl) * 4;
#pragma unroll
                for (int c = 0; c < 4; c++) o[c] = t[c];
            }
        }
    }
}

// U and V from the slice partials, summed in slice order.
__global__ void k_qv_uv_sum(const double *__restrict__ partial, int64_t n_pk, int na, int n_sl, double df,
                            double2 *__restrict__ U, double2 *__restrict__ V) {
    const int npair = na * (na + 1) / 2;
    const int64_t total = n_pk * npair;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t pk = e / npair;
        int a, b;
        uv_pair((int)(e % npair), na, a, b);
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        for (int sl = 0; sl < n_sl; sl++)
#pragma unroll
            for (int c = 0; c < 4; c++) s[c] += partial[(e * n_sl + sl) * 4 + c];
        uv_store(U, V, pk * na * na, na, a, b, 2.0 * df, s);
    }
}

// U and V (k_qv_uv, then k_qv_uv_sum over its band slices): band slices so
// that the grid is one round of resident blocks (three to a CU by LDS), at
// least one chunk and at most 32 of them, the slice partials held in `part`
// (part_bytes long; free once Q has been reduced from it).  The band is the
// bins m_lo .. m_lo + n_half - 1 and their mirrors.
struct UvPlan {
    int n_dg, n_sg, n_strip, lcb, n_sl;   // lcb: log2 of the chunk's bins
    int64_t per_sl;                       // bytes of one slice's partials
};
// Beside the direct sum a block takes two chunks by itself where that is at most
// twelve bins per lane: the sum's launch costs more (one point and mode, 161
// bins 97 us a call against 110; 9 modes 111, 117).  The windowed route's calls
// are shorter and lose by it (9 modes, 252 bins 42 us, 48).
UvPlan uv_plan(int64_t n_half, int na, int nd, int np, bool win) {
    UvPlan u;
    const int npair = na * (na + 1) / 2;
    u.n_dg = (nd + kUvDet - 1) / kUvDet;
    u.n_strip = uv_strips(na);
    u.n_sg = (u.n_strip + kQvThreads - 1) / kQvThreads;
    u.lcb = 0;
    while ((2 << u.lcb) <= kUvChunk && ((int64_t)(2 << u.lcb) + 1) * ((int64_t)na * 32 + kUvDet * 16) <= 49152) u.lcb++;
    const int64_t cb = (int64_t)1 << u.lcb, blocks1 = (int64_t)np * u.n_dg * u.n_sg;
    const int64_t chunks = (n_half + cb - 1) / cb, lanes = kQvThreads / std::min(u.n_strip, kQvThreads);
    const bool one = !win && chunks <= 2 && n_half <= 12 * lanes;
    u.n_sl = one ? 1 : (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(768 / blocks1, 32), chunks));
    u.per_sl = (int64_t)np * nd * npair * 32;
    return u;
}
void launch_uv(const void *hlm, const double *inv_psd, int64_t m_lo, int64_t n_half, int64_t n, int na, int nd, int np,
               double df, double *part, int64_t part_bytes, void *U, void *V, bool win, hipStream_t st) {
    const int npair = na * (na + 1) / 2;
    const UvPlan u = uv_plan(n_half, na, nd, np, win);
    int64_t n_sl = std::min<int64_t>(u.n_sl, std::max<int64_t>(1, part_bytes / u.per_sl));
    const int64_t uslice = (n_half + n_sl - 1) / n_sl;
    n_sl = (n_half + uslice - 1) / uslice;
    const size_t lds = std::max<size_t>((((size_t)1 << u.lcb) + 1) * ((size_t)na * 32 + kUvDet * 16),
                                        (size_t)kQvThreads * kUvDet * 4 * 8);
    // accumulators for as many detectors as a group holds
    auto go = [&](auto ND_) {
        hipLaunchKernelGGL(k_qv_uv<decltype(ND_)::value>, dim3((unsigned)np, (unsigned)n_sl, (unsigned)(u.n_dg * u.n_sg)),
                           dim3(kQvThreads), lds, st, (const double2 *)hlm, inv_psd, m_lo, n_half, n, na, nd, df, uslice,
                           (int)n_sl, u.lcb, u.n_dg, u.n_strip, part, (double2 *)U, (double2 *)V);
    };
    if (nd <= 2)
        go(std::integral_constant<int, 2>{});
    else if (nd == 3)
        go(std::integral_constant<int, 3>{});
    else
        go(std::integral_constant<int, 4>{});
    if (n_sl > 1) {
        const int64_t ue = (int64_t)np * nd * npair;
        hipLaunchKernelGGL(k_qv_uv_sum, dim3((unsigned)std::min<int64_t>((ue + 255) / 256, 65536)), dim3(256), 0, st,
                           part, (int64_t)np * nd, na, (int)n_sl, df, (double2 *)U, (double2 *)V);
    }
}

// --------------------------------------------------------- windowed FFT route
// Q over the window as M = n / 512 transforms of 512 points each: with the
// window in blocks of 512 times, j = 512 blk - win_half + i (0 <= i < 512),
// and the grid index m = M m2 + m1 (0 <= m2 < 512, 0 <= m1 < M),
//   e^{2 pi i m j / n} = e^{2 pi i m (512 blk - win_half) / n} e^{2 pi i m2 i / 512} e^{2 pi i m1 i / n},
//   Q(j) = sum_m1 zeta_i^m1 FFT512[ conj(h)(M m2 + m1) D(M m2 + m1) ](i),  zeta_i = e^{2 pi i i / n},
// with D = 2 df d w e^{2 pi i m (512 blk - win_half) / n} on the band, 0 off it
// (k_qv_wprep, once per call).  The sum over m1 is Horner's rule with the
// factor zeta_i^4 (the four waves of a block take m1 mod 4), so nothing but
// the window is ever written: the radix stage of the decimated route writes
// and reads n elements per column.  Work per column and bin: 9 radix-2 stages
// of a 512-point transform (three radix-8 steps in registers) against a
// 32-row matrix product over every bin.
// One wave holds one transform, 8 points per lane: step 1 over r of m2 =
// 64 r + l, step 2 over a and step 3 over b of l = 8 a + b, output
// i = k + 8 k2 + 64 k3.  Between the steps the real and then the imaginary
// parts change lanes through 576 doubles of LDS; the strides 72 and 9 keep
// every access conflict-free.  A block is one column; it stages h, kWinC
// consecutive m1 of every m2 at a time (runs of 64 bytes), straight into LDS.
// The blocks of one mode row's detectors are neighbours on one XCD, so that
// its L2 serves all but the first.  Small blocks (one wave per SIMD) so that
// three fit a CU by registers and LDS and one's staging hides behind the
// others' transforms: a block of two waves for each of three detectors, which
// reads h once, ran one to a CU (518 us on the shape below).
// Measured, 256 points x 9 modes x 3 detectors on 16,384 bins (20-1024 Hz, 410
// window times): 0.32 ms where the radix stage, the product and the slice sum
// of the decimated route take 1.36 ms.  The vector unit and the LDS are each
// busy about 55 % of it.
constexpr int kWinP = 512;
constexpr int kWinC = 4;                   // m1 per staged chunk, and waves per block
constexpr int kWinSlab = 64 * kWinC;       // staged elements of 64 m2
constexpr int kWinThreads = 64 * kWinC;
constexpr int kWinX = 576;                 // exchange buffer of a wave (doubles)
// Cost per bin, column and window block in the unit of dec_cost (a complex
// product of the matrix-core kernel): 0.32 ms for 6,912 columns of 16,384
// bins, where the direct sum's 497 per band bin (8,034) take 4.0 ms.
constexpr int kWinCost = 20;

__device__ __forceinline__ double2 cmul(double2 x, double2 w) {
    return make_double2(x.x * w.x - x.y * w.y, x.x * w.y + x.y * w.x);
}

// tw[r] = e^{2 pi i r / n}, and D[blk][k][m1][m2].
__global__ void __launch_bounds__(kQvThreads)
    k_qv_wprep(const double2 *__restrict__ data, const double *__restrict__ inv_psd, int64_t n, int nd, double df,
               int64_t m_lo, int64_t m_hi, int win_half, double2 *__restrict__ tw, double2 *__restrict__ D) {
    const int64_t M = n / kWinP;
    const int k = blockIdx.y, blk = blockIdx.z;
    for (int64_t e = (int64_t)blockIdx.x * kQvThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kQvThreads) {
        double s, c;
        if (k == 0 && blk == 0) {
            sincospi(2.0 * (double)e / (double)n, &s, &c);
            tw[e] = make_double2(c, s);
        }
        const int64_t m = M * (e % kWinP) + e / kWinP;
        const int64_t mm = 2 * m > n ? n - m : m;   // |signed index|
        double2 v = make_double2(0.0, 0.0);
        if (mm >= m_lo && mm <= m_hi) {
            int64_t r = (m * ((int64_t)kWinP * blk - win_half)) % n;
            r = r < 0 ? r + n : r;
            sincospi(2.0 * (double)r / (double)n, &s, &c);
            const double w = 2.0 * df * (inv_psd ? inv_psd[(int64_t)k * n + m] : 1.0);
            const double2 d = data[(int64_t)k * n + m];
            v = cmul(make_double2(d.x * w, d.y * w), make_double2(c, s));
        }
        D[((int64_t)blk * nd + k) * n + e] = v;
    }
}

// v[k] <- sum_j v[j] e^{2 pi i j k / 8}
__device__ __forceinline__ void dft8(double2 (&v)[8]) {
    constexpr double h = 0.70710678118654752440;
    auto add = [](double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); };
    auto sub = [](double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); };
    auto rot = [](double2 a) { return make_double2(-a.y, a.x); };   // i a
    const double2 a0 = add(v[0], v[4]), a1 = sub(v[0], v[4]), a2 = add(v[2], v[6]), a3 = rot(sub(v[2], v[6]));
    const double2 a4 = add(v[1], v[5]), a5 = sub(v[1], v[5]), a6 = add(v[3], v[7]), a7 = rot(sub(v[3], v[7]));
    const double2 b0 = add(a0, a2), b2 = sub(a0, a2), b1 = add(a1, a3), b3 = sub(a1, a3);
    const double2 c0 = add(a4, a6), c2 = rot(sub(a4, a6)), o1 = add(a5, a7), o3 = sub(a5, a7);
    const double2 c1 = make_double2((o1.x - o1.y) * h, (o1.x + o1.y) * h);      // e^{i pi / 4} o1
    const double2 c3 = make_double2((-o3.x - o3.y) * h, (o3.x - o3.y) * h);     // e^{3 i pi / 4} o3
    v[0] = add(b0, c0);
    v[4] = sub(b0, c0);
    v[2] = add(b2, c2);
    v[6] = sub(b2, c2);
    v[1] = add(b1, c1);
    v[5] = sub(b1, c1);
    v[3] = add(b3, c3);
    v[7] = sub(b3, c3);
}

// Lanes of one wave exchange through LDS: its accesses stay in program order
// on either side (the LDS serves one wave's instructions in order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v[j] of lane w0 + j ws is written, v[j] is read from r0 + j rs (both parts
// through the same doubles, one after the other).
template <int WS, int RS>
__device__ __forceinline__ void wave_exchange(double2 (&v)[8], double *x, int w0, int r0) {
#pragma unroll
    for (int j = 0; j < 8; j++) x[w0 + j * WS] = v[j].x;
    wave_sync();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j].x = x[r0 + j * RS];
    wave_sync();
#pragma unroll
    for (int j = 0; j < 8; j++) x[w0 + j * WS] = v[j].y;
    wave_sync();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j].y = x[r0 + j * RS];
    wave_sync();
}

// Block: column (p, a, k) x window block x m1 slice.  slabs: bit r is set when
// some bin with m2 in [64 r, 64 r + 64) is on the band; the staging area holds
// those slabs only.  out: [slice][col][n_time].
__global__ void __launch_bounds__(kWinThreads, 4)
    k_qv_win(const double2 *__restrict__ hlm, const double2 *__restrict__ D, const double2 *__restrict__ tw, int64_t n,
             int na, int nd, int64_t n_pa, int n_blk, int n_sl, int64_t m1_per, int64_t m_lo, int64_t m_hi, int slabs,
             int n_time, double2 *__restrict__ out) {
    extern __shared__ __align__(16) double2 win_lds[];
    const int64_t M = n / kWinP;
    // blocks of one mode row run on one XCD and share its L2
    const int64_t nb = gridDim.x, hb = blockIdx.x;
    int64_t lid = nb % 8 == 0 ? (hb % 8) * (nb / 8) + hb / 8 : hb;
    const int k = (int)(lid % nd);
    lid /= nd;
    const int sl = (int)(lid % n_sl);
    lid /= n_sl;
    const int blk = (int)(lid % n_blk);
    const int64_t pa = lid / n_blk;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_slab = __popc(slabs);
    // [exchange buffers][step-2 twiddles][staged slabs], the twiddles
    // e^{2 pi i b k2 / 64} at [k2][b]
    double *xb = (double *)win_lds + wv * kWinX;
    double2 *sT = win_lds + kWinC * (kWinX / 2);
    double2 *sH = sT + 64;
    const double2 *h = hlm + pa * n;
    const double2 *Dk = D + ((int64_t)blk * nd + k) * n;
    const int i0 = (lane >> 3) + 8 * (lane & 7);                       // output i = i0 + 64 k3
    if (wv == 0) sT[lane] = tw[(int64_t)(lane & 7) * (lane >> 3) * 8 * M];
    // zeta_i^4 = z0 zc[k3] (i = i0 + 64 k3): a lane factor and a uniform one,
    // the latter in scalar registers
    auto mod_n = [&](int64_t r) {   // of an index below 4 n
        while (r >= n) r -= n;
        return r;
    };
    const double2 z0 = tw[mod_n(kWinC * i0)];
    double2 t1[8], zc[8], acc[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        if (j > 0) t1[j] = tw[(int64_t)lane * j * M];             // e^{2 pi i l k / 512}
        if (j > 0) zc[j] = tw[mod_n(kWinC * 64 * j)];
        acc[j] = make_double2(0.0, 0.0);
    }
    // this lane's staged m1 of a chunk and M m2 of the first slab (n < 2^31)
    const unsigned m2l = 16 * wv + (lane >> 2), m1x = (lane & 3) ^ ((m2l >> 1) & 3), mb = (unsigned)M * m2l;
    const unsigned m_w = (unsigned)(m_hi - m_lo);
    const int64_t s_lo = (int64_t)sl * m1_per, s_hi = s_lo + m1_per < M ? s_lo + m1_per : M;
    for (int64_t c0 = s_lo + (s_hi - s_lo - 1) / kWinC * kWinC; c0 >= s_lo; c0 -= kWinC) {
        __syncthreads();   // the previous chunk's reads are done
        // The chunk goes straight to LDS, all of it in flight at once, 16 m2 x
        // 4 m1 per wave instruction.  Slot (m2, c) holds m1 = c0 +
        // (c ^ (m2 / 2 mod 4)), so that the lanes of a transform, on
        // consecutive m2 at one m1, read different banks.  An element off the
        // band or past the slice is not read: its lane loads the band's first
        // bin instead (D is zero there, and no m1 past the slice is used).
        const unsigned m1 = (unsigned)c0 + m1x;
        const unsigned mf = (int64_t)m1 < s_hi ? m1 + mb : ~0u;
        int bits = slabs;
        for (int g = 0; g < n_slab; g++, bits &= bits - 1) {
            const unsigned m = mf + (unsigned)(64 * (__ffs(bits) - 1)) * (unsigned)M;
            const unsigned mm = m < (unsigned)n - m ? m : (unsigned)n - m;
            const double2 *src = h + (mf != ~0u && mm - (unsigned)m_lo <= m_w ? m : (unsigned)m_lo);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                             (__attribute__((address_space(3))) void *)(sH + g * kWinSlab + wv * 64), 16,
                                             0, 0);
        }
        // the wave's row of D travels with them (a wave past the slice reads a
        // valid row that it does not use)
        double2 v[8];
        const double2 *dj = Dk + (c0 + wv < s_hi ? c0 + wv : c0) * kWinP + lane;
#pragma unroll
        for (int r = 0; r < 8; r++) {
            v[r] = make_double2(0.0, 0.0);
            if ((slabs >> r) & 1) v[r] = dj[64 * r];
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's loads have reached LDS
        __syncthreads();
        if (c0 + wv >= s_hi) continue;
        const double2 *hj = sH + lane * kWinC + (wv ^ ((lane >> 1) & 3));
#pragma unroll
        for (int r = 0; r < 8; r++)
            if ((slabs >> r) & 1) {
                const double2 d = v[r], x = *hj;
                v[r] = make_double2(x.x * d.x + x.y * d.y, x.x * d.y - x.y * d.x);   // conj(h) D
                hj += kWinSlab;
            }
        dft8(v);
#pragma unroll
        for (int q = 1; q < 8; q++) v[q] = cmul(v[q], t1[q]);
        wave_exchange<72, 8>(v, xb, lane, (lane >> 3) * 72 + (lane & 7));
        dft8(v);
#pragma unroll
        for (int q = 1; q < 8; q++) v[q] = cmul(v[q], sT[q * 8 + (lane & 7)]);
        wave_exchange<9, 1>(v, xb, (lane >> 3) * 72 + (lane & 7), lane * 9);
        dft8(v);
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const double2 o = q > 0 ? cmul(acc[q], zc[q]) : acc[q];
            acc[q].x = fma(-o.y, z0.y, fma(o.x, z0.x, v[q].x));
            acc[q].y = fma(o.x, z0.y, fma(o.y, z0.x, v[q].y));
        }
    }
    // the wave's own power of zeta_i, then the four waves summed in order
    // through LDS (two at a time: the exchange buffers hold two waves' values)
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int64_t m1 = s_lo + wv < M ? s_lo + wv : 0;   // m1 i < n (a wave past the slice holds zeros)
        acc[q] = cmul(acc[q], tw[m1 * (i0 + 64 * q)]);
    }
#pragma unroll
    for (int h2 = 2; h2 > 0; h2 >>= 1) {
        double2 *sum = win_lds + (wv & (h2 - 1)) * kWinP;
        __syncthreads();
        if (wv >= h2 && wv < 2 * h2) {
#pragma unroll
            for (int q = 0; q < 8; q++) sum[q * 64 + lane] = acc[q];
        }
        __syncthreads();
        if (wv < h2) {
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const double2 w = sum[q * 64 + lane];
                acc[q] = make_double2(acc[q].x + w.x, acc[q].y + w.y);
            }
        }
    }
    if (wv != 0) return;
    const int64_t p = pa / na, a = pa % na, col = (p * nd + k) * na + a, cols = n_pa * nd;
    double2 *o = out + ((int64_t)sl * cols + col) * n_time;
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int t = blk * kWinP + i0 + 64 * q;
        if (t < n_time) o[t] = acc[q];
    }
}

}  // namespace

size_t qv_scratch_bytes(int64_t n, int64_t n_band, int64_t cols, int n_time, int n_slices) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    return al((size_t)n * 16) + al((size_t)n_band * 8) * 2 + al((size_t)n_band * cols * 16) +
           al((size_t)n_slices * cols * n_time * 16);
}

namespace {

// Band slices per call: at least two rounds of resident blocks (256 CUs x 2
// blocks of k_qv_q), at least 128 bins per slice, and the fewest slices whose
// last round is at least 90 % full.

int slices_for(int64_t n_band, int64_t tiles) {
    constexpr int64_t kResident = 256 * 2;
    int64_t smax = (n_band + 127) / 128;
    smax = smax < 1 ? 1 : smax;
    int64_t best = 1;
    double best_eff = -1.0;
    for (int64_t s = 1; s <= smax && s <= 64; s++) {
        const int64_t blocks = tiles * s;
        const int64_t rounds = (blocks + kResident - 1) / kResident;
        const double eff = (double)blocks / (double)(rounds * kResident);
        if (blocks >= 2 * kResident && eff >= 0.9) return (int)s;
        if (eff > best_eff + 1e-9) {
            best_eff = eff;
            best = s;
        }
    }
    return (int)best;
}

}  // namespace

int qv_slices(int64_t n_band, int64_t cols, int n_time) {
    return slices_for(n_band, (int64_t)((n_time + kQvTT - 1) / kQvTT) * ((cols + kQvTC - 1) / kQvTC));
}

hipError_t launch_qv(const void *hlm, const void *data, const double *inv_psd, int64_t n, int na, int nd, int np,
                     double df, const int64_t *h_band, const int64_t *h_msig, int64_t n_band, int64_t m_lo,
                     int64_t n_half, int n_time, int win_half, void *Q, void *U, void *V, void *scratch,
                     int n_slices, hipStream_t st) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    char *w = (char *)scratch;
    double2 *tw = (double2 *)w;
    w += al((size_t)n * 16);
    int64_t *band = (int64_t *)w;
    w += al((size_t)n_band * 8);
    int64_t *msig = (int64_t *)w;
    w += al((size_t)n_band * 8);
    const int64_t cols = (int64_t)np * nd * na;
    double2 *X = (double2 *)w;
    w += al((size_t)n_band * cols * 16);
    double2 *part = (double2 *)w;
    hipError_t e = hipMemcpyAsync(band, h_band, (size_t)n_band * 8, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(msig, h_msig, (size_t)n_band * 8, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_qv_twiddle, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, tw, n);
    const int64_t xruns = std::min<int64_t>((n_band + kQvXRun - 1) / kQvXRun, 65535);
    hipLaunchKernelGGL(k_qv_x, dim3((unsigned)((cols + kQvThreads - 1) / kQvThreads), (unsigned)xruns),
                       dim3(kQvThreads), 0, st, (const double2 *)hlm, (const double2 *)data, inv_psd, band, n_band, n,
                       na, nd, np, df, X);
    const int64_t slice = ((n_band + n_slices - 1) / n_slices + kQvKB - 1) / kQvKB * kQvKB;
    const int ns = (int)((n_band + slice - 1) / slice);
    const int n_tt = (n_time + kQvTT - 1) / kQvTT;
    const int n_tc = (int)((cols + kQvTC - 1) / kQvTC);
    hipLaunchKernelGGL(k_qv_q<kQvTT>, dim3((unsigned)((int64_t)n_tt * n_tc * ns)), dim3(kQvThreads), 0, st, X, tw, msig,
                       n_band, n, cols, n_time, win_half, slice, n_tt, n_tc, part);
    const int64_t qe = cols * n_time;
    hipLaunchKernelGGL(k_qv_reduce, dim3((unsigned)std::min<int64_t>((qe + 255) / 256, 65536)), dim3(256), 0, st,
                       part, ns, cols, n_time, (double2 *)Q);
    launch_uv(hlm, inv_psd, m_lo, n_half, n, na, nd, np, df, (double *)part, (int64_t)ns * cols * n_time * 16, U, V,
              false, st);
    return hipGetLastError();
}

namespace {

int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

// The decimated times p_lo .. p_lo + n_t2 - 1 that the window covers.
void dec_window(int n_time, int win_half, int radix, int &p_lo, int &n_t2) {
    p_lo = floor_div(-win_half, radix);
    n_t2 = floor_div(n_time - 1 - win_half, radix) - p_lo + 1;
}

// The decimated times' tile height (32 or 64; 0 when they do not fit one).
int dec_tile(int n_t2) { return n_t2 <= 32 ? 32 : (n_t2 <= 64 ? 64 : 0); }

// Cost per column in complex matrix-core products: the direct sum takes
// (padded window) x n_band; the decimated one (tile height) x n for the
// product, about 49 per bin for the radix partial sums' 16-byte element
// written and read back (Y against X), at the measured rates (6.1e12
// products/s, 4 TB/s), and 2R per bin for their R-point sums on the vector
// units.
double dec_cost(int64_t n, int tile, int radix) { return (double)(tile + 49 + 2 * radix) * (double)n; }

}  // namespace

int qv_radix(int64_t n, int64_t n_band, int n_time, int win_half, bool force) {
    int best = 0;
    double best_cost = 0.0;
    for (int r = 2; r <= 16; r *= 2) {
        if (n % r != 0) continue;
        int p_lo, n_t2;
        dec_window(n_time, win_half, r, p_lo, n_t2);
        const int tile = dec_tile(n_t2);
        if (tile == 0) continue;
        const double c = dec_cost(n, tile, r);
        if (best == 0 || c < best_cost) {
            best = r;
            best_cost = c;
        }
    }
    if (best == 0 || force) return best;
    const double direct = (double)((n_time + kQvTT - 1) / kQvTT * kQvTT + 49) * (double)n_band;
    return best_cost < direct ? best : 0;
}

int qv_dec_slices(int64_t n, int64_t cols, int n_time, int win_half, int radix) {
    int p_lo, n_t2;
    dec_window(n_time, win_half, radix, p_lo, n_t2);
    const int64_t tc = qv_tc(dec_tile(n_t2));
    return slices_for(n / radix, (cols * radix + tc - 1) / tc);
}

size_t qv_dec_scratch_bytes(int64_t n, int64_t cols, int n_time, int win_half, int radix, int n_slices) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    int p_lo, n_t2;
    dec_window(n_time, win_half, radix, p_lo, n_t2);
    return al((size_t)n * 16) + al((size_t)(n / radix) * 16) + al((size_t)n * cols * 16) +
           al((size_t)n_slices * cols * radix * n_t2 * 16);
}

hipError_t launch_qv_dec(const void *hlm, const void *data, const double *inv_psd, int64_t n, int na, int nd,
                         int np, double df, double f_lo, double f_hi, int64_t m_lo, int64_t n_half,
                         int n_time, int win_half, int radix, void *Q, void *U, void *V, void *scratch,
                         int n_slices, hipStream_t st) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const int64_t n2 = n / radix;
    const int64_t cols = (int64_t)np * nd * na;
    const int64_t cols2 = cols * radix;
    int p_lo, n_t2;
    dec_window(n_time, win_half, radix, p_lo, n_t2);
    char *w = (char *)scratch;
    double2 *tw = (double2 *)w;
    w += al((size_t)n * 16);
    double2 *tw2 = (double2 *)w;
    w += al((size_t)n2 * 16);
    double2 *Y = (double2 *)w;
    w += al((size_t)n * cols * 16);
    double2 *part = (double2 *)w;
    hipLaunchKernelGGL(k_qv_twiddle, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, tw, n);
    hipLaunchKernelGGL(k_qv_twiddle, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, st, tw2, n2);
    const int64_t n_mt = (n2 + kDecM - 1) / kDecM;
    const dim3 g1((unsigned)(n_mt * ((cols + kDecC - 1) / kDecC)));
    switch (radix) {
    case 2:
        hipLaunchKernelGGL(k_qv_dec1<2>, g1, dim3(kQvThreads), 0, st, (const double2 *)hlm, (const double2 *)data,
                           inv_psd, tw, n, na, nd, np, df, f_lo, f_hi, n_mt, Y);
        break;
    case 4:
        hipLaunchKernelGGL(k_qv_dec1<4>, g1, dim3(kQvThreads), 0, st, (const double2 *)hlm, (const double2 *)data,
                           inv_psd, tw, n, na, nd, np, df, f_lo, f_hi, n_mt, Y);
        break;
    case 8:
        hipLaunchKernelGGL(k_qv_dec1<8>, g1, dim3(kQvThreads), 0, st, (const double2 *)hlm, (const double2 *)data,
                           inv_psd, tw, n, na, nd, np, df, f_lo, f_hi, n_mt, Y);
        break;
    case 16:
        hipLaunchKernelGGL(k_qv_dec1<16>, g1, dim3(kQvThreads), 0, st, (const double2 *)hlm, (const double2 *)data,
                           inv_psd, tw, n, na, nd, np, df, f_lo, f_hi, n_mt, Y);
        break;
    default:
        return hipErrorInvalidValue;
    }
    // the product over the N2 decimated bins (m2 itself as the signed index:
    // its phase only enters modulo N2) at decimated times p = t + p_lo
    const int64_t slice = ((n2 + n_slices - 1) / n_slices + kQvKB - 1) / kQvKB * kQvKB;
    const int ns = (int)((n2 + slice - 1) / slice);
    const int tile = dec_tile(n_t2);
    const int n_tc = (int)((cols2 + qv_tc(tile) - 1) / qv_tc(tile));
    if (tile == 32)
        hipLaunchKernelGGL(k_qv_q<32>, dim3((unsigned)((int64_t)n_tc * ns)), dim3(kQvThreads), 0, st, Y, tw2,
                           (const int64_t *)nullptr, n2, n2, cols2, n_t2, -p_lo, slice, 1, n_tc, part);
    else if (tile == 64)
        hipLaunchKernelGGL(k_qv_q<64>, dim3((unsigned)((int64_t)n_tc * ns)), dim3(kQvThreads), 0, st, Y, tw2,
                           (const int64_t *)nullptr, n2, n2, cols2, n_t2, -p_lo, slice, 1, n_tc, part);
    else
        return hipErrorInvalidValue;
    const int64_t qe = cols * n_time;
    hipLaunchKernelGGL(k_qv_dec_reduce, dim3((unsigned)std::min<int64_t>((qe + 255) / 256, 65536)), dim3(256), 0, st,
                       part, ns, cols, radix, n_t2, n_time, win_half, p_lo, (double2 *)Q);
    launch_uv(hlm, inv_psd, m_lo, n_half, n, na, nd, np, df, (double *)part, (int64_t)ns * cols2 * n_t2 * 16, U, V,
              false, st);
    return hipGetLastError();
}

namespace {

// m1 slices of the windowed route: about three blocks per CU, whole chunks of
// kWinC per slice.
struct WinPlan {
    int n_blk, n_sl;
    int64_t m1_per;
};
WinPlan win_plan(int64_t n, int64_t cols, int n_time) {
    WinPlan w;
    const int64_t M = n / kWinP;
    w.n_blk = (n_time + kWinP - 1) / kWinP;
    const int64_t blocks = cols * w.n_blk, chunks = (M + kWinC - 1) / kWinC;
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(chunks, (768 + blocks - 1) / blocks));
    w.m1_per = (chunks + want - 1) / want * kWinC;
    w.n_sl = (int)((M + w.m1_per - 1) / w.m1_per);
    return w;
}

}  // namespace

bool qv_win_ok(int64_t n, int64_t n_band, int64_t cols, int n_time) {
    if (n % kWinP != 0 || n >= ((int64_t)1 << 31)) return false;
    const WinPlan w = win_plan(n, cols, n_time);
    // a launch's grid holds it: the blocks of k_qv_win in x, the window blocks of
    // k_qv_wprep in z
    if (cols * w.n_blk * w.n_sl > INT32_MAX || w.n_blk > 65535) return false;
    return (double)kWinCost * (double)(n * w.n_blk) <
           (double)((n_time + kQvTT - 1) / kQvTT * kQvTT + 49) * (double)n_band;
}

size_t qv_win_scratch_bytes(int64_t n, int64_t n_half, int na, int nd, int np, int n_time) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const WinPlan w = win_plan(n, (int64_t)np * na * nd, n_time);
    const UvPlan u = uv_plan(n_half, na, nd, np, true);
    const size_t part = w.n_sl > 1 ? (size_t)w.n_sl * np * nd * na * n_time * 16 : 0;
    return al((size_t)n * 16) + al((size_t)n * nd * w.n_blk * 16) +
           al(std::max<size_t>(part, u.n_sl > 1 ? (size_t)u.n_sl * (size_t)u.per_sl : 0));
}

hipError_t launch_qv_win(const void *hlm, const void *data, const double *inv_psd, int64_t n, int na, int nd, int np,
                         double df, int64_t m_lo, int64_t n_half, int n_time, int win_half, void *Q, void *U, void *V,
                         void *scratch, hipStream_t st) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const int64_t M = n / kWinP, n_pa = (int64_t)np * na, cols = n_pa * nd, m_hi = m_lo + n_half - 1;
    const WinPlan w = win_plan(n, cols, n_time);
    const UvPlan u = uv_plan(n_half, na, nd, np, true);
    char *b = (char *)scratch;
    double2 *tw = (double2 *)b;
    b += al((size_t)n * 16);
    double2 *D = (double2 *)b;
    b += al((size_t)n * nd * w.n_blk * 16);
    double2 *part = (double2 *)b;
    // the slabs of 64 m2 that hold a bin of the band (m2 = m / M)
    int slabs = 0;
    for (int r = 0; r < 8; r++) {
        const int64_t lo = M * 64 * r, hi = M * 64 * (r + 1) - 1;
        const bool pos = lo <= m_hi && hi >= m_lo, neg = lo <= n - m_lo && hi >= n - m_hi;
        if (pos || neg) slabs |= 1 << r;
    }
    const unsigned pb = (unsigned)std::min<int64_t>((n + kQvThreads - 1) / kQvThreads, 4096);
    hipLaunchKernelGGL(k_qv_wprep, dim3(pb, (unsigned)nd, (unsigned)w.n_blk), dim3(kQvThreads), 0, st,
                       (const double2 *)data, inv_psd, n, nd, df, m_lo, m_hi, win_half, tw, D);
    const int64_t blocks = cols * w.n_blk * w.n_sl;   // qv_win_ok: a grid holds them
    const size_t lds = (size_t)kWinC * kWinX * 8 + 64 * 16 + (size_t)__builtin_popcount(slabs) * kWinSlab * 16;
    hipError_t e = hipFuncSetAttribute((const void *)k_qv_win, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_qv_win, dim3((unsigned)blocks), dim3(kWinThreads), lds, st, (const double2 *)hlm, D, tw, n, na,
                       nd, n_pa, w.n_blk, w.n_sl, w.m1_per, m_lo, m_hi, slabs, n_time,
                       w.n_sl > 1 ? part : (double2 *)Q);
    if (w.n_sl > 1) {
        const int64_t qe = cols * n_time;
        hipLaunchKernelGGL(k_qv_reduce, dim3((unsigned)std::min<int64_t>((qe + 255) / 256, 65536)), dim3(256), 0, st,
                           part, w.n_sl, cols, n_time, (double2 *)Q);
    }
    launch_uv(hlm, inv_psd, m_lo, n_half, n, na, nd, np, df, (double *)part, (int64_t)u.n_sl * u.per_sl, U, V, true,
              st);
    return hipGetLastError();
}

}  // namespace ile
