// Time-marginalised likelihood per extrinsic sample: the (time) x (extrinsic)
// array of eq. (lnL:MatrixForm) integrated over the geocentric time prior,
//   ln L_t = ln sum_j (dt / (R 2 t_w)) exp( s T1(t_j) - s^2 T2 / 4 ),
// on the nodes t_j = j dt / R, |j| <= tm_half (dt: the window's sample step).
// T2 does not depend on t.  With tau_k(t) = t - x_k.n/c, the window position
// of node j = R q + r in detector k is u0_k + q + r/R, so the integer part is
// i0_k + q + c_kr (c_kr in {0, 1}) and the four Lagrange weights depend only
// on (k, r): they are computed once per sample as five-tap weights over the
// samples i0_k + q - 1 .. i0_k + q + 3.  Per lattice step q each detector
// needs one new
//   G_k(i) = sum_a Re[ conj(F_k) y_a e^{i m_a phi} Q_k,a(i) ],
// and each node costs five FMAs per detector plus one exponential; the sum
// over nodes is a chunked log-sum-exp (one rescale per lattice step at most)
// accumulated in FP64.  A node whose stencil leaves the window contributes
// nothing (its pointwise lnL is -inf).
// With the distance integrated (DM) every node's value is the table's
// ln L_D(T1(t_j), T2) instead of s T1(t_j) - s^2 T2 / 4 (T1, T2 at s = 1):
//   ln L_{t,D} = ln sum_j (dt / (R 2 t_w)) L_D(T1(t_j), T2),
// the time and distance integrals taken together; the table row of T2 is
// set up once per sample and each node interpolates along a only (FP64).
#pragma once

#include <cfloat>

#include "k_lnl_impl.h"

namespace ile {

template <int S, int K, int POL, bool LDS, int R, bool DM>
struct TmargKernel {
    using LK = LnlKernel<S, K, POL, LDS, false>;
    using Tp = PolTypes<POL>;
    using TT = typename Tp::TT;
    using TS = typename Tp::TS;
    using TG = typename Tp::TG;
    using TE = typename Tp::TE;
    using TA = typename Tp::TA;
    using TO = typename Tp::TO;
    using ccpx = typename LK::ccpx;
    static constexpr int NM = LK::NM;
    static constexpr int NE = LK::NE;
    static constexpr bool kT2First = sizeof(TA) == 8 || DM;   // DM: the table row needs T2 first
    using TV = std::conditional_t<DM, double, TA>;             // node values
    // With the window in LDS the G rows (a different row per lane) load the
    // LDS beyond its bandwidth; reading the first detector through L1/L2
    // instead balances the two paths (measured, 256 x 2^16 samples: HLV 9
    // modes 33.8 -> 25.5 ms, two of three detectors through L1/L2 39.5 ms;
    // HL 5 modes 16.0 -> 14.5 ms).  Only the other detectors are staged.
    static constexpr int kGlobalDets = LDS ? tmarg_global_dets(S, K, POL) : K;

    typedef __attribute__((address_space(1))) const cpx<TA> gcpx;
    // FP32: exponents in units of ln 2, so that e^{s T1 - m} is one FMA and
    // v_exp_f32; the origin m is the same FP32 number in the sum and in the
    // result, so its rounding cancels.  It follows the maximum only in strides
    // of kStride (a new origin costs an exponential and an FP64 product, and
    // every lane rises to its maximum through many), which keeps an exponent's
    // rounding below 2^-21.  Masks only at the steps where a lane of the wave
    // has a node outside.  Bound by the vector unit (189 instructions per
    // step); 16 x 16,384 samples, HLV 9 modes, R = 4: 391 to 364 us.
    static constexpr bool kExp2 = sizeof(TV) == 4;
    static constexpr float kStride = 8.0f;

    __device__ __forceinline__ static void run(const EvalJob &J, const int64_t begin, const int64_t end,
                                               cpx<TA> *smem) {
        const int T = J.n_time;
        const cpx<TA> *__restrict__ Qg = (const cpx<TA> *)J.Q;
        if constexpr (LDS) {
            const size_t nwords = (size_t)(K - kGlobalDets) * T * NM * sizeof(cpx<TA>) / 8;
            const uint2 *src = (const uint2 *)(Qg + (size_t)kGlobalDets * T * NM);
            uint2 *dst = (uint2 *)smem;
            for (size_t w = threadIdx.x; w < nwords; w += blockDim.x) dst[w] = src[w];
            __syncthreads();
        }
        ccpx *Ut = (ccpx *)J.Ut;
        ccpx *Vt = (ccpx *)J.Vt;
        const TT *__restrict__ th = (const TT *)J.theta;
        const TT *__restrict__ lr = (const TT *)J.lnpmps;
        TO *__restrict__ outL = (TO *)J.lnL;
        TO *__restrict__ outW = (TO *)J.lw;
        const int64_t ld = J.ld;
        const int jh = J.tm_half;
        // lattice steps covering nodes -jh..jh (floor division)
        const int q_lo = (-jh >= 0) ? (-jh) / R : -((jh + R - 1) / R);
        const int q_hi = jh / R;

        for (int64_t i = begin + threadIdx.x; i < end; i += blockDim.x) {
            asm volatile("" : "+s"(Ut), "+s"(Vt));
            const TT al = th[i], de = th[ld + i], DD = th[3 * ld + i];
            const TT ci = th[4 * ld + i], ph = th[5 * ld + i], ps = th[6 * ld + i];
            const bool ok = DD > (TT)0 && ci >= (TT)-1 && ci <= (TT)1;

            TG Fr[K], Fi[K];
            TS uu[K];
            TG y[NM];
            TE Er[NE], Ei[NE];
            LK::geometry(J, al, de, (TT)0, ci, ph, ps, Fr, Fi, uu, y, Er, Ei);
            const TA s = pick<TA>(J.d_ref, J.d_reff) / (TA)DD;
            // T2 does not depend on t.  FP32: formed after the time loop, so its
            // temporaries never coexist with the loop state; FP64 (one wave per
            // SIMD, registers to spare): before it, like the pointwise kernel.
            TA T2 = (TA)0;
            if constexpr (kT2First) T2 = LK::template quad_T2<false>(Fr, Fi, y, Er, Ei, Ut, Vt);
            DistRow drow{};
            if constexpr (DM) drow = dist_row(J.dt, (double)T2);

            // c_k,a = conj(F_k) y_a e^{i m_a phi}: Re(c Q) = cr Q.re - cm Q.im
            TA cr[K][NM], cm[K][NM];
#pragma unroll
            for (int k = 0; k < K; k++) {
                static_for<0, NM>([&](auto A_) {
                    constexpr int a = decltype(A_)::value;
                    constexpr int m = kSets[S].m[a];
                    const TA er = (TA)Er[m < 0 ? -m : m];
                    const TA ei = (m < 0) ? -(TA)Ei[-m] : (TA)Ei[m];
                    const TA zr = (TA)y[a] * er, zi = (TA)y[a] * ei;
                    cr[k][a] = (TA)Fr[k] * zr + (TA)Fi[k] * zi;
                    cm[k][a] = (TA)Fr[k] * zi - (TA)Fi[k] * zr;
                });
            }
            // per detector: base index, five-tap weights per sub-step r, and
            // the lattice steps q for which every detector's stencil is inside
            int i0[K];
            TA w5[K][R][5];
            int qmin[R], qmax[R];
#pragma unroll
            for (int r = 0; r < R; r++) {
                qmin[r] = INT32_MIN / 2;
                qmax[r] = INT32_MAX / 2;
            }
#pragma unroll
            for (int k = 0; k < K; k++) {
                const TS fl = dfloor(uu[k]);
                // keep the base index representable; a sample this far out has no valid node
                const TS flc = fmin(fmax(fl, (TS)(-4 * T)), (TS)(4 * T));
                i0[k] = (int)flc;
                const TA f0 = (TA)(uu[k] - fl);
#pragma unroll
                for (int r = 0; r < R; r++) {
                    TA f = f0 + (TA)r / (TA)R;
                    const int c = f >= (TA)1 ? 1 : 0;
                    f -= (TA)c;
                    const TA fm1 = f - (TA)1, fm2 = f - (TA)2, fp1 = f + (TA)1;
                    const TA w0 = -f * fm1 * fm2 * (TA)(1.0 / 6.0);
                    const TA w1 = fp1 * fm1 * fm2 * (TA)0.5;
                    const TA w2 = -fp1 * f * fm2 * (TA)0.5;
                    const TA w3 = fp1 * f * fm1 * (TA)(1.0 / 6.0);
                    w5[k][r][0] = c ? (TA)0 : w0;
                    w5[k][r][1] = c ? w0 : w1;
                    w5[k][r][2] = c ? w1 : w2;
                    w5[k][r][3] = c ? w2 : w3;
                    w5[k][r][4] = c ? w3 : (TA)0;
                    // node (q, r) of detector k uses samples i0 + q + c - 1 .. i0 + q + c + 2
                    const int lo = 1 - i0[k] - c, hi = T - 3 - i0[k] - c;
                    qmin[r] = max(qmin[r], lo);
                    qmax[r] = min(qmax[r], hi);
                }
            }
            // nodes j = R q + r in [-jh, jh], and the steps at which every lane of
            // the wave has all its nodes
            int in_lo = INT32_MIN, in_hi = INT32_MAX;
#pragma unroll
            for (int r = 0; r < R; r++) {
                qmin[r] = max(qmin[r], -((jh + r) / R));
                qmax[r] = min(qmax[r], jh >= r ? (jh - r) / R : -1 - (r - jh - 1) / R);
                in_lo = max(in_lo, qmin[r]);
                in_hi = min(in_hi, qmax[r]);
            }
            // s in the units of the exponents
            TV se = (TV)s;
            if constexpr (kExp2) {
                se = (TV)((double)s * 1.4426950408889634074);
                if (!(se > (TV)0)) in_lo = INT32_MAX;   // D infinite: every step as one at an edge
                // (whatever lanes past the last sample give can only narrow the range)
#pragma unroll
                for (int m = 1; m < 64; m <<= 1) {
                    in_lo = max(in_lo, __shfl_xor(in_lo, m));
                    in_hi = min(in_hi, __shfl_xor(in_hi, m));
                }
                in_lo = __builtin_amdgcn_readfirstlane(in_lo);
                in_hi = __builtin_amdgcn_readfirstlane(in_hi);
            }
            // window G_k(i0 + q - 1 + t), t = 0..4: each step appends the
            // newest sample; the four steps before q_lo only fill the window
            // (their nodes lie below -tm_half and are masked)
            TA G[K][5];
#pragma unroll
            for (int k = 0; k < K; k++)
#pragma unroll
                for (int t = 0; t < 5; t++) G[k][t] = (TA)0;
            TV mx = (TV)-INFINITY;
            double sum = 0.0;
#pragma unroll 1
            for (int q = q_lo - 4; q <= q_hi; q++) {
                // The newest window row of the detectors.  In FP32, up to 27
                // complex values (3 detectors x 9 modes), every detector's row
                // is loaded before any is used: left to itself the allocator
                // recycled one destination register and waited for every
                // load in turn (37 against 24 ms, 256 x 2^16 samples, HLV 9
                // modes).  Larger sets, and FP64, go one detector at a time:
                // holding all their rows costs more registers than it saves.  Four
                // modes at a time, so that the row arrives in the order of its use
                // (the scheduler turned it round and waited for all of it: 16,384
                // samples, HL 21 modes, R = 1, 178 us against 147).
                constexpr int kGroup = (sizeof(TA) == 4 && K * NM <= 27) ? K : 1;
#pragma unroll
                for (int k0 = 0; k0 < K; k0 += kGroup) {
                    if constexpr (kGroup == 1) fence();
                    cpx<TA> qv[kGroup][NM];
#pragma unroll
                    for (int kk = 0; kk < kGroup; kk++) {
                        const int k = k0 + kk;
                        const int ic = min(max(i0[k] + q + 3, 0), T - 1);
                        // (a pointer that may be either would make both loads flat ones)
                        if (k < kGlobalDets) {
                            gcpx *qr = (gcpx *)Qg + ((size_t)k * T + ic) * NM;
                            static_for<0, NM>([&](auto A_) {
                                constexpr int a = decltype(A_)::value;
                                if constexpr (kGroup == 1 && a > 0 && a % 4 == 0) fence();
                                qv[kk][a].re = qr[a].re;
                                qv[kk][a].im = qr[a].im;
                            });
                        } else {
                            const cpx<TA> *qr = smem + ((size_t)(k - kGlobalDets) * T + ic) * NM;
                            static_for<0, NM>([&](auto A_) {
                                constexpr int a = decltype(A_)::value;
                                if constexpr (kGroup == 1 && a > 0 && a % 4 == 0) fence();
                                qv[kk][a] = qr[a];
                            });
                        }
                    }
#pragma unroll
                    for (int kk = 0; kk < kGroup; kk++) {
                        const int k = k0 + kk;
#pragma unroll
                        for (int t = 0; t < 4; t++) G[k][t] = G[k][t + 1];
                        TA g = (TA)0;
                        static_for<0, NM>([&](auto A_) {
                            constexpr int a = decltype(A_)::value;
                            g = fma(cr[k][a], qv[kk][a].re, g);
                            g = fma(-cm[k][a], qv[kk][a].im, g);
                        });
                        G[k][4] = g;
                    }
                }
                if constexpr (kExp2) {
                    TV t1[R];
                    TV tm = -FLT_MAX;
#pragma unroll
                    for (int r = 0; r < R; r++) {
                        TA v = (TA)0;
#pragma unroll
                        for (int k = 0; k < K; k++)
#pragma unroll
                            for (int t = 0; t < 5; t++) v = fma(w5[k][r][t], G[k][t], v);
                        // a NaN or -inf counts as no node: its exponential is 0
                        t1[r] = fmax(v, -FLT_MAX);
                    }
                    const bool edge = q < in_lo || q > in_hi;   // (the same for the wave)
                    if (edge) {
#pragma unroll
                        for (int r = 0; r < R; r++)
                            t1[r] = q >= qmin[r] && q <= qmax[r] ? t1[r] : -FLT_MAX;
                    }
#pragma unroll
                    for (int r = 0; r < R; r++) tm = fmax(tm, t1[r]);
                    const TV xm = se * tm;
                    if (xm > mx + kStride && tm > -FLT_MAX) {
                        asm volatile("");   // a branch: not the exponential and the product at every step
                        sum = (mx > -INFINITY) ? sum * (double)__builtin_amdgcn_exp2f(mx - xm) : 0.0;
                        mx = xm;
                    }
                    TV part = (TV)0;
                    if (edge) {
#pragma unroll
                        for (int r = 0; r < R; r++)
                            part += t1[r] > -FLT_MAX ? __builtin_amdgcn_exp2f(fma(se, t1[r], -mx)) : (TV)0;
                    } else {
#pragma unroll
                        for (int r = 0; r < R; r++) part += __builtin_amdgcn_exp2f(fma(se, t1[r], -mx));
                    }
                    sum += (double)part;
                } else {   // (node values in FP64)
                    TV x[R];
                    TV cmax = (TV)-INFINITY;
#pragma unroll
                    for (int r = 0; r < R; r++) {
                        const bool valid = q >= qmin[r] && q <= qmax[r];
                        TA t1 = (TA)0;
#pragma unroll
                        for (int k = 0; k < K; k++)
#pragma unroll
                            for (int t = 0; t < 5; t++) t1 = fma(w5[k][r][t], G[k][t], t1);
                        if constexpr (DM)
                            x[r] = valid ? dist_at(J.dt, drow, (double)t1) : -INFINITY;
                        else
                            x[r] = valid ? s * t1 : (TA)-INFINITY;
                        cmax = fmax(cmax, x[r]);
                    }
                    if (cmax > mx) {
                        sum = (mx > -INFINITY) ? sum * exp(mx - cmax) : 0.0;
                        mx = cmax;
                    }
                    double part = 0.0;
#pragma unroll
                    for (int r = 0; r < R; r++) part += (x[r] > -INFINITY) ? exp(x[r] - mx) : 0.0;
                    sum += part;
                }
            }
            if constexpr (!kT2First) {
                // the table pointers look redefined here, so the scalar loads
                // of the pair tables are not hoisted over the time loop
                fence();
                asm volatile("" : "+s"(Ut), "+s"(Vt));
                T2 = LK::template quad_T2<false>(Fr, Fi, y, Er, Ei, Ut, Vt);
            }
            double lnLt = -INFINITY;
            if constexpr (DM) {
                if (ok && mx > -INFINITY) lnLt = (double)mx + log(sum) + J.tm_lnw;
            } else {
                if (ok && mx > (TA)-INFINITY)
                    lnLt = (double)mx * (kExp2 ? 0.69314718055994530942 : 1.0) + log(sum) -
                           (double)(s * s * T2 * (TA)0.25) + J.tm_lnw;
            }
            const TO outv = (TO)lnLt;
            if (outL) outL[i] = outv;
            if (outW) outW[i] = outv + (lr ? (TO)lr[i] : (TO)0);
        }
    }
};

// --------------------------------------- FP64: samples by rounds of sixteen
// The same sums with the window read once per sixteen samples instead of once
// per sample, and with lanes along time.  Sixteen samples form the columns of a
// matrix product over the window times they share,
//   G_k(i, n) = sum_a Re[ c_k,a(n) Q_k,a(i) ]       (window time i, sample n),
// on the matrix cores (v_mfma_f64_16x16x4: 16 times x 16 samples, four of the
// 2 NM real products per instruction), one detector after the other into LDS;
// then a wave takes a sample at a time, each lane a lattice step and the five G
// of its stencil from consecutive LDS words.
// With a sample per lane instead, a step gathers 64 window rows of 16 NM bytes,
// one cache line at a time, the registers allow one wave per SIMD and there are
// only samples / 64 waves.  HLV 9 modes, R = 4, whole step: 4 x 8,191 samples
// 375 us with a sample per lane, 144 by rounds.  In FP32 the same scheme (with
// the interpolation on the matrix cores too) took 451 us against 391 with a
// sample per lane (16 x 16,384 samples): its rows are half as long, two waves
// fit a SIMD, and the matrix products are 1.6 times those that the samples
// need (the times that sixteen scattered samples share), so FP32 keeps the
// sample per lane.  So does the 5-mode set with one node per step, where the
// rounds have too little to do between their barriers (8 x 65,536 samples, HL:
// 892 us against 717).
//
// A block of eight waves sets up sr samples (a sample per lane, a detector per
// wave: c_k,a, stencil position, part of T2) in LDS, runs them in rounds of
// sixteen, two samples per wave, and passes of tm_chunks x 64 steps, and forms
// the logarithms and stores with a lane per sample again.  A sample's value
// depends on its own column only, whichever samples share its round.
//
// Rows of G: row p is window time ib + p, ib the first time that a sample of
// the round needs; times outside the window (-1 and T at most) repeat the
// nearest one and meet weights of zero.  The light travel time between the
// detector and the geocentre bounds the samples' spread, and with the pass
// length the rows to allocate.
template <int C, int RM>
__device__ __forceinline__ double dpp_row(double old, double v) {
    const int2 o = __builtin_bit_cast(int2, old), x = __builtin_bit_cast(int2, v);
    int2 r;
    r.x = __builtin_amdgcn_update_dpp(o.x, x.x, C, RM, 0xf, false);
    r.y = __builtin_amdgcn_update_dpp(o.y, x.y, C, RM, 0xf, false);
    return __builtin_bit_cast(double, r);
}
// Reduction over the 64 lanes, in every lane: row_shr 1, 2, 4, 8, then the row
// broadcasts; none: the value that changes nothing.
template <class F>
__device__ __forceinline__ double wave_fold(double v, const double none, F f) {
    v = f(v, dpp_row<0x111, 0xf>(none, v));
    v = f(v, dpp_row<0x112, 0xf>(none, v));
    v = f(v, dpp_row<0x114, 0xf>(none, v));
    v = f(v, dpp_row<0x118, 0xf>(none, v));
    v = f(v, dpp_row<0x142, 0xa>(none, v));
    v = f(v, dpp_row<0x143, 0xc>(none, v));
    int2 x = __builtin_bit_cast(int2, v);
    x.x = __builtin_amdgcn_readlane(x.x, 63);
    x.y = __builtin_amdgcn_readlane(x.y, 63);
    return __builtin_bit_cast(double, x);
}

typedef double tm_d4 __attribute__((ext_vector_type(4)));

template <int S, int K, int R, bool DM>
struct TmargRounds {
    using LK = LnlKernel<S, K, kFP64, false, false>;
    using ccpx = typename LK::ccpx;
    typedef __attribute__((address_space(1))) const double gdouble;
    static constexpr int NM = LK::NM;
    static constexpr int NE = LK::NE;
    static constexpr int N2 = 2 * NM;                // real products per G
    static constexpr int EK = (N2 + 3) / 4;          // matrix instructions per tile
    static constexpr int kOver = 4 * EK - N2;
    static constexpr int kAhead = 2;   // tiles of a wave whose rows are in flight
    static constexpr int PER = kTmCols / kTmWaves;   // samples of a wave per round
    static constexpr int CS = K * N2 + 1;            // a sample's coefficients; odd against bank conflicts
    static constexpr int kNever = 1 << 30;           // a lattice step past every pass
    static constexpr int kNone = -(1 << 30);         // i0 of a sample without a position

    // The LDS of a block (tm_lds_bytes).
    struct Lds {
        double *resS, *resM;   // [128] sums of exponentials, and the exponents' origins
        double *wtab;          // [16][K][5][R]
        double *f0s;           // [K][128]
        double *sv;            // [128] d_ref / D, NaN for a sample outside the support
        double *t2s;           // [K][128] parts of T2
        int *i0s;              // [K][128]
        int *rng;              // [K][8][2] least and largest i0 of a round
        int *qlim;             // [16][R][2] first and last step of the nodes
        double *coef;          // [sr][CS]: [K][N2]
        double *G;             // [16][gs], with coef before it and kTmPad values after it (see taps)
    };
    // T1 at a lane's nodes of a pass: steps qa + 64 c + lane.
    typedef double Nodes[kTmChunks][R];

    __device__ __forceinline__ static void run(const EvalJob *Jp, const int64_t begin, const int64_t end, char *smem,
                                               const int sr, const int gs) {
        const EvalJob &J = *Jp;
        const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int T = J.n_time, jh = J.tm_half;
        Lds L;
        L.resS = (double *)smem;
        L.resM = L.resS + kTmSetup;
        L.wtab = L.resM + kTmSetup;
        L.f0s = L.wtab + kTmCols * K * 5 * R;
        L.sv = L.f0s + K * kTmSetup;
        L.t2s = L.sv + kTmSetup;
        L.i0s = (int *)(L.t2s + K * kTmSetup);
        L.rng = L.i0s + K * kTmSetup;
        L.qlim = L.rng + K * (kTmSetup / kTmCols) * 2;
        L.coef = (double *)(L.qlim + kTmCols * R * 2);
        L.G = L.coef + sr * CS;
        gdouble *const Q = (gdouble *)J.Q;
        const double *__restrict__ th = (const double *)J.theta;
        const double *__restrict__ lr = (const double *)J.lnpmps;
        double *__restrict__ outL = (double *)J.lnL;
        double *__restrict__ outW = (double *)J.lw;
        const int64_t ld = J.ld;
        // lattice steps covering nodes -jh..jh (floor division)
        const int q_lo = -((jh + R - 1) / R), q_hi = jh / R;
        const int pass = 64 * J.tm_chunks;

        for (int64_t b0 = begin; b0 < end; b0 += sr) {
            const int ns = (int)(end - b0 < sr ? end - b0 : sr);
            // the job looks redefined here: what the set-up reads and derives
            // from it is not kept in registers over the rounds
            asm volatile("" : "+s"(Jp));
            __syncthreads();
            // a wave per detector and 64 samples
            const int sk = wave % K, t = wave / K * 64 + lane;
            if (t < sr) {
                int i0 = kNone;
                if (t < ns) i0 = setup(*Jp, th, ld, b0 + t, t, sk, L);
                L.i0s[sk * kTmSetup + t] = i0;
                int lo = i0 == kNone ? INT32_MAX : i0, hi = i0 == kNone ? INT32_MIN : i0;
#pragma unroll
                for (int m = 1; m < kTmCols; m <<= 1) {
                    lo = min(lo, __shfl_xor(lo, m));
                    hi = max(hi, __shfl_xor(hi, m));
                }
                if (t % kTmCols == 0) {
                    L.rng[(sk * (kTmSetup / kTmCols) + t / kTmCols) * 2] = lo;
                    L.rng[(sk * (kTmSetup / kTmCols) + t / kTmCols) * 2 + 1] = hi;
                }
            }
            __syncthreads();

            double mrun[PER], srun[PER];
            double a[kAhead][EK];
            int g = 0, qa = q_lo;   // the pass from lattice step qa of the round from sample g
            int ib, np;             // first window time of G, and how many
            extent(L, g, qa, 0, gs, T, q_hi, pass, ib, np);
            load_rows(Q, ib, np, T, lane, wave, a);
            bool more = true;
            while (more) {
                if (qa == q_lo) {
#pragma unroll
                    for (int i = 0; i < PER; i++) {
                        mrun[i] = -INFINITY;
                        srun[i] = 0.0;
                    }
                }
                // the pass after this one
                int ng = g, nqa = qa + pass;
                if (nqa > q_hi) {
                    nqa = q_lo;
                    ng += kTmCols;
                }
                more = ng < ns;
                const int nc = (min(pass - 1, q_hi - qa) >> 6) + 1;   // its chunks
                Nodes acc[PER];
                static_for<0, K>([&](auto K_) {
                    constexpr int k = decltype(K_)::value;
                    constexpr int kn = (k + 1) % K;
                    if (k == 0 && qa == q_lo) tables(g, T, jh, L);
                    rows(Q + (size_t)k * T * N2, L, g, k, gs, ib, np, T, lane, wave, a);
                    __syncthreads();
                    // the first window rows of the next G are in flight beside the use of this one
                    int nib = 0, nnp = 0;
                    if (kn || more) {
                        extent(L, kn ? g : ng, kn ? qa : nqa, kn, gs, T, q_hi, pass, nib, nnp);
                        load_rows(Q + (size_t)kn * T * N2, nib, nnp, T, lane, wave, a);
                    }
#pragma unroll
                    for (int i = 0; i < PER; i++) {
                        if constexpr (R > 1) fence();   // one sample's weights at a time
                        taps<k>(L, g, qa, wave * PER + i, gs, ib, np, nc, lane, acc[i]);
                    }
                    if constexpr (k == K - 1) {
                        constexpr int NB = R > 1 ? 1 : PER;
#pragma unroll
                        for (int i = 0; i < PER; i += NB) {
                            if constexpr (R > 1) fence();
                            nodes<NB>(J, L, g, qa, qa + pass - 1, wave * PER + i, nc, lane, acc + i, mrun + i, srun + i);
                        }
                        if (lane == 0 && qa + pass > q_hi) {
#pragma unroll
                            for (int i = 0; i < PER; i++) {
                                L.resM[g + wave * PER + i] = mrun[i];
                                L.resS[g + wave * PER + i] = srun[i];
                            }
                        }
                    }
                    ib = nib;
                    np = nnp;
                    __syncthreads();
                });
                g = ng;
                qa = nqa;
            }
            if (tid < ns) {
                const int64_t i = b0 + tid;
                const double mx = L.resM[tid], s = L.sv[tid];
                double lnLt = -INFINITY;
                if (s == s && mx > -INFINITY) {
                    lnLt = mx + log(L.resS[tid]);
                    if constexpr (!DM) lnLt -= s * s * total_T2(L, tid) * 0.25;
                    lnLt += J.tm_lnw;
                }
                if (outL) outL[i] = lnLt;
                if (outW) outW[i] = lnLt + (lr ? lr[i] : 0.0);
            }
        }
    }

    // Detector k's part of T1 at the nodes of the pass, column n (also for a
    // column without a sample: any rows, no result).
    template <int k>
    __device__ __forceinline__ static void taps(const Lds &L, const int g, const int qa, const int n, const int gs,
                                                const int ib, const int np, const int nc, const int lane,
                                                Nodes &acc) {
        // Lane q's stencil starts at row st0 + q of its column.  Rows outside the
        // column belong to nodes outside the window or the pass and may hold
        // anything: the start is only kept so that every address is inside the
        // block's LDS (from a start below -260 no lane reaches the column).
        const int i0 = __builtin_amdgcn_readfirstlane(L.i0s[k * kTmSetup + g + n]);
        const int st0 = min(max(i0 + qa - 1 - ib, -(64 * kTmChunks + 4)), np);
        const double *w = L.wtab + (n * K + k) * 5 * R;
        const double *gp = L.G + n * gs + st0 + lane;
        double wr[5][R];
#pragma unroll
        for (int t = 0; t < 5; t++)
#pragma unroll
            for (int r = 0; r < R; r++) wr[t][r] = w[t * R + r];
#pragma unroll
        for (int c = 0; c < kTmChunks; c++) {
            if constexpr (k == 0) {
#pragma unroll
                for (int r = 0; r < R; r++) acc[c][r] = 0.0;
            }
            // (the branch also keeps the registers to one chunk's at a time)
            if (R > 1 && c >= nc) continue;
#pragma unroll
            for (int t = 0; t < 5; t++) {
                const double gv = gp[64 * c + t];
#pragma unroll
                for (int r = 0; r < R; r++) acc[c][r] = fma(wr[t][r], gv, acc[c][r]);
            }
        }
    }

    // Node values of a pass, their maximum and the sum of their exponentials,
    // for NB of a wave's samples in step.  One node per step: both samples, and
    // no branch between the chunks (the exponentials are latency-bound: 1,645 to
    // 1,484 us, 8 x 65,536 samples, HLV 9 modes).  Four nodes per step: one sample and
    // one chunk at a time, for the registers.
    template <int NB>
    __device__ __forceinline__ static void nodes(const EvalJob &J, const Lds &L, const int g, const int qa,
                                                 const int q_end, const int n0, const int nc, const int lane, Nodes *x,
                                                 double *mrun, double *srun) {
        const int ncb = R > 1 ? nc : kTmChunks;
        double s[NB], m[NB], sum[NB];
        bool any[NB], plain[NB];
#pragma unroll
        for (int i = 0; i < NB; i++) {
            const int *ql = L.qlim + (n0 + i) * R * 2;
            int lo[R], sp[R];
            int in_lo = INT32_MIN, in_hi = INT32_MAX;   // steps with every node inside
#pragma unroll
            for (int r = 0; r < R; r++) {
                lo[r] = __builtin_amdgcn_readfirstlane(ql[2 * r]);
                const int hi = min(__builtin_amdgcn_readfirstlane(ql[2 * r + 1]), q_end);
                if (hi < lo[r]) lo[r] = kNever;
                sp[r] = max(hi - lo[r], 0);
                in_lo = max(in_lo, lo[r]);
                in_hi = min(in_hi, hi);
            }
            s[i] = L.sv[g + n0 + i];
            DistRow drow{};
            if constexpr (DM) {
                drow = dist_row(J.dt, total_T2(L, g + n0 + i));
                s[i] = s[i] == s[i] ? 1.0 : s[i];
            }
            m[i] = -INFINITY;
#pragma unroll
            for (int c = 0; c < kTmChunks; c++) {
                if (c >= ncb) break;
                const int q0 = qa + 64 * c;
                if constexpr (DM) {
#pragma unroll
                    for (int r = 0; r < R; r++) x[i][c][r] = dist_at(J.dt, drow, x[i][c][r]);
                }
                if (R == 1 || q0 < in_lo || q0 + 63 > in_hi) {
#pragma unroll
                    for (int r = 0; r < R; r++)
                        x[i][c][r] = (unsigned)(q0 + lane - lo[r]) <= (unsigned)sp[r] ? x[i][c][r] : -INFINITY;
                }
#pragma unroll
                for (int r = 0; r < R; r++) m[i] = fmax(m[i], x[i][c][r]);
            }
        }
#pragma unroll
        for (int i = 0; i < NB; i++) {
            m[i] = wave_fold(m[i], -INFINITY, [](double a, double b) { return fmax(a, b); });
            // false: no node, none with a value, or a sample outside the support
            any[i] = m[i] > -INFINITY && s[i] == s[i];
            m[i] = fmax(any[i] ? s[i] * m[i] : -INFINITY, mrun[i]);
            plain[i] = !any[i];
        }
        bool again;
#pragma unroll 1
        do {
#pragma unroll
            for (int i = 0; i < NB; i++) {
                sum[i] = 0.0;
#pragma unroll
                for (int c = 0; c < kTmChunks; c++) {
                    if (c >= ncb) break;
#pragma unroll
                    for (int r = 0; r < R; r++) sum[i] += exp(fma(s[i], x[i][c][r], -m[i]));
                }
            }
#pragma unroll
            for (int i = 0; i < NB; i++) sum[i] = wave_fold(sum[i], 0.0, [](double a, double b) { return a + b; });
            again = false;
#pragma unroll
            for (int i = 0; i < NB; i++) {
                if (sum[i] == sum[i] || plain[i]) continue;
                // a node's value is NaN (it counts as no node), or D is so small or so
                // large that s is infinite or zero: once more on plain values
#pragma unroll
                for (int c = 0; c < kTmChunks; c++) {
                    if (c >= ncb) break;
#pragma unroll
                    for (int r = 0; r < R; r++) {
                        const double v = s[i] * x[i][c][r];
                        x[i][c][r] = v > -INFINITY ? v : -INFINITY;
                    }
                }
                s[i] = 1.0;
                plain[i] = true;
                again = true;
            }
        } while (again);
#pragma unroll
        for (int i = 0; i < NB; i++) {
            if (!any[i]) continue;
            if (m[i] > mrun[i] && mrun[i] > -INFINITY) srun[i] *= exp(mrun[i] - m[i]);
            mrun[i] = m[i];
            srun[i] += sum[i];
        }
    }

    __device__ __forceinline__ static double total_T2(const Lds &L, const int t) {
        double T2 = L.t2s[t];
#pragma unroll
        for (int k = 1; k < K; k++) T2 += L.t2s[k * kTmSetup + t];
        return T2;
    }

    // Window times ib .. ib + np - 1 that the samples of a pass need of detector k.
    __device__ __forceinline__ static void extent(const Lds &L, const int g, const int qa, const int k, const int gs,
                                                  const int T, const int q_hi, const int pass, int &ib, int &np) {
        const int *u = L.rng + (k * (kTmSetup / kTmCols) + g / kTmCols) * 2;
        const int lo = __builtin_amdgcn_readfirstlane(u[0]), hi = __builtin_amdgcn_readfirstlane(u[1]);
        const int qb = min(qa + pass - 1, q_hi);
        ib = lo > hi ? T - 4 : min(max(lo + qa - 1, -1), T - 4);
        const int ie = lo > hi ? T : max(min(hi + qb + 3, T), ib + 4);
        np = min(ie - ib + 1, gs - 4);
    }

    // One sample per lane and one detector per wave: coefficients, stencil
    // position (returned: its integer part), distance factor, the detector's
    // part of T2.  (Every wave forms the whole geometry; the quadratic form is
    // the longer part, and a block waits for its set-up.)
    __device__ __forceinline__ static int setup(const EvalJob &J, const double *th, const int64_t ld, const int64_t i,
                                                const int t, const int k, const Lds &L) {
        const int T = J.n_time;
        const double al = th[i], de = th[ld + i], DD = th[3 * ld + i];
        const double ci = th[4 * ld + i], ph = th[5 * ld + i], ps = th[6 * ld + i];
        const bool ok = DD > 0.0 && ci >= -1.0 && ci <= 1.0;
        double Fr[K], Fi[K], uu[K], y[NM], Er[NE], Ei[NE];
        LK::geometry(J, al, de, 0.0, ci, ph, ps, Fr, Fi, uu, y, Er, Ei);
        double fr[1] = {Fr[0]}, fi[1] = {Fi[0]}, u = uu[0];
#pragma unroll
        for (int j = 1; j < K; j++) {
            fr[0] = j == k ? Fr[j] : fr[0];
            fi[0] = j == k ? Fi[j] : fi[0];
            u = j == k ? uu[j] : u;
        }
        if (k == 0) L.sv[t] = ok ? J.d_ref / DD : NAN;
        // c_a = conj(F) y_a e^{i m_a phi}: Re(c Q) = cr Q.re - cm Q.im
        double *const c = L.coef + t * CS + k * N2;
        static_for<0, NM>([&](auto A_) {
            constexpr int a = decltype(A_)::value;
            constexpr int m = kSets[S].m[a];
            const double er = Er[m < 0 ? -m : m], ei = (m < 0) ? -Ei[-m] : Ei[m];
            const double zr = y[a] * er, zi = y[a] * ei;
            c[2 * a] = fr[0] * zr + fi[0] * zi;
            c[2 * a + 1] = -(fr[0] * zi - fi[0] * zr);
        });
        const double fl = dfloor(u);
        // keep the base index representable; a sample this far out has no valid node
        const double flc = fmin(fmax(fl, (double)(-4 * T)), (double)(4 * T));
        L.f0s[k * kTmSetup + t] = u - fl;
        fence();
        L.t2s[k * kTmSetup + t] = LK::template quad_T2<true, 1>(fr, fi, y, Er, Ei, (ccpx *)J.Ut + k, (ccpx *)J.Vt + k);
        return u == u ? (int)flc : kNone;
    }

    // Five-tap weights of every (detector, sample, sub-step) of the round, one
    // per thread, and by the last threads the lattice steps (first, last) whose
    // stencils are inside the window in every detector and whose nodes are
    // inside the time prior.
    __device__ __forceinline__ static int tap_split(const double f0, const int r, double &f) {
        f = f0 + (double)r / (double)R;
        const int c = f >= 1.0 ? 1 : 0;
        f -= (double)c;
        return c;
    }
    __device__ __forceinline__ static void tables(const int g, const int T, const int jh, const Lds &L) {
        const int tid = threadIdx.x;
        if (tid < K * kTmCols * R) {
            const int r = tid % R, n = tid / R % kTmCols, k = tid / (R * kTmCols);
            double f;
            const int c = tap_split(L.f0s[k * kTmSetup + g + n], r, f);
            const double fm1 = f - 1.0, fm2 = f - 2.0, fp1 = f + 1.0;
            const double w0 = -f * fm1 * fm2 * (1.0 / 6.0), w1 = fp1 * fm1 * fm2 * 0.5;
            const double w2 = -fp1 * f * fm2 * 0.5, w3 = fp1 * f * fm1 * (1.0 / 6.0);
            double *w = L.wtab + (n * K + k) * 5 * R + r;
            w[0] = c ? 0.0 : w0;
            w[R] = c ? w0 : w1;
            w[2 * R] = c ? w1 : w2;
            w[3 * R] = c ? w2 : w3;
            w[4 * R] = c ? w3 : 0.0;
        }
        const int t0 = tid - (kTmWaves * 64 - kTmCols * R);
        if (t0 >= 0) {
            const int n = t0 / R, r = t0 % R;
            // nodes j = R q + r in [-jh, jh]
            int lo = -((jh + r) / R), hi = jh >= r ? (jh - r) / R : -1 - (r - jh - 1) / R;
#pragma unroll
            for (int k = 0; k < K; k++) {
                // node (q, r) of detector k uses samples i0 + q + c - 1 .. i0 + q + c + 2
                const int i0 = L.i0s[k * kTmSetup + g + n];
                double f;
                const int c = tap_split(L.f0s[k * kTmSetup + g + n], r, f);
                lo = i0 == kNone ? kNever : max(lo, 1 - i0 - c);
                hi = i0 == kNone ? -kNever : min(hi, T - 3 - i0 - c);
            }
            L.qlim[(n * R + r) * 2] = lo;
            L.qlim[(n * R + r) * 2 + 1] = hi;
        }
    }

    // The window rows of a tile of sixteen times from time row0: lane l holds
    // products first_product(l) .. + EK - 1 of time l % 16.  The last lane
    // group's run ends with the row, so that its first kOver products are the
    // group before's again: cleared at their use.
    __device__ __forceinline__ static int first_product(const int lane) { return min((lane >> 4) * EK, N2 - EK); }
    __device__ __forceinline__ static void load_tile(gdouble *Qk, const int row0, const int T, const int lane,
                                                     double (&a)[EK]) {
        const unsigned row = min(max(row0 + (lane & 15), 0), T - 1);
        gdouble *q = Qk + (row * (unsigned)N2 + (unsigned)first_product(lane));
#pragma unroll
        for (int s = 0; s < EK; s++) a[s] = q[s];
    }
    // The rows of a wave's first tiles, to be in flight before their use.
    __device__ __forceinline__ static void load_rows(gdouble *Qk, const int ib, const int np, const int T,
                                                     const int lane, const int wave, double (&a)[kAhead][EK]) {
#pragma unroll
        for (int j = 0; j < kAhead; j++)
            if (16 * (wave + j * kTmWaves) < np) load_tile(Qk, ib + 16 * (wave + j * kTmWaves), T, lane, a[j]);
    }
    // G_k of the round's columns at window times ib .. ib + np - 1, a wave per
    // tile of sixteen times, kAhead tiles' rows ahead (in a).
    __device__ __forceinline__ static void rows(gdouble *Qk, const Lds &L, const int g, const int k, const int gs,
                                                const int ib, const int np, const int T, const int lane,
                                                const int wave, double (&a)[kAhead][EK]) {
        const int col = lane & 15;
        const bool last = lane >= 48;
        const double *cf = L.coef + (g + col) * CS + k * N2 + first_product(lane);
        double b[EK];
#pragma unroll
        for (int s = 0; s < EK; s++) b[s] = s < kOver && last ? 0.0 : cf[s];
        for (int p0 = wave * 16; p0 < np; p0 += 16 * kAhead * kTmWaves) {
#pragma unroll
            for (int j = 0; j < kAhead; j++) {
                const int p = p0 + 16 * kTmWaves * j;
                if (p >= np) break;
                tm_d4 d = tm_d4{0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < EK; s++) {
                    const double v = s < kOver && last ? 0.0 : a[j][s];
                    d = __builtin_amdgcn_mfma_f64_16x16x4f64(v, b[s], d, 0, 0, 0);
                }
                if (p + 16 * kAhead * kTmWaves < np) load_tile(Qk, ib + p + 16 * kAhead * kTmWaves, T, lane, a[j]);
                // D: column lane % 16, rows lane / 16 + 4 r
#pragma unroll
                for (int r = 0; r < 4; r++) L.G[col * gs + p + (lane >> 4) + 4 * r] = d[r];
            }
        }
    }
};

template <int S, int K, int R, bool DM>
__global__ void __launch_bounds__(kTmWaves * 64)
    k_tmarg_rounds(const EvalJob *__restrict__ jobs, const Tile *__restrict__ tiles, int sr, int gs) {
    extern __shared__ __align__(16) char ile_smem[];
    const Tile tl = tiles[blockIdx.x];
    TmargRounds<S, K, R, DM>::run(jobs + tl.job, tl.begin, tl.end, ile_smem, sr, gs);
}

template <int S, int K, int POL, bool LDS, int R, bool DM>
__global__ void __launch_bounds__(tmarg_block_threads(POL), 1)
    k_lnl_tmarg(const EvalJob *__restrict__ jobs, const Tile *__restrict__ tiles) {
    extern __shared__ __align__(16) char ile_smem[];
    using TA = typename PolTypes<POL>::TA;
    const Tile tl = tiles[blockIdx.x];
    TmargKernel<S, K, POL, LDS, R, DM>::run(jobs[tl.job], tl.begin, tl.end, (cpx<TA> *)ile_smem);
}

// Launch the time-marginalised kernel of mode set S and policy POL (FP32 or
// FP64) for oversampling R in {1, 4}, with the distance integrated (dm) or not:
// a sample per lane, with lds_bytes the window staged in LDS, or with gs > 0
// (where tm_rounds) by rounds of sixteen, sr samples set up at a time and gs values
// of G per sample.
template <int S, int POL>
hipError_t launch_tmarg_sp(int kdet, int R, bool dm, size_t lds_bytes, int sr, int gs, const EvalJob *jobs,
                           const Tile *tiles, int n_tiles, int nthreads, hipStream_t st) {
    if (n_tiles <= 0) return hipSuccess;
    auto go = [&](auto KK, auto RR, auto DD) -> hipError_t {
        constexpr int K = decltype(KK)::value;
        constexpr int RV = decltype(RR)::value;
        constexpr bool DMV = decltype(DD)::value;
        if (gs > 0) {
            if constexpr (tm_rounds(S, POL, RV, DMV)) {
                if (nthreads != kTmWaves * 64 || sr < kTmCols || sr > kTmSetup || sr % kTmCols ||
                    lds_bytes < tm_lds_bytes(S, K, RV, sr, gs))
                    return hipErrorInvalidValue;
                auto fn = k_tmarg_rounds<S, K, RV, DMV>;
                hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   (int)lds_bytes);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(fn, dim3(n_tiles), dim3(nthreads), lds_bytes, st, jobs, tiles, sr, gs);
                return hipGetLastError();
            } else {
                return hipErrorInvalidValue;
            }
        }
        if (nthreads <= 0 || nthreads > tmarg_block_threads(POL) || nthreads % 64) return hipErrorInvalidValue;
        if (lds_bytes > 0) {
            if constexpr (tmarg_lds_compiled(S, K, POL, RV, DMV)) {
                auto fn = k_lnl_tmarg<S, K, POL, true, RV, DMV>;
                hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   (int)lds_bytes);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(fn, dim3(n_tiles), dim3(nthreads), lds_bytes, st, jobs, tiles);
                return hipGetLastError();
            } else {
                return hipErrorInvalidValue;
            }
        }
        hipLaunchKernelGGL((k_lnl_tmarg<S, K, POL, false, RV, DMV>), dim3(n_tiles), dim3(nthreads), 0, st, jobs, tiles);
        return hipGetLastError();
    };
    using T2 = std::integral_constant<int, 2>;
    using T3 = std::integral_constant<int, 3>;
    using R1 = std::integral_constant<int, 1>;
    using R4 = std::integral_constant<int, 4>;
    if (R != 1 && R != 4) return hipErrorInvalidValue;
    auto go_r = [&](auto KK) -> hipError_t {
        if (R == 1) return dm ? go(KK, R1{}, std::true_type{}) : go(KK, R1{}, std::false_type{});
        return dm ? go(KK, R4{}, std::true_type{}) : go(KK, R4{}, std::false_type{});
    };
    if (kdet == 2) return go_r(T2{});
    if (kdet == 3) return go_r(T3{});
    return hipErrorInvalidValue;
}

}  // namespace ile
