// The windowed-FFT and the decimated route for Q of eq. (QUV) (k_qv.hip); the
// direct route's launcher is declared with the other kernels.  Every route
// takes the band as the bins m_lo .. m_lo + n_half - 1 (0 <= m <= n / 2) and
// their mirrors n - m.
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

namespace ile {

// The radix R of the decimated route for a grid of n bins, a band of n_band
// bins and the window (n_time, win_half): of the R in {2, 4, 8, 16} that
// divide n and put the window on at most 64 decimated times
// floor((i - win_half) / R) (one 32- or 64-row time tile), the one of lowest
// estimated cost, or 0 when there is none.  With `force` false it is also 0
// when that cost exceeds the direct sum's.
int qv_radix(int64_t n, int64_t n_band, int n_time, int win_half, bool force);

// Whether the windowed-FFT route applies (n a multiple of its 512-point
// transforms, its launches within a grid) and its estimated cost is below the
// direct sum's; its scratch; Q by this route, U and V.
bool qv_win_ok(int64_t n, int64_t n_band, int64_t cols, int n_time);
size_t qv_win_scratch_bytes(int64_t n, int64_t n_half, int na, int nd, int np, int n_time);
hipError_t launch_qv_win(const void *hlm, const void *data, const double *inv_psd, int64_t n, int na, int nd, int np,
                         double df, int64_t m_lo, int64_t n_half, int n_time, int win_half, void *Q, void *U, void *V,
                         void *scratch, hipStream_t st);

// Band slices of the decimated route's matrix-core stage and its scratch
// (twiddles, the radix-R partial sums and the slice partials, each 256-byte
// aligned).
int qv_dec_slices(int64_t n, int64_t cols, int n_time, int win_half, int radix);
size_t qv_dec_scratch_bytes(int64_t n, int64_t cols, int n_time, int win_half, int radix, int n_slices);

// Q (decimated route), U and V.  The band is f_lo <= |m' df| <= f_hi (m' the
// signed index), tested on the device with the host's expression.
hipError_t launch_qv_dec(const void *hlm, const void *data, const double *inv_psd, int64_t n, int na, int nd,
                         int np, double df, double f_lo, double f_hi, int64_t m_lo, int64_t n_half, int n_time,
                         int win_half, int radix, void *Q, void *U, void *V, void *scratch,
                         int n_slices, hipStream_t st);

}  // namespace ile
