// Pieces the FFT-score kernels share: launch arguments, complex arithmetic, the
// centred samples of a sequence, and a lag's D(T) (or score) from its
// autocorrelation.  Included only by translation units compiled with
// -ffp-contract=off.
#pragma once

#include "internal.h"

namespace gpoeo {
namespace {

struct FftArgs {
    const float* x;
    const double* fstat;       // [S][4]: mean, sum y^2, sum |y|, unused (window statistics)
    double* edge;              // [S][tmax + 1]: E1(T) + E2(T)
    const double2* tw;         // twiddle tables
    double* l1;                // column kernel: partial sums of |y| by wavefront, or null
    double2* tw_out;           // the edge kernel's extra workgroups write W_4096^e here, or null
    double2* z;                // [pairs][len]
    double* part;              // [S][lags]: D(T)
    double* amp;               // spectra: [S][len/2 + 1] amplitudes |X_s(k)|
    int64_t seqs;              // S = B * C
    int64_t n_all, window_stride, channel_stride;
    int64_t len;
    int64_t tw_a, tw_b, tw_lo, tw_hi;
    int32_t num_channels;
    int32_t tmin, tmax, lags;
    int32_t lg, lg1, lg2, lgc, lgr;
    WindowTable tab;
    int64_t zstride;           // transform z of pair p sits at z + p * zstride
    // Loads of a transform see samples [seg_start, seg_start + seg_len) of
    // each sequence (seg_len 0: all of it): the heads and tails of the wrap
    // correction.
    int64_t seg_start, seg_len;
    // Wrap correction: the inverse column kernel of the head-tail transform
    // writes the cross-correlations cc(s), s < wm, to wout ([S][wm]); the one
    // of the main transform subtracts wrap[s][Tmax - T] from r(T) for T > wrap_w.
    double* wout;
    const double* wrap;
    int64_t wrap_w;
    int32_t wm;
    // Fused finalisation (one channel, uniform batch): S(T) to s64 and scores.
    double* s64;
    float* scores;
    float w0;
};

__device__ __forceinline__ double2 cadd(double2 a, double2 b) {
    return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 csub(double2 a, double2 b) {
    return make_double2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmul_conj(double2 a, double2 b) {   // a * conj(b)
    return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
struct Seq {
    const float* p;
    int64_t n;
    double mu;
};

__device__ __forceinline__ Seq seq_of(const FftArgs& a, int64_t s) {
    Seq q;
    if (s >= a.seqs) {
        q.p = nullptr;
        q.n = 0;
        q.mu = 0.0;
        return q;
    }
    const int64_t b = s / a.num_channels;
    const int64_t c = s % a.num_channels;
    q.n = table_n(a.tab, b, a.n_all);
    q.p = a.x + table_off(a.tab, b, a.window_stride) + c * a.channel_stride;
    q.mu = a.fstat[4 * s];
    if (a.seg_len > 0) {
        q.p += a.seg_start;
        q.n = min(q.n - a.seg_start, a.seg_len);
    }
    return q;
}

__device__ __forceinline__ double centred(const Seq& q, int64_t i) {
    return i < q.n ? (double)q.p[i] - q.mu : 0.0;
}

// E1(T) + E2(T) of sequence s: the energies of its first and last N - T samples
// (0 for a lag that write_lag leaves out or an empty slot).
__device__ __forceinline__ double lag_energy(const FftArgs& a, int64_t s, int64_t t) {
    if (s >= a.seqs || t < a.tmin || t > a.tmax) return 0.0;
    const int64_t b = s / a.num_channels;
    if (table_n(a.tab, b, a.n_all) <= 0 || t > table_tmax(a.tab, b, a.tmax)) return 0.0;
    return a.edge[s * (int64_t)(a.tmax + 1) + t];
}

// D(T) of sequence s from its energies and the scaled inverse transform value
// w = 4 L r(T).
__device__ __forceinline__ void write_lag(const FftArgs& a, int64_t s, int64_t t, double energy,
                                          double w) {
    if (s >= a.seqs || t < a.tmin || t > a.tmax) return;
    const int64_t b = s / a.num_channels;
    const int64_t n = table_n(a.tab, b, a.n_all);
    const bool live = n > 0 && t <= table_tmax(a.tab, b, a.tmax);
    double d = 0.0;
    if (live) {
        double r = ldexp(w, -(a.lg + 2));
        if (a.wrap && t > a.wrap_w) r -= a.wrap[s * a.wm + (a.tmax - t)];   // circular term
        d = energy - 2.0 * r;
    }
    const int64_t k = s * a.lags + (t - a.tmin);
    if (a.s64) {   // the finalisation of a single channel, in its own arithmetic
        if (!live && !a.scores) return;   // past a table window's lags: left unwritten
        const double v = 0.0 + (double)a.w0 * (d / (double)(n - t));
        a.s64[k] = v;
        if (a.scores) a.scores[k] = (float)v;
    } else {
        a.part[k] = d;
    }
}
__device__ __forceinline__ void write_d(const FftArgs& a, int64_t s, int64_t t, double w) {
    write_lag(a, s, t, lag_energy(a, s, t), w);
}

}  // namespace
}  // namespace gpoeo
