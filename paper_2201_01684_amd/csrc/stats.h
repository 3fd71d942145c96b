// Window statistics helpers shared by the statistics kernel and the fused
// small-window kernel, so that both compute the same bits: a fixed visiting
// order of a window's samples and fixed-order merges.  Every translation unit
// that includes this header is compiled with -ffp-contract=off.
#pragma once

#include "internal.h"

namespace gpoeo {
namespace stats {

constexpr int kStatsThreads = 256;          // the fused kernel, and windows it could take
constexpr int kStatsLongThreads = 1024;     // longer windows

// Count, mean and sum of squared deviations of a set of samples.
struct Moments {
    double n, mean, m2;
};

// 1 / x of a whole number x >= 1 (the hardware estimate refined by two Newton
// steps): a chain half as long as the division's.
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// Moments of two sets together (Chan, Golub and LeVeque's pairwise update).
__device__ __forceinline__ Moments merge(const Moments& a, const Moments& b) {
    if (b.n == 0.0) return a;
    if (a.n == 0.0) return b;
    const double n = a.n + b.n;
    const double f = b.n * recip(n);
    const double d = b.mean - a.mean;
    Moments r;
    r.n = n;
    r.mean = a.mean + d * f;
    r.m2 = (a.m2 + b.m2) + d * d * (a.n * f);
    return r;
}

// Mean, population variance and mean |x| of one channel of one window, as
// written by the statistics kernel (var[0] = variance, var[1] = mean |x|); also
// the sum of squared deviations and a bound of the sum of absolute ones, at
// most sqrt(n) times its root (fstat).  Every thread of the kT-wide workgroup
// returns the same values; red holds 4 kT / 64 doubles.
//
// One pass: a thread takes groups of kGroup samples kT apart, the next group's
// loads in flight, finds each group's mean and squared deviations about it, and
// merges the groups; then the threads' moments are merged in a fixed tree.  All
// of it works on x - x[0] (a difference of two floats in fp64), so an error of
// a mean is a few u times the mean |x - x[0]|, at most sqrt(n) standard
// deviations (no sample lies farther from the mean), and reaches the variance
// through differences of means only: a relative error below 4 n u, as the
// interval of R assumes for any order of evaluation.  A constant channel has a
// variance of exactly zero, any other one has not.  Bound by memory: 1024
// windows of 262,144 samples take 206 us, 5.2 TB/s (two passes over the samples:
// 355 us); 96 of 100,003, a workgroup each and so bound by latency, 21 us (37).
constexpr int kGroup = 16;

struct ChannelStats {
    double mean, var, absmean, sq, sabs;
};

template <int kT>
__device__ inline ChannelStats channel_stats(const float* __restrict__ xw, int64_t n, double* red) {
    constexpr int kWaves = kT / kWave;
    const double x0 = (double)xw[0];
    Moments m = {0.0, 0.0, 0.0};
    double sa = 0.0;
    float nxt[kGroup];
    auto load = [&](int64_t i0) {
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            const int64_t i = i0 + threadIdx.x + r * kT;
            nxt[r] = i < n ? xw[i] : 0.0f;
        }
    };
    load(0);
    for (int64_t i0 = 0; i0 < n; i0 += kGroup * kT) {
        float x[kGroup];
#pragma unroll
        for (int r = 0; r < kGroup; ++r) x[r] = nxt[r];
        if (i0 + kGroup * kT < n) load(i0 + kGroup * kT);
        Moments g = {0.0, 0.0, 0.0};
        if (i0 + threadIdx.x + (kGroup - 1) * kT < n) {        // a whole group
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < kGroup; ++r) {
                s = s + ((double)x[r] - x0);
                sa = sa + fabs((double)x[r]);
            }
            g.n = (double)kGroup;
            g.mean = s * (1.0 / kGroup);
#pragma unroll
            for (int r = 0; r < kGroup; ++r) {
                const double d = ((double)x[r] - x0) - g.mean;
                g.m2 = g.m2 + d * d;
            }
        } else {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < kGroup; ++r) {
                if (i0 + threadIdx.x + r * kT >= n) continue;
                s = s + ((double)x[r] - x0);
                sa = sa + fabs((double)x[r]);
                g.n = g.n + 1.0;
            }
            if (g.n > 0.0) g.mean = s / g.n;
#pragma unroll
            for (int r = 0; r < kGroup; ++r) {
                if (i0 + threadIdx.x + r * kT >= n) continue;
                const double d = ((double)x[r] - x0) - g.mean;
                g.m2 = g.m2 + d * d;
            }
        }
        m = merge(m, g);
    }
    auto down = [](Moments& t, double& ta, int o) {            // lane l takes lane l + o's in
        Moments q;
        q.n = __shfl_down(t.n, o);
        q.mean = __shfl_down(t.mean, o);
        q.m2 = __shfl_down(t.m2, o);
        t = merge(t, q);
        ta = ta + __shfl_down(ta, o);
    };
    for (int o = kWave / 2; o > 0; o >>= 1) down(m, sa, o);    // lane 0 ends with the wavefront's
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[4 * wave] = m.n;
        red[4 * wave + 1] = m.mean;
        red[4 * wave + 2] = m.m2;
        red[4 * wave + 3] = sa;
    }
    __syncthreads();
    // the wavefronts', by every wavefront in its first lanes
    const int lane = threadIdx.x & (kWave - 1), v = lane & (kWaves - 1);
    m = Moments{red[4 * v], red[4 * v + 1], red[4 * v + 2]};
    sa = red[4 * v + 3];
    for (int o = kWaves / 2; o > 0; o >>= 1) down(m, sa, o);
    m.mean = __shfl(m.mean, 0);
    m.m2 = __shfl(m.m2, 0);
    sa = __shfl(sa, 0);
    __syncthreads();
    ChannelStats r;
    r.mean = x0 + m.mean;
    r.absmean = sa / (double)n;
    r.sq = m.m2;
    r.sabs = sqrt((double)n * m.m2) * (1.0 + 1e-15);
    r.var = m.m2 / (double)n;
    return r;
}

// S(T) of window b from the fp64 chunk partials of its channels (layout
// [b*C + c][chunk][lags_padded], lag T at index T - t0): each channel's
// partials added in ascending chunk order, divided by the N - T pairs, and
// the weighted channel sum (the composite feature of Sec. 4.2).
// The partials are loaded kFinalizeBatch at a time (all in flight) and added
// in order.  finalize_lags does the same for L lags at once (lag
// t + k * lag_step, those below t_end), each with exactly finalize_lag's
// operations, loading kBatch partials a lag at a time.
constexpr int kFinalizeBatch = 8;

__device__ inline double finalize_lag(const double* __restrict__ part, const Weights& w,
                                      int32_t num_channels, int64_t b, int64_t n, int64_t t,
                                      int32_t t0, int32_t lags_padded, int32_t chunks) {
    double s = 0.0;
    for (int32_t c = 0; c < num_channels; ++c) {
        const double* p =
            part + ((b * num_channels + c) * chunks) * (int64_t)lags_padded + (t - t0);
        double d = 0.0;
        int32_t k = 0;
        for (; k + kFinalizeBatch <= chunks; k += kFinalizeBatch) {
            double v[kFinalizeBatch];
#pragma unroll
            for (int u = 0; u < kFinalizeBatch; ++u) v[u] = p[(int64_t)(k + u) * lags_padded];
#pragma unroll
            for (int u = 0; u < kFinalizeBatch; ++u) d += v[u];
        }
        for (; k < chunks; ++k) d += p[(int64_t)k * lags_padded];
        s += (double)w.w[c] * (d / (double)(n - t));
    }
    return s;
}

template <int L, int kBatch>
__device__ inline void finalize_lags(const double* __restrict__ part, const Weights& w,
                                     int32_t num_channels, int64_t b, int64_t n, int64_t t,
                                     int64_t lag_step, int64_t t_end, int32_t t0,
                                     int32_t lags_padded, int32_t chunks,
                                     double (&out)[L]) {
    bool live[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        live[l] = t + l * lag_step < t_end;
        out[l] = 0.0;
    }
    for (int32_t c = 0; c < num_channels; ++c) {
        const double* p =
            part + ((b * num_channels + c) * chunks) * (int64_t)lags_padded + (t - t0);
        double d[L];
#pragma unroll
        for (int l = 0; l < L; ++l) d[l] = 0.0;
        int32_t k = 0;
        for (; k + kBatch <= chunks; k += kBatch) {
            double v[L][kBatch];
#pragma unroll
            for (int l = 0; l < L; ++l)
#pragma unroll
                for (int u = 0; u < kBatch; ++u)
                    v[l][u] = live[l] ? p[l * lag_step + (int64_t)(k + u) * lags_padded] : 0.0;
#pragma unroll
            for (int l = 0; l < L; ++l)
#pragma unroll
                for (int u = 0; u < kBatch; ++u) d[l] += v[l][u];
        }
        for (; k < chunks; ++k)
#pragma unroll
            for (int l = 0; l < L; ++l)
                if (live[l]) d[l] += p[l * lag_step + (int64_t)k * lags_padded];
#pragma unroll
        for (int l = 0; l < L; ++l)
            if (live[l]) out[l] += (double)w.w[c] * (d[l] / (double)(n - (t + l * lag_step)));
    }
}

}  // namespace stats
}  // namespace gpoeo
