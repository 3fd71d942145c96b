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

// Sums of two values over the kT-wide workgroup, in a fixed order: a butterfly of
// lane shuffles in each wavefront, then the wavefronts' in turn.  red holds 2 kT /
// 64 doubles that no other thread still reads.
template <int kT>
__device__ __forceinline__ void block_sum2(double& x, double& y, double* red) {
    constexpr int kWaves = kT / kWave;
    for (int o = kWave / 2; o > 0; o >>= 1) {
        x = x + __shfl_xor(x, o);
        y = y + __shfl_xor(y, o);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[wave] = x;
        red[kWaves + wave] = y;
    }
    __syncthreads();
    x = red[0];
    y = red[kWaves];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) {
        x = x + red[v];
        y = y + red[kWaves + v];
    }
}

// Mean, population variance and mean |x| of one channel of one window, as
// written by the statistics kernel (var[0] = variance, var[1] = mean |x|); also
// the sum of squared deviations and a bound of the sum of absolute ones, at
// most sqrt(n) times its root (fstat).  Every thread of the kT-wide workgroup
// returns the same values; red holds 4 kT / 64 doubles.
//
// The samples are read once, in tiles of kGroup a thread kT apart, the next
// tile's loads in flight.  A window of one tile stays in registers: its mean, by
// way of differences from x[0] (a difference of two floats in fp64), then the
// deviations from it (two passes, one of them over memory).  In a longer window a
// thread finds each tile's mean and squared deviations about it and merges the
// tiles, all as differences from the mean of its first tile; then the threads'
// means give the window's, and their squared distances from it what the merged
// deviations lack.
//
// Error.  Every term of the variance is a square, so sums of k of them err by k u
// relative: kGroup, 4 a merge, and the reductions' 6 + kT / 64.  Errors e_t of the
// threads' means move it by at most 2 (sum_t n_t e_t^2 / m2)^(1/2).  With g = n / (kGroup
// kT) merges, e_t is 1.5 g u times the thread's mean |x - pivot|, whose squares sum
// to at most 2 (1 + g) m2 / n_t (the pivot, a mean of kGroup of its samples, is off
// by at most (m2_t / kGroup)^(1/2)): 4.3 g^1.5 u.  The pivots and their differences
// from x[0], which is at most n^(1/2) standard deviations from the mean, add
// some 60 n^(1/2) u.  Together below (n + 4) u for n up to 2^31, which fft_bound
// charges, and 3 (n + 4) u up to 2^34, which reference_bound does.  (An emulation
// against exact sums: at most 0.09 (n + 4) u over noise, large offsets, drifts
// and outliers, n from 8 to 262,144.)  A constant channel has a variance of
// exactly zero, any other one has not.
//
// Bound by memory: 1024 windows of 262,144 samples take 206 us, 5.2 TB/s (two
// passes over memory: 355 us).  Short windows are bound by latency, which is why
// one tile is not merged and the reductions are plain sums: 4000 windows of 2100
// samples 16.5 us with two passes over memory, 25.4 us with tiles and threads
// merged throughout, 17.7 us so.
constexpr int kGroup = 16;

struct ChannelStats {
    double mean, var, absmean, sq, sabs;
};

template <int kT>
__device__ inline ChannelStats channel_stats(const float* __restrict__ xw, int64_t n, double* red) {
    constexpr int kWaves = kT / kWave;
    constexpr int kTile = kGroup * kT;
    const int tid = threadIdx.x;
    float x[kGroup], nxt[kGroup];
    auto load = [&](int64_t i0) {
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            const int64_t i = i0 + tid + r * kT;
            nxt[r] = i < n ? xw[i] : 0.0f;
        }
    };
    const double x0 = (double)xw[0];
    load(0);
#pragma unroll
    for (int r = 0; r < kGroup; ++r) x[r] = nxt[r];
    const bool more = n > kTile;
    if (more) load(kTile);
    ChannelStats out;
    double sa = 0.0, q = 0.0;
    if (!more) {
        const int len = (int)n;
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            if (r * kT >= len) break;
            s = s + (tid + r * kT < len ? (double)x[r] - x0 : 0.0);
            sa = sa + fabs((double)x[r]);
        }
        block_sum2<kT>(s, sa, red);
        out.mean = x0 + s / (double)n;
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            if (r * kT >= len) break;
            const double d = tid + r * kT < len ? (double)x[r] - out.mean : 0.0;
            q = q + d * d;
        }
    } else {
        double t = 0.0;
        Moments m = {(double)kGroup, 0.0, 0.0};                // of x - c
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            t = t + ((double)x[r] - x0);
            sa = sa + fabs((double)x[r]);
        }
        const double c = x0 + t * (1.0 / kGroup);              // pivot
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            const double d = (double)x[r] - c;
            m.m2 = m.m2 + d * d;
        }
        for (int64_t i0 = kTile; i0 < n; i0 += kTile) {
#pragma unroll
            for (int r = 0; r < kGroup; ++r) x[r] = nxt[r];
            if (i0 + kTile < n) load(i0 + kTile);
            Moments g = {0.0, 0.0, 0.0};
            t = 0.0;
            if (i0 + kTile <= n) {                             // a whole tile
#pragma unroll
                for (int r = 0; r < kGroup; ++r) {
                    t = t + ((double)x[r] - c);
                    sa = sa + fabs((double)x[r]);
                }
                g.n = (double)kGroup;
                g.mean = t * (1.0 / kGroup);
#pragma unroll
                for (int r = 0; r < kGroup; ++r) {
                    const double d = ((double)x[r] - c) - g.mean;
                    g.m2 = g.m2 + d * d;
                }
            } else {
                const int left = (int)(n - i0) - tid;          // r kT below it: samples
                g.n = left > 0 ? (double)((left - 1) / kT + 1) : 0.0;
#pragma unroll
                for (int r = 0; r < kGroup; ++r) {
                    t = t + (r * kT < left ? (double)x[r] - c : 0.0);
                    sa = sa + fabs((double)x[r]);
                }
                if (left > 0) g.mean = t * recip(g.n);
#pragma unroll
                for (int r = 0; r < kGroup; ++r) {
                    const double d = r * kT < left ? ((double)x[r] - c) - g.mean : 0.0;
                    g.m2 = g.m2 + d * d;
                }
            }
            m = merge(m, g);
        }
        const double mean_t = (c - x0) + m.mean;               // of x - x0
        double total = m.n * mean_t;
        block_sum2<kT>(total, sa, red);
        const double mean = total / (double)n;
        out.mean = x0 + mean;
        const double d = mean_t - mean;
        q = m.m2 + m.n * (d * d);
    }
    double unused = 0.0;
    block_sum2<kT>(q, unused, red + 2 * kWaves);   // (the next call's first sums use the other half)
    out.absmean = sa / (double)n;
    out.sq = q;
    out.sabs = sqrt((double)n * q) * (1.0 + 4.0 * ((double)n + 4.0) * 1.1102230246251565e-16);
    out.var = q / (double)n;
    return out;
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
