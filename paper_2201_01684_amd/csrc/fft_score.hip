// Scores of every lag from an fp64 FFT autocorrelation.
//
// The spectrum of the trace is the starting point of period detection in
// Sec. 4.1.1 (Algorithm 1 transforms the samples and looks for amplitude
// peaks).  Here the transform serves the lag domain instead: for one window's
// channel y (centred by its fp64 mean, zero-padded to L = 2^lg >= N + Tmax
// points so that no lag up to Tmax wraps around),
//   D(T) = sum_{i<N-T} (y_i - y_{i+T})^2 = E1(T) + E2(T) - 2 r(T),
//   E1(T) = sum_{i<N-T} y_i^2,  E2(T) = sum_{i>=T} y_i^2,  r(T) = sum_i y_i y_{i+T},
// with r the inverse transform of |FFT(y)|^2.  Two real sequences a, b travel
// as one complex one, z = y_a + i y_b: from Z = FFT(z) the spectra of a and b
// are (Z(k) + conj Z(L-k)) / 2 and (Z(k) - conj Z(L-k)) / 2i, and the inverse
// transform of |X_a|^2 + i |X_b|^2 returns r_a + i r_b.
//
// Transforms: radix-2 butterflies in LDS, decimation in frequency forward
// (natural order in, bit-reversed out) and in time inverse (bit-reversed in,
// natural out), so no permutation pass is needed.  Up to 2^12 points one
// workgroup holds a whole pair.  Longer transforms use L = L1 * L2 (index
// n = n1 L2 + n2, frequency k = k1 + L1 k2): L2 column transforms of L1
// points, the twiddles W_L^(k1 n2), then L1 row transforms of L2 points.  The
// row kernel holds row k1 together with its mirror row L1 - k1, so the
// separation of the two sequences, the power spectrum, the inverse row
// transform and the inverse twiddles all happen while the two rows are in LDS;
// the inverse column kernel then forms D(T) for the lags it produces.
//
// Accuracy: every lag's D(T) is within an absolute bound derived from the
// sequence norms (fft_bound below); the lags for which that bound is not a
// small fraction of the score are re-scored in fp64 before any decision.
#include <algorithm>
#include <cmath>

#include "exact.h"
#include "fft_common.h"
#include "internal.h"

namespace gpoeo {
namespace {

constexpr int kThreads = 256;                          // edge and fix-up kernels
constexpr int kTThreads = 1 << kFftThreadsLog2;        // transform kernels


__device__ __forceinline__ uint32_t bitrev(uint32_t v, int lg) {
    return lg == 0 ? 0u : (__builtin_bitreverse32(v) >> (32 - lg));
}

// Consecutive workgroups of a launch go round-robin to the 8 XCDs; this maps
// them so that each XCD takes a contiguous range of logical ids (neighbouring
// column groups of one pair then share that XCD's L2).
__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nblk) {
    if (nblk % 8 != 0) return bid;
    return (bid & 7) * (nblk >> 3) + (bid >> 3);
}

// Transforms of `cols` interleaved sequences of L = 2^lg points, s[i * cols + q],
// as radix-2 butterflies: forward by decimation in frequency (natural order
// in, bit-reversed out), at stage h = 2^st the pair (i, i + h) becomes
// (a + b, (a - b) W_2h^j), j = i mod h; inverse by decimation in time
// (bit-reversed in, natural out), (a + b conj(W_2h^j), a - b conj(W_2h^j)).
// tw[m] = exp(-2 pi i m / L), m < L/2, so W_2h^j = tw[j L / 2h].
//
// A pass runs 2^R-point groups through R consecutive stages in registers (the
// same butterflies, so the same roundings as stage-by-stage): the points of a
// group share every index bit outside the pass's stages.  Passes hold up to 4
// stages, with at least 256 groups when the LDS tile allows (all threads busy).
template <int R, bool kInverse>
__device__ __forceinline__ void fft_pass(double2* s, int lg, int lgc, int st_lo,
                                         const double2* __restrict__ tw) {
    constexpr int kR = 1 << R;
    const int cols = 1 << lgc;
    const int groups = 1 << (lg - R + lgc);
    const int lo_mask = (1 << st_lo) - 1;
    for (int gi = threadIdx.x; gi < groups; gi += kTThreads) {
        const int q = gi & (cols - 1);
        const int g = gi >> lgc;
        const int blo = g & lo_mask;
        const int base = ((g >> st_lo) << (st_lo + R)) | blo;
        // the twiddles of all R stages first: stage k uses 2^k of them,
        // W_2h^(blo + u 2^st_lo) for u < 2^k, at wt[2^k - 1 + u]
        double2 wt[kR - 1];
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
            for (int u = 0; u < (1 << k); ++u)
                wt[(1 << k) - 1 + u] = tw[(blo + (u << st_lo)) << (lg - 1 - (st_lo + k))];
        double2 v[kR];
#pragma unroll
        for (int m = 0; m < kR; ++m) v[m] = s[(base + (m << st_lo)) * cols + q];
#pragma unroll
        for (int kk = 0; kk < R; ++kk) {
            const int k = kInverse ? kk : R - 1 - kk;   // stage st_lo + k
#pragma unroll
            for (int m = 0; m < kR; ++m) {
                if (m & (1 << k)) continue;
                const double2 w = wt[(1 << k) - 1 + (m & ((1 << k) - 1))];
                const double2 a = v[m];
                if (kInverse) {
                    const double2 b = cmul_conj(v[m + (1 << k)], w);
                    v[m] = cadd(a, b);
                    v[m + (1 << k)] = csub(a, b);
                } else {
                    const double2 b = v[m + (1 << k)];
                    v[m] = cadd(a, b);
                    v[m + (1 << k)] = cmul(csub(a, b), w);
                }
            }
        }
#pragma unroll
        for (int m = 0; m < kR; ++m) s[(base + (m << st_lo)) * cols + q] = v[m];
    }
}

template <bool kInverse, int kMaxR>
__device__ void lds_fft(double2* s, int lg, int lgc, const double2* __restrict__ tw) {
    int rmax = lg + lgc - kFftThreadsLog2;   // log2 of the points per thread
    rmax = rmax < 1 ? 1 : (rmax > kMaxR ? kMaxR : rmax);
    const int np = (lg + rmax - 1) / rmax;
    const int base = lg / np, extra = lg % np;
    int st = kInverse ? 0 : lg;
    for (int p = 0; p < np; ++p) {
        const int r = base + (p < extra ? 1 : 0);
        const int st_lo = kInverse ? st : st - r;
        if (r == 1) fft_pass<1, kInverse>(s, lg, lgc, st_lo, tw);
        else if (r == 2 || kMaxR < 3) fft_pass<(kMaxR < 2 ? 1 : 2), kInverse>(s, lg, lgc, st_lo, tw);
        else if (r == 3 || kMaxR < 4) fft_pass<(kMaxR < 3 ? 1 : 3), kInverse>(s, lg, lgc, st_lo, tw);
        else fft_pass<(kMaxR < 4 ? 1 : 4), kInverse>(s, lg, lgc, st_lo, tw);
        __syncthreads();
        st = kInverse ? st + r : st_lo;
    }
}

// A workgroup of 2^kFftThreadsLog2 threads on a tile of 2^kTile points holds
// 2^(kTile - kFftThreadsLog2) points per thread: the largest useful pass radix.
template <int kTile>
__device__ __forceinline__ void lds_fft_fwd(double2* s, int lg, int lgc, const double2* tw) {
    lds_fft<false, kTile - kFftThreadsLog2>(s, lg, lgc, tw);
}
template <int kTile>
__device__ __forceinline__ void lds_fft_inv(double2* s, int lg, int lgc, const double2* tw) {
    lds_fft<true, kTile - kFftThreadsLog2>(s, lg, lgc, tw);
}

// W_L^e = exp(-2 pi i e / L) for e < L from two tables split at bit lg2.
__device__ __forceinline__ double2 twiddle(const FftArgs& a, int64_t e) {
    return cmul(a.tw[a.tw_hi + (e >> a.lg2)], a.tw[a.tw_lo + (e & ((int64_t(1) << a.lg2) - 1))]);
}

// The pass twiddles of one 2^lg-point sub-transform (tw[m], m < 2^(lg-1)),
// copied to LDS at twl by the workgroup: load() issues the loads into
// registers (with the caller's data loads, all in flight together), store()
// writes them; the caller's barrier before the transform orders them.
template <int kTile>
struct TwiddleCopy {
    static constexpr int kPer = ((1 << (kTile - 1)) + kTThreads - 1) / kTThreads;
    double2 v[kPer];
    __device__ __forceinline__ void load(const double2* __restrict__ tw, int lg) {
        const int count = 1 << (lg - 1);
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int k = threadIdx.x + r * kTThreads;
            v[r] = k < count ? tw[k] : make_double2(0.0, 0.0);
        }
    }
    __device__ __forceinline__ void store(double2* twl, int lg) const {
        const int count = 1 << (lg - 1);
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int k = threadIdx.x + r * kTThreads;
            if (k < count) twl[k] = v[r];
        }
    }
};

// The four-step twiddle tables (tw_lo, 2^lg2 entries, then tw_hi, 2^lg1) in
// LDS at tl when together they hold at most kFourStepLds entries: copied like
// the pass twiddles, then read by twiddle_at with the same operations as
// twiddle().  (The forward column and row kernels; the wrap correction's row
// kernel keeps the global tables, whose LDS would cost it a workgroup per CU.)
constexpr int kFourStepLds = 1024;
__host__ __device__ inline bool four_step_in_lds(int lg1, int lg2) {
    return (1 << lg1) + (1 << lg2) <= kFourStepLds;
}
struct FourStepCopy {
    static constexpr int kPer = kFourStepLds / kTThreads;
    double2 v[kPer];
    __device__ __forceinline__ void load(const FftArgs& a) {
        const int count = (1 << a.lg1) + (1 << a.lg2);
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int k = threadIdx.x + r * kTThreads;
            v[r] = k < count ? a.tw[a.tw_lo + k] : make_double2(0.0, 0.0);
        }
    }
    __device__ __forceinline__ void store(const FftArgs& a, double2* tl) const {
        const int count = (1 << a.lg1) + (1 << a.lg2);
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int k = threadIdx.x + r * kTThreads;
            if (k < count) tl[k] = v[r];
        }
    }
};
__device__ __forceinline__ double2 twiddle_at(const FftArgs& a, const double2* tl, bool lds4,
                                              int64_t e) {
    if (!lds4) return twiddle(a, e);
    return cmul(tl[(1 << a.lg2) + (e >> a.lg2)], tl[e & ((int64_t(1) << a.lg2) - 1)]);
}

// 4 (|X_a|^2 + i |X_b|^2) at frequency k from Z(k) and Z(L - k).
__device__ __forceinline__ double2 power_pair(double2 zk, double2 zm) {
    const double ux = zk.x + zm.x, uy = zk.y - zm.y;
    const double vx = zk.x - zm.x, vy = zk.y + zm.y;
    return make_double2(ux * ux + uy * uy, vx * vx + vy * vy);
}

// Energies of the first and the last N - T samples of a sequence, E1(T) + E2(T)
// = (E - tail(T)) + (E - head(T)) for T = 0..Tmax of its window, with head and
// tail the sums of y^2 over the first and the last T samples; one workgroup per
// sequence, half of its threads a side.  Tiles of 4096 terms a side are loaded
// (all of a thread's loads in flight at once) and staged in LDS; each thread
// adds 16 consecutive terms, an exclusive scan of the side's thread totals
// (lane shuffles within each wavefront, then the wavefront totals in order)
// gives each thread its offset, and the running sums of both sides go through
// LDS for coalesced stores of their combination.  (The mean and E come from the
// window statistics, computed with the same mean.)
constexpr int kEdgeTile = 4096;
constexpr int kEdgePer = kEdgeTile / kThreads;   // 16 terms per thread
constexpr int kEdgeWaves = kThreads / kWave;
constexpr int64_t kEdgeTwGroups = kFftBlockPoints / 2 / (2 * kThreads);   // W_4096^e, e < 2048

__device__ __forceinline__ int edge_slot(int k) { return k + (k >> 4); }   // padded: no bank clash

__global__ __launch_bounds__(2 * kThreads) void fft_edge_kernel(FftArgs a) {
    __shared__ double tiles[2][kEdgeTile + kEdgeTile / 16];
    __shared__ double wsum[2][kEdgeWaves];
    const int64_t s = blockIdx.x;
    if (a.tw_out && s < kEdgeTwGroups) {   // the twiddles of the block transforms, by the first
        const int e = (int)s * 2 * kThreads + (int)threadIdx.x;
        double sn, cs;
        sincospi(ldexp(2.0 * (double)e, -kFftBlockLog2), &sn, &cs);   // exact argument
        a.tw_out[e] = make_double2(cs, -sn);
    }
    if (s >= a.seqs) return;
    const int side = threadIdx.x / kThreads, tid = threadIdx.x % kThreads;
    double* tile = tiles[side];
    const int64_t b = s / a.num_channels;
    const int64_t c = s % a.num_channels;
    const int64_t n = table_n(a.tab, b, a.n_all);
    if (n <= 0) return;
    const float* __restrict__ p = a.x + table_off(a.tab, b, a.window_stride) + c * a.channel_stride;
    const double mu = a.fstat[4 * s], e = a.fstat[4 * s + 1];
    double* __restrict__ out = a.edge + s * ((int64_t)a.tmax + 1);   // out[T]
    // T = 0 .. this window's largest lag
    const int64_t span = (int64_t)min(table_tmax(a.tab, b, a.tmax), a.tmax) + 1;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    if (threadIdx.x == 0) out[0] = e + e;
    double carry = 0.0;
    // the next tile's samples are loaded while this tile is scanned
    float nxt[kEdgePer];
    auto load_tile = [&](int64_t k0, float (&v)[kEdgePer]) {
#pragma unroll
        for (int r = 0; r < kEdgePer; ++r) {
            const int64_t kk = k0 + tid + r * kThreads;
            const bool in = kk < n && kk < span - 1;
            v[r] = in ? p[side == 0 ? kk : n - 1 - kk] : 0.0f;
        }
    };
    if (span - 1 > 0) load_tile(0, nxt);
    for (int64_t k0 = 0; k0 < span - 1; k0 += kEdgeTile) {   // terms k0 .. k0 + 4095
        {
            float v[kEdgePer];
#pragma unroll
            for (int r = 0; r < kEdgePer; ++r) v[r] = nxt[r];
            if (k0 + kEdgeTile < span - 1) load_tile(k0 + kEdgeTile, nxt);
#pragma unroll
            for (int r = 0; r < kEdgePer; ++r) {
                const int k = tid + r * kThreads;
                const int64_t kk = k0 + k;
                const double y = (kk < n && kk < span - 1) ? (double)v[r] - mu : 0.0;
                tile[edge_slot(k)] = y * y;
            }
        }
        __syncthreads();
        double part = 0.0;
        for (int r = 0; r < kEdgePer; ++r) part += tile[edge_slot(tid * kEdgePer + r)];
        double inc = part;   // inclusive scan within the wavefront
        for (int o = 1; o < kWave; o <<= 1) {
            const double u = __shfl_up(inc, o);
            if (lane >= o) inc += u;
        }
        if (lane == kWave - 1) wsum[side][wave] = inc;
        __syncthreads();
        double run = carry, total = carry;
        for (int w = 0; w < kEdgeWaves; ++w) {
            if (w < wave) run += wsum[side][w];
            total += wsum[side][w];
        }
        run += inc - part;   // this thread's exclusive offset
        for (int r = 0; r < kEdgePer; ++r) {
            const int k = tid * kEdgePer + r;
            run += tile[edge_slot(k)];
            tile[edge_slot(k)] = run;   // sum of terms 0 .. k0 + k: the value at T = k0 + k + 1
        }
        __syncthreads();
        for (int r = 0; r < kEdgePer / 2; ++r) {
            const int k = (int)threadIdx.x + r * 2 * kThreads;
            const int64_t t = k0 + k + 1;
            if (t < span)
                out[t] = (e - tiles[1][edge_slot(k)]) + (e - tiles[0][edge_slot(k)]);
        }
        carry = total;
        __syncthreads();
    }
}

// Twiddle tables: A (transforms of 2^lga points), B (2^lgb points, if any),
// and the two halves of W_L^e for the split transform.
__global__ void fft_twiddle_kernel(double2* tw, int lga, int lgb, int lg, int lg2, int64_t nb,
                                   int64_t nlo, int64_t nhi) {
    const int64_t na = int64_t(1) << (lga - 1);
    const int64_t total = na + nb + nlo + nhi;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        int64_t m;
        int lgl;
        if (e < na) {
            m = e;
            lgl = lga;
        } else if (e < na + nb) {
            m = e - na;
            lgl = lgb;
        } else if (e < na + nb + nlo) {
            m = e - na - nb;
            lgl = lg;
        } else {
            m = e - na - nb - nlo;
            lgl = lg - lg2;
        }
        double sn, cs;
        sincospi(ldexp(2.0 * (double)m, -lgl), &sn, &cs);   // exact argument 2m / 2^lgl
        tw[e] = make_double2(cs, -sn);
    }
}

// Whole transform of one pair in one workgroup (L <= 2^12).
template <int kTile>
__global__ __launch_bounds__(kTThreads) void fft_single_kernel(FftArgs a) {
    constexpr int kRegPoints = (1 << kTile) / kTThreads;
    extern __shared__ double2 lds[];
    const int64_t pair = blockIdx.x;
    const Seq qa = seq_of(a, 2 * pair), qb = seq_of(a, 2 * pair + 1);
    if (qa.n <= 0 && qb.n <= 0) return;                    // empty slots of a window table
    const int lg = a.lg;
    const int len = 1 << lg;
    const double2* tw = a.tw + a.tw_a;
    {   // all loads of a thread in flight before its LDS writes
        double2 v[kRegPoints];
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int i = threadIdx.x + r * kTThreads;
            v[r] = make_double2(centred(qa, i), centred(qb, i));
        }
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int i = threadIdx.x + r * kTThreads;
            if (i < len) lds[i] = v[r];
        }
    }
    __syncthreads();
    lds_fft_fwd<kTile>(lds, lg, 0, tw);
    double2 wv[kRegPoints];
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int pos = threadIdx.x + r * kTThreads;
        if (pos < len) {
            const uint32_t k = bitrev(pos, lg);
            const uint32_t km = (len - k) & (len - 1);
            wv[r] = power_pair(lds[pos], lds[bitrev(km, lg)]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int pos = threadIdx.x + r * kTThreads;
        if (pos < len) lds[pos] = wv[r];
    }
    __syncthreads();
    lds_fft_inv<kTile>(lds, lg, 0, tw);
    const int64_t tend = min((int64_t)a.tmax, (int64_t)len - 1);
    for (int64_t t = a.tmin + threadIdx.x; t <= tend; t += kTThreads) {
        write_d(a, 2 * pair, t, lds[t].x);
        write_d(a, 2 * pair + 1, t, lds[t].y);
    }
}

// Split transform, step 1: column transforms (L1 points, stride L2) of
// 2^lgc neighbouring columns, then the twiddles W_L^(k1 n2).  Row p of the
// output holds frequency k1 = bitrev(p).
template <int kTile>
__global__ __launch_bounds__(kTThreads) void fft_cols_fwd_kernel(FftArgs a) {
    constexpr int kRegPoints = (1 << kTile) / kTThreads;
    extern __shared__ double2 lds[];
    const int64_t groups = int64_t(1) << (a.lg2 - a.lgc);
    const int64_t id = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t pair = id / groups;
    const int64_t c0 = (id % groups) << a.lgc;
    const int cols = 1 << a.lgc;
    const int npts = (1 << a.lg1) * cols;
    const int64_t l2 = int64_t(1) << a.lg2;
    const Seq qa = seq_of(a, 2 * pair), qb = seq_of(a, 2 * pair + 1);
    double2* twl = lds + npts;   // the pass twiddles, after the tile
    // Tiles of four or more columns whose rows start on 16-byte boundaries: a
    // thread takes runs of four points of a row (their four samples of each
    // sequence in one 16-byte load) instead of single points.
    auto aligned = [&](const Seq& q) {
        return q.n == 0 || ((reinterpret_cast<uintptr_t>(q.p + c0) & 15) == 0);
    };
    const bool rows4 = a.lgc >= 2 && npts == kRegPoints * kTThreads && (l2 & 3) == 0 &&
                       aligned(qa) && aligned(qb);
    const bool lds4 = four_step_in_lds(a.lg1, a.lg2);
    double2* tl = twl + (1 << (a.lg1 - 1));   // the four-step twiddles, after the pass ones
    FourStepCopy fc;
    if (lds4) fc.load(a);
    double la = 0.0, lb = 0.0;
    if (rows4) {   // all loads of a thread in flight before its LDS writes
        constexpr int kRows = kRegPoints / 4;   // runs of four points a thread
        const int quads = cols >> 2;            // runs in a row of the tile
        TwiddleCopy<kTile> tc;
        tc.load(a.tw + a.tw_a, a.lg1);
        auto row_of = [&](const Seq& q, int64_t i) -> float4 {
            if (i + 3 < q.n) return *reinterpret_cast<const float4*>(q.p + i);
            float4 f4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (i < q.n) f4.x = q.p[i];
            if (i + 1 < q.n) f4.y = q.p[i + 1];
            if (i + 2 < q.n) f4.z = q.p[i + 2];
            return f4;
        };
        float4 va[kRows], vb[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int qd = threadIdx.x + k * kTThreads;   // points 4 qd .. 4 qd + 3
            const int64_t i = (int64_t)(qd / quads) * l2 + c0 + 4 * (qd % quads);
            va[k] = row_of(qa, i);
            vb[k] = row_of(qb, i);
        }
        tc.store(twl, a.lg1);
        if (lds4) fc.store(a, tl);
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int qd = threadIdx.x + k * kTThreads;
            const int f = 4 * qd;
            const int64_t i = (int64_t)(qd / quads) * l2 + c0 + 4 * (qd % quads);
            // the same values as centred(): (double)x - mu inside the sequence, 0 past it
            auto cv = [&](const Seq& q, float x, int64_t ii) {
                return ii < q.n ? (double)x - q.mu : 0.0;
            };
            const double2 y[4] = {make_double2(cv(qa, va[k].x, i), cv(qb, vb[k].x, i)),
                                  make_double2(cv(qa, va[k].y, i + 1), cv(qb, vb[k].y, i + 1)),
                                  make_double2(cv(qa, va[k].z, i + 2), cv(qb, vb[k].z, i + 2)),
                                  make_double2(cv(qa, va[k].w, i + 3), cv(qb, vb[k].w, i + 3))};
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                lds[f + m] = y[m];
                la += fabs(y[m].x);
                lb += fabs(y[m].y);
            }
        }
    } else {   // all loads of a thread in flight before its LDS writes
        TwiddleCopy<kTile> tc;
        tc.load(a.tw + a.tw_a, a.lg1);
        double2 v[kRegPoints];
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            const int64_t i = f < npts ? (int64_t)(f >> a.lgc) * l2 + c0 + (f & (cols - 1)) : a.len;
            v[r] = make_double2(centred(qa, i), centred(qb, i));
        }
        tc.store(twl, a.lg1);
        if (lds4) fc.store(a, tl);
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            if (f < npts) lds[f] = v[r];
            la += fabs(v[r].x);   // (0 past the tile)
            lb += fabs(v[r].y);
        }
    }
    if (a.l1) {   // sums of |y| by wavefront, for the fix-up's bound
        for (int o = kWave / 2; o > 0; o >>= 1) {
            la += __shfl_xor(la, o);
            lb += __shfl_xor(lb, o);
        }
        const int64_t parts = groups * (kTThreads / kWave);
        const int64_t part = (id % groups) * (kTThreads / kWave) + threadIdx.x / kWave;
        if ((threadIdx.x & (kWave - 1)) == 0) {
            a.l1[2 * pair * parts + part] = la;
            a.l1[(2 * pair + 1) * parts + part] = lb;
        }
    }
    __syncthreads();
    lds_fft_fwd<kTile>(lds, a.lg1, a.lgc, twl);
    double2* __restrict__ zp = a.z + pair * a.zstride;
    double2 w[kRegPoints];
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {   // twiddle loads first
        const int f = threadIdx.x + r * kTThreads;
        const int64_t k1 = bitrev(f >> a.lgc, a.lg1);
        w[r] = f < npts ? twiddle_at(a, tl, lds4, k1 * (c0 + (f & (cols - 1))))
                        : make_double2(1.0, 0.0);
    }
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int f = threadIdx.x + r * kTThreads;
        if (f < npts) zp[(int64_t)(f >> a.lgc) * l2 + c0 + (f & (cols - 1))] = cmul(lds[f], w[r]);
    }
}

// Split transform, step 2: row k1 and its mirror row L1 - k1 (frequencies k
// and L - k pair up between them): forward row transforms, separation into
// the two sequences' power spectra, inverse row transforms, inverse twiddles.
// A workgroup takes 2^lgr consecutive row pairs (4096 points in LDS).
template <int kTile>
__global__ __launch_bounds__(kTThreads) void fft_rows_kernel(FftArgs a) {
    constexpr int kRegPoints = (1 << kTile) / kTThreads;
    extern __shared__ double2 lds[];   // point i of slot q at i * 2^(lgr+1) + q
    const int64_t per = (int64_t(1) << (a.lg1 - 1)) + 1;   // row pairs per transform
    const int64_t wgs = (per + (1 << a.lgr) - 1) >> a.lgr;
    const int64_t id = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t pair = id / wgs;
    const int64_t g0 = (id % wgs) << a.lgr;
    const uint32_t l1 = 1u << a.lg1;
    const int lgs = a.lgr + 1;                 // log2 of the slots
    const int slots = 1 << lgs;
    const int l2 = 1 << a.lg2;
    const int npts = l2 << lgs;
    double2* __restrict__ zp = a.z + pair * a.zstride;
    // slot q: row pair g0 + (q >> 1), side q & 1 (0: k1 = g, 1: k1 = L1 - g)
    auto k1_of = [&](int q, bool& valid, bool& self) -> uint32_t {
        const int64_t g = g0 + (q >> 1);
        valid = g < per;
        const uint32_t ka = (uint32_t)g, kb = (l1 - (uint32_t)g) & (l1 - 1);
        self = ka == kb;
        return (q & 1) ? kb : ka;
    };
    double2* twl = lds + npts;   // the pass twiddles, after the tile
    const bool lds4 = four_step_in_lds(a.lg1, a.lg2);
    double2* tl = twl + (1 << (a.lg2 - 1));   // the four-step twiddles, after the pass ones
    {   // all loads of a thread in flight before its LDS writes
        TwiddleCopy<kTile> tc;
        tc.load(a.tw + a.tw_b, a.lg2);
        FourStepCopy fc;
        if (lds4) fc.load(a);
        double2 v[kRegPoints];
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            bool valid, self;
            const uint32_t k1 = k1_of(f & (slots - 1), valid, self);
            v[r] = (valid && f < npts) ? zp[(int64_t)bitrev(k1, a.lg1) * l2 + (f >> lgs)]
                                       : make_double2(0.0, 0.0);
        }
        tc.store(twl, a.lg2);
        if (lds4) fc.store(a, tl);
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            if (f < npts) lds[f] = v[r];
        }
    }
    __syncthreads();
    lds_fft_fwd<kTile>(lds, a.lg2, lgs, twl);
    double2 wv[kRegPoints];
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int f = threadIdx.x + r * kTThreads;
        if (f < npts) {
            const int q = f & (slots - 1);
            bool valid, self;
            const uint32_t k1 = k1_of(q, valid, self);
            const uint32_t k2 = bitrev(f >> lgs, a.lg2);
            const uint32_t k2m = k1 == 0 ? ((l2 - k2) & (l2 - 1)) : (l2 - 1 - k2);
            const int qm = self ? q : (q ^ 1);
            wv[r] = power_pair(lds[f], lds[(bitrev(k2m, a.lg2) << lgs) + qm]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int f = threadIdx.x + r * kTThreads;
        if (f < npts) lds[f] = wv[r];
    }
    __syncthreads();
    lds_fft_inv<kTile>(lds, a.lg2, lgs, twl);
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {   // twiddle loads first (wv is free again)
        const int f = threadIdx.x + r * kTThreads;
        bool valid, self;
        const uint32_t k1 = k1_of(f & (slots - 1), valid, self);
        wv[r] = (f < npts && valid) ? twiddle_at(a, tl, lds4, (int64_t)k1 * (f >> lgs))
                                    : make_double2(1.0, 0.0);
    }
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int f = threadIdx.x + r * kTThreads;
        const int q = f & (slots - 1);
        bool valid, self;
        const uint32_t k1 = k1_of(q, valid, self);
        if (f >= npts || !valid || ((q & 1) && self)) continue;
        zp[(int64_t)bitrev(k1, a.lg1) * l2 + (f >> lgs)] = cmul_conj(lds[f], wv[r]);
    }
}

// 4 Q(k) of the wrap correction from the head transform Z1 = FFT(h_a + i h_b)
// and the tail transform Z2 = FFT(u_a + i u_b) at k and L - k:
// with H_a = (Z1(k) + conj Z1(L-k)) / 2, H_b = (Z1(k) - conj Z1(L-k)) / 2i and
// U_a, U_b likewise from Z2, Q = U_a conj(H_a) + i U_b conj(H_b), whose
// inverse transform is cc_a + i cc_b, cc(s) = sum_j h_j u_{j+s}.
__device__ __forceinline__ double2 cross_pair(double2 z1k, double2 z1m, double2 z2k, double2 z2m) {
    const double2 ha = make_double2(z1k.x + z1m.x, z1k.y - z1m.y);   // 2 H_a
    const double2 hb = make_double2(z1k.y + z1m.y, z1m.x - z1k.x);   // 2 H_b
    const double2 ua = make_double2(z2k.x + z2m.x, z2k.y - z2m.y);   // 2 U_a
    const double2 ub = make_double2(z2k.y + z2m.y, z2m.x - z2k.x);   // 2 U_b
    const double2 pa = cmul_conj(ua, ha), pb = cmul_conj(ub, hb);
    return make_double2(pa.x - pb.y, pa.y + pb.x);
}

// Wrap correction, step 2: rows k1 and L1 - k1 of both the head transform
// (at z) and the tail transform (at z + zoff2) of 2^lgr consecutive row pairs:
// forward row transforms, the cross spectrum Q of the pair, inverse row
// transforms of Q and the inverse twiddles; Q's rows go over the head
// transform's rows.  LDS: point i of slot q at i * 4 * 2^lgr + q, slot q =
// (row pair, side, transform) from the high bits down; Q then takes the
// layout of two slots per row pair.
template <int kTile>
__global__ __launch_bounds__(kTThreads) void fft_wrap_rows_kernel(FftArgs a, int64_t zoff2) {
    constexpr int kRegPoints = (1 << kTile) / kTThreads;
    extern __shared__ double2 lds[];
    const int64_t per = (int64_t(1) << (a.lg1 - 1)) + 1;
    const int64_t wgs = (per + (1 << a.lgr) - 1) >> a.lgr;
    const int64_t id = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t pair = id / wgs;
    const int64_t g0 = (id % wgs) << a.lgr;
    const uint32_t l1 = 1u << a.lg1;
    const int lgs = a.lgr + 2;
    const int slots = 1 << lgs;
    const int l2 = 1 << a.lg2;
    const int npts = l2 << lgs;
    double2* __restrict__ z1 = a.z + pair * a.zstride;
    const double2* __restrict__ z2 = z1 + zoff2;
    auto k1_of = [&](int64_t g, int side, bool& valid, bool& self) -> uint32_t {
        valid = g < per;
        const uint32_t ka = (uint32_t)g, kb = (l1 - (uint32_t)g) & (l1 - 1);
        self = ka == kb;
        return side ? kb : ka;
    };
    double2* twl = lds + npts;   // the pass twiddles, after the tile
    {
        TwiddleCopy<kTile> tc;
        tc.load(a.tw + a.tw_b, a.lg2);
        double2 v[kRegPoints];
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            const int q = f & (slots - 1);
            bool valid, self;
            const uint32_t k1 = k1_of(g0 + (q >> 2), (q >> 1) & 1, valid, self);
            const double2* src = (q & 1) ? z2 : z1;
            v[r] = (valid && f < npts) ? src[(int64_t)bitrev(k1, a.lg1) * l2 + (f >> lgs)]
                                       : make_double2(0.0, 0.0);
        }
        tc.store(twl, a.lg2);
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            if (f < npts) lds[f] = v[r];
        }
    }
    __syncthreads();
    lds_fft_fwd<kTile>(lds, a.lg2, lgs, twl);
    double2 wv[kRegPoints];
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {   // at the head transform's slots
        const int f = threadIdx.x + r * kTThreads;
        const int q = f & (slots - 1);
        if (f < npts && (q & 1) == 0) {
            bool valid, self;
            const uint32_t k1 = k1_of(g0 + (q >> 2), (q >> 1) & 1, valid, self);
            const uint32_t k2 = bitrev(f >> lgs, a.lg2);
            const uint32_t k2m = k1 == 0 ? ((l2 - k2) & (l2 - 1)) : (l2 - 1 - k2);
            const int qm = self ? q : (q ^ 2);
            const int fm = (int)(bitrev(k2m, a.lg2) << lgs) + qm;
            wv[r] = cross_pair(lds[f], lds[fm], lds[f + 1], lds[fm + 1]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {   // Q: point i of slot q >> 1 at i * slots / 2 + (q >> 1)
        const int f = threadIdx.x + r * kTThreads;
        const int q = f & (slots - 1);
        if (f < npts && (q & 1) == 0) lds[(f >> lgs) * (slots >> 1) + (q >> 1)] = wv[r];
    }
    __syncthreads();
    lds_fft_inv<kTile>(lds, a.lg2, lgs - 1, twl);
    const int half = npts >> 1;
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {   // twiddle loads first
        const int f = threadIdx.x + r * kTThreads;
        const int q2 = f & ((slots >> 1) - 1);
        bool valid, self;
        const uint32_t k1 = k1_of(g0 + (q2 >> 1), q2 & 1, valid, self);
        wv[r] = (f < half && valid) ? twiddle(a, (int64_t)k1 * (f >> (lgs - 1)))
                                    : make_double2(1.0, 0.0);
    }
#pragma unroll
    for (int r = 0; r < kRegPoints; ++r) {
        const int f = threadIdx.x + r * kTThreads;
        const int q2 = f & ((slots >> 1) - 1);
        bool valid, self;
        const uint32_t k1 = k1_of(g0 + (q2 >> 1), q2 & 1, valid, self);
        if (f >= half || !valid || ((q2 & 1) && self)) continue;
        z1[(int64_t)bitrev(k1, a.lg1) * l2 + (f >> (lgs - 1))] = cmul_conj(lds[f], wv[r]);
    }
}

// Split transform, step 3: inverse column transforms (row p holds k1 =
// bitrev(p): the bit-reversed input order of the decimation in time), and
// D(T) for the lags T = n1 L2 + n2 in [tmin, tmax].
template <int kTile>
__global__ __launch_bounds__(kTThreads) void fft_cols_inv_kernel(FftArgs a) {
    constexpr int kRegPoints = (1 << kTile) / kTThreads;
    extern __shared__ double2 lds[];
    const int64_t groups = int64_t(1) << (a.lg2 - a.lgc);
    const int64_t id = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t pair = id / groups;
    const int64_t c0 = (id % groups) << a.lgc;
    const int cols = 1 << a.lgc;
    const int npts = (1 << a.lg1) * cols;
    const int64_t l2 = int64_t(1) << a.lg2;
    const double2* __restrict__ zp = a.z + pair * a.zstride;
    double2* twl = lds + npts;   // the pass twiddles, after the tile
    {   // all loads of a thread in flight before its LDS writes
        TwiddleCopy<kTile> tc;
        tc.load(a.tw + a.tw_a, a.lg1);
        double2 v[kRegPoints];
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            v[r] = f < npts ? zp[(int64_t)(f >> a.lgc) * l2 + c0 + (f & (cols - 1))]
                            : make_double2(0.0, 0.0);
        }
        tc.store(twl, a.lg1);
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int f = threadIdx.x + r * kTThreads;
            if (f < npts) lds[f] = v[r];
        }
    }
    __syncthreads();
    lds_fft_inv<kTile>(lds, a.lg1, a.lgc, twl);
    if (a.wout) {   // head-tail transform: cc_a(s) + i cc_b(s) for shifts s < wm
        const int rows = (int)min((int64_t)((a.wm - 1) / l2) + 1, int64_t(1) << a.lg1);
        for (int f = threadIdx.x; f < rows * cols; f += kTThreads) {
            const int64_t sh = (int64_t)(f >> a.lgc) * l2 + c0 + (f & (cols - 1));
            if (sh >= a.wm) continue;
            a.wout[2 * pair * a.wm + sh] = ldexp(lds[f].x, -(a.lg + 2));
            if (2 * pair + 1 < a.seqs) a.wout[(2 * pair + 1) * a.wm + sh] = ldexp(lds[f].y, -(a.lg + 2));
        }
    } else {
        const int rows = (int)min((int64_t)(a.tmax / l2) + 1, int64_t(1) << a.lg1);
        for (int f = threadIdx.x; f < rows * cols; f += kTThreads) {
            const int64_t t = (int64_t)(f >> a.lgc) * l2 + c0 + (f & (cols - 1));
            write_d(a, 2 * pair, t, lds[f].x);
            write_d(a, 2 * pair + 1, t, lds[f].y);
        }
    }
}

// Amplitudes |X_a(k)| and |X_b(k)| of the two sequences of a pair at
// frequency k <= L/2, from Z(k) and Z(L - k): |Z(k) + conj Z(L-k)| / 2 and
// |Z(k) - conj Z(L-k)| / 2.
__device__ __forceinline__ void write_amplitudes(const FftArgs& a, int64_t pair, int64_t k,
                                                 double2 zk, double2 zm) {
    const double ux = zk.x + zm.x, uy = zk.y - zm.y;
    const double vx = zk.x - zm.x, vy = zk.y + zm.y;
    const int64_t half = a.len / 2 + 1;
    const int64_t sa = 2 * pair, sb = sa + 1;
    a.amp[sa * half + k] = 0.5 * sqrt(ux * ux + uy * uy);
    if (sb < a.seqs) a.amp[sb * half + k] = 0.5 * sqrt(vx * vx + vy * vy);
}

// Spectrum of one pair in one workgroup (L up to one tile).
template <int kTile>
__global__ __launch_bounds__(kTThreads) void spec_single_kernel(FftArgs a) {
    constexpr int kRegPoints = (1 << kTile) / kTThreads;
    extern __shared__ double2 lds[];
    const int64_t pair = blockIdx.x;
    const Seq qa = seq_of(a, 2 * pair), qb = seq_of(a, 2 * pair + 1);
    const int lg = a.lg;
    const int len = 1 << lg;
    {
        double2 v[kRegPoints];
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int i = threadIdx.x + r * kTThreads;
            v[r] = make_double2(centred(qa, i), centred(qb, i));
        }
#pragma unroll
        for (int r = 0; r < kRegPoints; ++r) {
            const int i = threadIdx.x + r * kTThreads;
            if (i < len) lds[i] = v[r];
        }
    }
    __syncthreads();
    lds_fft_fwd<kTile>(lds, lg, 0, a.tw + a.tw_a);
    for (int pos = threadIdx.x; pos < len; pos += kTThreads) {
        const uint32_t k = bitrev(pos, lg);
        if (k > (uint32_t)(len / 2)) continue;
        const uint32_t km = (len - k) & (len - 1);
        write_amplitudes(a, pair, k, lds[pos], lds[bitrev(km, lg)]);
    }
}

// Absolute error bound of the computed D(T) of sequence s (any T), from the
// norms of s and of the sequence it shares the transform with.
//
// A radix-2 transform of L = 2^lg points with twiddles accurate to mu errs by
// at most phi ||exact||_2, phi = k eta / (1 - k eta), eta = mu + g4 (sqrt2 + mu)
// (Higham, Accuracy and Stability of Numerical Algorithms, Thm. 24.2), with k
// = lg + 1 stages (the split form adds the twiddle stage); mu = 16 u covers
// the table entries and the product of two of them.  Then, with zeta^2 =
// E_a + E_b, the spectrum of a errs by e1 sqrt(L) zeta (e1 = phi + 4u, with
// the separation); its power spectrum, summed over all frequencies and divided
// by L, errs by 2 e1 zeta |y_a| + (e1 zeta)^2 + g3 (|y_a| + e1 zeta)^2; the
// inverse transform adds phi (1 + g3) (|y_a|_1 + e1 sqrt(L) zeta)(|y_a| +
// e1 zeta) and the same for b.  Each bounds |r_computed(T) - r(T)|.  The
// energies E - head and E - tail are sums of at most 2N + 2 rounded terms
// (g_{2N+2} E each) plus the additions of the assembly, and centring in fp64
// moves D by at most 4u sqrt(D E) + 4 u^2 E <= 2u D + 3u E.  The result is
// doubled as a margin.  la and lb: |y_a|_1 and |y_b|_1, or bounds of them.
__device__ double fft_bound(const double* fstat, int64_t s, int64_t seqs, int64_t n, int lg,
                            double la, double lb) {
    const double u = 1.1102230246251565e-16;
    const double ea = fstat[4 * s + 1];
    const int64_t o = s ^ 1;
    const double eb = o < seqs ? fstat[4 * o + 1] : 0.0;
    const double ya = sqrt(ea), yb = sqrt(eb), zeta = sqrt(ea + eb);
    const double mu = 16.0 * u;
    const double g3 = 3.0 * u / (1.0 - 3.0 * u);
    const double g4 = 4.0 * u / (1.0 - 4.0 * u);
    const double eta = mu + g4 * (1.4142135623730951 + mu);
    const double keta = (double)(lg + 1) * eta;
    const double phi = keta / (1.0 - keta);
    const double e1 = phi + 4.0 * u;
    const double sl = sqrt(ldexp(1.0, lg));
    const double pa = ya + e1 * zeta, pb = yb + e1 * zeta;
    const double fwd = 2.0 * e1 * zeta * ya + e1 * e1 * zeta * zeta + g3 * pa * pa;
    const double inv = phi * (1.0 + g3) * ((la + e1 * sl * zeta) * pa + (lb + e1 * sl * zeta) * pb);
    const double k = 2.0 * (double)n + 2.0;
    const double ge = k * u / (1.0 - k * u);
    return 2.0 * (2.02 * (fwd + inv) + (2.0 * ge + 17.0 * u) * ea);
}

// Absolute error bound of the wrap term's share of D(T) (any T > W): the
// head-tail transform of 2^lg points takes z1 = h_a + i h_b and z2 = u_a + i u_b
// (the first and last M samples of a and of its partner b), whose norms the
// whole sequences' norms bound.  Each separated spectrum errs by e1 sqrt(L) zeta
// as in fft_bound; the products U conj H, summed over all frequencies and
// divided by L, err by 2 e1 zeta |y_a| + (e1 zeta)^2, their rounding and the
// assembly of Q (a product of two perturbed spectra and one addition each,
// within gamma_4) by g4 ((|y_a| + e1 zeta)^2 + (|y_b| + e1 zeta)^2), and the
// inverse transform by phi (1 + g3) ((|y_a|_1 + e1 sqrt(L) zeta)(|y_a| + e1 zeta)
// + the same for b).  The sum bounds |cc_computed(s) - cc(s)|; D takes it
// twice (D = ... - 2 (r_circ - cc)), with 1% margin, and the result is doubled.
__device__ double fft_bound_wrap(const double* fstat, int64_t s, int64_t seqs, int lg, double la,
                                 double lb) {
    const double u = 1.1102230246251565e-16;
    const double ea = fstat[4 * s + 1];
    const int64_t o = s ^ 1;
    const double eb = o < seqs ? fstat[4 * o + 1] : 0.0;
    const double ya = sqrt(ea), yb = sqrt(eb), zeta = sqrt(ea + eb);
    const double mu = 16.0 * u;
    const double g3 = 3.0 * u / (1.0 - 3.0 * u);
    const double g4 = 4.0 * u / (1.0 - 4.0 * u);
    const double eta = mu + g4 * (1.4142135623730951 + mu);
    const double keta = (double)(lg + 1) * eta;
    const double phi = keta / (1.0 - keta);
    const double e1 = phi + 4.0 * u;
    const double sl = sqrt(ldexp(1.0, lg));
    const double pa = ya + e1 * zeta, pb = yb + e1 * zeta;
    const double fwd = 2.0 * e1 * zeta * ya + e1 * e1 * zeta * zeta + g4 * (pa * pa + pb * pb);
    const double inv = phi * (1.0 + g3) * ((la + e1 * sl * zeta) * pa + (lb + e1 * sl * zeta) * pb);
    return 2.0 * (2.02 * (fwd + inv));
}

// The same for scores from transforms of sample blocks (P points, m samples a
// block, nb blocks).  With zeta_b and y_b the norms of block b (of the pair and
// of s), each separated spectrum errs by e1 sqrt(P) zeta_b; r comes from two
// sums over b of products of two spectra, whose errors, summed over all
// frequencies and divided by P, are at most 2 e1 zeta |y_a| + (e1 zeta)^2 each
// (Cauchy-Schwarz over b); the fp64 sums (2 nb fused multiply-adds a component,
// one more for R_j) add sqrt(2) gamma_{2 nb + 2} (|y_a| + e1 zeta)^2 each, and
// the assembly R_a + i R_b one rounding of both.  The inverse transform adds phi
// / sqrt(P) times the norm of R, at most the sum over b of the largest entry of
// one spectrum, sqrt(m) y_b (Cauchy-Schwarz over its samples), times the norm of
// the other, sqrt(P) times that of the samples of two blocks: phi sqrt(2 m)
// |y_a|^2 (Cauchy-Schwarz over b), each norm enlarged by its error.
__device__ double fft_bound_blocks(const double* fstat, int64_t s, int64_t seqs, int64_t n) {
    const double u = 1.1102230246251565e-16;
    const double ea = fstat[4 * s + 1];
    const int64_t o = s ^ 1;
    const double eb = o < seqs ? fstat[4 * o + 1] : 0.0;
    const double ya = sqrt(ea), yb = sqrt(eb), zeta = sqrt(ea + eb);
    const double nb = (double)((n + kFftBlockSamples - 1) / kFftBlockSamples);
    const double mu = 16.0 * u;
    const double g4 = 4.0 * u / (1.0 - 4.0 * u);
    const double gs = (2.0 * nb + 2.0) * u / (1.0 - (2.0 * nb + 2.0) * u);
    const double eta = mu + g4 * (1.4142135623730951 + mu);
    const double keta = (double)(kFftBlockLog2 + 1) * eta;
    const double phi = keta / (1.0 - keta);
    const double e1 = phi + 4.0 * u;
    const double pa = ya + 2.0 * e1 * zeta, pb = yb + 2.0 * e1 * zeta;
    const double fwd = 2.0 * (2.0 * e1 * zeta * ya + e1 * e1 * zeta * zeta) +
                       (2.0 * 1.4142135623730951 * gs + 2.0 * u) * pa * pa + 2.0 * u * pb * pb;
    const double inv = phi * (1.0 + gs + g4) * sqrt(2.0 * (double)kFftBlockSamples) *
                       (pa * pa + pb * pb);
    const double k = 2.0 * (double)n + 2.0;
    const double ge = k * u / (1.0 - k * u);
    return 2.0 * (2.02 * (fwd + inv) + (2.0 * ge + 17.0 * u) * ea);
}

struct FixArgs {
    const float* x;
    const double* fstat;
    double* s64;
    float* scores;
    uint32_t* tier1;
    WinState* state;
    int64_t seqs;
    int64_t n_all, window_stride, channel_stride;
    int32_t num_channels, tmin, tmax, lags, words, lg;
    double tau0;
    WindowTable tab;
    int32_t blocks;            // transforms of sample blocks
    int32_t wrap_lg;           // log2 of the head-tail transform (wrap correction), or -1
    const double* l1;          // split transforms: [S][l1_parts], partial sums of |y|; or null
    int32_t l1_parts;
};

// sum_i |x_i - mean| of sequence s from the column kernel's partial sums, by the
// whole workgroup.
__device__ double centred_abs_sum(const FixArgs& a, int64_t s, double* red) {
    if (s >= a.seqs) return 0.0;
    double acc = 0.0;
    for (int32_t k = threadIdx.x; k < a.l1_parts; k += kThreads) acc += a.l1[s * a.l1_parts + k];
    for (int o = kWave / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    __syncthreads();                                       // red is free
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = acc;
    __syncthreads();
    acc = red[0];
    for (int v = 1; v < kThreads / kWave; ++v) acc += red[v];
    return acc;
}

// The bound of one channel's D(T) times its weight, with long transforms.
__device__ double channel_bound(const FixArgs& a, const Weights& w, int32_t c, int64_t sq,
                                int64_t n, double la, double lb) {
    double e = fft_bound(a.fstat, sq, a.seqs, n, a.lg, la, lb);
    if (a.wrap_lg >= 0) e += fft_bound_wrap(a.fstat, sq, a.seqs, a.wrap_lg, la, lb);
    return (double)w.w[c] * e;
}

// One workgroup per window and kFixLags lags: lags whose score the FFT bound cannot place within
// tau0 / 2 of itself (the other half covers the rounding of the finalisation
// and of the sequential evaluation) are re-scored by a wavefront in fp64 and
// marked tier 1.  A score of exactly zero always lands here.
//
// The bound of the long transforms takes the sums of absolute deviations, of
// which the statistics give only sqrt(N) times the norm, up to several times as
// much.  Where a lag would be re-scored by that and not with the least bound there
// can be (no such term), the workgroup of a split transform takes the sums
// themselves (a detection of 2^21 samples, three such lags: 7.3 -> 1.9 ms).  Up to 2048
// samples the re-scores cost less than that test.
__global__ __launch_bounds__(kThreads) void fft_fixup_kernel(FixArgs a, Weights w) {
    __shared__ double abound, aleast;
    __shared__ double red[kThreads / kWave];
    const int64_t b = blockIdx.x;
    const int64_t n = table_n(a.tab, b, a.n_all);
    if (n == 0) return;
    const int32_t tm = table_tmax(a.tab, b, a.tmax);
    const int32_t nlags = tm - a.tmin + 1;
    if (threadIdx.x == 0) {
        double acc = 0.0, least = 0.0;
        for (int32_t c = 0; c < a.num_channels; ++c) {
            const int64_t sq = b * a.num_channels + c, o = sq ^ 1;
            acc += a.blocks ? (double)w.w[c] * fft_bound_blocks(a.fstat, sq, a.seqs, n)
                            : channel_bound(a, w, c, sq, n, a.fstat[4 * sq + 2],
                                            o < a.seqs ? a.fstat[4 * o + 2] : 0.0);
            if (a.l1) least += channel_bound(a, w, c, sq, n, 0.0, 0.0);
        }
        abound = acc * (1.0 + 1e-12);
        aleast = least;
    }
    if (a.l1) {
        __syncthreads();
        const double most = abound, least = aleast;
        bool open = false;
        for (int64_t j = (int64_t)blockIdx.y * kFixLags + threadIdx.x; j < nlags;
             j += (int64_t)gridDim.y * kFixLags)
#pragma unroll
            for (int r = 0; r < kFixBatch; ++r)
                if (j + r * kThreads < nlags) {
                    const double lim = 0.5 * a.tau0 * a.s64[b * a.lags + j + r * kThreads] *
                                       (double)(n - a.tmin - j - r * kThreads);
                    open = open || (!(most <= lim) && least <= lim);
                }
        if (__syncthreads_or(open)) {
            double acc = 0.0;
            for (int32_t c = 0; c < a.num_channels; ++c) {
                const int64_t sq = b * a.num_channels + c;
                const double la = centred_abs_sum(a, sq, red);
                const double lb = centred_abs_sum(a, sq ^ 1, red);
                acc += channel_bound(a, w, c, sq, n, la, lb);
            }
            if (threadIdx.x == 0) abound = acc * (1.0 + 1e-12);
        }
    }
    __syncthreads();
    const double ab = abound;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const float* __restrict__ xw = a.x + table_off(a.tab, b, a.window_stride);
    // wavefront w tests lags j0 + lane, j0 = 64 w + 256 k past the workgroup's
    // first; the scores of all kFixBatch k are loaded together, then tested
    for (int64_t jb = (int64_t)blockIdx.y * kFixLags + wave * kWave; jb < nlags;
         jb += (int64_t)gridDim.y * kFixLags) {
    double vb[kFixBatch];
#pragma unroll
    for (int r = 0; r < kFixBatch; ++r) {
        const int32_t j = (int32_t)jb + r * kThreads + lane;
        vb[r] = j < nlags ? a.s64[b * a.lags + j] : 0.0;
    }
    uint32_t fixes = 0;                                    // bit r: this lane's r-th lag
#pragma unroll
    for (int r = 0; r < kFixBatch; ++r) {
        const int32_t j = (int32_t)jb + r * kThreads + lane;
        bool fix = false;
        if (j < nlags) {
            const int64_t t = (int64_t)a.tmin + j;
            fix = !(ab / (double)(n - t) <= 0.5 * a.tau0 * vb[r]);
        }
        fixes |= fix ? 1u << r : 0u;
    }
#pragma unroll 1
    for (int r = 0; r < kFixBatch; ++r) {
        const int32_t j0 = (int32_t)jb + r * kThreads;
        uint64_t mask = __ballot((fixes >> r) & 1u);
        while (mask) {
            const int k = __builtin_ctzll(mask);
            mask &= mask - 1;
            const int32_t jj = j0 + k;
            const int64_t t = (int64_t)a.tmin + jj;
            const double v =
                exact::wave_score(xw, a.num_channels, a.channel_stride, n, t, w, lane);
            if (lane == 0) {
                a.s64[b * a.lags + jj] = v;
                if (a.scores) a.scores[b * a.lags + jj] = (float)v;
                atomicOr(&a.tier1[b * a.words + (jj >> 5)], 1u << (jj & 31));
                atomicAdd(&a.state[b].rescored, 1);
            }
        }
    }
    }
}

// What a chunk of kSpecChunk bins of one window's spectrum holds.
struct SpecChunk {
    double top;                // largest peak (0: none)
    double most;               // largest amplitude
    int64_t peaks;
};

struct SpecSelArgs {
    const double* amp;         // [S][stride]: per-channel amplitudes, by rows (rows > 0) or in order
    const double* fstat;       // [S][4]
    SpecChunk* chunk;          // [B][chunks]
    gpoeo_pd_spectral_result* out;
    int64_t seqs, half, len, stride;
    int32_t num_channels, tmin, tmax, k_max, lg, chunks;
    int32_t lg1;               // log2 of the rows, or -1
    int32_t scanned;           // spec_scan_kernel ran
    int64_t b0;                // first window of this scan launch
    double c_peak;
};

constexpr int kCandCap = 1024;   // candidates collected per window
// Spectra of more points are scanned by a launch of their own (8 windows of 20,000
// samples: 67 us a call, 103 with the scan in the selection; of 8000: 54 either way).
constexpr int64_t kSpecScanPoints = 8192;
constexpr int kSpecChunk = kSpecChunkBins;
constexpr int kSpecChunkLog2 = 11;
constexpr int kSpecMaxChunks = (1 << (kFftMaxLog2 - 1)) / kSpecChunk + 1;
static_assert(kSpecChunk == 1 << kSpecChunkLog2, "at least two entries of each of 1024 rows");

// A(k) = sum_c w_c |X_c(k)| of window b, in channel order.
__device__ __forceinline__ double spec_amp(const SpecSelArgs& a, const Weights& w, int64_t b,
                                           int64_t k) {
    const int64_t at =
        a.lg1 < 0 ? k : (k & ((int64_t(1) << a.lg1) - 1)) * kSpecRow + (k >> a.lg1);
    const double* __restrict__ amp = a.amp + b * a.num_channels * a.stride + at;
    double acc = 0.0;
    for (int32_t c = 0; c < a.num_channels; ++c) acc += (double)w.w[c] * amp[c * a.stride];
    return acc;
}

// Peaks of one chunk of one window's spectrum (2 <= k <= L/2 - 1, A(k) > A(k-1),
// A(k) >= A(k+1)): their number, the largest, and the largest amplitude.  A
// workgroup per chunk, so that few windows of long spectra fill the chip: the
// selection of 300 windows of 131,073 bins and two channels took 462 us with
// one workgroup a window, which wrote the channel sums back and read them twice;
// the scan and the selection take 210.
__global__ __launch_bounds__(kThreads) void spec_scan_kernel(SpecSelArgs a, Weights w) {
    constexpr int kPer = kSpecChunk / kThreads;
    __shared__ double s[kSpecChunk + 2 + (kSpecChunk + 2) / 32];
    // (padded: entries a row apart would meet in one bank)
    auto slot = [](int i) { return i + (i >> 5); };
    __shared__ double red[2][kThreads / kWave];
    __shared__ int32_t redi[kThreads / kWave];
    const int64_t b = a.b0 + blockIdx.x / a.chunks;
    const int32_t ch = (int32_t)(blockIdx.x % a.chunks);
    const int64_t k0 = (int64_t)ch * kSpecChunk;         // bins k0 .. k0 + kSpecChunk - 1
    const int tid = threadIdx.x;
    // bin of a thread's r-th entry, in the order the amplitudes are stored
    auto bin = [&](int r) {
        const int i = tid + r * kThreads;
        if (a.lg1 < 0) return i;
        const int per = kSpecChunkLog2 - a.lg1;           // log2 of a row's entries in the chunk
        return (i >> per) + ((i & ((1 << per) - 1)) << a.lg1);
    };
    double v[kPer], e = 0.0;                             // all loads in flight
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int64_t k = k0 + bin(r);
        v[r] = k < a.half ? spec_amp(a, w, b, k) : 0.0;
    }
    const int64_t ke = tid == 0 ? k0 - 1 : k0 + kSpecChunk;   // the neighbours
    if (tid < 2 && ke >= 0 && ke < a.half) e = spec_amp(a, w, b, ke);
#pragma unroll
    for (int r = 0; r < kPer; ++r) s[slot(1 + bin(r))] = v[r];
    if (tid < 2) s[slot(tid == 0 ? 0 : kSpecChunk + 1)] = e;
    __syncthreads();
    double top = 0.0, most = 0.0;
    int32_t peaks = 0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int i = 1 + bin(r);
        const int64_t k = k0 + i - 1;
        most = fmax(most, v[r]);
        if (k >= 2 && k <= a.half - 2 && v[r] > s[slot(i - 1)] && v[r] >= s[slot(i + 1)]) {
            ++peaks;
            top = fmax(top, v[r]);
        }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        top = fmax(top, __shfl_xor(top, o));
        most = fmax(most, __shfl_xor(most, o));
        peaks += __shfl_xor(peaks, o);
    }
    if ((tid & (kWave - 1)) == 0) {
        red[0][tid / kWave] = top;
        red[1][tid / kWave] = most;
        redi[tid / kWave] = peaks;
    }
    __syncthreads();
    if (tid == 0) {
        SpecChunk c = {top, most, peaks};
        for (int i = 1; i < kThreads / kWave; ++i) {
            c.top = fmax(c.top, red[0][i]);
            c.most = fmax(c.most, red[1][i]);
            c.peaks += redi[i];
        }
        a.chunk[b * a.chunks + ch] = c;
    }
}

// Candidates of one window from its amplitude spectrum: the peaks above c_peak
// times the largest one whose period round(L/k) is in [tmin, tmax], strongest
// first (ties: smaller k).  Only chunks whose largest amplitude reaches that
// threshold (within the error bound) are read again.  The window is flagged
// UNRESOLVED when a peak test, the threshold, or the order of the reported
// candidates lies within four times the amplitude error bound (the list a
// correctly rounded spectrum gives could then differ), or when more than
// kCandCap candidates qualify.
__global__ __launch_bounds__(kThreads) void spec_select_kernel(SpecSelArgs a, Weights w) {
    __shared__ double red[kThreads];
    __shared__ int32_t redi[kThreads];
    __shared__ double cand_a[kCandCap];
    __shared__ int32_t cand_k[kCandCap];
    __shared__ int32_t ncand;
    __shared__ int32_t flag;
    __shared__ gpoeo_pd_spectral_result res;
    __shared__ int32_t list[kSpecMaxChunks];               // chunks to read again
    __shared__ int32_t nlist;
    const int64_t b = blockIdx.x;
    const int tid = threadIdx.x;
    const SpecChunk* __restrict__ chunk = a.chunk + b * a.chunks;
    if (tid == 0) {
        ncand = 0;
        flag = 0;
        nlist = 0;
    }
    for (int i = tid; i < (int)(sizeof(res) / 4); i += kThreads) reinterpret_cast<int32_t*>(&res)[i] = 0;
    // 1. the largest peak and the number of peaks
    double mx = 0.0;
    int32_t npk = 0;
    if (a.scanned) {
        for (int32_t i = tid; i < a.chunks; i += kThreads) {
            mx = fmax(mx, chunk[i].top);
            npk += (int32_t)chunk[i].peaks;
        }
    } else {   // a short spectrum: here, instead of in a launch of its own
        for (int64_t k = 2 + tid; k <= a.half - 2; k += kThreads) {
            const double v = spec_amp(a, w, b, k);
            if (v > spec_amp(a, w, b, k - 1) && v >= spec_amp(a, w, b, k + 1)) {
                ++npk;
                mx = fmax(mx, v);
            }
        }
    }
    red[tid] = mx;
    redi[tid] = npk;
    __syncthreads();
    for (int st = kThreads / 2; st > 0; st >>= 1) {
        if (tid < st) {
            red[tid] = fmax(red[tid], red[tid + st]);
            redi[tid] += redi[tid + st];
        }
        __syncthreads();
    }
    const double top = red[0];
    const int32_t n_peaks = redi[0];
    __syncthreads();
    // 2. error bound of A (any k): the transform bound of each channel's pair
    // (as for the FFT scores: phi sqrt(L) zeta, plus the separation; more than
    // twice what the passes of longer spectra err by, fft_spectrum.hip), summed
    // with the weights, plus the rounding of the amplitude and the channel sum
    const double u = 1.1102230246251565e-16;
    const double mu = 16.0 * u;
    const double g4 = 4.0 * u / (1.0 - 4.0 * u);
    const double keta = (double)(a.lg + 1) * (mu + g4 * (1.4142135623730951 + mu));
    const double phi = keta / (1.0 - keta);
    double eps = 0.0;
    for (int32_t c = 0; c < a.num_channels; ++c) {
        const int64_t sq = b * a.num_channels + c, o = sq ^ 1;
        const double z2 = a.fstat[4 * sq + 1] + (o < a.seqs ? a.fstat[4 * o + 1] : 0.0);
        eps += (double)w.w[c] * (phi + 4.0 * u) * sqrt((double)a.len) * sqrt(z2);
    }
    eps = 2.0 * (eps + ((double)a.num_channels + 6.0) * u * top);
    const double m = 4.0 * eps;
    const double thr = a.c_peak * top;
    // 3. candidates, and decisions too close to call
    for (int32_t i = tid; i < a.chunks; i += kThreads)
        if (!a.scanned || !(chunk[i].most + m < a.c_peak * (top - m))) list[atomicAdd(&nlist, 1)] = i;
    __syncthreads();
    for (int32_t li = 0; li < nlist; ++li) {
        const int32_t i = list[li];
        const int64_t k0 = (int64_t)i * kSpecChunk;
        const int64_t k1 = min(k0 + (int64_t)kSpecChunk - 1, a.half - 2);
        for (int64_t k = max(k0, (int64_t)2) + tid; k <= k1; k += kThreads) {
            const double v = spec_amp(a, w, b, k);
            if (v + m < a.c_peak * (top - m)) continue;       // cannot matter
            const double l = spec_amp(a, w, b, k - 1), r = spec_amp(a, w, b, k + 1);
            const bool peak = v > l && v >= r;
            if (fabs(v - l) <= m || fabs(v - r) <= m) atomicOr(&flag, 1);
            if (!peak) continue;
            const int64_t t = (2 * a.len + k) / (2 * k);       // round(L / k), halves up
            if (t < a.tmin || t > a.tmax) continue;
            if (fabs(v - thr) <= m * (1.0 + a.c_peak)) atomicOr(&flag, 1);
            if (!(v > thr)) continue;
            const int slot = atomicAdd(&ncand, 1);
            if (slot < kCandCap) {
                cand_a[slot] = v;
                cand_k[slot] = (int32_t)k;
            } else {
                atomicOr(&flag, 2);
            }
        }
    }
    __syncthreads();
    const int nc = min(ncand, kCandCap);
    // 4. the strongest first: rounds of a block-wide arg-max (larger A, then smaller k)
    double prev = 0.0;
    int rounds = min(nc, a.k_max + 1);                     // one more to check the order
    for (int r = 0; r < rounds; ++r) {
        double bv = -1.0;
        int32_t bk = INT32_MAX, bi = -1;
        for (int i = tid; i < nc; i += kThreads) {
            const double v = cand_a[i];
            if (v > bv || (v == bv && cand_k[i] < bk)) {
                bv = v;
                bk = cand_k[i];
                bi = i;
            }
        }
        // wavefront arg-max, then the four wavefronts' in order
        for (int o = kWave / 2; o > 0; o >>= 1) {
            const double v1 = __shfl_xor(bv, o);
            const int32_t k1 = __shfl_xor(bk, o), i1 = __shfl_xor(bi, o);
            if (i1 >= 0 && (bi < 0 || v1 > bv || (v1 == bv && k1 < bk))) {
                bv = v1;
                bk = k1;
                bi = i1;
            }
        }
        if ((tid & (kWave - 1)) == 0) {
            red[tid / kWave] = bv;
            redi[tid / kWave] = bi;
        }
        __syncthreads();
        int best = redi[0];
        double bvv = red[0];
        for (int i = 1; i < kThreads / kWave; ++i) {
            const int i1 = redi[i];
            if (i1 >= 0 && (best < 0 || red[i] > bvv || (red[i] == bvv && cand_k[i1] < cand_k[best]))) {
                best = i1;
                bvv = red[i];
            }
        }
        __syncthreads();
        if (tid == 0) {
            if (r > 0 && prev - bvv <= m) flag |= 1;
            if (r < a.k_max) {
                const int32_t k = cand_k[best];
                res.periods[r] = (int32_t)((2 * a.len + k) / (2 * (int64_t)k));
                res.bins[r] = k;
                res.amplitudes[r] = bvv;
                res.count = r + 1;
            }
            cand_a[best] = -1.0;                           // taken
        }
        prev = bvv;
        __syncthreads();
    }
    if (tid == 0) {
        res.n_peaks = n_peaks;
        res.max_peak = top;
        res.flags = flag ? GPOEO_PD_UNRESOLVED : 0u;
    }
    __syncthreads();
    int32_t* out = reinterpret_cast<int32_t*>(a.out + b);
    for (int i = tid; i < (int)(sizeof(res) / 4); i += kThreads) out[i] = reinterpret_cast<int32_t*>(&res)[i];
}

// Transform geometry of 2^lg points in the launch arguments.
void set_geometry(FftArgs& a, int lg) {
    int32_t m1, m2, cols;
    fft_geometry(lg, &m1, &m2, &cols);
    a.lg = lg;
    a.len = int64_t(1) << lg;
    if (m2 == 1) {   // one workgroup per pair
        a.lg1 = lg;
        a.lg2 = 0;
        a.lgc = 0;
        a.lgr = 0;
        a.tw_a = 0;
        a.tw_b = a.tw_lo = a.tw_hi = 0;
    } else {
        a.lg1 = __builtin_ctz((unsigned)m1);
        a.lg2 = __builtin_ctz((unsigned)m2);
        a.lgc = __builtin_ctz((unsigned)cols);
        const int tile = fft_tile_log2(lg);
        a.lgr = a.lg2 >= tile - 1 ? 0 : tile - 1 - a.lg2;   // row pairs per tile
        a.tw_a = 0;
        a.tw_b = m1 / 2;
        a.tw_lo = a.tw_b + m2 / 2;
        a.tw_hi = a.tw_lo + m2;
    }
}

FftArgs args_of(const Plan& p, const float* x, double* fstat, double* edge, double* tw, double* z,
                double* part) {
    FftArgs a;
    a.x = x;
    a.fstat = fstat;
    a.edge = edge;
    a.tw = reinterpret_cast<const double2*>(tw);
    a.tw_out = nullptr;
    a.l1 = nullptr;
    a.z = reinterpret_cast<double2*>(z);
    a.part = part;
    a.amp = nullptr;
    a.seqs = p.num_windows * (int64_t)p.num_channels;
    a.n_all = p.n;
    a.window_stride = p.window_stride;
    a.channel_stride = p.channel_stride;
    a.num_channels = p.num_channels;
    a.tmin = p.tmin;
    a.tmax = p.tmax;
    a.lags = p.lags;
    a.tab = p.table;
    a.zstride = p.fft_len;
    a.seg_start = 0;
    a.seg_len = 0;
    a.wout = nullptr;
    a.wrap = nullptr;
    a.wrap_w = 0;
    a.wm = 0;
    a.s64 = nullptr;
    a.scores = nullptr;
    a.w0 = 1.0f;
    set_geometry(a, p.fft_log2);
    return a;
}

// The transform kernels for the geometry in `a`, over `pairs` pairs.
template <int kTile>
void launch_transforms(const FftArgs& a, int64_t pairs, hipStream_t s) {
    auto grid = [](int64_t items) { return dim3((unsigned)items); };
    if (a.lg2 == 0) {
        const size_t lds = sizeof(double2) * (size_t)a.len;
        hipLaunchKernelGGL((fft_single_kernel<kTile>), grid(pairs), dim3(kTThreads), lds,
                           s, a);
        return;
    }
    const int64_t m1 = int64_t(1) << a.lg1, m2 = int64_t(1) << a.lg2, cols = int64_t(1) << a.lgc;
    const int64_t col_groups = pairs * (m2 / cols);
    // tiles, then each kernel's pass twiddles (half a sub-transform), then for
    // the forward columns and the rows the four-step twiddles when they fit
    const size_t fs = four_step_in_lds(a.lg1, a.lg2) ? (size_t)(m1 + m2) : 0;
    const size_t lds_cols = sizeof(double2) * (size_t)(m1 * cols + m1 / 2);
    const size_t lds_cols_fwd = lds_cols + sizeof(double2) * fs;
    const int64_t rp = int64_t(1) << a.lgr;
    const size_t lds_rows = sizeof(double2) * ((size_t)(2 * rp * m2 + m2 / 2) + fs);
    const int64_t row_groups = pairs * ((m1 / 2 + 1 + rp - 1) / rp);
    hipLaunchKernelGGL((fft_cols_fwd_kernel<kTile>), grid(col_groups), dim3(kTThreads),
                       lds_cols_fwd, s, a);
    hipLaunchKernelGGL((fft_rows_kernel<kTile>), grid(row_groups), dim3(kTThreads),
                       lds_rows, s, a);
    hipLaunchKernelGGL((fft_cols_inv_kernel<kTile>), grid(col_groups), dim3(kTThreads),
                       lds_cols, s, a);
}

// Complex fp64 entries of the twiddle tables of one transform of 2^lg points.
int64_t twiddle_count_of(int lg) {
    int32_t m1, m2, cols;
    fft_geometry(lg, &m1, &m2, &cols);
    if (m2 == 1) return (int64_t)m1 / 2;
    return m1 / 2 + m2 / 2 + m2 + m1;
}

}  // namespace

int32_t fft_l1_parts(const Plan& p) {
    return p.fft_blocks || p.fft_m2 == 1 ? 0 : p.fft_m2 / p.fft_cols * (kTThreads / kWave);
}

// Complex fp64 entries of the twiddle tables of a plan.
int64_t fft_twiddle_count(const Plan& p) {
    if (p.fft_blocks) return kFftBlockPoints / 2;
    return twiddle_count_of(p.fft_log2) + (p.fft_wrap ? twiddle_count_of(p.fft_wrap_log2) : 0);
}

namespace {

// Twiddle tables of the geometry in `a`, written at `tw`.
void launch_twiddles(const FftArgs& a, double2* tw, hipStream_t s) {
    const int64_t count = twiddle_count_of(a.lg);
    int64_t tg = (count + 255) / 256;
    if (tg > 1024) tg = 1024;
    if (a.lg2 == 0) {
        hipLaunchKernelGGL(fft_twiddle_kernel, dim3((unsigned)tg), dim3(256), 0, s, tw, a.lg, 1,
                           a.lg, 0, (int64_t)0, (int64_t)0, (int64_t)0);
    } else {
        const int64_t m1 = int64_t(1) << a.lg1, m2 = int64_t(1) << a.lg2;
        hipLaunchKernelGGL(fft_twiddle_kernel, dim3((unsigned)tg), dim3(256), 0, s, tw, a.lg1,
                           a.lg2, a.lg, a.lg2, m2 / 2, m2, m1);
    }
}

}  // namespace

int64_t spectral_chunks(const Plan& p) { return (p.fft_len / 2 + kSpecChunk) / kSpecChunk; }
size_t spectral_chunk_bytes(const Plan& p) {
    return (size_t)(p.num_windows * spectral_chunks(p)) * sizeof(SpecChunk);
}

hipError_t launch_spectral(const Plan& p, const Weights& w, const float* x, const double* fstat,
                           double* tw, double* z, double* amp, void* chunk, double c_peak,
                           int32_t k_max, gpoeo_pd_spectral_result* out, hipStream_t s) {
    FftArgs a = args_of(p, x, const_cast<double*>(fstat), nullptr, tw, z, nullptr);
    a.amp = amp;
    a.lg = p.fft_log2;
    a.len = p.fft_len;
    a.tw_a = 0;
    const bool single = p.fft_log2 <= kSpecSingleLog2;
    if (single)   // (launch_spectrum_prepare computed those of the others)
        hipLaunchKernelGGL(fft_twiddle_kernel, dim3(8), dim3(256), 0, s,
                           reinterpret_cast<double2*>(tw), p.fft_log2, 1, p.fft_log2, 0, (int64_t)0,
                           (int64_t)0, (int64_t)0);
    if (!single) {
        const hipError_t err = launch_spectrum(p, x, fstat, tw, z, amp, s);
        if (err != hipSuccess) return err;   // (hipGetLastError has been read and cleared)
    } else if (p.fft_log2 <= kFftSmallTileLog2) {
        hipLaunchKernelGGL(spec_single_kernel<kFftSmallTileLog2>, dim3((unsigned)p.fft_pairs),
                           dim3(kTThreads), sizeof(double2) * (size_t)p.fft_len, s, a);
    } else {
        hipLaunchKernelGGL(spec_single_kernel<kFftTileLog2>, dim3((unsigned)p.fft_pairs),
                           dim3(kTThreads), sizeof(double2) * (size_t)p.fft_len, s, a);
    }
    SpecSelArgs sa;
    sa.amp = amp;
    sa.fstat = fstat;
    sa.out = out;
    sa.seqs = a.seqs;
    sa.half = p.fft_len / 2 + 1;
    sa.len = p.fft_len;
    sa.num_channels = p.num_channels;
    sa.tmin = p.tmin;
    sa.tmax = p.tmax;
    sa.k_max = k_max;
    sa.lg = p.fft_log2;
    sa.c_peak = c_peak;
    sa.stride = spectral_bins(p);
    sa.lg1 = single ? -1 : p.fft_log2 - kFftBlockLog2;
    sa.chunk = static_cast<SpecChunk*>(chunk);
    sa.chunks = (int32_t)spectral_chunks(p);
    sa.scanned = p.fft_len > kSpecScanPoints;
    if (sa.scanned) {   // in several launches past HIP's 32-bit global size
        const int64_t most = ((int64_t(1) << 32) - 1) / kThreads / sa.chunks;
        for (sa.b0 = 0; sa.b0 < p.num_windows; sa.b0 += most)
            hipLaunchKernelGGL(spec_scan_kernel,
                               dim3((unsigned)(std::min(most, p.num_windows - sa.b0) * sa.chunks)),
                               dim3(kThreads), 0, s, sa, w);
    }
    hipLaunchKernelGGL(spec_select_kernel, dim3((unsigned)p.num_windows), dim3(kThreads), 0, s,
                       sa, w);
    return hipGetLastError();
}

namespace {

// The wrap term of every sequence into `wrap` ([S][M]): head and tail
// transforms (column kernels on the segments), the cross spectrum and its
// inverse rows, then the inverse columns.  Twiddles of the 2^lgw geometry at
// `tw`.
template <int kTile>
void launch_wrap(const Plan& p, FftArgs aw, double2* tw, double2* zw, double* wrap,
                 hipStream_t s) {
    const int64_t lw = int64_t(1) << p.fft_wrap_log2;
    aw.tw = tw;
    aw.zstride = lw;
    aw.len = lw;
    launch_twiddles(aw, tw, s);
    const int64_t m1 = int64_t(1) << aw.lg1, m2 = int64_t(1) << aw.lg2, cols = int64_t(1) << aw.lgc;
    const int64_t col_groups = p.fft_pairs * (m2 / cols);
    const size_t fs = four_step_in_lds(aw.lg1, aw.lg2) ? (size_t)(m1 + m2) : 0;
    const size_t lds_cols = sizeof(double2) * (size_t)(m1 * cols + m1 / 2);
    const size_t lds_cols_fwd = lds_cols + sizeof(double2) * fs;
    aw.seg_len = p.fft_wrap_m;
    aw.seg_start = 0;                                  // heads
    aw.z = zw;
    hipLaunchKernelGGL((fft_cols_fwd_kernel<kTile>), dim3((unsigned)col_groups),
                       dim3(kTThreads), lds_cols_fwd, s, aw);
    aw.seg_start = p.n - p.fft_wrap_m;                 // tails
    aw.z = zw + p.fft_pairs * lw;
    hipLaunchKernelGGL((fft_cols_fwd_kernel<kTile>), dim3((unsigned)col_groups),
                       dim3(kTThreads), lds_cols_fwd, s, aw);
    aw.seg_len = 0;
    aw.z = zw;
    // a row pair holds four rows of m2 points: its two rows in each transform
    const int rows_tile = 4 * m2 <= (int64_t(1) << kFftSmallTileLog2) ? kFftSmallTileLog2
                                                                       : kFftTileLog2;
    aw.lgr = rows_tile - 2 - aw.lg2;
    if (aw.lgr > aw.lg1 - 1) aw.lgr = aw.lg1 - 1;
    const int64_t rp = int64_t(1) << aw.lgr;
    const int64_t row_groups = p.fft_pairs * ((m1 / 2 + 1 + rp - 1) / rp);
    const size_t lds_rows = sizeof(double2) * (size_t)(4 * rp * m2 + m2 / 2);
    if (rows_tile == kFftSmallTileLog2)
        hipLaunchKernelGGL((fft_wrap_rows_kernel<kFftSmallTileLog2>), dim3((unsigned)row_groups),
                           dim3(kTThreads), lds_rows, s, aw, p.fft_pairs * lw);
    else
        hipLaunchKernelGGL((fft_wrap_rows_kernel<kFftTileLog2>), dim3((unsigned)row_groups),
                           dim3(kTThreads), lds_rows, s, aw, p.fft_pairs * lw);
    aw.wout = wrap;
    aw.wm = p.fft_wrap_m;
    hipLaunchKernelGGL((fft_cols_inv_kernel<kTile>), dim3((unsigned)col_groups),
                       dim3(kTThreads), lds_cols, s, aw);
}

}  // namespace

hipError_t launch_fft_scores(const Plan& p, const float* x, double* fstat, double* edge,
                             double* tw, double* z, double* part, double* zw,
                             double* wrap, double* l1, double* s64, float* scores, float w0,
                             hipStream_t s) {
    FftArgs a = args_of(p, x, fstat, edge, tw, z, part);
    double2* const tw2 = reinterpret_cast<double2*>(tw);
    if (fft_fused_finalize(p, scores != nullptr)) {
        a.s64 = s64;
        a.scores = scores;
        a.w0 = w0;
    }
    if (p.fft_blocks) {
        a.tw_out = tw2;
        hipLaunchKernelGGL(fft_edge_kernel, dim3((unsigned)std::max(a.seqs, kEdgeTwGroups)),
                           dim3(2 * kThreads), 0, s, a);
        return launch_fft_blocks(p, FftBlockBuffers{tw, z, zw}, x, fstat, edge, part, a.s64,
                                 a.scores, w0, s);
    }
    launch_twiddles(a, tw2, s);
    hipLaunchKernelGGL(fft_edge_kernel, dim3((unsigned)a.seqs), dim3(2 * kThreads), 0, s, a);
    if (p.fft_wrap) {
        FftArgs aw = a;
        set_geometry(aw, p.fft_wrap_log2);
        double2* const tww = tw2 + twiddle_count_of(p.fft_log2);
        double2* const zw2 = reinterpret_cast<double2*>(zw);
        if (fft_tile_log2(p.fft_wrap_log2) == kFftSmallTileLog2)
            launch_wrap<kFftSmallTileLog2>(p, aw, tww, zw2, wrap, s);
        else
            launch_wrap<kFftTileLog2>(p, aw, tww, zw2, wrap, s);
        a.wrap = wrap;
        a.wrap_w = p.fft_len - p.n;
        a.wm = p.fft_wrap_m;
    }
    a.l1 = l1;
    if (fft_tile_log2(a.lg) == kFftSmallTileLog2)
        launch_transforms<kFftSmallTileLog2>(a, p.fft_pairs, s);
    else
        launch_transforms<kFftTileLog2>(a, p.fft_pairs, s);
    return hipGetLastError();
}

hipError_t launch_fft_fixup(const Plan& p, const Weights& w, const float* x, const double* fstat,
                            const double* l1, double* s64, float* scores, const SelectBuffers& sb,
                            hipStream_t s) {
    FixArgs a;
    a.x = x;
    a.fstat = fstat;
    a.s64 = s64;
    a.scores = scores;
    a.tier1 = sb.tier1;
    a.state = sb.state;
    a.seqs = p.num_windows * (int64_t)p.num_channels;
    a.n_all = p.n;
    a.window_stride = p.window_stride;
    a.channel_stride = p.channel_stride;
    a.num_channels = p.num_channels;
    a.tmin = p.tmin;
    a.tmax = p.tmax;
    a.lags = p.lags;
    a.words = p.bitmap_words;
    a.lg = p.fft_log2;
    a.tau0 = kFftRelBound;
    a.tab = p.table;
    a.blocks = p.fft_blocks;
    a.wrap_lg = p.fft_wrap ? p.fft_wrap_log2 : -1;
    a.l1 = l1;
    a.l1_parts = fft_l1_parts(p);
    hipLaunchKernelGGL(fft_fixup_kernel,
                       dim3((unsigned)p.num_windows, (unsigned)std::min((p.lags + kFixLags - 1) / kFixLags, 65535)),
                       dim3(kThreads), 0, s, a,
                       w);
    return hipGetLastError();
}

}  // namespace gpoeo
