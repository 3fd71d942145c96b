// Amplitude spectra |X_s(k)|, k <= L/2, of a batch of sequences, L = 2^lg > 4096
// points a pair of sequences (z = y_a + i y_b).  L = L1 * 4096, sample n = 4096 n1
// + n2 and frequency k = k1 + L1 k2:
//   spectrum_cols_kernel  L1-point transforms over n1 of 4096 / L1 neighbouring
//                         n2 a workgroup, and the twiddles W_L^(n2 k1)
//   spectrum_rows_kernel  4096-point transforms of the rows k1 and L1 - k1, whose
//                         frequencies mirror each other, and their amplitudes
// Every access is a contiguous run (at least 256 bytes of samples and 1 KB of
// transforms up to L = 2^18, 16 times less at 2^22), and the amplitudes are
// stored by rows, [k1][k2], which the selection's scan reads back in bins.
//
// Rounding, in units u of the norm (fft_core.h): four passes of the rows, 4 x 6 u
// and 3 x 19 u; up to four passes of the columns, 6 u each and 19 u but for the
// last; and the twiddles W_L^(n2 k1), powers of two table entries by repeated
// squaring, within 48 u at W^(7 ..) (f[7] below: 23 u for each of its factors), and
// their product, 2.3 u.  L = 2^18 has 81 + 31 + 50 = 162 u and 2^22 213 u at most;
// the selection's bound charges (lg L + 1) 21.7 u, 412 and 499 u.
//
// Measured on 300 windows of two channels and 150,001 samples (L = 2^18):
// 345 us for the columns (1.6 GB, 4.7 TB/s) and 560 us for the rows (1.9 GB, 3.4
// TB/s: one workgroup a CU), where even splits of L with radix-2 passes between
// LDS tiles took 752 and 805 us (16-byte pieces of samples, 64-byte pieces of
// transforms, 8-byte pieces of amplitudes).
#include <algorithm>

#include "fft_common.h"
#include "fft_core.h"
#include "internal.h"
#include "stats.h"

namespace gpoeo {
namespace {

struct SpectrumArgs {
    FftArgs f;                 // x, fstat, layout; tw: the tables of spectrum_prepare_kernel
    double2* z;                // [pairs][L1][4096]
    double* amp;               // [S][L1][kSpecRow]
    int32_t lg1;
};

__device__ __forceinline__ double2 turn_fwd(double2 z) { return make_double2(z.y, -z.x); }

// 2^r-point forward transforms in registers, natural order.
template <int r>
__device__ __forceinline__ void dft(double2* v) {
    if constexpr (r == 1) {
        const double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (r == 2) {
        const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
        const double2 c = cadd(v[1], v[3]), d = turn_fwd(csub(v[1], v[3]));
        v[0] = cadd(a, c);
        v[1] = cadd(b, d);
        v[2] = csub(a, c);
        v[3] = csub(b, d);
    } else {
        double2 w[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) w[m] = v[m];
        dft8<false, false>(w);
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = w[m];
    }
}

// log2 of the radix of the next pass with `left` bits of the length to go
// (threes, and one or two twos at the end).
constexpr int next_radix(int left) {
    return left % 3 == 0 || left == 5 || left > 5 ? 3 : (left >= 2 ? 2 : 1);
}

// Frequency (without its last digit) of group g of the last pass.
template <int kLg>
__device__ __forceinline__ int reverse_digits(int g) {
    int last = kLg, done = 0;
    while (next_radix(last) < last) last -= next_radix(last);
    int left = kLg, k = 0;
    while (left > last) {
        const int r = next_radix(left);
        k |= ((g >> (left - last - r)) & ((1 << r) - 1)) << done;
        done += r;
        left -= r;
    }
    return k;
}

// One pass of the L1-point transforms of a tile: point pos of column q at LDS
// slot of pos * Q + q.  Calls itself for the passes that follow.
template <int kLg, int kLeft>
__device__ __forceinline__ void column_passes(double2* lds, const SpectrumArgs& a, double2 (&v)[8],
                                              int64_t pair, int n20) {
    constexpr int r = next_radix(kLeft), kR = 1 << r, kSets = 8 / kR;
    constexpr int kLgQ = 12 - kLg;                          // columns of the tile
    const int t = (int)threadIdx.x;
    auto slot = [](int e) { return e + (e >> 3) + (e >> 6); };
#pragma unroll
    for (int u = 0; u < kSets; ++u) {
        const int gid = t + kT * u, q = gid & ((1 << kLgQ) - 1), g = gid >> kLgQ;
        const int c = g & ((1 << (kLeft - r)) - 1), blk = g >> (kLeft - r);
        const int e0 = (((blk << kLeft) + c) << kLgQ) + q;
        double2* w = v + kR * u;
        if constexpr (kLeft < kLg) {
#pragma unroll
            for (int m = 0; m < kR; ++m) w[m] = lds[slot(e0 + (m << (kLeft - r + kLgQ)))];
        }
        dft<r>(w);
        if constexpr (kLeft > r) {
            const double2* __restrict__ tw = a.f.tw;
            const int e = c << (12 - kLeft);                // W_(2^left)^c
            const double2 w1 = tw[e];
            w[1] = cmul(w[1], w1);
            if constexpr (r >= 2) {
                const double2 w2 = tw[2 * e], w3 = cmul(w1, w2);
                w[2] = cmul(w[2], w2);
                w[3] = cmul(w[3], w3);
                if constexpr (r == 3) {
                    const double2 w4 = tw[4 * e];
                    w[4] = cmul(w[4], w4);
                    w[5] = cmul(w[5], cmul(w1, w4));
                    w[6] = cmul(w[6], cmul(w2, w4));
                    w[7] = cmul(w[7], cmul(w3, w4));
                }
            }
#pragma unroll
            for (int m = 0; m < kR; ++m) lds[slot(e0 + (m << (kLeft - r + kLgQ)))] = w[m];
        } else {                                            // the last pass: rows of z
            // W_L^(n2 k1), k1 = kr + 2^(lg L1 - r) m, as W_L^(n2 kr) times powers of
            // W^n2 of 2^(12 + r): two contiguous reads a thread
            const int kr = reverse_digits<kLg>(g), n2 = n20 + q;
            double2 f[kR];
            f[0] = a.f.tw[kTw + kP + ((int64_t)kr << 12) + n2];
            const double2 s1 = a.f.tw[kTw + n2];
            f[1] = cmul(f[0], s1);
            if constexpr (r >= 2) {
                const double2 s2 = cmul(s1, s1);
                f[2] = cmul(f[0], s2);
                f[3] = cmul(f[1], s2);
                if constexpr (r == 3) {
                    const double2 s4 = cmul(s2, s2);
#pragma unroll
                    for (int m = 0; m < 4; ++m) f[4 + m] = cmul(f[m], s4);
                }
            }
            double2* __restrict__ zp = a.z + ((pair << kLg) << 12) + n2;
#pragma unroll
            for (int m = 0; m < kR; ++m)
                zp[(int64_t)(kr + (m << (kLg - r))) << 12] = cmul(w[m], f[m]);
        }
    }
    if constexpr (kLeft > r) {
        __syncthreads();
        column_passes<kLg, kLeft - r>(lds, a, v, pair, n20);
    }
}

// Workgroups of either launch, if there is as much work: each takes several
// tiles (row pairs) in turn, the next one's loads in flight meanwhile (columns
// 496 -> 345 us, rows 667 -> 560 us; 512 to 2048 row workgroups within 3%).
constexpr int64_t kColGroups = 2048, kRowGroups = 1024;

template <int kLg>
__global__ __launch_bounds__(kT, 4) void spectrum_cols_kernel(SpectrumArgs a) {
    constexpr int r = next_radix(kLg), kR = 1 << r, kSets = 8 / kR, kLgQ = 12 - kLg;
    __shared__ double2 lds[kSlots];
    const int64_t total = ((a.f.seqs + 1) / 2) << kLg;
    auto index = [&](int64_t id, int u, int m) {            // sample of point m of set u
        const int gid = (int)threadIdx.x + kT * u, q = gid & ((1 << kLgQ) - 1), g = gid >> kLgQ;
        return ((int64_t)(g + (m << (kLg - r))) << 12) + ((id & ((1 << kLg) - 1)) << kLgQ) + q;
    };
    float xa[8], xb[8];
    auto samples = [&](int64_t id) {
        const Seq qa = seq_of(a.f, 2 * (id >> kLg)), qb = seq_of(a.f, 2 * (id >> kLg) + 1);
#pragma unroll
        for (int u = 0; u < kSets; ++u)
#pragma unroll
            for (int m = 0; m < kR; ++m) {
                const int64_t i = index(id, u, m);
                xa[kR * u + m] = i < qa.n ? qa.p[i] : 0.0f;
                xb[kR * u + m] = i < qb.n ? qb.p[i] : 0.0f;
            }
    };
    int64_t id = blockIdx.x;
    samples(id);
    while (true) {
        const int64_t pair = id >> kLg;
        const Seq qa = seq_of(a.f, 2 * pair), qb = seq_of(a.f, 2 * pair + 1);
        double2 v[8];
#pragma unroll
        for (int u = 0; u < kSets; ++u)
#pragma unroll
            for (int m = 0; m < kR; ++m) {
                const int64_t i = index(id, u, m);
                v[kR * u + m] = make_double2(i < qa.n ? (double)xa[kR * u + m] - qa.mu : 0.0,
                                             i < qb.n ? (double)xb[kR * u + m] - qb.mu : 0.0);
            }
        const int64_t next = id + gridDim.x;
        if (next < total) samples(next);
        column_passes<kLg, kLg>(lds, a, v, pair, (int)(id & ((1 << kLg) - 1)) << kLgQ);
        if (next >= total) break;
        id = next;
        if constexpr (kLg > r) __syncthreads();             // all points read
    }
}

// Rows g and L1 - g of a pair (g = 0: rows 0 and L1 / 2, each its own mirror), one
// by either half of the workgroup.  (Both in turn by 512 threads, the first row's
// frequencies spill while the second is transformed: 1470 us.)
__global__ __launch_bounds__(2 * kT) void spectrum_rows_kernel(SpectrumArgs a) {
    __shared__ double2 tile[2][kSlots];
    __shared__ double2 tw512[256];
    const int32_t l1 = 1 << a.lg1, half = l1 >> 1;
    const int64_t total = ((a.f.seqs + 1) / 2) * half;
    const int side = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kT);
    double2* lds = tile[side];
    const Lanes at((int)threadIdx.x % kT);
    auto row_of = [&](int32_t g) { return side == 0 ? g : (g == 0 ? half : l1 - g); };
    double2 nxt[8];
    auto load = [&](int64_t id) {
        const double2* __restrict__ zp =
            a.z + ((((id / half) << a.lg1) + row_of((int32_t)(id % half))) << 12) + at.t;
#pragma unroll
        for (int r = 0; r < 8; ++r) nxt[r] = zp[kT * r];
    };
    if (threadIdx.x < 256) tw512[threadIdx.x] = a.f.tw[8 * threadIdx.x];
    load(blockIdx.x);
    for (int64_t id = blockIdx.x; id < total; id += gridDim.x) {
    const int64_t pair = id / half;
    const int32_t g = (int32_t)(id % half);
    const int32_t row = row_of(g);
    double2 v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = nxt[r];
    Twiddles t1;                                            // (kept, they would spill)
    t1.load(a.f.tw, at.t);
    forward_first<false>(lds, at, v, t1);
    __syncthreads();
    forward_rest(lds, at, v, tw512);
    __syncthreads();                                        // all points read
    // upper half (k2 >= 2048) of this row
#pragma unroll
    for (int r = 4; r < 8; ++r) lds[at.sk + 584 * (r - 4)] = v[r];
    __syncthreads();
    const double2 at_half = v[4];
    if (id + gridDim.x < total) load(id + gridDim.x);       // (earlier, the registers would spill)
    // mirror of (k1, k2): (L1 - k1, 4095 - k2); of row 0: (0, 4096 - k2)
    const int kappa = (at.t >> 6) + (at.t & 56) + 64 * (at.t & 7);   // k2 = kappa + 512 r
    const int u = kT - 1 - kappa;
    const int sm = u + (u >> 3) + (u >> 6);                 // + 584 (3 - r): 4095 - k2
    const double2* other = g == 0 ? lds : tile[1 - side];
    const bool zero = row == 0;
    double amp[2][4];                                       // of both sequences
    auto amplitudes = [](double2 zk, double2 zm, double& fa, double& fb) {
        const double ux = zk.x + zm.x, uy = zk.y - zm.y;
        const double vx = zk.x - zm.x, vy = zk.y + zm.y;
        fa = 0.5 * sqrt(ux * ux + uy * uy);
        fb = 0.5 * sqrt(vx * vx + vy * vy);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int s0 = kappa == 0 ? 584 * (4 - r) : at.sm + 584 * (3 - r);
        double2 m = other[zero ? s0 : sm + 584 * (3 - r)];
        const bool self = r == 0 && zero && kappa == 0;     // k = 0
        m.x = self ? v[r].x : m.x;
        m.y = self ? v[r].y : m.y;
        amplitudes(v[r], m, amp[0][r], amp[1][r]);
    }
    const int64_t seq_stride = (int64_t)kSpecRow << a.lg1;
    double* __restrict__ out = a.amp + 2 * pair * seq_stride;
    const bool pair_b = 2 * pair + 1 < a.f.seqs;
    if (zero && at.t == 0) {                                // k = L / 2
        double fa, fb;
        amplitudes(at_half, at_half, fa, fb);
        out[kP / 2] = fa;
        if (pair_b) out[seq_stride + kP / 2] = fb;
    }
    __syncthreads();                                        // all mirrors read
    double* flat = reinterpret_cast<double*>(lds);          // two lists of 2048 in order of k2
    constexpr int kList = 584 * 4;
#pragma unroll
    for (int l = 0; l < 2; ++l)
#pragma unroll
        for (int r = 0; r < 4; ++r) flat[kList * l + at.sk + 584 * r] = amp[l][r];
    __syncthreads();
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        if (l == 1 && !pair_b) continue;
        double* __restrict__ o = out + l * seq_stride + (int64_t)row * kSpecRow + at.t;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[kT * r] = flat[kList * l + at.s1 + 584 * r];
    }
    __syncthreads();                                        // the next rows reuse the LDS
    }
}

// The twiddle tables, W_4096^e (e < 2048); W^n2 of 2^(12 + r) (n2 < 4096, r = log2
// of the columns' last radix); W_L^(kr n2), kr < L1 / 2^r; and beside them, in
// the first workgroups, the statistics of every sequence as the statistics
// kernel computes them (one launch less).
template <int kT>
__global__ __launch_bounds__(kT) void spectrum_prepare_kernel(FftArgs a, double* var, double* fstat,
                                                              double2* tw, int lg, int r,
                                                              int64_t total) {
    __shared__ double red[4 * kT / kWave];
    if ((int64_t)blockIdx.x < a.seqs) {
        const int64_t s = blockIdx.x;
        const stats::ChannelStats st =
            stats::channel_stats<kT>(a.x + s / a.num_channels * a.window_stride +
                                         s % a.num_channels * a.channel_stride,
                                     a.n_all, red);
        if (threadIdx.x == 0) {
            var[2 * s] = st.var;
            var[2 * s + 1] = st.absmean;
            fstat[4 * s] = st.mean;
            fstat[4 * s + 1] = st.sq;
            fstat[4 * s + 2] = st.sabs;
            fstat[4 * s + 3] = 0.0;
        }
        return;
    }
    for (int64_t e = (blockIdx.x - a.seqs) * (int64_t)kT + threadIdx.x; e < total;
         e += (gridDim.x - a.seqs) * (int64_t)kT) {
        int64_t m = e;
        int lgl = 12;
        if (e >= kTw + kP) {
            const int64_t i = e - kTw - kP;
            m = (i >> 12) * (i & (kP - 1));
            lgl = lg;
        } else if (e >= kTw) {
            m = e - kTw;
            lgl = 12 + r;
        }
        double sn, cs;
        sincospi(ldexp(2.0 * (double)m, -lgl), &sn, &cs);   // exact argument
        tw[e] = make_double2(cs, -sn);
    }
}

constexpr int last_radix(int lg1) {
    while (next_radix(lg1) < lg1) lg1 -= next_radix(lg1);
    return lg1;
}

template <int kLg>
void launch_cols(const SpectrumArgs& a, int64_t pairs, hipStream_t s) {
    hipLaunchKernelGGL(spectrum_cols_kernel<kLg>,
                       dim3((unsigned)std::min(pairs << kLg, kColGroups)), dim3(kT), 0, s, a);
}

}  // namespace

int64_t spectrum_twiddles(int32_t lg) {
    return kTw + kP + ((int64_t(1) << lg) >> last_radix(lg - kFftBlockLog2));
}

namespace {

SpectrumArgs spectrum_args(const Plan& p, const float* x) {
    SpectrumArgs a = {};
    a.f.x = x;
    a.f.seqs = p.num_windows * (int64_t)p.num_channels;
    a.f.n_all = p.n;
    a.f.window_stride = p.window_stride;
    a.f.channel_stride = p.channel_stride;
    a.f.num_channels = p.num_channels;
    a.lg1 = p.fft_log2 - kFftBlockLog2;
    return a;
}

}  // namespace

hipError_t launch_spectrum_prepare(const Plan& p, const float* x, double* var, double* fstat,
                                   double* tw, hipStream_t s) {
    const SpectrumArgs a = spectrum_args(p, x);
    const int64_t entries = spectrum_twiddles(p.fft_log2);
    const int r = last_radix(a.lg1);
    double2* const tw2 = reinterpret_cast<double2*>(tw);
    const unsigned groups = (unsigned)a.f.seqs;
    if (p.n > kFusedMaxN && a.f.seqs <= kStatsLongMaxSeqs)
        hipLaunchKernelGGL(spectrum_prepare_kernel<stats::kStatsLongThreads>,
                           dim3(groups + (unsigned)std::min<int64_t>(entries / 1024, 1024)),
                           dim3(stats::kStatsLongThreads), 0, s, a.f, var, fstat, tw2, p.fft_log2,
                           r, entries);
    else
        hipLaunchKernelGGL(spectrum_prepare_kernel<stats::kStatsThreads>,
                           dim3(groups + (unsigned)std::min<int64_t>(entries / 256, 4096)),
                           dim3(stats::kStatsThreads), 0, s, a.f, var, fstat, tw2, p.fft_log2, r,
                           entries);
    return hipGetLastError();
}

hipError_t launch_spectrum(const Plan& p, const float* x, const double* fstat, const double* tw,
                           double* z, double* amp, hipStream_t s) {
    SpectrumArgs a = spectrum_args(p, x);
    a.f.fstat = fstat;
    a.f.tw = reinterpret_cast<const double2*>(tw);
    a.z = reinterpret_cast<double2*>(z);
    a.amp = amp;
    switch (a.lg1) {
        case 1: launch_cols<1>(a, p.fft_pairs, s); break;
        case 2: launch_cols<2>(a, p.fft_pairs, s); break;
        case 3: launch_cols<3>(a, p.fft_pairs, s); break;
        case 4: launch_cols<4>(a, p.fft_pairs, s); break;
        case 5: launch_cols<5>(a, p.fft_pairs, s); break;
        case 6: launch_cols<6>(a, p.fft_pairs, s); break;
        case 7: launch_cols<7>(a, p.fft_pairs, s); break;
        case 8: launch_cols<8>(a, p.fft_pairs, s); break;
        case 9: launch_cols<9>(a, p.fft_pairs, s); break;
        default: launch_cols<10>(a, p.fft_pairs, s); break;
    }
    hipLaunchKernelGGL(spectrum_rows_kernel,
                       dim3((unsigned)std::min(p.fft_pairs << (a.lg1 - 1), kRowGroups)),
                       dim3(2 * kT), 0, s, a);
    return hipGetLastError();
}

}  // namespace gpoeo
