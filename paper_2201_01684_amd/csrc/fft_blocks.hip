// FFT scores of a batch from short transforms of sample blocks.
//
// r(T) = sum_i y_i y_{i+T} is needed only for T <= Tmax, a fraction of N, so the
// sequence is cut into blocks x_b of m = 2048 samples and
//   r(j m + n) = sum_b sum_{i<m} x_b(i) s_{b+j}(i + n),   0 < n <= m,
// with s_b the 2m samples of blocks b and b + 1.  With X_b the 2m-point
// transform of the zero-padded block, the transform of s_b is X_b(k) +
// (-1)^k X_{b+1}(k), so that the spectrum of r over lags j m + 1 .. (j + 1) m is
//   R_j(k) = C_j(k) + (-1)^k C_{j+1}(k),   C_j(k) = sum_b conj(X_b(k)) X_{b+j}(k).
// Three launches do it:
//   blocks_fwd_kernel   X_b of every block, one 4096-point transform a workgroup
//   blocks_corr_kernel  C_j along the blocks, every frequency on its own
//   blocks_inv_kernel   r of m lags from R_j, and their D(T)
// and a pair whose sequences fit one transform is done by the last of them alone.
//
// Against one transform of N + Tmax points split into columns and rows, the
// spectra take two sweeps of 2N points instead of four of 2^k >= N + Tmax (or of
// 2^k >= N and six of the head-tail transform), every access is a contiguous
// run of at least 512 bytes, and N is padded to a multiple of 2048 instead of a
// power of two.  The sums over the blocks cost 4 N Tmax / 2048 multiply-adds a
// sequence, below the memory time up to Tmax of about 100,000.
//
// Measured on 1024 windows of 262,144 samples, T up to 32,768 (all three are
// bound by memory; a 2 GiB copy runs at 4.9 TB/s): forward 1.08 ms for 5.4 GB,
// block sums 1.15 ms for 4.8 GB, inverse 0.29 ms for 1.2 GB, where the long
// transforms and their wrap term took 4.38 ms for 15.3 GB.
#include <algorithm>
#include <cmath>

#include "fft_common.h"
#include "fft_core.h"
#include "internal.h"

namespace gpoeo {
namespace {

constexpr int kM = kFftBlockSamples;         // 2048 samples a block
static_assert(kP == kFftBlockPoints && kP == 2 * kM, "a block and as many zeros");

struct BlockArgs {
    FftArgs f;                 // x, fstat, edge, part, s64, scores, layout (f.lg = log2 kP)
    // The entry t + 512 r of a spectrum, r < 4, is the frequency thread t of a
    // transform ends with (Lanes): all of them below 2048 once.
    double2* z;                // [2 pairs of this launch][nb][kM]: 2 X_b(k) of each sequence
    double2* r;                // [2 pairs of this launch][jmax][kM]: 4 R_j(k)
    int64_t pair0;             // first pair of this launch
    int32_t nb, jmax;          // blocks and lag tiles of the longest window
    int32_t one;               // the inverse launch does the pairs of one transform alone
    int32_t step;              // workgroups per pair of the forward launch
};

// Samples, blocks and lag tiles of sequence s (none for an empty slot or past
// the last sequence).
struct Span {
    int64_t n;
    int32_t nb, j;
    bool whole;                // n + Tmax points fit one transform
};
__device__ __forceinline__ Span span_of(const FftArgs& a, int64_t s) {
    Span v = {0, 0, 0, true};
    if (s >= a.seqs) return v;
    const int64_t b = s / a.num_channels;
    v.n = table_n(a.tab, b, a.n_all);
    if (v.n <= 0) return v;
    const int32_t tmax = min(table_tmax(a.tab, b, a.tmax), a.tmax);
    v.nb = (int32_t)((v.n + kM - 1) / kM);
    v.j = (tmax + kM - 1) / kM;
    v.whole = v.n + tmax <= kP;
    return v;
}

// Passes of an inverse transform from the frequencies of this thread in v (the
// forward one's backwards) to the points t + 512 r; the first barrier is after
// the reads that filled v.
__device__ __forceinline__ void inverse_passes(double2* lds, const Lanes& at, double2 (&v)[8],
                                               const Twiddles& t1, const Twiddles& t2,
                                               const Twiddles& t3) {
    dft8<true, false>(v);
    __syncthreads();                                              // all mirrors read
    put8<1>(lds, at.s4, v);
    wave_exchange();
    get8<9>(lds, at.s3, v);
    twiddle8<true>(v, t3);
    dft8<true, false>(v);
    put8<9>(lds, at.s3, v);
    wave_exchange();
    get8<73>(lds, at.s2, v);
    twiddle8<true>(v, t2);
    dft8<true, false>(v);
    put8<73>(lds, at.s2, v);
    __syncthreads();
    get8<584>(lds, at.s1, v);
    twiddle8<true>(v, t1);
    dft8<true, false>(v);
}

// A pair whose sequences fit one transform (N + Tmax up to 4096 points): its
// spectrum, the power spectra 4 |A|^2 + 4 i |B|^2 and their inverse transform, the
// autocorrelations of all its lags, in one workgroup of the inverse launch; the
// other two leave the pair out.  Neither spectra nor lag tiles pass through
// memory: rolling detection of 1024 windows of 2048 samples 582 -> 393 us a call, of
// 8000 (suffixes of 45 to 1260) 623 -> 449; detection of 4000 windows of 2100, T up
// to 200, 322 -> 168.  (In the forward launch, whose loop it slows, 256 windows of
// 8000 took 344 instead of 286 us; a launch of its own costs 5 us.)
__device__ __forceinline__ void one_transform(const BlockArgs& a, double2* lds, double2* tw512,
                                              const Lanes& at, int64_t sa, int64_t sb) {
    const Seq qa = seq_of(a.f, sa), qb = seq_of(a.f, sb);
    const int c = at.t & 63;
    double2 v[8], q[4];
#pragma unroll
    for (int r = 0; r < 8; ++r)
        v[r] = make_double2(centred(qa, at.t + kT * r), centred(qb, at.t + kT * r));
    if (at.t < 256) tw512[at.t] = a.f.tw[8 * at.t];
    Twiddles t1, t2, t3;
    t1.load(a.f.tw, at.t);
    forward_first<false>(lds, at, v, t1);
    __syncthreads();
    forward_rest(lds, at, v, tw512);
    __syncthreads();                                              // all points read
#pragma unroll
    for (int r = 4; r < 8; ++r) lds[at.sk + 584 * r] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool edge = r == 0 && at.t == 0;                    // k = 0, with k = 2048
        const double2 zk = v[r];
        const double2 zm = lds[edge ? 584 * 4 : at.sm + 584 * (7 - r)];
        const double ux = zk.x + zm.x, uy = zk.y - zm.y, vx = zk.x - zm.x, vy = zk.y + zm.y;
        v[r] = make_double2(ux * ux + uy * uy, vx * vx + vy * vy);
        q[r] = v[r];
        if (edge) {
            v[r] = make_double2(4.0 * (zk.x * zk.x), 4.0 * (zk.y * zk.y));
            q[r] = make_double2(4.0 * (zm.x * zm.x), 4.0 * (zm.y * zm.y));
        }
    }
    __syncthreads();                                              // all mirrors read
#pragma unroll
    for (int r = 0; r < 4; ++r) lds[r == 0 && at.t == 0 ? 584 * 4 : at.sm + 584 * (7 - r)] = q[r];
    __syncthreads();
#pragma unroll
    for (int r = 4; r < 8; ++r) v[r] = lds[at.sk + 584 * r];
    t3.load(tw512, 8 * (c & 7));
    t2.load(tw512, c);
    inverse_passes(lds, at, v, t1, t2, t3);
#pragma unroll
    for (int r = 0; r < 3; ++r) {                                 // T <= 4096 / 3 < 1536
        write_d(a.f, sa, at.t + kT * r, v[r].x);
        write_d(a.f, sb, at.t + kT * r, v[r].y);
    }
}

// Workgroups of a forward launch (two fit a CU), if there are as many blocks
// (1024 to 8192 differ by 3% on 1024 x 262144 and 256 x 8 x 131072).
constexpr int64_t kFwdGroups = 4096;

// Transforms of blocks of a pair (a, b): z = y_a + i y_b, then the two spectra
// 2 A(k) = Z(k) + conj Z(P - k), 2 B(k) = (Z(k) - conj Z(P - k)) / i for k <
// 2048; the entry of k = 0 holds the two real values at k = 0 and k = 2048.  A
// workgroup takes every step-th block; the next one's samples are loaded while
// this one is transformed and the twiddles stay on chip (1.39 -> 1.08 ms on the
// batch above; 1.83 ms before the mirror exchange was halved to the upper four
// values).
__global__ __launch_bounds__(kT, 4) void blocks_fwd_kernel(BlockArgs a) {
    __shared__ double2 lds[kSlots];
    const int64_t pl = blockIdx.x / a.step;                       // pair within the launch
    const int64_t sa = 2 * (a.pair0 + pl), sb = sa + 1;
    const Seq qa = seq_of(a.f, sa), qb = seq_of(a.f, sb);
    const Span pa = span_of(a.f, sa), pb = span_of(a.f, sb);
    const int32_t na = pa.nb, nbb = pb.nb;
    const int32_t nb = max(na, nbb);
    if (a.one && pa.whole && pb.whole) return;
    const Lanes at((int)threadIdx.x);
    float xa[4], xb[4];
    auto samples = [&](int32_t b) {
        const int64_t i0 = (int64_t)b * kM + at.t;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = i0 + kT * r;
            xa[r] = i < qa.n ? qa.p[i] : 0.0f;
            xb[r] = i < qb.n ? qb.p[i] : 0.0f;
        }
    };
    int32_t b = (int32_t)(blockIdx.x % a.step);
    if (b >= nb) return;
    samples(b);
    // the first pass's twiddles stay in registers, W_512^e for the others in LDS
    // (ordered before its first reads by the first pass's barrier)
    __shared__ double2 tw512[256];
    Twiddles t1;
    t1.load(a.f.tw, at.t);
    if (at.t < 256) tw512[at.t] = a.f.tw[8 * at.t];
    while (true) {
        double2 v[8];
        const int64_t i0 = (int64_t)b * kM + at.t;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = i0 + kT * r;
            v[r] = make_double2(i < qa.n ? (double)xa[r] - qa.mu : 0.0,
                                i < qb.n ? (double)xb[r] - qb.mu : 0.0);
        }
        const int32_t next = b + a.step;
        if (next < nb) samples(next);
        forward_first<true>(lds, at, v, t1);
        __syncthreads();
        forward_rest(lds, at, v, tw512);
        __syncthreads();                                          // all points read
#pragma unroll
        for (int r = 4; r < 8; ++r) lds[at.sk + 584 * r] = v[r];
        __syncthreads();
        double2* __restrict__ za = a.z + ((2 * pl) * a.nb + b) * (int64_t)kM + at.t;
        double2* __restrict__ zb = za + (int64_t)a.nb * kM;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool edge = r == 0 && at.t == 0;                // k = 0, with k = 2048
            const double2 zk = v[r];
            const double2 zm = lds[edge ? 584 * 4 : at.sm + 584 * (7 - r)];
            double2 va = make_double2(zk.x + zm.x, zk.y - zm.y);
            double2 vb = make_double2(zk.y + zm.y, zm.x - zk.x);
            if (edge) {
                va = make_double2(2.0 * zk.x, 2.0 * zm.x);
                vb = make_double2(2.0 * zk.y, 2.0 * zm.y);
            }
            if (b < na) za[kT * r] = va;
            if (b < nbb) zb[kT * r] = vb;
        }
        if (next >= nb) break;
        b = next;
        __syncthreads();                                          // all mirrors read
    }
}

// C_j0 .. C_{j0+kJ} of one sequence and frequency a thread, then R_j.  The
// spectra of consecutive blocks stream through a ring of registers, kAhead of
// them loaded before they are needed.  With more than kJ lag tiles (kOffset) a
// workgroup takes kJ of them, from j0 = kJ blockIdx.y on, and block b's own
// spectrum is a second stream.  Entry 0's two real values are multiplied
// separately (p, q below).
constexpr int kCorrThreads = 256;
template <int kJ, bool kOffset>
__global__ __launch_bounds__(kCorrThreads) void blocks_corr_kernel(BlockArgs a) {
    constexpr int kAhead = kOffset ? 2 : 3;
    constexpr int kRing = kJ + 1 + kAhead;
    constexpr int kParts = kM / kCorrThreads;
    const int64_t sl = blockIdx.x / kParts;
    const Span sp = span_of(a.f, 2 * a.pair0 + sl);
    if (a.one && sp.whole && span_of(a.f, (2 * a.pair0 + sl) ^ 1).whole) return;
    const int32_t j0 = kOffset ? kJ * (int32_t)blockIdx.y : 0;
    if (j0 >= sp.j) return;
    const int k = (int)(blockIdx.x % kParts) * kCorrThreads + (int)threadIdx.x;
    const double2* __restrict__ zp = a.z + sl * a.nb * (int64_t)kM + k;
    const bool real2 = k == 0;
    auto spectrum = [&](int32_t b) {
        return b < sp.nb ? zp[(int64_t)b * kM] : make_double2(0.0, 0.0);
    };
    double2 ring[kRing], acc[kJ + 1];
#pragma unroll
    for (int i = 0; i <= kJ; ++i) acc[i] = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < kRing; ++i) ring[i] = spectrum(j0 + i);
    double2 own = kOffset ? spectrum(0) : make_double2(0.0, 0.0);
    const int32_t last = sp.nb - j0;      // blocks past it have no partner
    for (int32_t b0 = 0; b0 < last; b0 += kRing) {
#pragma unroll
        for (int u = 0; u < kRing; ++u) {
            const int32_t b = b0 + u;
            if (b < last) {               // the same for every thread
                const double2 x = kOffset ? own : ring[u];
                if (kOffset) own = spectrum(b + 1);
                const double p = real2 ? 0.0 : x.y, q = real2 ? x.y : x.x, h = real2 ? 0.0 : -x.y;
#pragma unroll
                for (int j = 0; j <= kJ; ++j) {
                    const double2 y = ring[(u + j) % kRing];
                    acc[j].x = fma(x.x, y.x, acc[j].x);
                    acc[j].y = fma(q, y.y, acc[j].y);
                    acc[j].x = fma(p, y.y, acc[j].x);
                    acc[j].y = fma(h, y.x, acc[j].y);
                }
                ring[u] = spectrum(b + j0 + kRing);
            }
        }
    }
    // entry k holds a frequency of parity w = k / 64 (mod 8)
    const double sign = (k & 64) ? -1.0 : 1.0;
    double2* __restrict__ out = a.r + (sl * a.jmax + j0) * (int64_t)kM + k;
#pragma unroll
    for (int j = 0; j < kJ; ++j)
        if (j0 + j < sp.j)
            out[(int64_t)j * kM] = make_double2(fma(sign, acc[j + 1].x, acc[j].x),
                                                fma(sign, acc[j + 1].y, acc[j].y));
}

// r(T) of both sequences of a pair for one tile of lags: Q = R_a + i R_b over
// all 4096 frequencies, its inverse transform (the passes of the forward one
// backwards), and D(T) for T = 2048 j + n, 0 < n <= 2048.  The energies of
// those lags are loaded before the transform (0.32 -> 0.29 ms).
template <bool kOne>
__global__ __launch_bounds__(kT, 4) void blocks_inv_kernel(BlockArgs a) {
    __shared__ double2 lds[kSlots];
    // pairs in turn; or lag tiles in turn where whole pairs, which take twice as
    // long, are among the first tiles, so that none of them starts last (rolling
    // detection of 128 windows of 100,001 samples 662 -> 606 us a call)
    const uint32_t pairs = gridDim.x / (uint32_t)a.jmax;
    const int64_t pl = kOne ? blockIdx.x % pairs : blockIdx.x / a.jmax;
    const int32_t j = (int32_t)(kOne ? blockIdx.x / pairs : blockIdx.x % a.jmax);
    const int64_t sa = 2 * (a.pair0 + pl), sb = sa + 1;
    const Span pa = span_of(a.f, sa), pb = span_of(a.f, sb);
    if (j >= max(pa.j, pb.j)) return;
    const Lanes at((int)threadIdx.x);
    if constexpr (kOne) {
        __shared__ double2 tw512[256];
        if (pa.whole && pb.whole) {
            one_transform(a, lds, tw512, at, sa, sb);
            return;
        }
    }
    const int c = at.t & 63;
    const double2* __restrict__ ra = a.r + ((2 * pl) * a.jmax + j) * (int64_t)kM + at.t;
    const double2* __restrict__ rb = ra + (int64_t)a.jmax * kM;
    double2 va[4], vb[4], v[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        va[r] = j < pa.j ? ra[kT * r] : make_double2(0.0, 0.0);
        vb[r] = j < pb.j ? rb[kT * r] : make_double2(0.0, 0.0);
    }
    Twiddles t3, t2, t1;
    t3.load(a.f.tw, 64 * (c & 7));
    t2.load(a.f.tw, 8 * c);
    t1.load(a.f.tw, at.t);
    const int64_t t0 = (int64_t)j * kM + at.t;
    // lags t0 + 512 r, r < 4 (n = 0 is another tile's: thread 0 takes n = 2048
    // in its place)
    auto lag_of = [&](int r) { return r == 0 && at.t == 0 ? t0 + kM : t0 + kT * r; };
    double ea[4], eb[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        ea[r] = lag_energy(a.f, sa, lag_of(r));
        eb[r] = lag_energy(a.f, sb, lag_of(r));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool edge = r == 0 && at.t == 0;
        double2 qm = make_double2(va[r].x + vb[r].y, vb[r].x - va[r].y);
        v[r] = make_double2(va[r].x - vb[r].y, va[r].y + vb[r].x);
        if (edge) {                                               // k = 0 and k = 2048
            v[r] = make_double2(va[r].x, vb[r].x);
            qm = make_double2(va[r].y, vb[r].y);
        }
        lds[edge ? 584 * 4 : at.sm + 584 * (7 - r)] = qm;
    }
    __syncthreads();
#pragma unroll
    for (int r = 4; r < 8; ++r) v[r] = lds[at.sk + 584 * r];
    inverse_passes(lds, at, v, t1, t2, t3);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double2 y = r == 0 && at.t == 0 ? v[4] : v[r];
        write_lag(a.f, sa, lag_of(r), ea[r], y.x);
        write_lag(a.f, sb, lag_of(r), eb[r], y.y);
    }
}

}  // namespace

hipError_t launch_fft_blocks(const Plan& p, const FftBlockBuffers& u, const float* x,
                             const double* fstat, double* edge, double* part, double* s64,
                             float* scores, float w0, hipStream_t s) {
    BlockArgs a = {};
    a.f.x = x;
    a.f.fstat = fstat;
    a.f.edge = edge;
    a.f.tw = reinterpret_cast<const double2*>(u.tw);
    a.f.part = part;
    a.f.seqs = p.num_windows * (int64_t)p.num_channels;
    a.f.n_all = p.n;
    a.f.window_stride = p.window_stride;
    a.f.channel_stride = p.channel_stride;
    a.f.num_channels = p.num_channels;
    a.f.tmin = p.tmin;
    a.f.tmax = p.tmax;
    a.f.lags = p.lags;
    a.f.tab = p.table;
    a.f.lg = kFftBlockLog2;
    a.f.len = kP;
    a.f.s64 = s64;
    a.f.scores = scores;
    a.f.w0 = w0;
    a.z = reinterpret_cast<double2*>(u.z);
    a.r = reinterpret_cast<double2*>(u.r);
    a.nb = p.blk_nb;
    a.jmax = p.blk_j;
    a.one = p.blk_whole || p.fft_table;
    for (int64_t p0 = 0; p0 < p.fft_pairs; p0 += p.blk_pairs) {
        const int64_t pc = std::min(p.blk_pairs, p.fft_pairs - p0);
        a.pair0 = p0;
        a.step = (int32_t)std::min<int64_t>(p.blk_nb, (kFwdGroups + pc - 1) / pc);
        const dim3 inv((unsigned)(pc * a.jmax));
        if (p.blk_whole) {
            hipLaunchKernelGGL(blocks_inv_kernel<true>, inv, dim3(kT), 0, s, a);
            continue;
        }
        hipLaunchKernelGGL(blocks_fwd_kernel, dim3((unsigned)(pc * a.step)), dim3(kT), 0, s, a);
        const dim3 grid((unsigned)(2 * pc * (kM / kCorrThreads))), block(kCorrThreads);
        if (p.blk_j > 16)
            hipLaunchKernelGGL((blocks_corr_kernel<16, true>),
                               dim3(grid.x, (unsigned)((p.blk_j + 15) / 16)), block, 0, s, a);
        else if (p.blk_j > 8)
            hipLaunchKernelGGL((blocks_corr_kernel<16, false>), grid, block, 0, s, a);
        else if (p.blk_j > 4)
            hipLaunchKernelGGL((blocks_corr_kernel<8, false>), grid, block, 0, s, a);
        else if (p.blk_j > 2)
            hipLaunchKernelGGL((blocks_corr_kernel<4, false>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((blocks_corr_kernel<2, false>), grid, block, 0, s, a);
        if (a.one)
            hipLaunchKernelGGL(blocks_inv_kernel<true>, inv, dim3(kT), 0, s, a);
        else
            hipLaunchKernelGGL(blocks_inv_kernel<false>, inv, dim3(kT), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace gpoeo
