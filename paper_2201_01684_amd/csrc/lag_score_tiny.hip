// Lag scores of tiny problems (one short trace, a few lags: the online case of
// Algorithm 3): one workgroup per (sequence, block of kTinyLags lags, chunk of
// kTinyChunk samples).  The chunk x[i0 .. i0 + kTinyChunk) and its partners
// x[i0 + T0 .. i0 + T0 + kTinyChunk + kTinyLags) are staged in LDS once (zeros
// past the window).  Wavefront w takes a quarter of the chunk's samples and lane
// l the lags T0 + 4 l .. + 3: four samples and four new partners (two 16-byte
// reads) make sixteen pairs, each quarter an fp32 run of at most 64 terms per
// lag (within the main kernel's bound), and the four quarters are added in
// fp64.  Every load is issued at the start, so the kernel takes about one memory
// round trip plus 16 steps (one window of 4096 samples, 1023 lags: 5.0 us; 6.4
// with one lag a lane, two LDS reads a pair and 256 steps).
//
// The statistics of every sequence (stats::channel_stats) ride along in
// workgroups of their own when the fused finish kernel will need them: they run
// beside the scores instead of in front of the selection.
#include "internal.h"
#include "stats.h"

namespace gpoeo {
namespace {

struct TinyArgs {
    const float* x;
    double* part;              // [window*C + channel][chunk][lags_padded]
    double* var;               // [window*C + channel][2], or null
    int64_t n, window_stride, channel_stride, seqs;
    int32_t num_channels, t0, lag_blocks, lags_padded, chunks;
};

constexpr int kWaves = kTinyLags / kWave;
constexpr int kQuarter = kTinyChunk / kWaves;
static_assert(kTinyLags == 4 * kWave && kTinyLags == stats::kStatsThreads && kQuarter % 4 == 0,
              "four lags a lane, four samples a step, a statistics workgroup as wide");

__global__ __launch_bounds__(kTinyLags) void lag_score_tiny_kernel(TinyArgs a) {
    __shared__ __attribute__((aligned(16))) float xa[kTinyChunk];
    __shared__ __attribute__((aligned(16))) float xb[kTinyChunk + kTinyLags];
    __shared__ __attribute__((aligned(16))) float sums[kWaves][kTinyLags];
    __shared__ double red[4 * kWaves];
    const int tid = threadIdx.x;
    int64_t task = blockIdx.x;
    if (a.var) {                          // the first workgroups: statistics
        if (task < a.seqs) {
            const int64_t b = task / a.num_channels;
            const int64_t c = task % a.num_channels;
            const stats::ChannelStats st = stats::channel_stats<kTinyLags>(
                a.x + b * a.window_stride + c * a.channel_stride, a.n, red);
            if (tid == 0) {
                a.var[2 * task] = st.var;
                a.var[2 * task + 1] = st.absmean;
            }
            return;
        }
        task -= a.seqs;
    }
    const int32_t k = (int32_t)(task % a.chunks);
    const int64_t rest = task / a.chunks;
    const int32_t blk = (int32_t)(rest % a.lag_blocks);
    const int64_t bc = rest / a.lag_blocks;
    const int64_t b = bc / a.num_channels;
    const int32_t c = (int32_t)(bc % a.num_channels);
    const float* __restrict__ xw = a.x + b * a.window_stride + (int64_t)c * a.channel_stride;
    const int64_t n = a.n;
    const int64_t i0 = (int64_t)k * kTinyChunk;
    const int64_t t_blk = (int64_t)a.t0 + (int64_t)blk * kTinyLags;
    for (int j = tid; j < kTinyChunk; j += kTinyLags) xa[j] = i0 + j < n ? xw[i0 + j] : 0.0f;
    for (int j = tid; j < kTinyChunk + kTinyLags; j += kTinyLags) {
        const int64_t idx = i0 + t_blk + j;
        xb[j] = idx < n ? xw[idx] : 0.0f;
    }
    __syncthreads();
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    // pair (i, lag 4 lane + j) of the chunk counts iff i + 4 lane + j < rem
    const int64_t left = n - i0 - t_blk;
    const int rem = (int)min(left, (int64_t)(2 * kTinyChunk + kTinyLags)) - 4 * lane;
    const float4* __restrict__ a4 = reinterpret_cast<const float4*>(xa) + wave * (kQuarter / 4);
    const float4* __restrict__ b4 =
        reinterpret_cast<const float4*>(xb) + wave * (kQuarter / 4) + lane;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float4 lo = b4[0];
    auto steps = [&](auto&& valid) {
#pragma unroll 4
        for (int q = 0; q < kQuarter / 4; ++q) {
            const float4 u4 = a4[q], hi = b4[q + 1];
            const float u[4] = {u4.x, u4.y, u4.z, u4.w};
            const float y[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d = valid(wave * kQuarter + 4 * q + i + j) ? u[i] - y[i + j] : 0.0f;
                    acc[j] = __builtin_fmaf(d, d, acc[j]);
                }
            lo = hi;
        }
    };
    if (left >= kTinyChunk + kTinyLags)   // every pair of the workgroup
        steps([](int) { return true; });
    else
        steps([&](int s) { return s < rem; });
    *reinterpret_cast<float4*>(&sums[wave][4 * lane]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    __syncthreads();
    double d = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) d = d + (double)sums[w][tid];
    a.part[(bc * a.chunks + k) * (int64_t)a.lags_padded + (t_blk - a.t0) + tid] = d;
}

}  // namespace

hipError_t launch_lag_score_tiny(const Plan& p, const float* x, double* part, double* var,
                                 hipStream_t s) {
    TinyArgs a;
    a.x = x;
    a.part = part;
    a.var = var;
    a.n = p.n;
    a.window_stride = p.window_stride;
    a.channel_stride = p.channel_stride;
    a.seqs = p.num_windows * (int64_t)p.num_channels;
    a.num_channels = p.num_channels;
    a.t0 = p.t0;
    a.lag_blocks = p.lag_blocks;
    a.lags_padded = p.lags_padded;
    a.chunks = p.chunks;
    const int64_t groups = a.seqs * p.lag_blocks * (int64_t)p.chunks + (var ? a.seqs : 0);
    hipLaunchKernelGGL(lag_score_tiny_kernel, dim3((unsigned)groups), dim3(kTinyLags), 0, s, a);
    return hipGetLastError();
}

}  // namespace gpoeo
