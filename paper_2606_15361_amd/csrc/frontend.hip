// On-device front end for gfx950: delta encoders, storage cast, time scrunch, clipped channel
// statistics, normalisation, channel flagging and zero-DM subtraction (Methods, "Input encoding",
// "Multi-rate extension"; Results, "False-positive rate").
//
// Every kernel here streams a filterbank once or twice and is bound by memory, so each one keeps
// several independent 16-byte (or whole-line) loads per lane in flight and writes whole dwords; rows
// need no alignment beyond their element's (unaligned 16-byte accesses are native).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "snd_internal.h"
#include "stage_common.h"

namespace snd {
namespace {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32u __attribute__((aligned(1)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));

__device__ inline f32x4u load4(global_ptr<const float> p) { return *reinterpret_cast<global_ptr<const f32x4u>>(p); }

constexpr int kRow = 4096;  // samples of a row per workgroup: 256 threads, four 16-byte loads each

// A workgroup's kRow samples of a row from t0 (n: the row's samples; row_threads threads): f(t, x) for every
// whole group of four, one(t, x) for the samples of the last, partial one.
template <typename F, typename G>
__device__ inline void row_quads(const float *row, int64_t t0, int64_t n, F &&f, G &&one)
{
    const auto src = as_global(row);
    const int64_t t = t0 + 4 * (int)threadIdx.x;
    if (t0 + kRow <= n) {  // uniform
        f32x4u v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load4(src + t + 1024 * u);
#pragma unroll
        for (int u = 0; u < 4; ++u) f(t + 1024 * u, v[u]);
        return;
    }
    for (int u = 0; u < 4; ++u) {
        const int64_t tu = t + 1024 * u;
        if (tu + 4 <= n) f(tu, load4(src + tu));
        else
            for (int64_t i = tu; i < n; ++i) one(i, src[i]);
    }
}

// ---------------------------------------------------------------------------------------
// Delta encoder (Methods, "Input encoding"): level = number of thresholds z exceeds.
// ---------------------------------------------------------------------------------------
struct Thresholds { float v[8]; int n; };

__device__ inline uint32_t level(const Thresholds &th, float x)
{
    uint32_t l = 0;
    for (int j = 0; j < th.n; ++j) l += x > th.v[j];
    return l;
}

// Channel-major input: four samples per dword store (one byte per lane and store took 0.30 ms for
// 1024 x 131,072 samples, this 0.13).
__global__ __launch_bounds__(256) void k_encode_cm(const float *z, int64_t zp, int64_t nsamp, Thresholds th,
                                                   uint8_t *out, int64_t op)
{
    const int c = blockIdx.y;
    const auto dst = as_global(out + (int64_t)c * op);
    row_quads(
        z + (int64_t)c * zp, (int64_t)blockIdx.x * kRow, nsamp,
        [&](int64_t t, f32x4u x) {
            const uint32_t w = level(th, x.x) | level(th, x.y) << 8 | level(th, x.z) << 16 | level(th, x.w) << 24;
            *reinterpret_cast<global_ptr<u32u>>(dst + t) = w;
        },
        [&](int64_t t, float x) { dst[t] = (uint8_t)level(th, x); });
}

// Time-major input, transposed through LDS: a tile of 64 channels x T samples.  A lane reads one
// channel of T / 4 consecutive samples (a wave reads whole 256-byte lines), packs four levels per dword
// and writes them to its channel's LDS row; the rows leave as runs of T bytes (64 x 64 tiles of bytes
// took 0.26 ms for 1024 x 131,072 samples, T = 256 takes 0.17).  Blocks of fewer than kTmBlocks such tiles
// take T = 64, since a wave's loads come in rounds of sixteen (four thresholds: 64 channels x 4000 samples
// 14.6 us by 256, 9.1 by 64; 1024 x 8192 16.0 and 10.9).
constexpr int64_t kTmBlocks = 1024, kTmBitBlocks = 512;

template <int T>
__global__ __launch_bounds__(256) void k_encode_tm(const float *z, int64_t zp, int nchan, int64_t nsamp, Thresholds th,
                                                   uint8_t *out, int64_t op)
{
    constexpr int W = T / 4, pitch = W + 1;  // dwords of an LDS row; odd pitch: a column of lanes spreads over the banks
    __shared__ uint32_t tile[64 * pitch];
    const int64_t tb = (int64_t)blockIdx.x * T;
    const int cb = blockIdx.y * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = cb + lane;
    const auto src = as_global(z) + c;
    const bool inside = tb + T <= nsamp && cb + 64 <= nchan;  // uniform
#pragma unroll 1
    for (int g = 0; g < W / 16; ++g) {  // 16 samples of the wave's T / 4 at a time
        const int64_t t = tb + W * wave + 16 * g;
        float x[16];
        if (inside) {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = src[(t + i) * zp];
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = t + i < nsamp && c < nchan ? src[(t + i) * zp] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            tile[lane * pitch + W / 4 * wave + 4 * g + q] =
                level(th, x[4 * q]) | level(th, x[4 * q + 1]) << 8 | level(th, x[4 * q + 2]) << 16 |
                level(th, x[4 * q + 3]) << 24;
    }
    __syncthreads();
    const int wl = lane & (W - 1);
    const int64_t t = tb + 4 * wl;
#pragma unroll 4
    for (int i = 0; i < 16; i += 64 / W) {
        const int r = 16 * wave + i + lane / W;  // channel within the tile
        if (cb + r >= nchan) break;
        const uint32_t w = tile[r * pitch + wl];
        const auto dst = as_global(out + (int64_t)(cb + r) * op + t);
        if (t + 4 <= nsamp) *reinterpret_cast<global_ptr<u32u>>(dst) = w;
        else
            for (int b = 0; b < 4 && t + b < nsamp; ++b) dst[b] = (uint8_t)(w >> (8 * b));
    }
}

// Bits: a wave tests 1024 consecutive samples of a channel, 64 per ballot (sixteen loads in flight),
// and writes their 32 words as one 128-byte store (one ballot and an 8-byte store per wave took
// 0.27 ms for 1024 x 131,072 samples, this 0.10).  Rows short of kRow take no more waves than they fill.
__global__ __launch_bounds__(256) void k_encode_bits_cm(const float *z, int64_t zp, int64_t nsamp, float th,
                                                        uint32_t *out, int64_t ow)
{
    const int c = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int64_t tb = (int64_t)blockIdx.x * kRow + (threadIdx.x >> 6) * 1024;  // first sample of the wave
    const auto src = as_global(z + (int64_t)c * zp) + tb + lane;
    float x[16];
    if (tb + 1024 <= nsamp) {  // uniform per wave
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = src[64 * u];
    } else {
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = tb + lane + 64 * u < nsamp ? src[64 * u] : -__builtin_inff();
    }
    uint32_t w = 0;  // lane l: word l of the wave
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const uint64_t mask = __ballot(x[u] > th && tb + lane + 64 * u < nsamp);
        w = lane == 2 * u ? (uint32_t)mask : lane == 2 * u + 1 ? (uint32_t)(mask >> 32) : w;
    }
    const int64_t wi = (tb >> 5) + lane;
    if (lane < 32 && 32 * wi < nsamp) as_global(out + (int64_t)c * ow)[wi] = w;
}

// Bits from time-major input: a lane builds the words of one channel from the samples it reads (a
// wave reads whole 256-byte lines), 32 samples each; the words of 64 channels x 128 K samples leave
// through LDS as runs of 4 K words of each row.  Blocks of fewer than kTmBitBlocks tiles of K = 8 take
// K = 2 (3 channels x 100,000 samples: 29 us by 8, with a branch for the last channels, 7.9).
template <int K>
__global__ __launch_bounds__(256) void k_encode_bits_tm(const float *z, int64_t zp, int nchan, int64_t nsamp,
                                                        float th, uint32_t *out, int64_t ow)
{
    constexpr int W = 4 * K;  // words of an LDS row
    __shared__ uint32_t tile[64 * (W + 1)];
    const int64_t tb = (int64_t)blockIdx.x * (32 * W);
    const int cb = blockIdx.y * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // lanes past the last channel read the last one's samples: their words are not stored
    const auto src = as_global(z) + (cb + lane < nchan ? cb + lane : nchan - 1);
#pragma unroll 1
    for (int k = 0; k < K; ++k) {  // the wave's words K wave + k
        const int64_t t = tb + 32 * (K * wave + k);
        float x[32];
        if (t + 32 <= nsamp) {  // uniform
#pragma unroll
            for (int i = 0; i < 32; ++i) x[i] = src[(t + i) * zp];
        } else {
#pragma unroll
            for (int i = 0; i < 32; ++i) x[i] = t + i < nsamp ? src[(t + i) * zp] : -__builtin_inff();
        }
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) w |= (uint32_t)(x[i] > th && t + i < nsamp) << i;
        tile[lane * (W + 1) + K * wave + k] = w;
    }
    __syncthreads();
    const int wl = lane & (W - 1);
    const int64_t wi = (tb >> 5) + wl;
    for (int r = 64 / W * wave + lane / W; r < 64; r += 256 / W)
        if (cb + r < nchan && 32 * wi < nsamp) as_global(out + (int64_t)(cb + r) * ow)[wi] = tile[r * (W + 1) + wl];
}

// Time scrunch: output t is the sum of s consecutive samples of one channel in order (FP32, no
// contraction), scaled by r.  S > 0: s known at compile time; a thread's outputs are 256 apart and
// each is S / 4 16-byte loads (S = 2: two neighbouring outputs per load).  One sample per load took
// 0.20 ms for 1024 x 131,072 samples at S = 2, 4 and 8, this 0.13, 0.12 and 0.11.
template <int S>
__global__ __launch_bounds__(256) void k_scrunch(const float *z, int64_t zp, int64_t nout, int s_, float r, float *out,
                                                 int64_t op)
{
    constexpr int U = S == 0 ? 1 : S <= 4 ? 8 : 32 / S;  // outputs per thread
    const int c = blockIdx.y;
    const int64_t t0 = (int64_t)blockIdx.x * 256 * U;
    const auto src = as_global(z + (int64_t)c * zp);
    const auto dst = as_global(out + (int64_t)c * op);
    auto one = [&](int64_t t) {
        const int s = S ? S : s_;
        const auto p = src + t * s;
        float acc = p[0];
        for (int j = 1; j < s; ++j) acc = acc + p[j];
        dst[t] = acc * r;
    };
    if constexpr (S >= 2) {
        if (t0 + 256 * U <= nout) {  // uniform
            constexpr int Q = S == 2 ? 1 : S / 4;     // loads per step
            constexpr int N = S == 2 ? U / 2 : U;     // steps
            f32x4u v[N][Q];
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    v[u][q] = load4(src + (S == 2 ? 2 * (t0 + 2 * (int)threadIdx.x + 512 * u)
                                                  : S * (t0 + (int)threadIdx.x + 256 * u) + 4 * q));
#pragma unroll
            for (int u = 0; u < N; ++u) {
                if constexpr (S == 2) {
                    const int64_t t = t0 + 2 * (int)threadIdx.x + 512 * u;
                    dst[t] = (v[u][0].x + v[u][0].y) * r;
                    dst[t + 1] = (v[u][0].z + v[u][0].w) * r;
                } else {
                    float acc = v[u][0].x;
#pragma unroll
                    for (int j = 1; j < S; ++j) acc = acc + v[u][j / 4][j % 4];
                    dst[t0 + (int)threadIdx.x + 256 * u] = acc * r;
                }
            }
            return;
        }
    }
    for (int u = 0; u < U; ++u) {
        const int64_t t = t0 + (int)threadIdx.x + 256 * u;
        if (t < nout) one(t);
    }
}

// Sum of one FP64 pair per thread over a workgroup of T threads, returned to every thread.
template <int T>
__device__ inline void block_sum2(double &a, double &b, double (*sh)[T / 64])
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = a;
        sh[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    a = sh[0][0];
    b = sh[1][0];
#pragma unroll
    for (int w = 1; w < T / 64; ++w) {
        a += sh[0][w];
        b += sh[1][w];
    }
    __syncthreads();
}

// Sigma-clip statistics of one channel per workgroup: a first FP64 pass about the channel's
// first sample gives mu0 and sigma0, a second pass the same statistics of the clipped values
// (about the clip range's centre, mu0).  Two workgroups of T = 1024 threads fill a CU, four 16-byte loads
// per lane in flight (256 threads with one 4-byte load each took 0.53 ms for 1024 x 131,072,
// this 0.18).  Shorter rows take T = 256 (up to 16,384 samples) or one wave (up to 1024), since all of a
// large workgroup's threads take part in its sums: 4096 x 1000 samples 64 us by 1024, 12 by 256, 8 by 64;
// 4096 x 8200 85 by 1024, 39 by 256.
template <int T, typename F>
__device__ inline void stat_fold(global_ptr<const float> row, int64_t n, F &&f)
{
    const int tid = threadIdx.x;
    const int64_t nv = n / 4;
    int64_t i = tid;
    for (; i + 3 * T < nv; i += 4 * T) {
        f32x4u v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load4(row + 4 * (i + u * T));
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) f(v[u][j]);
    }
    for (; i < nv; i += T) {
        const f32x4u v = load4(row + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) f(v[j]);
    }
    if (4 * nv + tid < n) f(row[4 * nv + tid]);
}

template <int T>
__global__ __launch_bounds__(T) void k_chanstats(const float *p, int64_t pp, int64_t n, double clip,
                                                            double *stats)
{
    __shared__ double sh[2][T / 64];
    const int c = blockIdx.x;
    const auto row = as_global(p + (int64_t)c * pp);
    const double shift = (double)row[0];
    double a = 0.0, b = 0.0;
    stat_fold<T>(row, n, [&](float x) {
        const double d = (double)x - shift;
        a += d;
        b += d * d;
    });
    block_sum2<T>(a, b, sh);
    const double dn = (double)n;
    const double m1 = a / dn;
    const double mu0 = shift + m1;
    const double v0 = b / dn - m1 * m1;
    const double s0 = v0 > 0.0 ? sqrt(v0) : 0.0;
    const double lo = mu0 - clip * s0, hi = mu0 + clip * s0;
    a = 0.0;
    b = 0.0;
    stat_fold<T>(row, n, [&](float x) {
        double v = (double)x;
        v = v < lo ? lo : (v > hi ? hi : v);
        const double d = v - mu0;
        a += d;
        b += d * d;
    });
    block_sum2<T>(a, b, sh);
    if (threadIdx.x == 0) {
        const double m = a / dn;
        const double v = b / dn - m * m;
        stats[2 * c] = mu0 + m;
        stats[2 * c + 1] = v > 0.0 ? sqrt(v) : 0.0;
    }
}

// (p - mu) / sigma as one FP64 quotient, rounded once (1024 x 131,072 samples: 0.17 ms, 6.5 TB/s; one
// sample per thread took 0.30).
__global__ __launch_bounds__(256) void k_normalize(const float *p, int64_t pp, int64_t n, const double *stats,
                                                   float *z, int64_t zp)
{
    const int c = blockIdx.y;
    const double mu = stats[2 * c], sg = stats[2 * c + 1];
    const auto dst = as_global(z + (int64_t)c * zp);
    auto norm = [&](float x) { return (float)(((double)x - mu) / sg); };
    row_quads(
        p + (int64_t)c * pp, (int64_t)blockIdx.x * kRow, n,
        [&](int64_t t, f32x4u x) {
            *reinterpret_cast<global_ptr<f32x4u>>(dst + t) = f32x4u{norm(x.x), norm(x.y), norm(x.z), norm(x.w)};
        },
        [&](int64_t t, float x) { dst[t] = norm(x); });
}

// Zero-DM subtraction: one lane per sample t sums the channels in order in FP64 (a wave reads
// whole lines of a channel row, kZdLoads rows in flight; one row at a time took 0.71 ms for
// 1024 x 131,072, this 0.10); when the zero-DM S/N |sum| / sqrt(nchan) exceeds gamma, the channel mean
// sum / nchan is subtracted from every channel, each result rounded once to FP32.  A few such
// samples of a wave are corrected one by one, a lane per channel; many of them as the sums were read.
constexpr int kZdLoads = 32;
constexpr int kZdFew = 8;
__global__ __launch_bounds__(64) void k_zero_dm(float *z, int64_t zp, int nchan, int64_t n, double gamma,
                                                int32_t *count)
{
    const int lane = threadIdx.x;
    const int64_t t = (int64_t)blockIdx.x * 64 + lane;
    const bool on = t < n;
    const auto col = as_global(z) + (on ? t : n - 1);
    double s = 0.0;
    int c = 0;
    for (; c + kZdLoads <= nchan; c += kZdLoads) {
        float v[kZdLoads];
#pragma unroll
        for (int u = 0; u < kZdLoads; ++u) v[u] = col[(int64_t)(c + u) * zp];
#pragma unroll
        for (int u = 0; u < kZdLoads; ++u) s += (double)v[u];
    }
    for (; c < nchan; ++c) s += (double)col[(int64_t)c * zp];
    const bool hit = on && __builtin_fabs(s) / __builtin_sqrt((double)nchan) > gamma;
    uint64_t hits = __ballot(hit);
    if (!hits) return;
    if (count && lane == 0) atomicAdd(count, (int)__popcll(hits));
    const double mean = s / (double)nchan;
    if (__popcll(hits) <= kZdFew) {  // uniform
        while (hits) {
            const int h = __builtin_ctzll(hits);
            hits &= hits - 1;
            const double m = __shfl(mean, h, 64);
            const auto p = as_global(z) + (int64_t)blockIdx.x * 64 + h;
            for (int c0 = 0; c0 < nchan; c0 += 256) {
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    v[u] = c0 + lane + 64 * u < nchan ? p[(int64_t)(c0 + lane + 64 * u) * zp] : 0.0f;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c0 + lane + 64 * u < nchan) p[(int64_t)(c0 + lane + 64 * u) * zp] = (float)((double)v[u] - m);
            }
        }
        return;
    }
    if (!hit) return;
    c = 0;
    for (; c + 8 <= nchan; c += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = col[(int64_t)(c + u) * zp];
#pragma unroll
        for (int u = 0; u < 8; ++u) col[(int64_t)(c + u) * zp] = (float)((double)v[u] - mean);
    }
    for (; c < nchan; ++c) col[(int64_t)c * zp] = (float)((double)col[(int64_t)c * zp] - mean);
}

// Windowed channel flagging by median absolute deviation, in two kernels.
// k_chan_window_sigma: one wave per (channel, window of w samples): s = the population standard
//   deviation over the window, each of its two FP64 sums (samples, then squared deviations from
//   the mean) taken as 64 interleaved partial sums -- lane j sums samples j, j + 64, ... in
//   order -- added in lane order.  Windows of up to 64 U samples stay in registers between the two
//   sums, so they are read once, with all their loads in flight; longer ones (U = 0) are read twice.
//   (Flagging 1024 x 131,072 samples in windows of 8192 took 0.71 ms with one load in flight, 0.18 this
//   way; with every window past 512 read twice 0.23, and 0.89 instead of 0.70 in windows of 1000.)
//   Writes sigma[window][channel].
// k_flag_window: each workgroup of a window finds m = the lower median of the window's s over the
//   channels and MAD = the lower median of |s_c - m|, then takes its share of the channels: channel c is
//   flagged when |s_c - m| > k * (kMad * MAD), kMad = 1 / Phi^-1(3/4), and its samples in the window are
//   set to 0.  Few windows take several workgroups each (one leaves most CUs idle while it zeroes: 0.17 ms
//   for 16 windows of 1024 channels, with sixteen 0.10), up to kFlagBlocks in all, one on each CU; since
//   each repeats the medians, more windows than that take one (512 windows of 256 samples: 4.3 ms
//   with sixteen each, 0.50).
constexpr double kFlagMadScale = 1.4826022185056018;
constexpr uint32_t kFlagSlices = 16, kFlagBlocks = 256;

__device__ inline double wave_sum_in_lane_order(double v, double *lds64)
{
    const int lane = threadIdx.x & 63;
    lds64[lane] = v;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double s = 0.0;
#pragma unroll 8
    for (int j = 0; j < 64; ++j) s += lds64[j];
    __builtin_amdgcn_wave_barrier();
    return s;
}

// f(x) for the lane's samples of the window in order, from registers (v) or from memory
template <int U, typename F>
__device__ inline void window_fold(global_ptr<const float> row, int64_t len, const float (&v)[U > 0 ? U : 1], F &&f)
{
    const int lane = threadIdx.x & 63;
    if constexpr (U > 0) {
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 8) {
            if (64 * (u0 + 8) <= len) {  // uniform
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u) f(v[u]);
            } else if (64 * u0 < len) {
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u)
                    if (lane + 64 * u < len) f(v[u]);
            }
        }
    } else {
        int64_t t = lane;
        for (; t + 64 * 31 < len; t += 64 * 32) {
            float x[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) x[u] = row[t + 64 * u];
#pragma unroll
            for (int u = 0; u < 32; ++u) f(x[u]);
        }
        for (; t < len; t += 64) f(row[t]);
    }
}

template <int U>
__global__ __launch_bounds__(256) void k_chan_window_sigma(const float *z, int64_t zp, int nchan, int64_t n,
                                                           int64_t w, double *sigma)
{
    __shared__ double part[4][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + wave;
    const int64_t b = blockIdx.y;
    if (c >= nchan) return;  // whole waves
    const int64_t t0 = b * w;
    const int64_t len = n - t0 < w ? n - t0 : w;
    const auto row = as_global(z + (int64_t)c * zp + t0);
    float v[U > 0 ? U : 1];
    if constexpr (U > 0) {
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 8) {
            if (64 * (u0 + 8) <= len) {  // uniform
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u) v[u] = row[lane + 64 * u];
            } else if (64 * u0 < len) {
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u) v[u] = lane + 64 * u < len ? row[lane + 64 * u] : 0.0f;
            }
        }
    }
    double a = 0.0;
    window_fold<U>(row, len, v, [&](float x) { a += (double)x; });
    const double mu = wave_sum_in_lane_order(a, part[wave]) / (double)len;
    double q = 0.0;
    window_fold<U>(row, len, v, [&](float x) {
        const double d = (double)x - mu;
        q += d * d;
    });
    const double qs = wave_sum_in_lane_order(q, part[wave]);
    if (lane == 0) sigma[b * nchan + c] = __builtin_sqrt(qs / (double)len);
}

// The value of rank r (0-based, increasing) among the non-negative v[0..n) in LDS: the largest of the
// values that at most r others lie below.  (Non-negative doubles order as their bits; NaNs never count.)
__device__ inline double lds_rank_value(const double *v, int n, int r, unsigned long long *best)
{
    if (threadIdx.x == 0) *best = 0ull;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const double x = v[i];
        int below = 0;
#pragma unroll 8
        for (int j = 0; j < n; ++j) below += v[j] < x;
        if (below <= r && x == x) atomicMax(best, (unsigned long long)__double_as_longlong(x));
    }
    __syncthreads();
    return __longlong_as_double((long long)*best);
}

__global__ __launch_bounds__(1024) void k_flag_window(float *z, int64_t zp, int nchan, int64_t n, int64_t w,
                                                      double k, const double *sigma, uint8_t *flags, int64_t fp)
{
    extern __shared__ double sv[];  // [nchan]: the window's sigmas, then their deviations
    __shared__ unsigned long long best;
    const int64_t b = blockIdx.x;
    const int64_t t0 = b * w;
    const int64_t len = n - t0 < w ? n - t0 : w;
    for (int c = threadIdx.x; c < nchan; c += blockDim.x) sv[c] = sigma[b * nchan + c];
    const int r = (nchan - 1) / 2;
    const double m = lds_rank_value(sv, nchan, r, &best);
    __syncthreads();
    for (int c = threadIdx.x; c < nchan; c += blockDim.x) sv[c] = __builtin_fabs(sv[c] - m);
    const double thr = k * (kFlagMadScale * lds_rank_value(sv, nchan, r, &best));
    const int c0 = (int)((int64_t)nchan * blockIdx.y / gridDim.y), c1 = (int)((int64_t)nchan * (blockIdx.y + 1) / gridDim.y);
    if (flags)
        for (int c = c0 + (int)threadIdx.x; c < c1; c += blockDim.x) flags[b * fp + c] = sv[c] > thr ? 1 : 0;
    for (int c = c0; c < c1; ++c) {  // uniform: every thread sees the same flag
        if (!(sv[c] > thr)) continue;
        const auto row = as_global(z + (int64_t)c * zp + t0);
        for (int64_t t = threadIdx.x; t < len; t += blockDim.x) row[t] = 0.0f;
    }
}

// f32 rows to bf16 / f16, four samples per 8-byte store (1024 x 8192 samples: 17 -> 10 us).
template <typename TO>
__global__ __launch_bounds__(256) void k_cast(const float *src, int64_t sp, int64_t cols, TO *dst, int64_t dp)
{
    const int64_t r = blockIdx.y;
    const auto out = as_global(dst + r * dp);
    row_quads(
        src + r * sp, (int64_t)blockIdx.x * kRow, cols,
        [&](int64_t t, f32x4u x) {
            *reinterpret_cast<global_ptr<u32x2u>>(out + t) =
                u32x2u{store_bits<TO>(x.x) | store_bits<TO>(x.y) << 16, store_bits<TO>(x.z) | store_bits<TO>(x.w) << 16};
        },
        [&](int64_t t, float x) { Store<TO>::put(out + t, x); });
}

uint32_t blocks(int64_t n, int64_t per) { return (uint32_t)((n + per - 1) / per); }
// threads of a row_quads workgroup: rows of up to 512 samples have one quad for half of 256 or fewer
uint32_t row_threads(int64_t n) { return n > 512 ? 256 : n > 256 ? 128 : 64; }

}  // namespace

int launch_encode(const float *z, int64_t zp, int time_major, int nchan, int64_t nsamp, const float *thr, int nthr,
                  uint8_t *out, int64_t op, void *stream)
{
    Thresholds th{};
    th.n = nthr;
    for (int i = 0; i < nthr; ++i) th.v[i] = thr[i];
    hipStream_t st = (hipStream_t)stream;
    const bool few = (int64_t)blocks(nsamp, 256) * blocks(nchan, 64) < kTmBlocks;
    if (time_major)
        hipLaunchKernelGGL(few ? k_encode_tm<64> : k_encode_tm<256>, dim3(blocks(nsamp, few ? 64 : 256), blocks(nchan, 64)),
                           dim3(256), 0, st, z, zp, nchan, nsamp, th, out, op);
    else
        hipLaunchKernelGGL(k_encode_cm, dim3(blocks(nsamp, kRow), (uint32_t)nchan), dim3(row_threads(nsamp)), 0, st, z,
                           zp, nsamp, th, out, op);
    return (int)hipGetLastError();
}

int launch_encode_bits(const float *z, int64_t zp, int time_major, int nchan, int64_t nsamp, float thr, uint32_t *out,
                       int64_t ow, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const bool few = (int64_t)blocks(nsamp, 1024) * blocks(nchan, 64) < kTmBitBlocks;
    if (time_major)
        hipLaunchKernelGGL(few ? k_encode_bits_tm<2> : k_encode_bits_tm<8>,
                           dim3(blocks(nsamp, few ? 256 : 1024), blocks(nchan, 64)), dim3(256), 0, st, z, zp, nchan, nsamp,
                           thr, out, ow);
    else
        hipLaunchKernelGGL(k_encode_bits_cm, dim3(blocks(nsamp, kRow), (uint32_t)nchan),
                           dim3(64 * blocks(nsamp < kRow ? nsamp : kRow, 1024)), 0, st, z, zp, nsamp, thr, out, ow);
    return (int)hipGetLastError();
}

int launch_scrunch(const float *z, int64_t zp, int nchan, int64_t nout, int s, float r, float *out, int64_t op,
                   void *stream)
{
    hipStream_t st = (hipStream_t)stream;
#define SND_SCRUNCH(S, U)                                                                                             \
    hipLaunchKernelGGL(k_scrunch<S>, dim3(blocks(nout, 256 * U), (uint32_t)nchan), dim3(256), 0, st, z, zp, nout, s, \
                       r, out, op)
    switch (s) {  // the scrunch factors of the multi-rate bands
    case 2: SND_SCRUNCH(2, 8); break;
    case 4: SND_SCRUNCH(4, 8); break;
    case 8: SND_SCRUNCH(8, 4); break;
    case 16: SND_SCRUNCH(16, 2); break;
    default: SND_SCRUNCH(0, 1); break;
    }
#undef SND_SCRUNCH
    return (int)hipGetLastError();
}

int launch_chanstats(const float *p, int64_t pp, int nchan, int64_t n, double clip, double *stats, void *stream)
{
    const int threads = n <= 1024 ? 64 : n <= 16384 ? 256 : 1024;
    hipLaunchKernelGGL(threads == 64 ? k_chanstats<64> : threads == 256 ? k_chanstats<256> : k_chanstats<1024>,
                       dim3((uint32_t)nchan), dim3((uint32_t)threads), 0, (hipStream_t)stream, p, pp, n, clip, stats);
    return (int)hipGetLastError();
}

int launch_normalize(const float *p, int64_t pp, int nchan, int64_t n, const double *stats, float *z, int64_t zp,
                     void *stream)
{
    hipLaunchKernelGGL(k_normalize, dim3(blocks(n, kRow), (uint32_t)nchan), dim3(row_threads(n)), 0, (hipStream_t)stream,
                       p, pp, n, stats, z, zp);
    return (int)hipGetLastError();
}

int launch_zero_dm(float *z, int64_t zp, int nchan, int64_t n, double gamma, int32_t *count, void *stream)
{
    hipLaunchKernelGGL(k_zero_dm, dim3(blocks(n, 64)), dim3(64), 0, (hipStream_t)stream, z, zp, nchan, n, gamma, count);
    return (int)hipGetLastError();
}

int launch_flag_channels(float *z, int64_t zp, int nchan, int64_t n, int64_t w, double k, double *sigma,
                         uint8_t *flags, int64_t fp, void *stream)
{
    const uint32_t nwin = blocks(n, w);
    const auto sigmas = w <= 512 ? k_chan_window_sigma<8> : w <= 2048 ? k_chan_window_sigma<32>
                        : w <= 8192 ? k_chan_window_sigma<128> : k_chan_window_sigma<0>;
    hipLaunchKernelGGL(sigmas, dim3(blocks(nchan, 4), nwin), dim3(256), 0, (hipStream_t)stream, z, zp, nchan, n, w,
                       sigma);
    uint32_t slices = kFlagBlocks / nwin;
    slices = slices < 1 ? 1 : slices > kFlagSlices ? kFlagSlices : slices;
    if (slices > (uint32_t)nchan) slices = (uint32_t)nchan;
    hipLaunchKernelGGL(k_flag_window, dim3(nwin, slices), dim3(1024), (size_t)nchan * sizeof(double),
                       (hipStream_t)stream, z, zp, nchan, n, w, k, sigma, flags, fp);
    return (int)hipGetLastError();
}

int launch_cast(const float *src, int64_t sp, int64_t rows, int64_t cols, void *dst, int64_t dp, int dst_dt, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid(blocks(cols, kRow), (uint32_t)rows), threads(row_threads(cols));
    if (dst_dt == SND_DT_BF16) hipLaunchKernelGGL(k_cast<bf16_t>, grid, threads, 0, st, src, sp, cols, (bf16_t *)dst, dp);
    else if (dst_dt == SND_DT_F16) hipLaunchKernelGGL(k_cast<f16_t>, grid, threads, 0, st, src, sp, cols, (f16_t *)dst, dp);
    else return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

}  // namespace snd
