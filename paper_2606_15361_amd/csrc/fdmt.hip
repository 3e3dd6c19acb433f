// FDMT merges for gfx950 (Methods, "Classical dedispersion algorithms"), K iterations per pass.
//
// One iteration writes every delay row of every sub-band and the next one reads them all, about 2 n
// samples of traffic per row and iteration, which is all the time there is (a pass over one iteration
// ran at the rate of a device copy).  So a pass evaluates K iterations at once: an output row is the
// sum of 2^K source rows, found by walking the K iterations' tables from the output row down, each
// read at the sum of the delays on its way and added in the iterations' own order (the same FP32 sums
// as K single passes, bit for bit).  Neighbouring delays share all but one of their source rows, so a
// workgroup's 16 waves take neighbouring rows of the same 256 samples, whose sources stay in the
// CU's cache, and step through a run of rows.  1024 channels x 65,536 samples to DM 1000 (14.2 k rows of
// 0.26 MB per iteration): 16.1 -> 7.8 ms with passes of 4, 3 and 3 iterations (3.5, 2.2, 2.2 ms; the
// last two move about 8 GB of new bytes each, at 3.5 TB/s, and 30 GB through the caches).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "snd_internal.h"
#include "stage_common.h"

namespace snd {

constexpr int kFdmtTile = 256;  // samples per workgroup: one 16-byte load per lane and source row

namespace {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// the K iterations' tables, the output's first: per row (upper source row, lower source row, delay of
// the lower one, 0)
template <int K>
struct FdmtTables {
    const int32_t *t[K];
};

template <int K>
__global__ __launch_bounds__(1024, K <= 3 ? 8 : 4) void k_fdmt(const float *src, int64_t sp, float *dst, int64_t dp, FdmtTables<K> tabs,
                                               int64_t rows, int64_t run, int64_t n)
{
    constexpr int N = 1 << K;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * kFdmtTile;
    const uint32_t i4 = 4u * lane;  // the lane's first sample in the tile
    const int64_t r1 = ((int64_t)blockIdx.y + 1) * run < rows ? ((int64_t)blockIdx.y + 1) * run : rows;
    for (int64_t r = (int64_t)blockIdx.y * run + wave; r < r1; r += 16) {
        int32_t row[N], sh[N];  // uniform: scalar loads and registers
        row[0] = (int32_t)r;
        sh[0] = 0;
        int32_t far = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const auto tab = as_const(tabs.t[k]);
#pragma unroll
            for (int j = (1 << k) - 1; j >= 0; --j) {
                const int64_t e = 4 * (int64_t)row[j];
                row[2 * j + 1] = tab[e + 1];
                sh[2 * j + 1] = sh[j] + tab[e + 2];
                row[2 * j] = tab[e];
                sh[2 * j] = sh[j];
            }
        }
#pragma unroll
        for (int j = 0; j < N; ++j) far = far > sh[j] ? far : sh[j];
        f32x4u v[N];
        if (t0 + kFdmtTile + far <= n) {  // uniform
#pragma unroll
            for (int j = 0; j < N; ++j)
                v[j] = *reinterpret_cast<global_ptr<const f32x4u>>(as_global(src + (row[j] * sp + sh[j] + t0)) + i4);
        } else {  // samples past the row are zero
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const auto p = as_global(src + (row[j] * sp + sh[j] + t0)) + i4;
                const int left = (int)(n - t0 - sh[j] < kFdmtTile ? n - t0 - sh[j] : kFdmtTile) - (int)i4;
                v[j] = f32x4u{0.0f, 0.0f, 0.0f, 0.0f};
                if (left >= 4) v[j] = *reinterpret_cast<global_ptr<const f32x4u>>(p);
                else
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (i < left) v[j][i] = p[i];
            }
        }
#pragma unroll
        for (int w = N / 2; w > 0; w >>= 1)
#pragma unroll
            for (int j = 0; j < w; ++j) v[j] = v[2 * j] + v[2 * j + 1];
        const auto o = as_global(dst + (r * dp + t0)) + i4;
        const int left = (int)(n - t0 < kFdmtTile ? n - t0 : kFdmtTile) - (int)i4;
        if (left >= 4) *reinterpret_cast<global_ptr<f32x4u>>(o) = v[0];
        else
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < left) o[i] = v[0][i];
    }
}

template <int K>
int launch_pass(const float *src, int64_t sp, float *dst, int64_t dp, const int32_t *const *tabs, int64_t rows, int64_t n,
                hipStream_t st)
{
    FdmtTables<K> tb;
    for (int k = 0; k < K; ++k) tb.t[k] = tabs[k];
    const int64_t nx = (n + kFdmtTile - 1) / kFdmtTile;
    // 64 rows a workgroup (a source row's samples then serve about 64 / 2^K of them), 16 where that
    // would leave CUs without work
    int64_t run = nx * ((rows + 63) / 64) >= 1024 ? 64 : 16;
    while ((rows + run - 1) / run > 65535) run *= 2;
    const int64_t ny = (rows + run - 1) / run;
    hipLaunchKernelGGL(k_fdmt<K>, dim3((uint32_t)nx, (uint32_t)ny), dim3(1024), 0, st, src, sp, dst, dp, tb, rows, run, n);
    return (int)hipGetLastError();
}

}  // namespace

// One pass over k iterations; tabs: their tables, the output's (the latest) first.
int launch_fdmt_pass(int k, const float *src, int64_t sp, float *dst, int64_t dp, const int32_t *const *tabs,
                     int64_t rows, int64_t n, void *stream)
{
    if (rows < 1) return 0;
    hipStream_t st = (hipStream_t)stream;
    switch (k) {
    case 1: return launch_pass<1>(src, sp, dst, dp, tabs, rows, n, st);
    case 2: return launch_pass<2>(src, sp, dst, dp, tabs, rows, n, st);
    case 3: return launch_pass<3>(src, sp, dst, dp, tabs, rows, n, st);
    case 4: return launch_pass<4>(src, sp, dst, dp, tabs, rows, n, st);
    default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace snd
