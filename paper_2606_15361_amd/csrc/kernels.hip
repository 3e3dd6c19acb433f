// SND tree kernels for gfx950 (CDNA4).
//
// One generic stage kernel evaluates, for a block of output rows and a time tile, the SND
// sub-tree between two materialised levels (Methods, "The Spiking Neural Dedispersion
// algorithm": leaf clusters, B-ary levels, shared-pattern neurons; "Tree activation modes").
// Each output row owns a list of (source row, time offset, closing depth) entries in
// depth-first tree order.  A wave walks that list with scalar loads, reads the 64 x V
// shifted source samples of each entry with coalesced vector loads, and keeps one partial
// sum per open tree level in registers; when an entry closes k levels the node activation
// (quorum, clip or none) is applied level by level exactly as in the tree.  The node
// arithmetic, its order and its association are those of a level-by-level evaluation, so
// the result does not depend on which levels are materialised.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "snd_internal.h"
#include "stage_common.h"

namespace snd {
namespace {

constexpr int kWaves = 4;      // output rows per workgroup (one per wave)
constexpr int kV = 4;          // time samples per lane (strided by 64)
constexpr int kTile = 64 * kV; // time samples per wave
constexpr int kUnroll = 8;     // entries whose loads are issued together

template <int MODE, typename TI, typename TO, int MAXD>
__global__ __launch_bounds__(256) void k_stage(StageArgs s0, Multi m)
{
    using A = typename Acc<MODE>::type;
    StageArgs s;
    uint32_t bid, nblk;
    select_record(s0, m, s, bid, nblk);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const uint32_t L = xcd_remap(bid, nblk);
    const int rg = (int)(L % (uint32_t)s.n_rgroups);
    const int tt = (int)(L / (uint32_t)s.n_rgroups);
    int row = rg * kWaves + wave;
    if (row >= s.rows) return;
    row = __builtin_amdgcn_readfirstlane(row);
    const int len = s.row_len[row] - s.len_cut;
    const int t0 = tt * kTile;
    if (t0 >= len) return;
    const uint32_t beg = s.row_ptr[row], end = s.row_ptr[row + 1];
    const int depth = s.depth;

    bool ok[kV];
#pragma unroll
    for (int v = 0; v < kV; ++v) ok[v] = t0 + lane + 64 * v < len;

    A acc[MAXD][kV];
    A out[kV];
#pragma unroll
    for (int j = 0; j < MAXD; ++j)
#pragma unroll
        for (int v = 0; v < kV; ++v) acc[j][v] = 0;
#pragma unroll
    for (int v = 0; v < kV; ++v) out[v] = 0;

    const TI *src = static_cast<const TI *>(s.src);
    uint32_t e0 = beg;
    // full chunks: all table entries, then all loads, then the sums (no per-entry guards, so the
    // loads of a chunk are in flight together)
    for (; e0 + kUnroll <= end; e0 += kUnroll) {
        Entry en[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) en[u] = s.ent[e0 + u];
        A val[kUnroll][kV];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const TI *p = src + (int64_t)(en[u].rowc & kRowMask) * s.src_pitch + en[u].off + t0 + lane;
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                A x = 0;
                if (ok[v]) x = (A)Load<TI>::get(p + 64 * v);
                if constexpr (MODE == SND_MODE_BINARY) x = x != 0;
                val[u][v] = x;
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
#pragma unroll
            for (int v = 0; v < kV; ++v) acc[0][v] += val[u][v];
            close_levels<MODE, A, MAXD, kV>(acc, out, (int)(en[u].rowc >> 24), depth, s.src_is_input, s.k_leaf,
                                            s.k_int, s.cap);
        }
    }
    for (; e0 < end; ++e0) {
        const Entry en = s.ent[e0];
        const TI *p = src + (int64_t)(en.rowc & kRowMask) * s.src_pitch + en.off + t0 + lane;
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            A x = 0;
            if (ok[v]) x = (A)Load<TI>::get(p + 64 * v);
            if constexpr (MODE == SND_MODE_BINARY) x = x != 0;
            acc[0][v] += x;
        }
        close_levels<MODE, A, MAXD, kV>(acc, out, (int)(en.rowc >> 24), depth, s.src_is_input, s.k_leaf, s.k_int,
                                        s.cap);
    }

    TO *dst = static_cast<TO *>(s.dst) + (int64_t)row * s.dst_pitch + t0 + lane;
#pragma unroll
    for (int v = 0; v < kV; ++v) {
        if (ok[v]) {
            if constexpr (MODE == SND_MODE_FLOAT) Store<TO>::put(dst + 64 * v, out[v] * s.scale);
            else Store<TO>::put(dst + 64 * v, out[v]);
        }
    }
}

template <int MODE, typename TI, typename TO>
int launch_typed(const StageArgs &a, int64_t max_len, hipStream_t st, const Multi &m, int64_t nb_multi)
{
    StageArgs s = a;
    const int64_t nblocks = m.n > 0 ? nb_multi : stage_blocks(s, max_len);
    if (nblocks <= 0) return 0;
    if (nblocks > 0x7fffffffLL || max_len > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    dim3 grid((uint32_t)nblocks), block(256);
    if (a.depth <= 1) hipLaunchKernelGGL((k_stage<MODE, TI, TO, 1>), grid, block, 0, st, s, m);
    else if (a.depth <= 2) hipLaunchKernelGGL((k_stage<MODE, TI, TO, 2>), grid, block, 0, st, s, m);
    else if (a.depth <= 4) hipLaunchKernelGGL((k_stage<MODE, TI, TO, 4>), grid, block, 0, st, s, m);
    else if (a.depth <= 8) hipLaunchKernelGGL((k_stage<MODE, TI, TO, 8>), grid, block, 0, st, s, m);
    else hipLaunchKernelGGL((k_stage<MODE, TI, TO, 16>), grid, block, 0, st, s, m);
    return (int)hipGetLastError();
}

struct StageLauncher {
    const StageArgs &a;
    int64_t max_len;
    const Multi &m;
    int64_t nblocks;
    template <int MODE, typename TI, typename TO> int run(hipStream_t st) const
    {
        return launch_typed<MODE, TI, TO>(a, max_len, st, m, nblocks);
    }
};

}  // namespace

int64_t stage_blocks(StageArgs &a, int64_t max_len)
{
    const int64_t ntt = (max_len + kTile - 1) / kTile;
    a.n_ttiles = (int32_t)ntt;
    a.n_rgroups = (a.rows + kWaves - 1) / kWaves;
    return (int64_t)a.n_rgroups * ntt;
}

int launch_stage(int mode, int src_dt, int dst_dt, const StageArgs &a, int64_t max_len, void *stream, const Multi &m,
                 int64_t nblocks)
{
    return dispatch_types(mode, src_dt, dst_dt, StageLauncher{a, max_len, m, nblocks}, (hipStream_t)stream);
}

// Approximate sub-band dedispersion, second step: out row k = sum over sub-bands s of row
// coarse[k] of sub-band plane s, read offs[k * nsub + s] samples later, in FP32 in sub-band
// order.  A workgroup covers 1024 samples of one row, 4 per lane (coalesced reads of each plane
// row); the table words are uniform (scalar loads).
__global__ __launch_bounds__(256) void k_subband_combine(const float *const *planes, const int64_t *pitches,
                                                         const int32_t *coarse, const int32_t *offs, int nsub,
                                                         float *out, int64_t op, int64_t n)
{
    const int k = blockIdx.y;
    const int64_t t0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const int j = coarse[k];
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < nsub; ++s) {
        const float *row = planes[s] + (int64_t)j * pitches[s] + offs[(int64_t)k * nsub + s];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t t = t0 + 256 * i;
            if (t < n) acc[i] += row[t];
        }
    }
    float *o = out + (int64_t)k * op;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (t0 + 256 * i < n) o[t0 + 256 * i] = acc[i];
}

int launch_subband_combine(const float *const *planes, const int64_t *pitches, const int32_t *coarse,
                           const int32_t *offs, int nsub, int ndm, float *out, int64_t op, int64_t n, void *stream)
{
    if (ndm < 1 || n < 1) return 0;
    hipLaunchKernelGGL(k_subband_combine, dim3((uint32_t)((n + 1023) / 1024), (uint32_t)ndm), dim3(256), 0,
                       (hipStream_t)stream, planes, pitches, coarse, offs, nsub, out, op, n);
    return (int)hipGetLastError();
}

}  // namespace snd
