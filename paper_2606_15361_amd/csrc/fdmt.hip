// FDMT merges for gfx950 (Methods, "Classical dedispersion algorithms"), K = 2 .. 5 iterations per pass.
//
// One iteration writes every delay row of every sub-band and the next one reads them all, about 2 n
// samples of traffic per row and iteration, which is all the time there is (a pass over one iteration
// ran at the rate of a device copy).  So a pass evaluates K iterations at once, through LDS.
// Neighbouring output rows of a sub-band use neighbouring rows of its halves, so a group of
// kFdmtRun of them needs at most kFdmtRun - 1 + 2^k rows of the 2^k sub-bands k iterations down, each
// shifted by less than kFdmtRun samples along the group.  A workgroup keeps those rows as 256-sample
// slots, reads the pass's source rows once for the iteration next to them, and forms the others slot from
// slot (the same FP32 sums as K single passes, bit for bit).  The sources of the next tile are on
// their way while a tile is formed; two workgroups share a CU.  1024 channels x 65,536 samples to DM 1000,
// ten iterations: in ten passes of one 16.0 ms, in four of up to three through registers 7.8, in two of
// five through LDS 3.6.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "snd_internal.h"
#include "stage_common.h"

namespace snd {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kSlot = 256;                      // samples of a slot: four per lane
constexpr int kSlotBytes = 4 * kSlot;
constexpr int kFdmtTile = kSlot - kFdmtRun;     // output samples: a slot less the largest shift
static_assert(kFdmtTile % 4 == 0, "whole quads");
constexpr int kWaves = 16;

// the K iterations' tables, the output's first: per row (upper source row, lower source row, delay of
// the lower one, first row of the iteration's group of this number)
template <int K>
struct FdmtTables {
    const int32_t *t[K];
};

// rows that a group can need k iterations down, and how many of them a wave forms
constexpr int slots_at(int k) { return kFdmtRun - 1 + (1 << k); }
constexpr int ops_at(int k) { return (slots_at(k) + kWaves - 1) / kWaves; }
// LDS: the rows of levels K - 1, K - 3, .. in one buffer, of K - 2, K - 4, .. in the other; a read of
// a shifted row may run a quad and the largest shift past its slot
constexpr int lds_bytes(int k)
{
    return (slots_at(k - 1) + (k > 2 ? slots_at(k - 2) : 0)) * kSlotBytes + 4 * kFdmtRun + 16;
}
static_assert(lds_bytes(kFdmtMaxIters) <= 81920, "two workgroups on a CU");

// Barrier for LDS only: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// four samples of a row from sample i on, zero past sample n
__device__ __forceinline__ f32x4 load4(const float *row, int64_t start, int lane, int64_t n)
{
    const auto p = as_global(row + start) + 4 * lane;
    if (start + kSlot <= n) return *reinterpret_cast<global_ptr<const f32x4u>>(p);  // uniform
    const int64_t left = n - start - 4 * lane;
    f32x4 v{0.0f, 0.0f, 0.0f, 0.0f};
    if (left >= 4) v = *reinterpret_cast<global_ptr<const f32x4u>>(p);
    else
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < left) v[i] = p[i];
    return v;
}

// a += the samples P .. P + 3 of the quads x, y
template <int P>
__device__ __forceinline__ void add_from(f32x4 &a, const f32x4 &x, const f32x4 &y)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] += j + P < 4 ? x[(j + P) & 3] : y[(j + P) & 3];
    asm volatile("; from %1" : "+v"(a) : "i"(P));  // keeps the variants' adds apart (no selects, no moves)
}

// the lane's quad of the row at LDS byte a plus that of the row read from byte b on (uniform)
__device__ __forceinline__ f32x4 sum_rows(const unsigned char *lds, uint32_t a, uint32_t b, int lane)
{
    const unsigned char *base = lds + 16 * lane;
    f32x4 s = *reinterpret_cast<const f32x4 *>(base + a);
    const f32x4 x = *reinterpret_cast<const f32x4 *>(base + (b & ~15u));
    const f32x4 y = *reinterpret_cast<const f32x4 *>(base + (b & ~15u) + 16);
    uint32_t p = b & 12u;
    if (p == 0u) add_from<0>(s, x, y);
    asm volatile("" : "+s"(p));
    if (p == 4u) add_from<1>(s, x, y);
    asm volatile("" : "+s"(p));
    if (p == 8u) add_from<2>(s, x, y);
    asm volatile("" : "+s"(p));
    if (p == 12u) add_from<3>(s, x, y);
    return s;
}

// One sub-band's rows of a group: the first row, their number, their first slot, and the shift of the
// sub-band's slots past the tile's first sample.
struct Node {
    int lo, cnt, slot, shift;
};

template <int K>
__global__ __launch_bounds__(64 * kWaves, 8) void k_fdmt(const float *src, int64_t sp, float *dst, int64_t dp,
                                                         FdmtTables<K> tabs, int64_t rows, int ngroups, int64_t ntiles,
                                                         int64_t per, int64_t n)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // neighbouring groups (which share source rows) of the same tiles on one XCD
    const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int g = (int)(L % (uint32_t)ngroups);
    const int64_t tile0 = (int64_t)(L / (uint32_t)ngroups) * per;
    const int64_t tile1 = tile0 + per < ntiles ? tile0 + per : ntiles;
    const auto tab0 = as_const(tabs.t[0]);
    const int r0 = tab0[4 * (int64_t)g + 3];
    const int r1 = g + 1 < ngroups ? tab0[4 * (int64_t)(g + 1) + 3] : (int)rows;

    // the group's sub-bands, level by level: node 2^k - 1 + j is sub-band j of level k
    Node *nodes = reinterpret_cast<Node *>(smem);
    if (tid == 0) nodes[0] = Node{r0, r1 - r0, 0, 0};
#pragma unroll
    for (int k = 0; k + 1 < K; ++k) {
        __syncthreads();
        Node *kids = nodes + (2 << k) - 1;
        if (tid < 1 << k) {
            const Node nd = nodes[(1 << k) - 1 + tid];
            const int32_t *e0 = tabs.t[k] + 4 * (int64_t)nd.lo, *e1 = e0 + 4 * (int64_t)(nd.cnt - 1);
            kids[2 * tid] = Node{e0[0], e1[0] - e0[0] + 1, 0, nd.shift};
            kids[2 * tid + 1] = Node{e0[1], e1[1] - e0[1] + 1, 0, nd.shift + e0[2]};
        }
        __syncthreads();
        if (tid < 2 << k) {
            int slot = 0;
            for (int j = 0; j < tid; ++j) slot += kids[j].cnt;
            kids[tid].slot = slot;
        }
    }
    __syncthreads();
    // this wave's rows wave + 16 m of every level: the source rows and shifts (level K - 1), or the
    // LDS bytes of the two rows to add; and the number of them
    auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    int cnt[K];
    int src_row[ops_at(K - 1)][2], src_shift[ops_at(K - 1)][2];
    uint32_t at[K][ops_at(K - 1)][2];
    constexpr int kOther = slots_at(K - 1) * kSlotBytes;  // second buffer
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const Node *nk = nodes + (1 << k) - 1;
        const int in = (K - 2 - k) % 2 ? kOther : 0;  // buffer of level k + 1
        const int total = uni(nk[(1 << k) - 1].slot + nk[(1 << k) - 1].cnt);
        cnt[k] = total > wave ? (total - wave + kWaves - 1) / kWaves : 0;
#pragma unroll
        for (int m = 0; m < ops_at(k); ++m) {
            const int x = wave + kWaves * m;
            if (x >= total) continue;
            int j = 0;
            while (j + 1 < 1 << k && x >= nk[j + 1].slot) ++j;
            const Node nd = nk[j];
            const int32_t *e = tabs.t[k] + 4 * (int64_t)(nd.lo + x - nd.slot);
            const int shift = nd.shift + e[2];
            if (k == K - 1) {
                src_row[m][0] = uni(e[0]);
                src_row[m][1] = uni(e[1]);
                src_shift[m][0] = uni(nd.shift);
                src_shift[m][1] = uni(shift);
            } else {
                const Node u = nodes[(2 << k) - 1 + 2 * j], l = nodes[(2 << k) - 1 + 2 * j + 1];
                at[k][m][0] = (uint32_t)uni(in + (u.slot + e[0] - u.lo) * kSlotBytes);
                at[k][m][1] = (uint32_t)uni(in + (l.slot + e[1] - l.lo) * kSlotBytes + 4 * (shift - l.shift));
            }
        }
    }
    __syncthreads();

    constexpr int M = ops_at(K - 1);
    f32x4 u[M], l[M];
    auto load = [&](int64_t tile) {
        const int64_t t0 = tile * kFdmtTile;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if (m >= cnt[K - 1]) break;
            u[m] = load4(src + src_row[m][0] * sp, t0 + src_shift[m][0], lane, n);
            l[m] = load4(src + src_row[m][1] * sp, t0 + src_shift[m][1], lane, n);
        }
    };
    auto store = [&](int m, int64_t tile, const f32x4 &v) {
        const int64_t t = tile * kFdmtTile + 4 * lane, left = n - t;
        if (lane >= kFdmtTile / 4) return;
        const auto o = as_global(dst + (int64_t)(r0 + wave + kWaves * m) * dp + t);
        if (left >= 4) *reinterpret_cast<global_ptr<f32x4u>>(o) = v;
        else
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < left) o[i] = v[i];
    };
    if (tile0 < tile1) load(tile0);
    for (int64_t tile = tile0; tile < tile1; ++tile) {
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (m < cnt[K - 1])
                *reinterpret_cast<f32x4 *>(smem + (wave + kWaves * m) * kSlotBytes + 16 * lane) = u[m] + l[m];
        lds_barrier();
        if (tile + 1 < tile1) load(tile + 1);
#pragma unroll
        for (int k = K - 2; k >= 0; --k) {
            unsigned char *out = smem + ((K - 1 - k) % 2 ? kOther : 0);
#pragma unroll
            for (int m = 0; m < ops_at(k); ++m) {
                if (m >= cnt[k]) break;
                const f32x4 s = sum_rows(smem, at[k][m][0], at[k][m][1], lane);
                if (k == 0) store(m, tile, s);
                else *reinterpret_cast<f32x4 *>(out + (wave + kWaves * m) * kSlotBytes + 16 * lane) = s;
            }
            // (level 0 reads the buffer that the next tile's level K - 1 writes where K is even)
            if (k > 0 || K % 2 == 0) lds_barrier();
        }
    }
}

// One merge alone (two channels): output row r = source row U (tab[4r]) plus source row L (tab[4r + 1]) read
// tab[4r + 2] samples later, zero past n.  Nothing to keep in LDS; a workgroup covers 2048 samples of a
// strided set of rows, and the table words are uniform (7089 rows of 100,000 samples: 0.51 ms, by tiles
// of the pass above 0.61).
__global__ __launch_bounds__(256) void k_fdmt_merge(const float *src, int64_t sp, float *dst, int64_t dp,
                                                    const int32_t *tab, int64_t rows, int64_t n)
{
    const int64_t t0 = (int64_t)blockIdx.x * 2048 + threadIdx.x;
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
        const int64_t ru = tab[4 * r], rl = tab[4 * r + 1], du = tab[4 * r + 2];
        const float *u = src + ru * sp;
        const float *l = src + rl * sp + du;
        float *o = dst + r * dp;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t t = t0 + 256 * j;
            if (t < n) o[t] = u[t] + (t + du < n ? l[t] : 0.0f);
        }
    }
}

template <int K>
int launch_pass(const float *src, int64_t sp, float *dst, int64_t dp, const int32_t *const *tabs, int64_t rows,
                int64_t ngroups, int64_t n, hipStream_t st)
{
    FdmtTables<K> tb;
    for (int k = 0; k < K; ++k) tb.t[k] = tabs[k];
    const int64_t ntiles = (n + kFdmtTile - 1) / kFdmtTile;
    // up to 16 tiles a workgroup (the group's tables are walked once for them), fewer where that would
    // leave CUs without work
    int64_t per = ngroups * ntiles / 2048;
    per = per < 1 ? 1 : per > 16 ? 16 : per;
    int64_t nb = ngroups * ((ntiles + per - 1) / per);
    while (nb > 0x7fffffffLL) {
        per *= 2;
        nb = ngroups * ((ntiles + per - 1) / per);
    }
    hipLaunchKernelGGL(k_fdmt<K>, dim3((uint32_t)nb), dim3(64 * kWaves), lds_bytes(K), st, src, sp, dst, dp, tb, rows,
                       (int)ngroups, ntiles, per, n);
    return (int)hipGetLastError();
}

}  // namespace

// One pass over k iterations; tabs: their tables, the output's (the latest) first; ngroups: groups of
// the output's rows.
int launch_fdmt_pass(int k, const float *src, int64_t sp, float *dst, int64_t dp, const int32_t *const *tabs,
                     int64_t rows, int64_t ngroups, int64_t n, void *stream)
{
    if (rows < 1) return 0;
    hipStream_t st = (hipStream_t)stream;
    switch (k) {
    case 1:
        hipLaunchKernelGGL(k_fdmt_merge, dim3((uint32_t)((n + 2047) / 2048), (uint32_t)(rows < 4096 ? rows : 4096)),
                           dim3(256), 0, st, src, sp, dst, dp, tabs[0], rows, n);
        return (int)hipGetLastError();
    case 2: return launch_pass<2>(src, sp, dst, dp, tabs, rows, ngroups, n, st);
    case 3: return launch_pass<3>(src, sp, dst, dp, tabs, rows, ngroups, n, st);
    case 4: return launch_pass<4>(src, sp, dst, dp, tabs, rows, ngroups, n, st);
    case 5: return launch_pass<5>(src, sp, dst, dp, tabs, rows, ngroups, n, st);
    default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace snd
