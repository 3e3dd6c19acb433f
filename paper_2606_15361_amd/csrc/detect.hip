// Boxcar matched filter and candidate-pixel compaction for gfx950 (Methods, "Matched
// filtering" and "Candidate detection").
//
// k_rowstats: mean and population standard deviation of each DM row over its valid samples.
//   Integer planes use exact 64-bit sums S1, S2 and sigma = sqrt(n*S2 - S1*S1)/n in one fixed
//   FP64 expression; float planes use one FP64 pass about the row's first sample.  A floor
//   sigma_min applies.
// k_snr: one workgroup per (row, tile of samples).  The tile plus the widest boxcar is staged in
//   LDS as an inclusive prefix sum (int32 for integer planes: exact; FP64 for float planes), every
//   sample then evaluates all widths with two LDS reads each:
//   SNR(t, W) = (S_W(t) - mu W) / (sigma sqrt W), maximum over widths (first width on ties).
//   Either the full S/N plane and width index are written, or the cells whose S/N reaches the
//   threshold are appended to a global pixel list, each workgroup's cells as one segment in
//   increasing t.  For the list, a per-width bound on the boxcar sum (in the prefix type)
//   skips the cells that cannot reach the threshold; every cell that can takes the exact
//   quotient.  The widths are the outer loop of the bound tests and a thread's cells the inner
//   one, so any list length runs the same straight-line inner code, and only the slabs of cells
//   past the last valid start of a width are tested against it.  Aligned u8 rows take the tests on
//   two cells per 32-bit lane (k_snr_pairs).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "snd_detect.h"

namespace snd {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <typename T> using global_ptr = __attribute__((address_space(1))) T *;
template <typename T> __device__ inline global_ptr<const T> as_global(const T *p) { return (global_ptr<const T>)p; }

constexpr int kThreads = 256;

template <typename T> struct IsInt { static constexpr bool value = true; };
template <> struct IsInt<float> { static constexpr bool value = false; };
// Samples of one row per S/N workgroup.  Integer planes carry a 4-byte prefix per sample (two or
// four bytes on the paired path) and little arithmetic per byte read, so their tiles are long
// (fewer workgroups, a smaller share of re-read halo; 4096 keeps seven workgroups on a CU, 8192 and
// 2048 measured slower).  Float planes carry an 8-byte prefix and take kFloatSlabs cells per thread:
// lists up to kFloatNarrow samples stage tile and halo as eight samples per thread (the tile gives up
// the halo, in whole 64-sample steps, so that rows of 64-sample pitch start every tile on a 16-byte
// boundary), wider ones twelve per thread over the whole slabs.
constexpr int kIntTile = 4096;
constexpr int kFloatSlabs = 8, kFloatNarrow = 192;
template <typename T> constexpr int snr_slabs() { return IsInt<T>::value ? kIntTile / kThreads : kFloatSlabs; }
template <typename T> constexpr int snr_per(bool wide)
{
    return IsInt<T>::value ? (kIntTile + kMaxWidth + kThreads - 1) / kThreads
                           : wide ? (kFloatSlabs * kThreads + kMaxWidth + kThreads - 1) / kThreads : kFloatSlabs;
}
template <typename T> int snr_tile(int wmax)
{
    return IsInt<T>::value || wmax > kFloatNarrow ? snr_slabs<T>() * kThreads
                                                  : (kThreads * kFloatSlabs - (wmax - 1)) / 64 * 64;
}
static_assert(kThreads * kFloatSlabs - kFloatNarrow - 63 > kThreads * (kFloatSlabs - 1), "only the last slab is partial");
// Prefix entry j of a float tile of the cell list sits at j + j / 8: a thread writes runs of consecutive
// entries, and the gap of one entry in eight spreads the lanes of a wave over the LDS banks.  (The whole
// plane's tiles have none: every cell reads every width there, and the gaps cost more than they save.)
template <bool GAPS> __device__ inline int pre_at(int j) { return GAPS ? j + (j >> 3) : j; }

// Row sums with 16-byte loads: a scalar head up to the first 16-byte boundary of the row, then
// 16-byte vectors (four in flight per thread), then a scalar tail.  f(x, j) folds one sample;
// j is its place in a vector (0 for the scalar head and tail), for independent accumulators.
template <typename T, typename F>
__device__ inline void row_fold(const T *row, int64_t n, int tid, F &&f)
{
    constexpr int E = 16 / (int)sizeof(T);  // samples per vector
    int64_t head = (int64_t)(((16u - ((uint32_t)(uintptr_t)row & 15u)) & 15u) / sizeof(T));
    if (((uintptr_t)row % sizeof(T)) != 0 || head > n) head = n;  // misaligned element type: all scalar
    if (tid < head) f(row[tid], 0);
    const int64_t nv = (n - head) / E;
    const auto vec = as_global(reinterpret_cast<const u32x4 *>(row + head));
    int64_t i = tid;
    for (; i + 3 * kThreads < nv; i += 4 * kThreads) {
        u32x4 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = vec[i + u * kThreads];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T *e = reinterpret_cast<const T *>(&q[u]);
#pragma unroll
            for (int j = 0; j < E; ++j) f(e[j], j);
        }
    }
    for (; i < nv; i += kThreads) {
        const u32x4 q = vec[i];
        const T *e = reinterpret_cast<const T *>(&q);
#pragma unroll
        for (int j = 0; j < E; ++j) f(e[j], j);
    }
    for (int64_t t = head + nv * E + tid; t < n; t += kThreads) f(row[t], 0);
}

// Row k of a launch: a row of the single plane, or (BATCH) batch row row0 + k of the plane
// whose row range holds it (a scan of the table: every value is wave-uniform, so scalar work).
template <bool BATCH, typename T>
__device__ inline void locate_row(const T *plane, int64_t pitch, int64_t n, const int32_t *row_nw, const DetBeam *beams,
                                  int nbeams, int row0, int k_launch, const T *&row, int64_t &nr, const int32_t *&nw,
                                  int &k, int &kl)
{
    k = row0 + k_launch;
    if constexpr (!BATCH) {
        row = plane + (int64_t)k * pitch;
        nr = n;
        nw = row_nw;
        kl = k;
        return;
    }
    int i = 0;
    while (i + 1 < nbeams && k >= beams[i + 1].row_base) ++i;
    const DetBeam b = beams[i];
    kl = k - b.row_base;
    row = static_cast<const T *>(b.plane) + (int64_t)kl * b.pitch;
    nr = b.n;
    nw = b.row_nw;
}

template <typename T, bool BATCH>
__global__ __launch_bounds__(kThreads) void k_rowstats(const T *plane, int64_t pitch, int64_t n_, double sigma_min,
                                                       double *stats, const DetBeam *beams, int nbeams, int row0)
{
    const T *row;
    int64_t n;
    const int32_t *nw_unused;
    int k, kl;
    locate_row<BATCH>(plane, pitch, n_, nullptr, beams, nbeams, row0, (int)blockIdx.x, row, n, nw_unused, k, kl);
    const int tid = threadIdx.x;
    if constexpr (IsInt<T>::value) {
        __shared__ unsigned long long s1[kThreads], s2[kThreads];
        // per-thread sums stay exact in 64 bits (at most n / kThreads + 1 samples of < 2^16 each)
        unsigned long long a = 0, b = 0;
        row_fold(row, n, tid, [&](T x, int) {
            const unsigned long long v = (unsigned long long)x;
            a += v;
            b += v * v;
        });
        s1[tid] = a;
        s2[tid] = b;
        __syncthreads();
        for (int s = kThreads / 2; s > 0; s >>= 1) {
            if (tid < s) {
                s1[tid] += s1[tid + s];
                s2[tid] += s2[tid + s];
            }
            __syncthreads();
        }
        if (tid == 0) {
            const double dn = (double)n;
            const double mu = (double)s1[0] / dn;
            const double num = __dsub_rn(__dmul_rn(dn, (double)s2[0]), __dmul_rn((double)s1[0], (double)s1[0]));
            double sg = num > 0.0 ? sqrt(num) / dn : 0.0;
            if (sg < sigma_min) sg = sigma_min;
            stats[2 * k] = mu;
            stats[2 * k + 1] = sg;
        }
    } else {
        // one pass in FP64 about a shift c (the row's first sample), so that a large mean does
        // not cancel: mu = c + S1 / n, sigma^2 = S2 / n - (S1 / n)^2 with S1, S2 the sums of
        // (y - c) and (y - c)^2; two accumulator pairs keep the FP64 adds independent
        __shared__ double r1[kThreads], r2[kThreads];
        const double c = (double)row[0];
        double a0 = 0.0, b0 = 0.0, a1 = 0.0, b1 = 0.0;
        row_fold(row, n, tid, [&](T x, int j) {
            const double d = (double)x - c;
            if (j & 1) {
                a1 += d;
                b1 += d * d;
            } else {
                a0 += d;
                b0 += d * d;
            }
        });
        r1[tid] = a0 + a1;
        r2[tid] = b0 + b1;
        __syncthreads();
        for (int s = kThreads / 2; s > 0; s >>= 1) {
            if (tid < s) {
                r1[tid] += r1[tid + s];
                r2[tid] += r2[tid + s];
            }
            __syncthreads();
        }
        if (tid == 0) {
            const double m1 = r1[0] / (double)n;
            const double var = r2[0] / (double)n - m1 * m1;
            double sg = var > 0.0 ? sqrt(var) : 0.0;
            if (sg < sigma_min) sg = sigma_min;
            stats[2 * k] = c + m1;
            stats[2 * k + 1] = sg;
        }
    }
}

// Per-row constants of S/N(t, W) = (S_W(t) - mu W) / (sigma sqrt W), for threads tid < nw:
// mu W, sigma sqrt W and the bound on the boxcar sum below which a cell cannot reach the
// threshold at width W.
template <typename P>
__device__ inline void row_constants(int tid, const SnrArgs &a, double mu, double sg, double *muw, double *den,
                                     P *sthr, bool is_int)
{
    if (tid >= a.nw) return;
    muw[tid] = __dmul_rn(mu, (double)a.w[tid]);
    den[tid] = __dmul_rn(sg, a.sqrtw[tid]);
    // S/N >= Theta needs S >= mu W + Theta sigma sqrt W up to the rounding of the exact
    // quotient (relative 1e-16); the bound takes a relative margin of 1e-9 below that
    const double b = muw[tid] + a.threshold * den[tid];
    const double thr = b - 1e-9 * (fabs(muw[tid]) + a.threshold * den[tid]);
    if (is_int) {  // integer sums: the largest integer at or below the bound
        sthr[tid] = thr <= -2147483648.0 ? (P)(-2147483647 - 1) : thr >= 2147483647.0 ? (P)2147483647 : (P)floor(thr);
    } else {
        sthr[tid] = (P)thr;
    }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pk_sub(uint32_t x, uint32_t y)  // two 16-bit differences modulo 2^16
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, x) - __builtin_bit_cast(u16x2, y));
}
__device__ inline uint32_t pk_sub_sat(uint32_t x, uint32_t y)  // two max(x - y, 0)
{
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, x), __builtin_bit_cast(u16x2, y)));
}
// (p mod 2^16, (p + x) mod 2^16) from p and a word whose byte 2 holds x (other bytes zero)
__device__ inline uint32_t pair_word(uint32_t p, uint32_t x_hi)
{
    return __builtin_amdgcn_perm(p, p, 0x01000100u) + x_hi;
}

// Inclusive sum over the 64 lanes of a wave with DPP moves: within each row of 16 lanes by
// shifts of 1, 2, 4 and 8 (lanes shifted in from outside the row add zero), then lane 15's total
// into rows 1 and 3, then lane 31's into rows 2 and 3.
__device__ inline uint32_t wave_inclusive_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// The same scan for FP64 values (each DPP move carries the two halves of a value).
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_f64(double x)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline double wave_inclusive_sum(double x)
{
    x += dpp_f64<0x111, 0xf>(x);
    x += dpp_f64<0x112, 0xf>(x);
    x += dpp_f64<0x114, 0xf>(x);
    x += dpp_f64<0x118, 0xf>(x);
    x += dpp_f64<0x142, 0xa>(x);
    x += dpp_f64<0x143, 0xc>(x);
    return x;
}
__device__ inline int32_t wave_inclusive_sum(int32_t x) { return (int32_t)wave_inclusive_sum((uint32_t)x); }

// ---- u8 rows, two cells per lane ----
// The prefix P of the tile is kept modulo 2^16 in 16-bit halves: a boxcar sum of at most 256 u8
// samples is below 2^16, so the difference of two such prefixes is the exact sum.  Longer boxcars
// (up to 1024 samples, sums below 2^18) use a second array, P / 4 modulo 2^16: the difference D of
// two of those lies within 3/4 of S / 4, so S >= b implies D >= b / 4 rounded down, which is the
// bound test, and the two differences together give S exactly (S = the value congruent to the first
// one modulo 2^16 nearest to 4 D).
constexpr int kPairExact = 256;                        // widest boxcar of the first array alone
constexpr int kPairs = kIntTile / 2 / kThreads;        // pairs of cells per thread
constexpr int kPairSlack = 8;                          // entries past tile + halo
static_assert(kIntTile == 16 * kThreads && kMaxWidth <= 4 * kThreads, "sixteen tile bytes and four halo bytes per thread");
constexpr int pair_entries(int wmax) { return kIntTile + (wmax > kPairExact ? kMaxWidth : kPairExact) + kPairSlack; }
inline int64_t pairs_lds_bytes(int wmax) { return (int64_t)pair_entries(wmax) * (wmax > kPairExact ? 4 : 2); }

// What the bound tests of one width read: the two 16-bit copies of the bound less one, all ones where
// every cell passes, the width's dword step and the width itself.
struct PairWidth {
    uint32_t t, all, step, w;
};

struct PairShared {
    int32_t wtot[2][kThreads / 64];
    int slab_off[kPairs][kThreads / 64];
    unsigned int base;
    double muw[kMaxWidths], den[kMaxWidths];
    int32_t sthr[kMaxWidths];
    uint64_t smask[kPairs][kThreads / 64][2];
    PairWidth rec[kMaxWidths];
};

// One tile of a row: avail samples from its first to the row's end, nwk leading widths of the list.
// EDGE: some width of the list does not fit every cell of the tile.
template <bool EDGE>
__device__ __forceinline__ void snr_pairs_tile(const uint8_t *row, int k, int64_t t0, int avail, int nwk,
                                               const double *stats, const SnrArgs &a, unsigned char *dyn, PairShared &sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wlist = a.wmax;
    const bool two = wlist > kPairExact;
    uint16_t *pre16 = reinterpret_cast<uint16_t *>(dyn);       // P(j) mod 2^16
    uint16_t *pre4 = pre16 + (two ? pair_entries(wlist) : 0);  // (P(j) / 4) mod 2^16
    // thread t: tile samples 16 t .. 16 t + 15 and halo samples 4096 + 4 t .. + 3; samples past the
    // row read as zero and feed prefix entries that no valid cell reads
    const auto grow = as_global(row);
    const int h0 = kIntTile + 4 * tid;
    u32x4 q = {0u, 0u, 0u, 0u};
    uint32_t hq = 0u;
    if (!EDGE) {
        q = as_global(reinterpret_cast<const u32x4 *>(row))[tid];
        if (4 * tid < wlist - 1 && h0 + 4 <= avail) {
            hq = as_global(reinterpret_cast<const uint32_t *>(row))[h0 >> 2];
        } else if (4 * tid < wlist - 1) {
            for (int b = 0; b < 4 && h0 + b < avail; ++b) hq |= (uint32_t)grow[h0 + b] << (8 * b);
        }
    } else {
        if (16 * tid + 16 <= avail) {
            q = as_global(reinterpret_cast<const u32x4 *>(row))[tid];
        } else if (16 * tid < avail) {  // one thread of the row's last tile
            uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll 1
                for (int b = 0; b < 4 && 16 * tid + 4 * i + b < avail; ++b)
                    d[i] |= (uint32_t)grow[16 * tid + 4 * i + b] << (8 * b);
            q = u32x4{d[0], d[1], d[2], d[3]};
        }
        if (4 * tid < wlist - 1) {
#pragma unroll 1
            for (int b = 0; b < 4 && h0 + b < avail; ++b) hq |= (uint32_t)grow[h0 + b] << (8 * b);
        }
    }
    const double mu = stats[2 * k], sg = stats[2 * k + 1];
    if (!(sg > 0.0)) return;  // uniform: no cell of the row has a non-zero S/N
    row_constants(tid, a, mu, sg, sh.muw, sh.den, sh.sthr, true);
    // a cell's sum (or its quarter) passes when max(sum - (bound - 1), 0) > 0; a bound at or below
    // zero passes every cell; widths past the row's set never pass
    if (tid < a.nw) {
        const int32_t w = a.w[tid], sb = w > kPairExact ? sh.sthr[tid] >> 2 : sh.sthr[tid];
        const bool all = sb <= 0 && tid < nwk;
        const uint32_t t = sb <= 0 || tid >= nwk ? 0xFFFFu : (uint32_t)min(sb - 1, 65535);
        sh.rec[tid] = PairWidth{t * 0x00010001u, all ? 0xFFFFFFFFu : 0u, (uint32_t)(w >> 1), (uint32_t)w};
    }
    constexpr uint32_t kOnes = 0x01010101u;
    uint32_t tot = __builtin_amdgcn_udot4(q.x, kOnes, 0u, false);
    tot = __builtin_amdgcn_udot4(q.y, kOnes, tot, false);
    tot = __builtin_amdgcn_udot4(q.z, kOnes, tot, false);
    tot = __builtin_amdgcn_udot4(q.w, kOnes, tot, false);
    const uint32_t htot = __builtin_amdgcn_udot4(hq, kOnes, 0u, false);
    const uint32_t inc = wave_inclusive_sum(tot);
    uint32_t hinc = htot;
    if (256 * wv < wlist - 1) hinc = wave_inclusive_sum(htot);  // uniform per wave: it holds halo samples
    if (lane == 63) {
        sh.wtot[0][wv] = (int32_t)inc;
        sh.wtot[1][wv] = (int32_t)hinc;
    }
    __syncthreads();
    uint32_t B = inc - tot, Bh = hinc - htot;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wv) {
            B += (uint32_t)sh.wtot[0][w];
            Bh += (uint32_t)sh.wtot[1][w];
        }
        Bh += (uint32_t)sh.wtot[0][w];
    }
    const uint32_t qd[4] = {q.x, q.y, q.z, q.w}, B0 = B;
    {
        uint32_t words[8];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint32_t d = qd[m];
            words[2 * m] = pair_word(B, __builtin_amdgcn_perm(0u, d, 0x0c000c0cu));  // P(4m), P(4m + 1)
            const uint32_t B2 = __builtin_amdgcn_udot4(d, 0x00000101u, B, false);
            words[2 * m + 1] = pair_word(B2, __builtin_amdgcn_perm(0u, d, 0x0c020c0cu));  // P(4m + 2), P(4m + 3)
            B = __builtin_amdgcn_udot4(d, kOnes, B, false);
        }
        u32x4 *p4 = reinterpret_cast<u32x4 *>(pre16 + 16 * tid);
        p4[0] = u32x4{words[0], words[1], words[2], words[3]};
        p4[1] = u32x4{words[4], words[5], words[6], words[7]};
    }
    if (4 * tid <= wlist) {  // the halo's prefixes, through the first entry past it
        uint32_t *h2 = reinterpret_cast<uint32_t *>(pre16 + h0);
        h2[0] = pair_word(Bh, __builtin_amdgcn_perm(0u, hq, 0x0c000c0cu));
        h2[1] = pair_word(__builtin_amdgcn_udot4(hq, 0x00000101u, Bh, false), __builtin_amdgcn_perm(0u, hq, 0x0c020c0cu));
    }
    const int nfine = a.nfine < nwk ? a.nfine : nwk;  // widths that the first array serves
    if (nfine < nwk) {  // uniform
        auto quarters = [](uint32_t d, uint32_t base, uint32_t &lo, uint32_t &hi) {
            const uint32_t p1 = base + (d & 0xffu), p2 = __builtin_amdgcn_udot4(d, 0x00000101u, base, false);
            const uint32_t p3 = __builtin_amdgcn_udot4(d, 0x00010101u, base, false);
            lo = __builtin_amdgcn_perm(p1 >> 2, base >> 2, 0x05040100u);
            hi = __builtin_amdgcn_perm(p3 >> 2, p2 >> 2, 0x05040100u);
        };
        uint32_t base = B0, words[8];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            quarters(qd[m], base, words[2 * m], words[2 * m + 1]);
            base = __builtin_amdgcn_udot4(qd[m], kOnes, base, false);
        }
        u32x4 *c4 = reinterpret_cast<u32x4 *>(pre4 + 16 * tid);
        c4[0] = u32x4{words[0], words[1], words[2], words[3]};
        c4[1] = u32x4{words[4], words[5], words[6], words[7]};
        if (4 * tid <= wlist) {
            uint32_t *h2 = reinterpret_cast<uint32_t *>(pre4 + h0);
            quarters(hq, Bh, h2[0], h2[1]);
        }
    }
    __syncthreads();
    // bound tests; m[j] is non-zero in the halves whose cell passes at some width.  Lane w holds the
    // record of width w.
    const uint32_t *dw = reinterpret_cast<const uint32_t *>(pre16);
    const uint32_t *dw4 = reinterpret_cast<const uint32_t *>(pre4);
    const PairWidth mine = sh.rec[lane & (kMaxWidths - 1)];
    const uint32_t odd = a.odd;  // bit w: width w of the list is odd
    uint32_t m[kPairs], d0[kPairs];
    const uint32_t all = __ballot(lane < nwk && mine.all != 0u) != 0 ? ~0u : 0u;  // uniform
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        m[j] = EDGE ? 0u : all;
        d0[j] = dw[tid + kThreads * j];
    }
    auto tests = [&](const uint32_t *src, int w0, int w1) {
        for (int w = w0; w < w1; ++w) {
            const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)mine.t, w);
            const uint32_t *p = src + tid + (uint32_t)__builtin_amdgcn_readlane((int)mine.step, w);
            uint32_t s[kPairs];
            if ((odd >> w) & 1u) {  // uniform
#pragma unroll
                for (int j = 0; j < kPairs; ++j)
                    s[j] = __builtin_amdgcn_alignbit(p[kThreads * j + 1], p[kThreads * j], 16);
            } else {
#pragma unroll
                for (int j = 0; j < kPairs; ++j) s[j] = p[kThreads * j];
            }
            if constexpr (!EDGE) {
#pragma unroll
                for (int j = 0; j < kPairs; ++j) m[j] |= pk_sub_sat(pk_sub(s[j], d0[j]), t);
            } else {
                // last cell of the tile that the width fits
                const int lim = avail - __builtin_amdgcn_readlane((int)mine.w, w);
                const uint32_t on = (uint32_t)__builtin_amdgcn_readlane((int)mine.all, w);
#pragma unroll
                for (int j = 0; j < kPairs; ++j) {
                    const int i = 2 * (tid + kThreads * j);
                    const uint32_t y = pk_sub_sat(pk_sub(s[j], d0[j]), t) | on;
                    m[j] |= i < lim ? y : i == lim ? y & 0xFFFFu : 0u;
                }
            }
        }
    };
    tests(dw, 0, nfine);
    if (nfine < nwk) {
#pragma unroll
        for (int j = 0; j < kPairs; ++j) d0[j] = dw4[tid + kThreads * j];
        tests(dw4, nfine, nwk);
    }
    uint32_t any = 0u;
#pragma unroll
    for (int j = 0; j < kPairs; ++j) any |= m[j];
    if (!__syncthreads_or(any != 0u)) return;  // most tiles hold no such cell
    auto exact16 = [&](int i, double &best, int &bi) {
        best = 0.0;
        bi = -1;
        for (int w = 0; w < nwk; ++w) {
            const int W = (int)sh.rec[w].w;
            if (EDGE && i + W > avail) break;
            int32_t sum = (int32_t)(uint16_t)(pre16[i + W] - pre16[i]);
            if (W > kPairExact) sum += ((4 * (int32_t)(uint16_t)(pre4[i + W] - pre4[i]) - sum + 32768) >> 16) << 16;
            const double val = __dsub_rn((double)sum, sh.muw[w]) / sh.den[w];
            if (bi < 0 || val > best) {
                best = val;
                bi = w;
            }
        }
    };
    // the marked pairs (few) take the exact quotient on both cells; bit 2 j + h of `flags`:
    // cell 2 (tid + 256 j) + h reaches the threshold
    uint32_t maybe = 0;
#pragma unroll
    for (int j = 0; j < kPairs; ++j) maybe |= (m[j] != 0u ? 1u : 0u) << j;
    uint32_t flags = 0;
    while (maybe) {
        const int j = __builtin_ctz(maybe);
        maybe &= maybe - 1u;
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            double best;
            int bi;
            exact16(2 * (tid + kThreads * j) + h, best, bi);
            if (bi >= 0 && best >= a.threshold) flags |= 1u << (2 * j + h);
        }
    }
    // ordered output: pairs in increasing t (slab j, then thread), the even cell first; each
    // wave's ballots of its even and odd cells per slab go through LDS for the output loop
#pragma unroll 1
    for (int j = 0; j < kPairs; ++j) {
        const uint64_t b0 = __ballot((flags >> (2 * j)) & 1u), b1 = __ballot((flags >> (2 * j + 1)) & 1u);
        if (lane == 0) {
            sh.slab_off[j][wv] = __popcll(b0) + __popcll(b1);
            sh.smask[j][wv][0] = b0;
            sh.smask[j][wv][1] = b1;
        }
    }
    __syncthreads();
    if (tid == 0) {
        int tsum = 0;
        for (int j = 0; j < kPairs; ++j)
            for (int w = 0; w < kThreads / 64; ++w) {
                const int c = sh.slab_off[j][w];
                sh.slab_off[j][w] = tsum;
                tsum += c;
            }
        sh.base = tsum ? atomicAdd(a.counter, (unsigned int)tsum) : 0u;
    }
    __syncthreads();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t f = flags;
    while (f) {
        const int b = __builtin_ctz(f);
        f &= f - 1u;
        const int j = b >> 1, h = b & 1;
        const int64_t pos = (int64_t)sh.base + sh.slab_off[j][wv] + __popcll(sh.smask[j][wv][0] & below) +
                            __popcll(sh.smask[j][wv][1] & below) + (h ? ((flags >> (2 * j)) & 1u) : 0u);
        if (pos < a.max_pixels) {
            // the flagged cells are few: their exact maximum is taken again rather than kept
            const int i = 2 * (tid + kThreads * j) + h;
            double best;
            int bi;
            exact16(i, best, bi);
            Pixel px;
            px.k = k;
            px.t = (int32_t)(t0 + i);
            px.snr = best;
            px.widx = bi;
            px.pad = 0;
            a.pixels[pos] = px;
        }
    }
}

// The cell list of u8 planes whose rows all start on a 16-byte boundary, any width list: one
// workgroup per (row, tile of kIntTile cells).  The cells whose bound test passes take the exact
// quotient, as on the general path; the list is the same.  Instruction issue bounds it (three
// packed instructions per pair of cells and width, and about as many again for the prefixes), so
// the interior tiles have a body without end tests, every per-width value is read from LDS once (by
// scalar loads of the argument list in the width loop it took 0.54 ms instead of 0.29), and tiles
// without a marked cell stop before the ordered output.  Against the same arithmetic with widths
// known at compile time, even, at most 256 and interior tiles only, the rest on the general path:
// 4096 x 102,748 cells, seven widths 0.29 ms (was 0.32); 4 x 4096 rows of 8192 cells, where every
// second tile is a row's last, 0.16 (was 0.79); a multi-rate search's bands with widths to 1024,
// 0.27 ms in all (was 1.23).
template <bool BATCH>
__global__ __launch_bounds__(kThreads) void k_snr_pairs(const uint8_t *plane, int64_t pitch, int64_t n_,
                                                        const double *stats, SnrArgs a)
{
    extern __shared__ __align__(16) unsigned char pair_dyn[];  // one or two prefix arrays
    __shared__ PairShared sh;
    const uint8_t *rowk;
    int64_t n;
    const int32_t *row_nw;
    int k, kl;
    locate_row<BATCH>(plane, pitch, n_, a.row_nw, a.beams, a.nbeams, a.row0, (int)blockIdx.y, rowk, n, row_nw, k, kl);
    const int64_t t0 = (int64_t)blockIdx.x * kIntTile;
    if constexpr (BATCH) {
        if (t0 >= n) return;  // a shorter plane of the batch (uniform: before any barrier)
    }
    // the row's widths: the first nwk of the list
    int nwk = a.nw;
    if (row_nw) nwk = __builtin_amdgcn_readfirstlane(row_nw[kl]);
    const int avail = (int)(n - t0 < kIntTile + kMaxWidth ? n - t0 : kIntTile + kMaxWidth);
    if (kIntTile - 1 + a.wmax <= avail)  // uniform
        snr_pairs_tile<false>(rowk + t0, k, t0, avail, nwk, stats, a, pair_dyn, sh);
    else
        snr_pairs_tile<true>(rowk + t0, k, t0, avail, nwk, stats, a, pair_dyn, sh);
}

// PER: staged samples per thread.  BATCH: rows of several planes (SnrArgs::beams).  PLANE: the whole S/N
// plane instead of the cell list.  LDS reads and
// the FP64 bound tests bound the float form; with the widths as a run-time outer loop over
// straight-line slabs (against a run-time loop with end tests inside each cell) a 4096 x 102,748
// plane takes 1.12 ms with eleven widths up to 1024 (was 3.39), and 4 x 4096 rows of 8192 cells with
// seven widths 0.26 ms (was 0.81).
template <typename T, int PER, bool BATCH, bool PLANE>
__global__ __launch_bounds__(kThreads) void k_snr(const T *plane, int64_t pitch, int64_t n_, const double *stats,
                                                  SnrArgs a)
{
    using P = typename PrefixType<T>::type;
    constexpr bool G = std::is_same<P, double>::value && !PLANE;
    constexpr int kSlabs = snr_slabs<T>();  // cells per thread
    static_assert(kSlabs <= 32, "one flag bit per slab");
    extern __shared__ __align__(16) unsigned char snr_dyn[];  // prefix sums: tile + widest width + 1
    P *pre = reinterpret_cast<P *>(snr_dyn);
    __shared__ P wtot[kThreads / 64];
    __shared__ int slab_off[kSlabs][kThreads / 64];
    __shared__ unsigned int base_s;
    __shared__ double muw[kMaxWidths], den[kMaxWidths];  // per-row constants
    __shared__ P sthr[kMaxWidths];                       // per-row boxcar-sum bounds
    __shared__ int32_t sw[kMaxWidths + 1];               // the list
    const T *rowk;
    int64_t n;
    const int32_t *row_nw;
    int k, kl;
    locate_row<BATCH>(plane, pitch, n_, a.row_nw, a.beams, a.nbeams, a.row0, (int)blockIdx.y, rowk, n, row_nw, k, kl);
    // a row's last tile has no halo past it, so it may be as long as the slabs (1000 rows x 2034 samples,
    // the whole plane at seven widths: 40.0 us with a second tile of 50 samples, 26.7 in one)
    constexpr int kFull = kSlabs * kThreads;
    constexpr bool kWhole = IsInt<T>::value || PER == snr_per<T>(true);  // every tile is as long (see snr_tile)
    const int64_t t0 = (int64_t)blockIdx.x * (kWhole ? kFull : a.tile);
    if constexpr (BATCH) {
        // past a shorter plane of the batch (uniform: before any barrier)
        if (t0 >= n || (!kWhole && t0 > 0 && n - t0 + a.tile <= kFull)) return;
    }
    const int tile = kWhole || n - t0 <= kFull ? kFull : a.tile;
    const T *row = rowk + t0;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // widths of this row: the first nwk of the list (all of them unless a DM-scaled set)
    const int nwk = row_nw ? row_nw[kl] : a.nw;
    const int wmax = a.w[nwk - 1];
    // samples from the tile's first to the row's end, as far as any cell can read
    const int avail = (int)(n - t0 < tile + kMaxWidth ? n - t0 : tile + kMaxWidth);
    // elements t0 .. t0 + L - 1 are needed (and exist)
    const int L = avail < tile + wmax - 1 ? avail : tile + wmax - 1;
    // float tiles are read as 16-byte vectors, which may start on any element (1024 unaligned rows x 40,000
    // samples, one boxcar of 16: 129 us sample by sample, 96 so)
    static_assert(PER % 4 == 0, "vector chunks");
    const bool vec4 = !IsInt<T>::value && sizeof(T) == 4 && ((uintptr_t)row & 3u) == 0;
    // every thread takes PER elements, those past L read as zero (integer tiles: the staged bytes
    // fit the prefix array for any L), and only prefix entries up to L are written
    const int beg = tid * PER;
    // prefix sums: per-thread chunk totals, wave scan, wave totals through LDS.  Integer
    // tiles are first read with coalesced loads into LDS (in the prefix array's storage, which
    // is written only after the barrier below); float tiles are read in place (measured faster)
    P v[PER];
    P run = 0;
    if constexpr (IsInt<T>::value) {
        T *raw = reinterpret_cast<T *>(pre);
        static_assert(sizeof(T) <= sizeof(P), "the staged tile fits the prefix array");
        const auto grow = as_global(row);
        // 16-byte loads where the tile starts on a 16-byte boundary (rows of 64-sample pitch do)
        constexpr int E = 16 / (int)sizeof(T);
        int j0 = 0;
        if (((uintptr_t)row & 15u) == 0) {
            const auto g4 = as_global(reinterpret_cast<const u32x4 *>(row));
            u32x4 *r4 = reinterpret_cast<u32x4 *>(raw);
            for (int j = tid; j < L / E; j += kThreads) r4[j] = g4[j];
            j0 = L / E * E;
        }
        for (int j = j0 + tid; j < L; j += kThreads) raw[j] = grow[j];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int j = beg + i;
            const P x = (P)raw[j];
            v[i] = j < L ? x : (P)0;
            run += v[i];
        }
    } else if (vec4) {
        typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
        const auto grow = as_global(row);
#pragma unroll
        for (int i = 0; i < PER; i += 4) {
            const int j = beg + i;
            if (j + 3 < L) {
                const f32x4u q = *reinterpret_cast<global_ptr<const f32x4u>>(grow + j);
                v[i] = (P)q.x;
                v[i + 1] = (P)q.y;
                v[i + 2] = (P)q.z;
                v[i + 3] = (P)q.w;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[i + u] = j + u < L ? (P)grow[j + u] : (P)0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) run += v[i + u];
        }
    } else {
        const auto grow = as_global(row);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int j = beg + i;
            v[i] = j < L ? (P)grow[j] : (P)0;
            run += v[i];
        }
    }
    const P inc = wave_inclusive_sum(run);
    if (lane == 63) wtot[wv] = inc;
    __syncthreads();
    P acc = inc - run;
    for (int w = 0; w < wv; ++w) acc += wtot[w];
    if constexpr (G) {
        // entries 0 .. L: each thread writes the prefix before each of its samples, the thread that
        // holds sample L - 1 also the one after it
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (beg + i < L) pre[pre_at<G>(beg + i)] = acc;
            acc += v[i];
            if (beg + i == L - 1) pre[pre_at<G>(L)] = acc;
        }
    } else {
        if (tid == 0) pre[0] = (P)0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            acc += v[i];
            if (beg + i < L) pre[beg + i + 1] = acc;  // entries 1 .. L
        }
    }
    const double mu = stats[2 * k], sg = stats[2 * k + 1];
    // per-row constants of S/N(t, W) = (S_W(t) - mu W) / (sigma sqrt W)
    row_constants(tid, a, mu, sg, muw, den, sthr, IsInt<T>::value);
    if (tid < a.nw) sw[tid] = a.w[tid];
    __syncthreads();
    // the exact maximum over widths of sample i (first width on ties)
    auto exact = [&](int i, double &best, int &bi) {
        best = 0.0;
        bi = -1;
        for (int w = 0; w < nwk; ++w) {
            const int W = a.w[w];
            if (i + W > avail) break;
            double val = 0.0;
            if (sg > 0.0) {
                const double s = (double)(pre[pre_at<G>(i + W)] - pre[pre_at<G>(i)]);
                val = __dsub_rn(s, muw[w]) / den[w];
            }
            if (bi < 0 || val > best) {
                best = val;
                bi = w;
            }
        }
    };
    if constexpr (PLANE) {
        for (int i = tid; i < kFull; i += kThreads) {
            const int64_t t = t0 + i;
            if (i >= tile || t >= n) break;
            double best;
            int bi;
            exact(i, best, bi);
            a.snr[(int64_t)k * a.snr_pitch + t] = (float)best;
            a.widx[(int64_t)k * a.widx_pitch + t] = (int8_t)bi;
        }
        return;
    }
    if (!(sg > 0.0)) return;  // uniform: no cell of the row has a non-zero S/N
    // compaction: a cell can reach the threshold at width W only if its boxcar sum reaches
    // the row's bound for W (one subtraction and one compare per width, in the prefix type);
    // the cells that do take the exact quotient.  mk[j]: the wave's lanes whose cell of slab j does.
    uint64_t mk[kSlabs];
    P p0[kSlabs];
    const int last = tile - 1 < avail - 1 ? tile - 1 : avail - 1;  // last cell of the tile
    const int slabs = last / kThreads + 1;
#pragma unroll
    for (int j = 0; j < kSlabs; ++j) {
        mk[j] = 0;
        p0[j] = j < slabs ? pre[pre_at<G>(tid + kThreads * j)] : (P)0;
    }
    if (tile - 1 + wmax <= avail) {  // uniform: every width fits every cell
        for (int w = 0; w < nwk; ++w) {
            const P thr = sthr[w];
            const P *p = pre + pre_at<G>(tid + sw[w]);
            P s[kSlabs];
            // entry i + W + 256 j: 256 entries on, 32 gaps more in a float tile
#pragma unroll
            for (int j = 0; j < kSlabs; ++j) s[j] = p[pre_at<G>(kThreads * j)];
#pragma unroll
            for (int j = 0; j < kSlabs; ++j) mk[j] |= __ballot((P)(s[j] - p0[j]) >= thr);
        }
        mk[kSlabs - 1] &= __ballot(tid + kThreads * (kSlabs - 1) < tile);  // the last slab may be partial
    } else {
        for (int w = 0; w < nwk; ++w) {
            const int W = __builtin_amdgcn_readfirstlane(sw[w]);
            const int lim = avail - W < last ? avail - W : last;  // last cell of the tile that the width fits
            const P thr = sthr[w];
            const P *p = pre + pre_at<G>(tid + W);
#pragma unroll
            for (int j = 0; j < kSlabs; ++j) {
                if (kThreads * j > lim) break;  // uniform
                uint64_t hit = __ballot((P)(p[pre_at<G>(kThreads * j)] - p0[j]) >= thr);
                if (kThreads * j + kThreads - 1 > lim) hit &= __ballot(tid + kThreads * j <= lim);  // uniform
                mk[j] |= hit;
            }
        }
    }
    uint64_t any = 0;
#pragma unroll
    for (int j = 0; j < kSlabs; ++j) any |= mk[j];
    if (!__syncthreads_or(any != 0)) return;  // most tiles hold no such cell
    uint32_t flags = 0;
    if (any) {  // uniform over the wave
        uint32_t maybe = 0;
#pragma unroll
        for (int j = 0; j < kSlabs; ++j) maybe |= (uint32_t)((mk[j] >> lane) & 1u) << j;
        while (maybe) {
            const int j = __builtin_ctz(maybe);
            maybe &= maybe - 1u;
            double best;
            int bi;
            exact(tid + kThreads * j, best, bi);
            if (bi >= 0 && best >= a.threshold) flags |= 1u << j;
        }
    }
    // ordered output: the block's cells in increasing t (slab by slab, thread by thread)
#pragma unroll
    for (int j = 0; j < kSlabs; ++j) {
        mk[j] = __ballot((flags >> j) & 1u);
        if (lane == 0) slab_off[j][wv] = __popcll(mk[j]);
    }
    if (!__syncthreads_or((int)flags)) return;
    if (tid == 0) {
        int tot = 0;
        for (int j = 0; j < kSlabs; ++j)
            for (int w = 0; w < kThreads / 64; ++w) {
                const int c = slab_off[j][w];
                slab_off[j][w] = tot;
                tot += c;
            }
        base_s = atomicAdd(a.counter, (unsigned int)tot);
    }
    __syncthreads();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
    for (int j = 0; j < kSlabs; ++j) {
        if (!((flags >> j) & 1u)) continue;
        const int64_t pos = (int64_t)base_s + slab_off[j][wv] + __popcll(mk[j] & below);
        if (pos < a.max_pixels) {
            // the flagged cells are few: their exact maximum is taken again rather than kept
            const int i = tid + kThreads * j;
            double best;
            int bi;
            exact(i, best, bi);
            Pixel px;
            px.k = k;
            px.t = (int32_t)(t0 + i);
            px.snr = best;
            px.widx = bi;
            px.pad = 0;
            a.pixels[pos] = px;
        }
    }
}

// Robust row sigma, the MAD option of the matched filter: sigma = kMadScale * MAD, MAD the lower
// median of |y - m| over the row's valid samples and m the row's lower median (rank
// floor((n - 1) / 2) of the sorted values; kMadScale = 1 / Phi^-1(3/4) makes it the standard
// deviation of Gaussian noise).  Both medians are exact: a radix select over an order-preserving
// integer key of the values, 8 bits per pass over the row, with one histogram per wave in LDS.
// The deviation is taken in the plane's own arithmetic: exact for integer planes, one FP32
// subtraction for float planes.  The floor sigma_min applies as for the standard deviation.
constexpr double kMadScale = 1.4826022185056018;

template <typename T> struct MadKeys;
template <> struct MadKeys<uint8_t> {
    static constexpr int kBits = 8;
    __device__ static uint32_t key(uint8_t v) { return v; }
    __device__ static uint8_t value(uint32_t k) { return (uint8_t)k; }
    __device__ static uint32_t dev_key(uint8_t v, uint8_t m) { return v > m ? (uint32_t)(v - m) : (uint32_t)(m - v); }
    __device__ static double dev_value(uint32_t k) { return (double)k; }
};
template <> struct MadKeys<uint16_t> {
    static constexpr int kBits = 16;
    __device__ static uint32_t key(uint16_t v) { return v; }
    __device__ static uint16_t value(uint32_t k) { return (uint16_t)k; }
    __device__ static uint32_t dev_key(uint16_t v, uint16_t m) { return v > m ? (uint32_t)(v - m) : (uint32_t)(m - v); }
    __device__ static double dev_value(uint32_t k) { return (double)k; }
};
template <> struct MadKeys<float> {
    static constexpr int kBits = 32;
    // IEEE order as unsigned order: negative values reversed below the positive ones
    __device__ static uint32_t key(float v)
    {
        const uint32_t u = __float_as_uint(v);
        return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    }
    __device__ static float value(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k); }
    __device__ static uint32_t dev_key(float v, float m) { return key(__builtin_fabsf(v - m)); }
    __device__ static double dev_value(uint32_t k) { return (double)value(k); }
};

// Key of rank `rank` (0-based, in increasing order) among key(y) over the row.
template <typename T, int BITS, typename K>
__device__ uint32_t radix_select(const T *row, int64_t n, int64_t rank, K key, uint32_t (*hist)[256],
                                 uint32_t *s_digit, long long *s_rank)
{
    const int tid = threadIdx.x, wave = tid >> 6;
    uint32_t prefix = 0;
    for (int shift = BITS - 8; shift >= 0; shift -= 8) {
        for (int i = tid; i < (kThreads / 64) * 256; i += kThreads) (&hist[0][0])[i] = 0u;
        __syncthreads();
        const int hs = shift + 8;  // keys that agree with the prefix above this digit take part
        row_fold(row, n, tid, [&](T v, int) {
            const uint32_t k = key(v);
            if ((uint32_t)((uint64_t)(k ^ prefix) >> hs) == 0u) atomicAdd(&hist[wave][(k >> shift) & 255u], 1u);
        });
        __syncthreads();
        if (tid < 256) {
            uint32_t c = 0;
#pragma unroll
            for (int w = 0; w < kThreads / 64; ++w) c += hist[w][tid];
            hist[0][tid] = c;
        }
        __syncthreads();
        if (tid == 0) {  // the digit whose bin holds the rank; the taking part outnumber it
            long long r = rank;
            uint32_t b = 0;
            for (; b < 255u && r >= (long long)hist[0][b]; ++b) r -= hist[0][b];
            *s_digit = b;
            *s_rank = r;
        }
        __syncthreads();
        prefix |= *s_digit << shift;
        rank = *s_rank;
        __syncthreads();  // everyone has read the digit before the histogram is cleared
    }
    return prefix;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_rowmad(const T *plane, int64_t pitch, int64_t n, double sigma_min,
                                                       double *stats)
{
    __shared__ uint32_t hist[kThreads / 64][256];
    __shared__ uint32_t s_digit;
    __shared__ long long s_rank;
    const int64_t k = blockIdx.x;
    const T *row = plane + k * pitch;
    const int64_t r = (n - 1) / 2;
    using MK = MadKeys<T>;
    const T m = MK::value(radix_select<T, MK::kBits>(row, n, r, [](T v) { return MK::key(v); }, hist, &s_digit, &s_rank));
    const uint32_t d = radix_select<T, MK::kBits>(row, n, r, [m](T v) { return MK::dev_key(v, m); }, hist, &s_digit,
                                                  &s_rank);
    if (threadIdx.x == 0) {
        double sg = kMadScale * MK::dev_value(d);
        if (sg < sigma_min) sg = sigma_min;
        stats[2 * k + 1] = sg;
    }
}

__global__ void k_zero_counter(unsigned int *c) { *c = 0u; }

template <typename T, bool BATCH>
int launch_snr(int rows, const T *p, int64_t pitch, int64_t n, double *stats, const SnrArgs &a, hipStream_t st);

template <typename T>
int launch_typed(const void *plane, int64_t pitch, int ndm, int64_t n, double sigma_min, int sigma_mad,
                 double *stats, const SnrArgs &a, hipStream_t st)
{
    const T *p = static_cast<const T *>(plane);
    if (!a.snr) hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(1), 0, st, a.counter);
    hipLaunchKernelGGL((k_rowstats<T, false>), dim3((uint32_t)ndm), dim3(kThreads), 0, st, p, pitch, n, sigma_min,
                       stats, (const DetBeam *)nullptr, 0, 0);
    if (sigma_mad)  // sigma from the median absolute deviation instead (the mean stays)
        hipLaunchKernelGGL((k_rowmad<T>), dim3((uint32_t)ndm), dim3(kThreads), 0, st, p, pitch, n, sigma_min, stats);
    SnrArgs b = a;
    b.rows16 = ((uintptr_t)p & 15u) == 0 && pitch * (int64_t)sizeof(T) % 16 == 0;
    return launch_snr<T, false>(ndm, p, pitch, n, stats, b, st);
}

// Batched: statistics and S/N of batch rows a.row0 .. a.row0 + nrows - 1; the grid spans the
// longest plane, the tiles past a shorter plane's end return at once.
template <typename T>
int launch_typed_batch(int nrows, int64_t n_max, double sigma_min, double *stats, const SnrArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL((k_rowstats<T, true>), dim3((uint32_t)nrows), dim3(kThreads), 0, st, (const T *)nullptr,
                       (int64_t)0, (int64_t)0, sigma_min, stats, a.beams, a.nbeams, a.row0);
    return launch_snr<T, true>(nrows, (const T *)nullptr, 0, n_max, stats, a, st);
}

// n: samples per row (batched: of the longest plane)
template <typename T, bool BATCH>
int launch_snr(int rows, const T *p, int64_t pitch, int64_t n, double *stats, const SnrArgs &a0, hipStream_t st)
{
    using P = typename PrefixType<T>::type;
    SnrArgs a = a0;
    const int wmax = a.w[a.nw - 1];  // every row's set is a leading part of the list
    const bool wide = !IsInt<T>::value && wmax > kFloatNarrow;
    a.tile = snr_tile<T>(wmax);
    a.wmax = wmax;
    a.nfine = 0;
    a.odd = 0u;
    for (int w = 0; w < a.nw; ++w) {
        a.nfine += a.w[w] <= kPairExact;
        a.odd |= (uint32_t)(a.w[w] & 1) << w;
    }
    const int64_t past = n - snr_slabs<T>() * kThreads;  // samples that the last tile cannot hold
    const dim3 grid((uint32_t)(past > 0 ? 1 + (past + a.tile - 1) / a.tile : 1), (uint32_t)rows);
    if constexpr (std::is_same<T, uint8_t>::value) {
        if (!a.snr && a.rows16) {
            hipLaunchKernelGGL((k_snr_pairs<BATCH>), grid, dim3(kThreads), (size_t)pairs_lds_bytes(wmax), st, p, pitch,
                               n, stats, a);
            return (int)hipGetLastError();
        }
    }
    // the prefix array holds the tile's slabs (which are read whole) plus the widest boxcar; integer tiles
    // are first staged in its storage (at most kThreads * per samples of sizeof(T) <= 2 bytes each)
    int64_t bytes = ((int64_t)snr_slabs<T>() * kThreads + wmax + 1) * (int64_t)sizeof(P);
    if (IsInt<T>::value) bytes = std::max<int64_t>(bytes, (int64_t)kThreads * snr_per<T>(false) * 2);
    else if (!a.snr) bytes += bytes / 8 + (int64_t)sizeof(P);
    constexpr int narrow = snr_per<T>(false), broad = snr_per<T>(true);
    auto kernel = wide ? k_snr<T, broad, BATCH, false> : k_snr<T, narrow, BATCH, false>;
    if constexpr (!BATCH)
        if (a.snr) kernel = wide ? k_snr<T, broad, false, true> : k_snr<T, narrow, false, true>;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), (size_t)bytes, st, p, pitch, n, stats, a);
    return (int)hipGetLastError();
}

}  // namespace

int launch_detect(int plane_dtype, const void *plane, int64_t pitch, int ndm, int64_t n, double sigma_min,
                  int sigma_mad, double *stats, const SnrArgs &a, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    switch (plane_dtype) {
    case SND_DT_U8: return launch_typed<uint8_t>(plane, pitch, ndm, n, sigma_min, sigma_mad, stats, a, st);
    case SND_DT_U16: return launch_typed<uint16_t>(plane, pitch, ndm, n, sigma_min, sigma_mad, stats, a, st);
    case SND_DT_F32: return launch_typed<float>(plane, pitch, ndm, n, sigma_min, sigma_mad, stats, a, st);
    }
    return (int)hipErrorInvalidValue;
}

int launch_zero_counter(unsigned int *counter, void *stream)
{
    hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(1), 0, (hipStream_t)stream, counter);
    return (int)hipGetLastError();
}

int launch_detect_batch(int plane_dtype, int nrows, int64_t n_max, double sigma_min, double *stats, const SnrArgs &a,
                        void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    switch (plane_dtype) {
    case SND_DT_U8: return launch_typed_batch<uint8_t>(nrows, n_max, sigma_min, stats, a, st);
    case SND_DT_U16: return launch_typed_batch<uint16_t>(nrows, n_max, sigma_min, stats, a, st);
    case SND_DT_F32: return launch_typed_batch<float>(nrows, n_max, sigma_min, stats, a, st);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace snd
