// Final stage of a float-mode plan as one sum per DM row (Methods, "Tree activation modes":
// float mode applies no activation, so the root of DM d is the plain sum of its leaf neurons,
// each read at its own delay; Eq. for y_d in "Incoherent dedispersion").
//
// Staging is that of the other row-group kernels: 16 waves of 1024 threads, leaf windows copied
// global -> LDS in double-buffered batches, full tiles by 64-unit chunks listed in the plan.  Each
// wave sums four DM rows (64 DM-adjacent rows share the staged windows) over a tile of 1008 (f32) or
// 1024 samples (16-bit rows):
//  * f32 rows: lane i owns samples 4 i .. 4 i + 3 of four blocks of 252.  An input is read as the
//    16-byte units that hold its samples (LDS gives 16-byte reads twice the bytes per clock of
//    4- and 8-byte ones: 121 TB/s against 67 and 71 over the chip), and where its first sample is
//    not the first of a unit, the adds take the last ones from the next lane (a DPP operand of the
//    add; lane 63 has no next one, hence 252).  Four variants of the adds, one per place in the unit,
//    behind uniform branches.  Sums alone went from 8.5 to 6.7 ms at 1024 channels x 4096 DMs x
//    102,748 samples, the kernel from 8.9 to 8.2: the copies, 46 GB from a plane of 20 GB, take 6.1 by
//    themselves, a batch holds 2.4 inputs, and its copies start only when the batch before is done.
//    Tiles of two blocks, or eight rows of 512 samples by dwords, where those fit the grid to the chip
//    (lin_blocks).
//  * bf16 / f16 rows: reads are dwords at o + 4 i + 256 v for an input at LDS byte offset o (v = 0 .. 7),
//    which pair into stride-64 reads of two.  Lane i owns the sample pairs (2 i + 128 v, 2 i + 1 + 128 v).
//    An input whose first sample sits in the upper half of a dword takes the upper half of that
//    dword and the lower half of the next one (a second read); the branch on that is uniform.
//    f16 samples are added by v_fma_mix_f32 with a multiplier of 1.0 (the f16 half widened
//    exactly, the product exact, one rounding: the FP32 add of the widened sample, in one
//    instruction).  bf16 inputs go in twos: one
//    byte permute puts the two inputs' samples of one output sample into one dword, and one
//    v_dot2_f32_bf16 with weights (1, 1) adds both to the FP32 sum (one instruction per sample
//    instead of a widening and an add).  Only samples of the output being formed enter a dot.
//
// Each row is summed in FP32 in the order the plan lists its inputs (16-bit rows: batch by batch,
// each batch's inputs that start a dword before the others): an association of the exact sum
// that differs from the tree's, within the float tolerance of the FP64 definition.  A bf16 dot
// does not round like FP32 adds: measured on gfx950, its error stays below 1.5 x 2^-23 times the
// sum of its three terms' magnitudes (against 2^-24 times the result for an add), with a slight
// bias toward -infinity.  A row of n inputs is therefore within n 2^-23 sum|x| of the exact sum,
// the bound the parity tests check element by element.
#include <hip/hip_runtime.h>

#include "group_tab.h"

namespace snd {

namespace {

// The policies below index the sums of a wave in a plain array of the pipeline (a struct
// holding them ended up in scratch memory).
//
// f32 rows: st[4 (q * V + v) + j] is sample 252 v + 4 lane + j of row q.  The next input's units are read
// while one is added.
// Interface shared with the linear 16-bit sums: output element types, words per (batch, wave),
// the batch's inputs n (and the 16-bit dword-phase counts) as per-batch scalars; each policy
// sets its rows per wave and tile.
struct LinBase {
    using A = float;
    using TO = float;
    static constexpr int kWords = kLinWords, kSmemWords = kLinSmemWords;
    struct Carry {
        int n;
        uint32_t even;
    };
    static __device__ __forceinline__ Carry carry(const uint32_t (&blk)[kLinSmemWords])
    {
        return Carry{(int)blk[kLinSmemWords - 1], blk[kLinSmemWords - 2]};
    }
};

// V: blocks of a tile (four, or two in short tiles).
template <int V>
struct LinF32 : LinBase {
    using TI = float;
    static constexpr int R = lin_rows(SND_DT_F32), kRows = R, kStep = V * kLinBlock;
    static constexpr int kState = R * V * 4;
    static_assert(kLinBlock == 4 * 63 && R % 2 == 0, "the last quad of a block only feeds its neighbour; rows in twos");

    typedef float f32x4 __attribute__((ext_vector_type(4)));
    // a += the samples P .. P + 3 of the lane's quad x and its neighbour's
    template <int P>
    static __device__ __forceinline__ void add_at(float *a, const f32x4 (&x)[V])
    {
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j + P < 4)
                    a[4 * v + j] += x[v][j + P];
                else
                    a[4 * v + j] += __int_as_float(__builtin_amdgcn_update_dpp(
                        0, __float_as_int(x[v][j + P - 4]), 0x130, 0xf, 0xf, true));  // wave_shl:1
            }
        // keeps the four variants' adds apart: merged behind the branch, each operand takes a move
#pragma unroll
        for (int v = 0; v < V; ++v)
            asm volatile("; phase %4" : "+v"(a[4 * v]), "+v"(a[4 * v + 1]), "+v"(a[4 * v + 2]), "+v"(a[4 * v + 3]) : "i"(P));
    }
    // the n inputs of every row of the wave from the batch at buf; w: the lane's offset word
    static __device__ __forceinline__ void add_batch(float (&st)[kState], const unsigned char *buf,
                                                     const uint32_t (&w)[1], int lane, const Carry &c,
                                                     const GroupArgs &)
    {
        const uint32_t vw = w[0];
        const int n = c.n;
        const unsigned char *base = buf + 16 * lane;
        f32x4 x[2][V];
        uint32_t o[2];
        auto load = [&](int u, int k) {
            o[u] = (uint32_t)__builtin_amdgcn_readlane((int)vw, k);
            const unsigned char *p = base + (o[u] & ~15u);
#pragma unroll
            for (int v = 0; v < V; ++v) x[u][v] = *reinterpret_cast<const f32x4 *>(p + 4 * kLinBlock * v);
        };
        load(0, 0);
        for (int i = 0; i < n; ++i) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int u = q & 1;
                if (q + 1 < R) load(u ^ 1, (q + 1) * n + i);
                else if (i + 1 < n) load(u ^ 1, i + 1);
                float *a = &st[4 * V * q];
                uint32_t ph = o[u] & 12u;  // (read afresh by each test: a four-way branch takes moves of the sums)
                if (ph == 0u) add_at<0>(a, x[u]);
                asm volatile("" : "+s"(ph));
                if (ph == 4u) add_at<1>(a, x[u]);
                asm volatile("" : "+s"(ph));
                if (ph == 8u) add_at<2>(a, x[u]);
                asm volatile("" : "+s"(ph));
                if (ph == 12u) add_at<3>(a, x[u]);
            }
        }
    }
    static __device__ __forceinline__ void store(const float (&st)[kState], int q, float *drow, int lane, int vt,
                                                 const GroupArgs &s)
    {
        auto d = as_global(drow);
        const bool vec = (reinterpret_cast<uintptr_t>(drow) & 15u) == 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float *a = &st[4 * (V * q + v)];
            const int t = kLinBlock * v + 4 * lane;
            if (lane == 63 || t >= vt) continue;
            if (vec && t + 3 < vt) {
                *reinterpret_cast<__attribute__((address_space(1))) f32x4 *>(d + t) =
                    f32x4{a[0] * s.scale, a[1] * s.scale, a[2] * s.scale, a[3] * s.scale};
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (t + j < vt) d[t + j] = a[j] * s.scale;
            }
        }
    }
};

// f32 rows, eight per wave: st[q * V + v] is sample lane + 64 v of row q, each read as a dword (stride-64
// reads of two).
struct LinDwords : LinBase {
    using TI = float;
    static constexpr int R = lin_rows(SND_DT_F32, kLinDwords), kRows = R, kStep = lin_tile(SND_DT_F32, kLinDwords);
    static constexpr int V = kStep / 64;
    static constexpr int kState = R * V;

    static __device__ __forceinline__ void add_batch(float (&st)[kState], const unsigned char *buf,
                                                     const uint32_t (&w)[1], int lane, const Carry &c,
                                                     const GroupArgs &)
    {
        const uint32_t vw = w[0];
        const int n = c.n;
        const unsigned char *lane_base = buf + 4 * lane;
        for (int i = 0; i < n; ++i) {
#pragma unroll
            for (int q0 = 0; q0 < R; q0 += 2) {
                float x[2][V];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)vw, (q0 + u) * n + i);
                    const float *p = reinterpret_cast<const float *>(lane_base + o);
#pragma unroll
                    for (int v = 0; v < V; ++v) x[u][v] = p[64 * v];
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < V; ++v) st[(q0 + u) * V + v] += x[u][v];
                __builtin_amdgcn_sched_barrier(0);  // two rows' reads at a time: all eight's spill
            }
        }
    }
    static __device__ __forceinline__ void store(const float (&st)[kState], int q, float *drow, int lane, int vt,
                                                 const GroupArgs &s)
    {
        auto d = as_global(drow);
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (lane + 64 * v < vt) d[lane + 64 * v] = st[q * V + v] * s.scale;
    }
};

// bf16 / f16 rows: st[LO + q * V + v] and st[HI + q * V + v] are samples 2 lane + 128 v and
// 2 lane + 1 + 128 v of row q.  An input whose first sample starts a dword is read as one
// dword per pair; one whose first sample sits in the upper half of a dword as the upper half of
// that dword and the lower half of the next (two reads per pair).  The plan lists each row's
// inputs of the first kind first.
template <bool F16>
struct Lin16 : LinBase {
    using TI = uint16_t;
    static constexpr int R = lin_rows(SND_DT_BF16), kRows = R, kStep = lin_tile(SND_DT_BF16, 0);
    static constexpr int V = kStep / 128;
    static constexpr int LO = 0, HI = R * V, kState = 2 * R * V;

    static __device__ inline float lower(uint32_t d)
    {
        if constexpr (F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)(d & 0xffffu));
        else return __uint_as_float(d << 16);
    }
    static __device__ inline float upper(uint32_t d)
    {
        if constexpr (F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)(d >> 16));
        else return __uint_as_float(d & 0xffff0000u);
    }
    // f16: acc + the lower or upper half of d, widened, as one FP32 add (v_fma_mix_f32 with a
    // multiplier of 1.0 in a scalar register)
    static __device__ __forceinline__ float mix_lo(float acc, uint32_t d, uint32_t one)
    {
        float r;
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(d), "s"(one), "v"(acc));
        return r;
    }
    static __device__ __forceinline__ float mix_hi(float acc, uint32_t d, uint32_t one)
    {
        float r;
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(d), "s"(one), "v"(acc));
        return r;
    }
    // acc + lower(d) / upper(d): one instruction for f16, widening and add for bf16
    static __device__ __forceinline__ float add_lo(float acc, uint32_t d, uint32_t one)
    {
        if constexpr (F16) return mix_lo(acc, d, one);
        else return acc + lower(d);
    }
    static __device__ __forceinline__ float add_hi(float acc, uint32_t d, uint32_t one)
    {
        if constexpr (F16) return mix_hi(acc, d, one);
        else return acc + upper(d);
    }
    // byte selectors of v_perm_b32 (a, b): the lower halves of b and a, or their upper halves
    static constexpr uint32_t kLoLo = 0x05040100u, kHiHi = 0x07060302u;
    // acc + the two bf16 samples that the selector picks from a and b (weights one2 = (1, 1))
    static __device__ __forceinline__ float add2(float acc, uint32_t a, uint32_t b, uint32_t sel, uint32_t one2)
    {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const uint32_t pr = __builtin_amdgcn_perm(a, b, sel);
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pr), __builtin_bit_cast(bf16x2, one2), acc,
                                               false);
    }
    // Row q's inputs that start a dword (the first even_q of its n words), then the others: two
    // loops per row without a branch per input, two inputs in flight.
    static __device__ __forceinline__ void add_batch(float (&st)[kState], const unsigned char *buf,
                                                     const uint32_t (&w)[1], int lane, const Carry &c,
                                                     const GroupArgs &)
    {
        const uint32_t vw = w[0];
        const int n = c.n;
        const uint32_t even = c.even;
        // (1.0, 1.0) in bf16, materialised in a scalar register so that the compiler cannot encode
        // it as an inline constant (which the hardware would apply to one half only); 1.0f for f16
        uint32_t one2;
        if constexpr (F16) asm volatile("s_mov_b32 %0, 0x3f800000" : "=s"(one2));
        else asm volatile("s_mov_b32 %0, 0x3f803f80" : "=s"(one2));
        const unsigned char *lane_base = buf + 4 * lane;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int k0 = q * n, ke = k0 + (int)((even >> (4 * q)) & 15u), k1 = k0 + n;
            int k = k0;
            for (; k + 2 <= ke; k += 2) {
                uint32_t x[2][V];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)vw, k + u);
                    const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + o);
#pragma unroll
                    for (int v = 0; v < V; ++v) x[u][v] = p[64 * v];
                }
                if constexpr (F16) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            st[LO + q * V + v] = add_lo(st[LO + q * V + v], x[u][v], one2);
                            st[HI + q * V + v] = add_hi(st[HI + q * V + v], x[u][v], one2);
                        }
                } else {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        st[LO + q * V + v] = add2(st[LO + q * V + v], x[1][v], x[0][v], kLoLo, one2);
                        st[HI + q * V + v] = add2(st[HI + q * V + v], x[1][v], x[0][v], kHiHi, one2);
                    }
                }
            }
            if (k < ke) {
                const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)vw, k);
                const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + o);
                uint32_t x[V];
#pragma unroll
                for (int v = 0; v < V; ++v) x[v] = p[64 * v];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    st[LO + q * V + v] = add_lo(st[LO + q * V + v], x[v], one2);
                    st[HI + q * V + v] = add_hi(st[HI + q * V + v], x[v], one2);
                }
                ++k;
            }
            // first sample in the upper half: that half of the dword, then the lower half of the next
            if constexpr (!F16) {
                for (; k + 2 <= k1; k += 2) {
                    uint32_t x[2][V], y[2][V];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)vw, k + u);
                        const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + (o & ~3u));
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            x[u][v] = p[64 * v];
                            y[u][v] = p[64 * v + 1];
                        }
                    }
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        st[LO + q * V + v] = add2(st[LO + q * V + v], x[1][v], x[0][v], kHiHi, one2);
                        st[HI + q * V + v] = add2(st[HI + q * V + v], y[1][v], y[0][v], kLoLo, one2);
                    }
                }
            }
            for (; k < k1; ++k) {
                const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)vw, k);
                const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + (o & ~3u));
                uint32_t x[V], y[V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    x[v] = p[64 * v];
                    y[v] = p[64 * v + 1];
                }
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    st[LO + q * V + v] = add_hi(st[LO + q * V + v], x[v], one2);
                    st[HI + q * V + v] = add_lo(st[HI + q * V + v], y[v], one2);
                }
            }
        }
    }
    static __device__ __forceinline__ void store(const float (&st)[kState], int q, float *drow, int lane, int vt,
                                                 const GroupArgs &s)
    {
        const float scale = s.scale;
        auto d = as_global(drow);
        const bool vec = (reinterpret_cast<uintptr_t>(drow) & 7u) == 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float y0 = st[LO + q * V + v] * scale, y1 = st[HI + q * V + v] * scale;
            const int t = 2 * lane + 128 * v;
            if (vec && t + 1 < vt) {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                *reinterpret_cast<__attribute__((address_space(1))) f32x2 *>(d + t) = f32x2{y0, y1};
            } else {
                if (t < vt) d[t] = y0;
                if (t + 1 < vt) d[t + 1] = y1;
            }
        }
    }
};

}  // namespace

// The last tile of a launch takes as few blocks as hold its samples, one or two (see lin_blocks; 1024
// channels x 4096 DMs x 16,384 samples, eight tiles twice and half a block: 1430 us with all four, 1376 so).
template <class Sum>
struct LastTile {
    static __device__ __forceinline__ void run(const GroupArgs &s, uint32_t bid, uint32_t nblk, int)
    {
        group_tab_run<Sum>(s, bid, nblk);
    }
};
template <int V>
struct LastTile<LinF32<V>> {
    static __device__ __forceinline__ void run(const GroupArgs &s, uint32_t bid, uint32_t nblk, int left)
    {
        if (left <= kLinBlock) group_tab_run<LinF32<1>, V * kLinBlock>(s, bid, nblk);
        else if (V > 2 && left <= 2 * kLinBlock) group_tab_run<LinF32<2>, V * kLinBlock>(s, bid, nblk);
        else group_tab_run<LinF32<V>>(s, bid, nblk);
    }
};

template <class Sum>
__global__ __launch_bounds__(1024) void k_group_lin(GroupArgs s0, Multi m)
{
    GroupArgs s;
    uint32_t bid, nblk;
    select_record(s0, m, s, bid, nblk);
    const int t0 = (int)(xcd_remap_chunked(bid, nblk, (uint32_t)s.xcd_chunk) / (uint32_t)s.ngroups) * Sum::kStep;
    LastTile<Sum>::run(s, bid, nblk, s.n_out - t0);
}

namespace {

template <class Sum>
int launch_lin(const GroupArgs &a, int64_t n_out, int lds, void *stream, const Multi &m, int64_t nb_multi)
{
    const int64_t ntt = (n_out + Sum::kStep - 1) / Sum::kStep;
    const int64_t nb = m.n > 0 ? nb_multi : (int64_t)a.ngroups * ntt;
    if (nb <= 0) return 0;
    if (nb > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(k_group_lin<Sum>, dim3((uint32_t)nb), dim3(1024), lds, (hipStream_t)stream, a, m);
    return (int)hipGetLastError();
}

}  // namespace

int launch_group_lin(int src_dt, const GroupArgs &a, int64_t n_out, int lds, void *stream, const Multi &m,
                     int64_t nblocks)
{
    switch (src_dt) {
    case SND_DT_F32:
        switch (a.lin_blocks) {
        case 2: return launch_lin<LinF32<2>>(a, n_out, lds, stream, m, nblocks);
        case 4: return launch_lin<LinF32<4>>(a, n_out, lds, stream, m, nblocks);
        case kLinDwords: return launch_lin<LinDwords>(a, n_out, lds, stream, m, nblocks);
        default: return (int)hipErrorInvalidValue;
        }
    case SND_DT_BF16: return launch_lin<Lin16<false>>(a, n_out, lds, stream, m, nblocks);
    case SND_DT_F16: return launch_lin<Lin16<true>>(a, n_out, lds, stream, m, nblocks);
    default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace snd
