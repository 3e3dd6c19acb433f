// Final stage of a graded-mode plan on u8 rows (Methods, "Tree activation modes": every node's output
// is the sum of its inputs clipped at the cap, at every level up to the root).  Integer arithmetic in
// the tree's own order throughout, or where no clip can apply in an order that gives the same integer:
// the result is the tree's, bit for bit.
//
// Staging is the table pipeline of the one-sum float kernel (group_tab.h); each wave computes two DM
// rows over 1008 samples, or four rows over 512 (depth 5, or level-1 nodes of eight inputs).  What
// bounds the sums is instruction issue (vector and scalar) and the waits of only four waves per SIMD, so the
// path is the one with the fewest instructions and reads per input that the plane's largest value m,
// which the stage that wrote it reports, allows; it is chosen per launch:
//
// * Wide sums (PackWide; two-row shapes): with n inputs in the largest super node (at most 16, two
//   levels of a tree of four) and n m < 256 no sum inside a super node passes a byte, and with the sums
//   one level below it at most the cap no clip inside it does anything.  So its inputs are added four
//   samples per instruction as the dwords that hold them, wherever their first sample sits in its dword:
//   grouped by that byte phase, highest first, the running sum is moved down by the difference (one
//   cross-lane move and one byte align) before the next group joins, at most three times per node
//   instead of once per input, and every input costs one dword read, not two.  Only the node's sum is
//   split into 16-bit counts, clipped and added to the levels above.  A lane needs its neighbour's dword
//   for those moves, so 63 lanes own samples and the 64th only feeds the 63rd.  1024 channels x 4096 DMs
//   x 102,748 samples: 4.5 ms (byte sums at level 1: 5.5); 1000 channels (a ragged tree) x 1021 DMs x
//   32.9 k samples: 0.47 ms (1.22 on the general row-group kernel, one byte per LDS read).
// * Byte sums at level 1 (BYTES; regular level-1 nodes of F1 inputs, F1 m < 256): each input's four
//   samples are aligned into one dword (v_alignbyte_b32) from the two that hold them, the F1 dwords are
//   added as four bytes at once, and the node's sum is split into 16-bit counts for the clip.
// * Any plane: one byte permute per pair of samples picks them out of two dwords as 16-bit counts,
//   (0, 2) and (1, 3); level sums are formed two samples per instruction (fan-in x cap < 2^16, so the
//   halves never carry into each other) and clipped with a packed 16-bit minimum.  Levels close with
//   compile-time control as the plan's closing counts say (PackGraded), or, where level-1 nodes are
//   irregular, input by input (PackAny).
//
// A sample position that holds no valid output (past the last tile's valid length) may carry out of
// its byte, but only into higher positions, which hold none either.
#include <hip/hip_runtime.h>

#include "group_tab.h"

namespace snd {

namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t pk_min_u16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                   __builtin_bit_cast(u16x2, b)));
}

// st[(j * R + q) * K + k]: j = 0 .. D - 2 the open partial sums of levels 2 .. D, j = D - 1 the
// root; k = 2 v + h holds samples (h, h + 2) of the lane's four in block v.  BYTES: level-1 sums
// as four bytes per dword (the input plane's bound allows it).
template <int F1, int D, bool BYTES>
struct PackGraded {
    using TI = uint8_t;
    using TO = uint8_t;
    using A = uint32_t;
    static constexpr int kRows = pack_rows(F1, D), kStep = pack_tile(F1, D), kWords = kPackWords,
                         kSmemWords = kPackSmemWords;
    static constexpr int R = kRows, V = (kStep + 255) / 256, K = 2 * V;
    static constexpr int OUT = D - 1;  // slot of the root
    static constexpr int kState = D * R * K;
    static_assert(F1 >= 3, "three-input adds");
    struct Carry {
        uint32_t close0, close1;  // levels completed by each level-1 node, 4 bits per node
        int n;
    };
    static __device__ __forceinline__ Carry carry(const uint32_t (&blk)[kPackSmemWords])
    {
        return Carry{blk[kPackCloses], blk[kPackCloses + 1], (int)blk[kPackSmemWords - 1]};
    }
    static __device__ __forceinline__ A &at(A (&st)[kState], int j, int q, int k) { return st[(j * R + q) * K + k]; }

    // close levels J .. D after a node that completes c levels (closing level j implies every
    // level below it)
    template <int J>
    static __device__ __forceinline__ void close_from(A (&st)[kState], int c, uint32_t cap2)
    {
        if constexpr (J <= D) {
            if (c >= J) {
#pragma unroll
                for (int q = 0; q < R; ++q)
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const uint32_t y = pk_min_u16(at(st, J - 2, q, k), cap2);
                        at(st, J - 2, q, k) = 0;
                        if constexpr (J == D) at(st, OUT, q, k) = y;
                        else at(st, J - 1, q, k) += y;
                    }
                close_from<J + 1>(st, c, cap2);
            }
        }
    }

    // the dword pairs holding the lane's samples of the F1 inputs of level-1 node j of one row
    // (offset words w), and per input the byte selector of its samples (0, 2); +0x00010001
    // gives samples (1, 3), and 0x0c fills a zero byte
    static __device__ __forceinline__ void load_row(uint32_t (&d)[F1][V][2], uint32_t (&sel)[F1], uint32_t w,
                                                    const unsigned char *lane_base, int j)
    {
#pragma unroll
        for (int u = 0; u < F1; ++u) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)w, j * F1 + u);
            sel[u] = 0x0c020c00u + (o & 3u) * 0x00010001u;
            const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + (o & ~3u));
#pragma unroll
            for (int v = 0; v < V; ++v) {
                d[u][v][0] = p[64 * v];
                d[u][v][1] = p[64 * v + 1];
            }
        }
    }

    // the same dword pairs, and per input its byte phase
    static __device__ __forceinline__ void load_row_bytes(uint32_t (&d)[F1][V][2], uint32_t (&ph)[F1], uint32_t w,
                                                          const unsigned char *lane_base, int j)
    {
#pragma unroll
        for (int u = 0; u < F1; ++u) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)w, j * F1 + u);
            ph[u] = o & 3u;
            const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + (o & ~3u));
#pragma unroll
            for (int v = 0; v < V; ++v) {
                d[u][v][0] = p[64 * v];
                d[u][v][1] = p[64 * v + 1];
            }
        }
    }

    // the level-1 nodes of one batch: for each, its F1 inputs per row, then the closes
    static __device__ __forceinline__ void add_batch(A (&st)[kState], const unsigned char *buf, const uint32_t (&w)[4],
                                                     int lane, const Carry &cr, const GroupArgs &s)
    {
        const uint32_t (&wq)[4] = w;  // component q: row q's input `lane`
        const uint32_t cap2 = (uint32_t)s.cap * 0x00010001u;
        const unsigned char *lane_base = buf + 4 * lane;
        const int nn = cr.n / F1;
        if constexpr (BYTES) {
            for (int j = 0; j < nn; ++j) {
                const int c = (int)(((j < 8 ? cr.close0 : cr.close1) >> (4 * (j & 7))) & 15u);
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    uint32_t d[F1][V][2], ph[F1];
                    load_row_bytes(d, ph, wq[q], lane_base, j);
                    uint32_t a[K];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        uint32_t x[F1];
#pragma unroll
                        for (int u = 0; u < F1; ++u) x[u] = __builtin_amdgcn_alignbyte(d[u][v][1], d[u][v][0], ph[u]);
                        // four byte sums below 256 each: no carries between valid samples
                        uint32_t acc = x[0] + x[1] + x[2];
#pragma unroll
                        for (int u = 3; u < F1; u += 2) acc = u + 1 < F1 ? acc + x[u] + x[u + 1] : acc + x[u];
                        a[2 * v] = __builtin_amdgcn_perm(0u, acc, 0x0c020c00u);      // samples (0, 2)
                        a[2 * v + 1] = __builtin_amdgcn_perm(0u, acc, 0x0c030c01u);  // samples (1, 3)
                    }
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const uint32_t y = pk_min_u16(a[k], cap2);
                        if constexpr (D == 1) at(st, OUT, q, k) = y;
                        else at(st, 0, q, k) += y;
                    }
                }
                close_from<2>(st, c, cap2);
            }
            return;
        }
        for (int j = 0; j < nn; ++j) {
            const int c = (int)(((j < 8 ? cr.close0 : cr.close1) >> (4 * (j & 7))) & 15u);
#pragma unroll
            for (int q = 0; q < R; ++q) {
                uint32_t d[F1][V][2], sel[F1];
                load_row(d, sel, wq[q], lane_base, j);
                // the node's sum of F1 permuted inputs, three at a time (v_add3_u32)
                uint32_t a[K];
#pragma unroll
                for (int v = 0; v < V; ++v)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        uint32_t x[F1];
#pragma unroll
                        for (int u = 0; u < F1; ++u)
                            x[u] = __builtin_amdgcn_perm(d[u][v][1], d[u][v][0], sel[u] + (h ? 0x00010001u : 0u));
                        uint32_t acc = x[0] + x[1] + x[2];
#pragma unroll
                        for (int u = 3; u < F1; u += 2) acc = u + 1 < F1 ? acc + x[u] + x[u + 1] : acc + x[u];
                        a[2 * v + h] = acc;
                    }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const uint32_t y = pk_min_u16(a[k], cap2);
                    if constexpr (D == 1) at(st, OUT, q, k) = y;
                    else at(st, 0, q, k) += y;
                }
            }
            close_from<2>(st, c, cap2);
        }
    }

    // root counts (<= cap <= 255) back to bytes: (s0, s2) | (s1, s3) << 8
    static __device__ __forceinline__ void store(const A (&st)[kState], int q, uint8_t *drow, int lane, int vt,
                                                 const GroupArgs &)
    {
        auto d = as_global(drow);
        const bool vec = (reinterpret_cast<uintptr_t>(drow) & 3u) == 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t x = st[(OUT * R + q) * K + 2 * v] | (st[(OUT * R + q) * K + 2 * v + 1] << 8);
            const int t = 4 * lane + 256 * v;
            if (vec && t + 4 <= vt) {
                *reinterpret_cast<__attribute__((address_space(1))) uint32_t *>(d + t) = x;
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (t + b < vt) d[t + b] = (uint8_t)(x >> (8 * b));
            }
        }
    }
};

// Two rows over four blocks of 252 samples: lane i owns samples 4 i + 252 v, lane 63 none.  U: levels
// above the super nodes.  st[(j * 2 + q) * 8 + 2 v + h], j < max(U, 1): the open sums of those levels as
// 16-bit counts of samples (h, h + 2) (U = 0: the root itself), then st[NB + 4 q + v]: the open super
// node's byte sums.
template <int U>
struct PackWide {
    using TI = uint8_t;
    using TO = uint8_t;
    using A = uint32_t;
    static constexpr int kRows = 2, kStep = kPackWideTile, kWords = kPackWords, kSmemWords = kPackSmemWords;
    static constexpr int V = 4, K = 2 * V, L = U > 0 ? U : 1;
    static constexpr int NB = L * 2 * K, kState = NB + 2 * V;
    struct Carry {
        uint32_t part[kPackMaxParts / 2];
        int n;
    };
    static __device__ __forceinline__ Carry carry(const uint32_t (&blk)[kPackSmemWords])
    {
        Carry c;
#pragma unroll
        for (int i = 0; i < kPackMaxParts / 2; ++i) c.part[i] = blk[kPackParts + i];
        c.n = (int)blk[kPackSmemWords - 2];
        return c;
    }
    // the sums moved down by `bytes` (1..3) byte positions, the next lane's low bytes coming in
    static __device__ __forceinline__ void drop(uint32_t (&acc)[V], uint32_t bytes)
    {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)acc[v], 0x130, 0xf, 0xf, true);  // wave_shl:1
            acc[v] = __builtin_amdgcn_alignbyte(next, acc[v], bytes);
        }
    }
    template <int C>
    static __device__ __forceinline__ void load(uint32_t (&x)[C][V], uint32_t (&d)[C], uint32_t words, int k,
                                                const unsigned char *lane_base)
    {
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)words, k + u);
            d[u] = o & 3u;
            const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + (o & ~3u));
#pragma unroll
            for (int v = 0; v < V; ++v) x[u][v] = p[63 * v];
        }
    }
    template <int C>
    static __device__ __forceinline__ void add(uint32_t (&acc)[V], const uint32_t (&x)[C][V], const uint32_t (&d)[C])
    {
        if constexpr (C == 4) {  // most groups of four hold one phase
            if ((d[0] | d[1] | d[2] | d[3]) == 0u) {
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = (acc[v] + x[0][v] + x[1][v]) + x[2][v] + x[3][v];
                return;
            }
        }
#pragma unroll
        for (int u = 0; u < C; u += 2) {  // every branch is uniform
            if (d[u]) drop(acc, d[u]);
            if (u + 1 < C && d[u + 1] == 0) {
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = acc[v] + x[u][v] + x[u + 1][v];
                continue;
            }
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] += x[u][v];
            if (u + 1 < C) {
                drop(acc, d[u + 1]);
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] += x[u + 1][v];
            }
        }
    }
    // levels J .. U above the super nodes, the last of which stays open (the root, clipped at the store)
    template <int J>
    static __device__ __forceinline__ void close_from(A (&st)[kState], int c, uint32_t cap2)
    {
        if constexpr (J < U) {
            if (c > J) {
#pragma unroll
                for (int i = 0; i < 2 * K; ++i) {
                    const uint32_t y = pk_min_u16(st[(J - 1) * 2 * K + i], cap2);
                    st[(J - 1) * 2 * K + i] = 0;
                    st[J * 2 * K + i] += y;
                }
                close_from<J + 1>(st, c, cap2);
            }
        }
    }
    static __device__ __forceinline__ void add_batch(A (&st)[kState], const unsigned char *buf, const uint32_t (&w)[4],
                                                     int lane, const Carry &cr, const GroupArgs &s)
    {
        const uint32_t cap2 = (uint32_t)s.cap * 0x00010001u;
        const unsigned char *lane_base = buf + 4 * lane;
        int k = 0;  // first input of the part
#pragma unroll 1
        for (int i = 0; i < cr.n; ++i) {
            const uint32_t word = i < 2 ? cr.part[0] : i < 4 ? cr.part[1] : i < 6 ? cr.part[2] : cr.part[3];
            const uint32_t part = i & 1 ? word >> 16 : word & 0xffffu;
            const int n = (int)(part & 31u), c = (int)((part >> 5) & 7u);
            uint32_t acc[2][V];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < V; ++v) acc[q][v] = 0u;
            int j = 0;
            for (; j + 4 <= n; j += 4) {  // four inputs of each row in flight
                uint32_t x0[4][V], x1[4][V], d0[4], d1[4];
                load(x0, d0, w[2], k + j, lane_base);
                load(x1, d1, w[3], k + j, lane_base);
                add(acc[0], x0, d0);
                add(acc[1], x1, d1);
            }
            for (; j < n; ++j) {
                uint32_t x0[1][V], x1[1][V], d0[1], d1[1];
                load(x0, d0, w[2], k + j, lane_base);
                load(x1, d1, w[3], k + j, lane_base);
                add(acc[0], x0, d0);
                add(acc[1], x1, d1);
            }
            k += n;
            const uint32_t last[2] = {(part >> 8) & 3u, (part >> 10) & 3u};
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (last[q]) drop(acc[q], last[q]);
#pragma unroll
                for (int v = 0; v < V; ++v) st[NB + V * q + v] += acc[q][v];
            }
            if (c == 0) continue;  // the super node goes on in the next batch
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const uint32_t b = st[NB + V * q + v];
                    st[NB + V * q + v] = 0u;
                    st[q * K + 2 * v] += pk_min_u16(__builtin_amdgcn_perm(0u, b, 0x0c020c00u), cap2);
                    st[q * K + 2 * v + 1] += pk_min_u16(__builtin_amdgcn_perm(0u, b, 0x0c030c01u), cap2);
                }
            close_from<1>(st, c, cap2);
        }
    }
    static __device__ __forceinline__ void store(const A (&st)[kState], int q, uint8_t *drow, int lane, int vt,
                                                 const GroupArgs &s)
    {
        const uint32_t cap2 = (uint32_t)s.cap * 0x00010001u;
        auto d = as_global(drow);
        const bool vec = (reinterpret_cast<uintptr_t>(drow) & 3u) == 0;
        if (lane == 63) return;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t x = pk_min_u16(st[((L - 1) * 2 + q) * K + 2 * v], cap2) |
                               pk_min_u16(st[((L - 1) * 2 + q) * K + 2 * v + 1], cap2) << 8;
            const int t = 4 * lane + 252 * v;
            if (vec && t + 4 <= vt) {
                *reinterpret_cast<__attribute__((address_space(1))) uint32_t *>(d + t) = x;
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (t + b < vt) d[t + b] = (uint8_t)(x >> (8 * b));
            }
        }
    }
};

// Any nodes: 16-bit counts, input by input, as the inputs' closing counts say.  Two rows, lane i
// owning samples 4 i + 256 v; st[(j * 2 + q) * 8 + 2 v + h]: the open sums of levels j + 1 = 1 .. D (the
// root is clipped at the store).
template <int D>
struct PackAny {
    using TI = uint8_t;
    using TO = uint8_t;
    using A = uint32_t;
    static constexpr int kRows = 2, kStep = kPackWideTile, kWords = kPackWords, kSmemWords = kPackSmemWords;
    static constexpr int V = 4, K = 2 * V, kState = D * 2 * K;
    struct Carry {
        uint32_t close[kPackMaxBatchEntries / 8];
        int n;
    };
    static __device__ __forceinline__ Carry carry(const uint32_t (&blk)[kPackSmemWords])
    {
        Carry c;
#pragma unroll
        for (int i = 0; i < kPackMaxBatchEntries / 8; ++i) c.close[i] = blk[kPackCloses + i];
        c.n = (int)blk[kPackSmemWords - 1];
        return c;
    }
    template <int J>
    static __device__ __forceinline__ void close_from(A (&st)[kState], int c, uint32_t cap2)
    {
        if constexpr (J < D) {
            if (c >= J) {
#pragma unroll
                for (int i = 0; i < 2 * K; ++i) {
                    const uint32_t y = pk_min_u16(st[(J - 1) * 2 * K + i], cap2);
                    st[(J - 1) * 2 * K + i] = 0;
                    st[J * 2 * K + i] += y;
                }
                close_from<J + 1>(st, c, cap2);
            }
        }
    }
    static __device__ __forceinline__ void add_batch(A (&st)[kState], const unsigned char *buf, const uint32_t (&w)[4],
                                                     int lane, const Carry &cr, const GroupArgs &s)
    {
        const uint32_t cap2 = (uint32_t)s.cap * 0x00010001u;
        const unsigned char *lane_base = buf + 4 * lane;
#pragma unroll
        for (int g = 0; g < kPackMaxBatchEntries / 8; ++g) {
            uint32_t closes = cr.close[g];
            for (int i = 8 * g; i < 8 * g + 8 && i < cr.n; ++i, closes >>= 4) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)(w[q]), i);
                    const uint32_t sel = 0x0c020c00u + (o & 3u) * 0x00010001u;
                    const uint32_t *p = reinterpret_cast<const uint32_t *>(lane_base + (o & ~3u));
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const uint32_t lo = p[64 * v], hi = p[64 * v + 1];
                        st[q * K + 2 * v] += __builtin_amdgcn_perm(hi, lo, sel);
                        st[q * K + 2 * v + 1] += __builtin_amdgcn_perm(hi, lo, sel + 0x00010001u);
                    }
                }
                close_from<1>(st, (int)(closes & 15u), cap2);
            }
        }
    }
    static __device__ __forceinline__ void store(const A (&st)[kState], int q, uint8_t *drow, int lane, int vt,
                                                 const GroupArgs &s)
    {
        const uint32_t cap2 = (uint32_t)s.cap * 0x00010001u;
        auto d = as_global(drow);
        const bool vec = (reinterpret_cast<uintptr_t>(drow) & 3u) == 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t x = pk_min_u16(st[((D - 1) * 2 + q) * K + 2 * v], cap2) |
                               pk_min_u16(st[((D - 1) * 2 + q) * K + 2 * v + 1], cap2) << 8;
            const int t = 4 * lane + 256 * v;
            if (vec && t + 4 <= vt) {
                *reinterpret_cast<__attribute__((address_space(1))) uint32_t *>(d + t) = x;
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (t + b < vt) d[t + b] = (uint8_t)(x >> (8 * b));
            }
        }
    }
};

}  // namespace

// F1 0: any nodes, U levels above the super nodes.  The bodies are separate, so that none holds
// another's registers; the choice is per record (uniform per workgroup).
template <int F1, int D, int U>
__global__ __launch_bounds__(1024) void k_group_pack(GroupArgs s0, Multi m)
{
    GroupArgs s;
    uint32_t bid, nblk;
    select_record(s0, m, s, bid, nblk);
    const uint32_t most = s.bound ? as_const(s.bound)[0] : 0xffffu;  // largest value of the input plane
    if constexpr (U >= 0) {
        if ((uint32_t)s.wide_inputs * most <= 255u && (uint32_t)s.wide_sub * most <= (uint32_t)s.cap) {
            group_tab_run<PackWide<U>>(s, bid, nblk);
            return;
        }
    }
    if constexpr (F1 == 0) {
        group_tab_run<PackAny<D>>(s, bid, nblk);
    } else {
        if ((uint32_t)F1 * most <= 255u) group_tab_run<PackGraded<F1, D, true>>(s, bid, nblk);
        else group_tab_run<PackGraded<F1, D, false>>(s, bid, nblk);
    }
}

namespace {

template <int F1, int D, int U>
int launch_pack(const GroupArgs &a, int64_t n_out, int lds, void *stream, const Multi &m, int64_t nb_multi)
{
    const int64_t ntt = (n_out + pack_tile(F1, D) - 1) / pack_tile(F1, D);
    const int64_t nb = m.n > 0 ? nb_multi : (int64_t)a.ngroups * ntt;
    if (nb <= 0) return 0;
    if (nb > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL((k_group_pack<F1, D, U>), dim3((uint32_t)nb), dim3(1024), lds, (hipStream_t)stream, a, m);
    return (int)hipGetLastError();
}

}  // namespace

// Every (inputs per level-1 node, depth) pair the plan builder admits for this kernel, and with
// irregular nodes every (depth, levels above the super nodes).  A tree of one level has no wide path: its
// nodes are single level-1 nodes, which the byte sums serve as they are (16 channels, 300 DMs x 29,987
// samples: 10.8 us by super nodes, 9.6).
int launch_group_pack(const GroupArgs &a, int64_t n_out, int lds, void *stream, const Multi &m, int64_t nblocks)
{
    const int u = a.depth - a.wide_level;
#define SND_PACK(F, DD, UU) \
    if (a.f1 == F && a.depth == DD && (UU < 0 || u == UU)) \
        return launch_pack<F, DD, UU>(a, n_out, lds, stream, m, nblocks);
    SND_PACK(4, 1, -1) SND_PACK(4, 2, 0) SND_PACK(4, 3, 1) SND_PACK(4, 4, 2) SND_PACK(4, 5, -1)
    SND_PACK(8, 1, -1) SND_PACK(8, 2, -1) SND_PACK(8, 3, -1) SND_PACK(8, 4, -1)
    SND_PACK(0, 1, 0)
    SND_PACK(0, 2, 0) SND_PACK(0, 2, 1)
    SND_PACK(0, 3, 0) SND_PACK(0, 3, 1) SND_PACK(0, 3, 2)
    SND_PACK(0, 4, 0) SND_PACK(0, 4, 1) SND_PACK(0, 4, 2) SND_PACK(0, 4, 3)
#undef SND_PACK
    return (int)hipErrorInvalidValue;
}

}  // namespace snd
