// Staging pipeline of the table-driven row-group kernels (the one-sum float kernel and the
// packed graded kernel): 16 waves of 1024 threads, each wave computing Sum::kRows DM rows of
// one DM group over a time tile of Sum::kStep samples.  The leaf windows of a batch of inputs
// are copied global -> LDS into one of two buffers while the other batch is summed: in full
// tiles by the 64-unit chunks the plan lists per (batch, wave), in the last tile window by
// window.  Each buffer also receives the wave's offset words of its batch (Sum::kWords per
// wave, Sum::kWords / 64 per lane); the scalar words of batch b + 1 (chunks, counts) are
// loaded while the wave waits for the barrier of batch b.
//
// A Sum policy provides the element types, the sizes above, the per-batch scalars it needs
// (Carry, taken from the scalar words before they are overwritten), the per-batch arithmetic
// and the store of one row; the sums live in a plain array of this function (`st`).
#pragma once

#include "group_common.h"

namespace snd {

// The pipeline for workgroup bid of nblk over the arguments s (its record, already selected).  T: samples of
// the launch's tiles (a Sum of fewer serves a last tile that it covers).
template <class Sum, int T = Sum::kStep>
__device__ __forceinline__ void group_tab_run(const GroupArgs &s, uint32_t bid, uint32_t nblk)
{
    using TI = typename Sum::TI;
    using A = typename Sum::A;
    constexpr int ES = (int)sizeof(TI);
    constexpr int R = Sum::kRows, NW = Sum::kWords, NSM = Sum::kSmemWords;
    constexpr int WPL = NW / 64;  // offset words per lane
    static_assert(WPL == 1 || WPL == 4, "one load of 4 or 16 bytes per lane");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // logical tile = time tile * ngroups + DM group, dealt so that the XCDs share time tiles
    const uint32_t L = xcd_remap_chunked(bid, nblk, (uint32_t)s.xcd_chunk);
    const int g = (int)(L % (uint32_t)s.ngroups);
    const int t0 = (int)(L / (uint32_t)s.ngroups) * T;
    const int vt = s.n_out - t0 < T ? s.n_out - t0 : T;
    int row[R];
#pragma unroll
    for (int q = 0; q < R; ++q)
        row[q] = __builtin_amdgcn_readfirstlane(as_const(s.grp_rows)[(g * kGroupRows + wave) * R + q]);
    const unsigned char *srcb = static_cast<const unsigned char *>(s.src);
    const_ptr<int32_t> batches = as_const(s.batches);
    const_ptr<int32_t> instrs = as_const(s.instrs);
    const int64_t pitch_bytes = s.src_pitch * (int64_t)ES;
    const int buf_bytes = s.buf_elems * ES;
    const int stride = buf_bytes;  // bytes of one buffer
    const bool full = vt == T;  // full tiles copy from the chunk table; the last tile by window

    A st[Sum::kState];
#pragma unroll
    for (int i = 0; i < Sum::kState; ++i) st[i] = 0;

    const_ptr<uint32_t> smem_tab = as_const(s.lin_smem);
    // the tile's first sample of the plane's first row (t0 is a multiple of a 16-byte unit's samples);
    // chunk sources add their unit index
    const unsigned char *tile_src = srcb + ((int64_t)t0 * ES - 16 * kChunkBias);
    // the lane's offset words of the next batch
    constexpr bool kCompact = lin_compact(WPL == 4, R);
    constexpr int kPerInput = lin_input_words(WPL == 4, R);
    auto next = as_global(s.lin + (kCompact ? ((int64_t)g * kGroupRows + wave) * s.n_entries * kPerInput : 0)) + WPL * lane;
    // Copies of batch bb into buffer j: this wave's chunks of its windows (scalar words blk), or
    // its windows one by one in the last tile; and the lane's offset words of the batch into w.
    auto issue = [&](int bb, const uint32_t (&blk)[NSM], int j, uint32_t (&w)[WPL]) {
        unsigned char *buf_base = smem + j * stride;
        if (full) {
            const int nch = (int)blk[0];
#pragma unroll
            for (int c = 0; c < kLinMaxChunks; ++c) {
                if (c >= nch) break;
                const uint32_t cw = blk[3 + 3 * c];
                const uint32_t ua = blk[1 + 3 * c], ub = blk[2 + 3 * c], u = ua < ub ? ua : ub;
                const uint32_t at = (uint32_t)lane + (lane < (int)((cw >> 16) & 127u) ? ua - u : ub - u);
                if (lane < (int)(cw >> 24)) copy_lds16(tile_src + 16 * (uint64_t)u, 16u * at, buf_base + 16u * (cw & 0xffffu));
            }
        } else {
            issue_batch<TI, true>(batches, instrs, bb, wave, lane, srcb, pitch_bytes, t0, vt,
                            reinterpret_cast<TI *>(buf_base));
        }
        typedef uint32_t words_t __attribute__((ext_vector_type(WPL)));
        auto take = [&](global_ptr<const uint32_t> wp) {
            const words_t t = *reinterpret_cast<global_ptr<const words_t>>(wp);
#pragma unroll
            for (int i = 0; i < WPL; ++i) w[i] = t[i];
        };
        if constexpr (kCompact) {
            take(next);
            next += (int)blk[NSM - 1] * kPerInput;
        } else {
            take(as_global(s.lin + ((int64_t)bb * kGroupRows + wave) * NW + WPL * lane));
        }
    };
    auto load_blk = [&](int bb, uint32_t (&blk)[NSM]) {
        const_ptr<uint32_t> p = smem_tab + ((int64_t)bb * kGroupRows + wave) * NSM;
#pragma unroll
        for (int i = 0; i < NSM; ++i) blk[i] = p[i];
    };

    const int b0 = as_const(s.batch_ptr)[g], b1 = as_const(s.batch_ptr)[g + 1];
    uint32_t blk[NSM];
    uint32_t w[WPL] = {}, wn[WPL] = {};  // the wave's offset words of batches b and b + 1
    typename Sum::Carry cur{};
    if (b0 < b1) {
        load_blk(b0, blk);
        issue(b0, blk, 0, w);
        cur = Sum::carry(blk);
    }
    int slot = 0;
    for (int b = b0; b < b1; ++b) {
        // the scalar words of batch b + 1 load while this wave waits for its copies and the barrier
        if (b + 1 < b1) load_blk(b + 1, blk);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies of batch b have landed
        stage_barrier();  // everyone's have; everyone is done reading batch b - 1
        typename Sum::Carry nxt{};
        if (b + 1 < b1) {  // into the buffer of batch b - 1
            issue(b + 1, blk, slot ^ 1, wn);
            nxt = Sum::carry(blk);
        }
        const unsigned char *buf_base = smem + slot * stride;
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): no scalar loads left, so that waits for LDS reads can count
        Sum::add_batch(st, buf_base, w, lane, cur, s);
        cur = nxt;
#pragma unroll
        for (int i = 0; i < WPL; ++i) w[i] = wn[i];
        slot ^= 1;
    }

#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (row[q] < 0) continue;
        Sum::store(st, q, static_cast<typename Sum::TO *>(s.dst) + (int64_t)row[q] * s.dst_pitch + t0, lane, vt, s);
    }
}

}  // namespace snd
