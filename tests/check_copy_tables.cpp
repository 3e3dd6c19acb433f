// Host check of the table kernels' plan tables: the copy chunks of every batch move exactly the units of
// its windows to their place in the LDS buffer, inside the source plane, and the offset words and parts
// of a wide packed plan name every input of a batch once, in phase order, with the drops between them.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "snd_internal.h"

#define CHECK(x)                                                              \
    do {                                                                      \
        if (!(x)) {                                                           \
            std::printf("failed at line %d: %s\n", __LINE__, #x);            \
            std::exit(1);                                                     \
        }                                                                     \
    } while (0)

using namespace snd;

static long check_stage(const PlanImpl &P, const Stage &S)
{
    const Stage &Q = P.stages[P.stages.size() - 2];
    const int es = dtype_size(S.src_dtype), epd = 16 / es;
    const int nw = S.group_lin ? kLinWords : kPackWords, nsm = S.group_lin ? kLinSmemWords : kPackSmemWords;
    const int cover = S.group_lin ? lin_cover(S.src_dtype)
                                  : S.group_rpw == 2 ? kPackReach : pack_tile(S.group_f1, S.depth) + 16;
    long windows = 0;
    for (size_t b = 0; b < S.batches.size() / 4; ++b) {
        const int n = S.batches[4 * b + 1] - S.batches[4 * b];
        std::vector<long> want((size_t)S.lds_buf_elems / epd, -1), got(want.size(), -1);
        for (int si = S.batches[4 * b + 2]; si < S.batches[4 * b + 3]; ++si, ++windows) {
            const int row = S.slots[4 * si], lo = S.slots[4 * si + 1], span = S.slots[4 * si + 2], at = S.slots[4 * si + 3];
            const int head = lo % epd, units = (head + span + cover + epd - 1) / epd;
            for (int u = 0; u < units; ++u) {
                CHECK((at - head) % epd == 0 && (size_t)((at - head) / epd + u) < want.size());
                want[(size_t)((at - head) / epd + u)] = ((long)row * Q.pitch + lo - head) / epd + u;
            }
        }
        for (int w = 0; w < kGroupRows; ++w) {
            const uint32_t *sm = &S.lin_smem[(b * kGroupRows + w) * nsm];
            CHECK(sm[0] <= (uint32_t)kLinMaxChunks && (int)sm[nsm - 1] == n);
            for (uint32_t c = 0; c < sm[0]; ++c) {
                const uint32_t cw = sm[3 + 3 * c];
                CHECK(std::labs((long)sm[2 + 3 * c] - (long)sm[1 + 3 * c]) <= kChunkReach + 64);
                for (uint32_t lane = 0; lane < cw >> 24; ++lane) {
                    const long src = (long)(lane < ((cw >> 16) & 127u) ? sm[1 + 3 * c] : sm[2 + 3 * c]) + lane - kChunkBias;
                    const size_t dst = (cw & 0xffffu) + lane;
                    CHECK(dst < got.size() && got[dst] == -1 && src >= 0);
                    got[dst] = src;
                }
            }
        }
        CHECK(want == got);
        if (!S.wide_level) continue;
        for (int w = 0; w < kGroupRows; ++w) {
            const uint32_t *sm = &S.lin_smem[(b * kGroupRows + w) * nsm];
            const uint32_t *words = &S.lin[(b * kGroupRows + w) * nw];
            int k = 0;
            CHECK(sm[nsm - 2] <= (uint32_t)kPackMaxParts);
            for (uint32_t p = 0; p < sm[nsm - 2]; ++p) {
                const uint32_t part = (sm[kPackParts + p / 2] >> (16 * (p % 2))) & 0xffffu;
                const int m = (int)(part & 31u);
                CHECK(m >= 1 && m <= kPackWideInputs && k + m <= n);
                const int closes = (int)(S.ent[(size_t)(S.batches[4 * b] + k + m - 1)].rowc >> 24);
                const int c = (int)((part >> 5) & 7u);
                CHECK(c == (closes >= S.wide_level ? closes - S.wide_level + 1 : 0));
                CHECK(c > 0 || p + 1 == sm[nsm - 2]);
                for (int q = 0; q < 2; ++q) {
                    std::vector<uint32_t> tree, sorted;
                    int phase = -1;
                    for (int i = k; i < k + m; ++i) tree.push_back(words[4 * i + q]);
                    uint32_t sum = 0;  // drops after input i: the phase it is read at, less the last phase
                    for (int i = k + m - 1; i >= k; --i) {
                        const uint32_t o = words[4 * i + 2 + q], at = (part >> (8 + 2 * q) & 3u) + sum;
                        CHECK(at <= 3 && (phase < 0 || (int)at >= phase));
                        phase = (int)at;
                        sorted.push_back((o & ~3u) | at);
                        sum += o & 3u;
                    }
                    CHECK((words[4 * k + 2 + q] & 3u) == 0);
                    for (uint32_t t : tree) {  // the same inputs, each once
                        size_t at = 0;
                        while (at < sorted.size() && sorted[at] != t) ++at;
                        CHECK(at < sorted.size());
                        sorted.erase(sorted.begin() + (long)at);
                    }
                }
                k += m;
            }
            CHECK(k == n);
        }
    }
    return windows;
}

int main()
{
    struct Shape { int nchan, ndm, branching, mode, dt; double dm_max; int chunk = 5000; };
    const Shape shapes[] = {
        {1024, 300, 4, SND_MODE_GRADED, SND_DT_U8, 500.0}, {1000, 70, 4, SND_MODE_GRADED, SND_DT_U8, 100.0},
        {999, 33, 8, SND_MODE_GRADED, SND_DT_U8, 60.0},    {1024, 200, 8, SND_MODE_GRADED, SND_DT_U8, 300.0},
        {97, 130, 3, SND_MODE_GRADED, SND_DT_U8, 80.0},    {203, 64, 5, SND_MODE_GRADED, SND_DT_U8, 40.0},
        {255, 65, 16, SND_MODE_GRADED, SND_DT_U8, 90.0},   {4096, 40, 4, SND_MODE_GRADED, SND_DT_U8, 30.0},
        {5, 40, 4, SND_MODE_GRADED, SND_DT_U8, 10.0},      {1024, 300, 4, SND_MODE_FLOAT, SND_DT_F32, 500.0},
        {1000, 129, 4, SND_MODE_FLOAT, SND_DT_BF16, 200.0}, {64, 260, 2, SND_MODE_FLOAT, SND_DT_F16, 60.0},
        {37, 300, 4, SND_MODE_FLOAT, SND_DT_F32, 700.0},
        {64, 1500, 4, SND_MODE_FLOAT, SND_DT_F32, 100.0, 4000000},  // windows of one batch gigabytes apart
    };
    long windows = 0;
    int stages = 0;
    for (const Shape &s : shapes) {
        std::vector<double> f((size_t)s.nchan), dm((size_t)s.ndm);
        for (int c = 0; c < s.nchan; ++c) f[(size_t)c] = 416.0 - (c + 0.5) * 16.0 / s.nchan;
        for (int k = 0; k < s.ndm; ++k) dm[(size_t)k] = s.dm_max * k / (s.ndm - 1);
        snd_plan_desc d{};
        d.nchan = s.nchan;
        d.freq_mhz = f.data();
        d.tsamp_s = 0.138e-3;
        d.ndm = s.ndm;
        d.dm = dm.data();
        d.branching = s.branching;
        d.cluster = 4;
        d.mode = s.mode;
        d.cap = 255;
        d.in_dtype = d.node_dtype = s.dt;
        d.chunk = s.chunk;
        PlanImpl P;
        std::string err;
        CHECK(build_plan(d, P, err) == SND_OK);
        const Stage &S = P.stages.back();
        if (P.stages.size() < 2 || !(S.group_lin || S.group_pack)) continue;
        windows += check_stage(P, S);
        ++stages;
    }
    std::printf("%d stages, %ld windows\n", stages, windows);
    return stages >= 10 ? 0 : 1;
}
