// Host check of the plan builder's choice of kernels: each shape below gets the schedule that it is
// measured faster on.
#include <cmath>
#include <cstdio>
#include <vector>

#include "snd_internal.h"

using namespace snd;

struct Shape {
    int mode, dt, nchan, branching, ndm;
    double dm_lo, dm_max;  // equal ratios from dm_lo > 0, else equal steps from 0
    int64_t n_out;
    bool chunk = false;
};

static PlanImpl plan_of(const Shape &s)
{
    std::vector<double> f((size_t)s.nchan), dm((size_t)s.ndm);
    for (int c = 0; c < s.nchan; ++c) f[(size_t)c] = 416.0 - (c + 0.5) * 16.0 / s.nchan;
    for (int k = 0; k < s.ndm; ++k) {
        const double x = s.ndm > 1 ? (double)k / (s.ndm - 1) : 0.0;
        dm[(size_t)k] = s.dm_lo > 0.0 ? s.dm_lo * std::pow(s.dm_max / s.dm_lo, x) : s.dm_max * x;
    }
    snd_plan_desc d{};
    d.nchan = s.nchan;
    d.freq_mhz = f.data();
    d.tsamp_s = 0.138e-3;
    d.ndm = s.ndm;
    d.dm = dm.data();
    d.branching = s.branching;
    d.cluster = 4;
    d.mode = s.mode;
    d.k_leaf = 2;
    d.k_int = 1;
    d.cap = 255;
    d.in_dtype = d.node_dtype = s.dt;
    if (s.chunk) d.chunk = (int32_t)s.n_out;
    else d.nsamp = s.n_out + (int64_t)(14.3 * s.dm_max);
    PlanImpl P;
    std::string err;
    if (build_plan(d, P, err) != SND_OK) {
        std::printf("no plan: %s\n", err.c_str());
        P.stages.clear();
    }
    return P;
}

static int bad = 0;
#define EXPECT(x, ...)                                                                  \
    do {                                                                                \
        const Shape s_ = Shape{__VA_ARGS__};                                            \
        const PlanImpl P = plan_of(s_);                                                 \
        if (P.stages.size() != 2 || !(x)) {                                             \
            std::printf("line %d: %s does not hold\n", __LINE__, #x);                   \
            ++bad;                                                                      \
        }                                                                               \
    } while (0)

int main()
{
    const int G = SND_MODE_GRADED, F = SND_MODE_FLOAT, U8 = SND_DT_U8, F32 = SND_DT_F32;
    // sparse grids from the input in one stage: regular nodes, and in float the general kernel too where
    // the tree does not outgrow the open levels of the final stage
    EXPECT(P.direct.size() == 1 && P.direct[0].group_f1 == 4, G, U8, 64, 4, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.size() == 1 && P.direct[0].group_f1 == 4, G, U8, 64, 2, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.size() == 1 && P.direct[0].group_f1 == 4, G, U8, 128, 8, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.size() == 1, F, F32, 64, 4, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.size() == 1, F, F32, 128, 4, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.size() == 1 && P.direct[0].group_f1 == 0, F, F32, 128, 2, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.size() == 1 && P.direct[0].group_f1 == 0, F, F32, 37, 2, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.empty(), G, U8, 37, 2, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.empty(), G, U8, 100, 2, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.empty(), G, U8, 128, 2, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.empty(), F, F32, 128, 3, 600, 2.0, 800.0, 30000);
    EXPECT(P.direct.empty(), F, F32, 64, 2, 600, 2.0, 800.0, 30000);
    // grids that share their leaf rows keep the leaf plane
    EXPECT(P.direct.empty(), F, F32, 64, 4, 600, 0.0, 100.0, 30000);
    // irregular nodes: the packed kernel where its workgroups fill half the chip; streaming plans below that
    // hold both, for pushes alone and in shared grids
    EXPECT(!P.stages[1].group_pack && P.alone.empty(), G, U8, 1000, 4, 20, 0.0, 100.0, 9000);
    EXPECT(!P.stages[1].group_pack && P.alone.empty(), G, U8, 1000, 4, 300, 0.0, 300.0, 9000);
    EXPECT(!P.stages[1].group_pack && P.alone.empty(), G, U8, 300, 3, 600, 0.0, 300.0, 2500);
    EXPECT(P.stages[1].group_pack && P.alone.empty(), G, U8, 1000, 4, 600, 0.0, 300.0, 9000);
    EXPECT(P.stages[1].group_pack && P.alone.empty(), G, U8, 100, 4, 200, 0.0, 300.0, 30000);
    EXPECT(P.stages[1].group_pack && P.alone.size() == 1 && !P.alone[0].group_pack, G, U8, 1000, 4, 300, 0.0, 300.0,
           8192, true);
    EXPECT(P.stages[1].group_pack && P.alone.empty(), G, U8, 1000, 4, 1000, 0.0, 300.0, 8192, true);
    EXPECT(P.stages[1].group_pack && P.alone.empty(), G, U8, 1024, 4, 20, 0.0, 100.0, 8192, true);
    // regular nodes whose windows nearly fill a buffer, likewise
    EXPECT(P.stages[1].group_pack, G, U8, 256, 4, 600, 0.0, 300.0, 2640);
    EXPECT(!P.stages[1].group_pack && P.stages[1].group_f1 == 4, G, U8, 256, 4, 600, 0.0, 780.0, 2640);
    EXPECT(!P.stages[1].group_pack && P.stages[1].group_f1 == 4, G, U8, 256, 4, 16, 0.0, 100.0, 9018);
    EXPECT(!P.stages[1].group_pack && P.stages[1].group_f1 == 4, G, U8, 64, 4, 300, 0.0, 100.0, 535);
    EXPECT(P.stages[1].group_pack && P.alone.empty(), G, U8, 256, 4, 600, 0.0, 780.0, 9000);
    EXPECT(P.stages[1].group_pack && P.alone.size() == 1 && P.alone[0].group_f1 == 4, G, U8, 256, 4, 600, 0.0, 780.0,
           2640, true);
    // device tables: a row-group stage's entry lists stay on the host, and offset words leave without padding
    EXPECT(P.stages[1].off_ent == 0 && P.table.size() < 6000000, G, U8, 1000, 4, 1000, 0.0, 500.0, 30000);
    EXPECT(P.stages[1].off_ent == 0 && P.table.size() < 2000000, F, F32, 1024, 4, 300, 0.0, 150.0, 30000);
    EXPECT(P.direct[0].off_ent == 0 && P.table.size() < 1500000, F, F32, 64, 4, 600, 2.0, 800.0, 30000);
    return bad;
}
