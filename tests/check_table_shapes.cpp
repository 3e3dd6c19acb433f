// Further host checks of the table kernels' plan tables, with the checks of check_copy_tables.cpp: shapes
// that must all build a table stage (the four-row packed ones and the short float tiles among them), every
// copied unit inside the source plane and the 64 bytes past it, and the packed launch's shapes all provided.
#define main check_copy_tables_main
#include "check_copy_tables.cpp"
#undef main

struct Wanted { int nchan, ndm, branching, cluster, mode, dt; double dm_max; int rpw; };

static PlanImpl plan_for(int nchan, int ndm, int branching, int cluster, int mode, int dt, double dm_max, int chunk)
{
    std::vector<double> f((size_t)nchan), dm((size_t)ndm);
    for (int c = 0; c < nchan; ++c) f[(size_t)c] = 416.0 - (c + 0.5) * 16.0 / nchan;
    for (int k = 0; k < ndm; ++k) dm[(size_t)k] = ndm > 1 ? dm_max * k / (ndm - 1) : dm_max;
    snd_plan_desc d{};
    d.nchan = nchan;
    d.freq_mhz = f.data();
    d.tsamp_s = 0.138e-3;
    d.ndm = ndm;
    d.dm = dm.data();
    d.branching = branching;
    d.cluster = cluster;
    d.mode = mode;
    d.cap = 255;
    d.in_dtype = d.node_dtype = dt;
    d.chunk = chunk;
    PlanImpl P;
    std::string err;
    CHECK(build_plan(d, P, err) == SND_OK);
    return P;
}

// 16-byte units that a full tile copies beyond the source plane: at most the four of its padding
static void check_reach(const PlanImpl &P, const Stage &S)
{
    const Stage &Q = P.stages[P.stages.size() - 2];
    const int es = dtype_size(S.src_dtype), epd = 16 / es;
    const int nsm = S.group_lin ? kLinSmemWords : kPackSmemWords;
    const long last_tile = (P.n_out / S.group_tile - 1) * S.group_tile;  // first sample of the last full tile
    if (last_tile < 0) return;
    const long plane = Q.rows * Q.pitch / epd;  // (rows start on units)
    CHECK(Q.pitch % epd == 0 && S.group_tile % epd == 0);
    for (size_t b = 0; b < S.batches.size() / 4; ++b)
        for (int w = 0; w < kGroupRows; ++w) {
            const uint32_t *sm = &S.lin_smem[(b * kGroupRows + w) * nsm];
            for (uint32_t c = 0; c < sm[0]; ++c) {
                const uint32_t cw = sm[3 + 3 * c], split = (cw >> 16) & 127u, lanes = cw >> 24;
                for (uint32_t lane = 0; lane < lanes; ++lane) {
                    const long u = (long)(lane < split ? sm[1 + 3 * c] : sm[2 + 3 * c]) + lane - kChunkBias + last_tile / epd;
                    CHECK(u >= 0 && u < plane + 4);
                }
            }
        }
}

int main()
{
    const int G = SND_MODE_GRADED, F = SND_MODE_FLOAT, U8 = SND_DT_U8, F32 = SND_DT_F32;
    const Wanted shapes[] = {
        {1024, 200, 8, 8, G, U8, 20.0, 4}, {512, 130, 8, 4, G, U8, 60.0, 4},  {4096, 40, 4, 4, G, U8, 30.0, 4},
        {64, 65, 8, 1, G, U8, 60.0, 4},     {1024, 300, 4, 4, G, U8, 500.0, 2}, {203, 64, 5, 4, G, U8, 40.0, 2},
        {1024, 300, 4, 4, F, F32, 150.0, 4}, {37, 300, 4, 4, F, F32, 20.0, 4},  {256, 64, 4, 4, F, F32, 10.0, 4},
        {1000, 129, 4, 4, F, SND_DT_BF16, 200.0, 4}, {64, 260, 2, 4, F, SND_DT_F16, 60.0, 4},
        {64, 1, 4, 4, F, F32, 5.0, 4},
    };
    for (const Wanted &s : shapes) {
        const PlanImpl P = plan_for(s.nchan, s.ndm, s.branching, s.cluster, s.mode, s.dt, s.dm_max, 5000);
        const Stage &S = P.stages.back();
        CHECK(P.stages.size() >= 2 && (s.mode == F ? S.group_lin : S.group_pack) && S.group_rpw == s.rpw);
        if (S.lin_blocks % 4 == 0 && S.lin_blocks <= 4) check_stage(P, S);  // (its cover is that of tiles of four blocks)
        check_reach(P, S);
        // offset words in the device image: each wave's inputs one after the other, as the kernel walks them
        const uint32_t *image = reinterpret_cast<const uint32_t *>(&P.table[(size_t)S.off_lin]);
        const int full = S.group_pack ? kPackWords : kLinWords, per = lin_input_words(S.group_pack, S.group_rpw);
        for (int g = 0; g < S.ngroups; ++g)
            for (int w = 0; w < kGroupRows; ++w) {
                long at = ((long)g * kGroupRows + w) * S.n_entries * per;
                for (int b = S.batch_ptr[(size_t)g]; b < S.batch_ptr[(size_t)g + 1]; ++b) {
                    const int words = (S.batches[4 * (size_t)b + 1] - S.batches[4 * (size_t)b]) * per;
                    const uint32_t *want = &S.lin[((size_t)b * kGroupRows + w) * full];
                    if (!lin_compact(S.group_pack, S.group_rpw)) at = ((long)b * kGroupRows + w) * full;
                    for (int i = 0; i < words; ++i) CHECK(image[at + i] == want[i]);
                    CHECK(S.off_lin + 4 * (at + (S.group_pack ? kPackWords : kLinWords)) <= (long)P.table.size());
                    at += words;
                }
            }
    }
    // every (inputs per level-1 node, depth, levels above the super nodes) of a packed stage is one of those
    // that its launch provides
    for (int nchan = 1; nchan < 700; nchan += nchan < 70 ? 1 : 37)
        for (int cluster : {1, 4})
            for (int branching : {2, 3, 4, 5, 8, 16}) {
                const PlanImpl P = plan_for(nchan, 33, branching, cluster, G, U8, 20.0, 1100);
                const Stage &S = P.stages.back();
                if (!S.group_pack) continue;
                const int f1 = S.group_f1, d = S.depth, u = d - S.wide_level;
                if (f1 == 4) CHECK(d == 5 || (d <= 4 && u == (d <= 2 ? 0 : d - 2)));
                else if (f1 == 8) CHECK(d <= 4);
                else CHECK(f1 == 0 && d <= kPackAnyDepth && S.wide_level >= 1 && u >= 0 && u < d);
            }
    std::printf("ok\n");
    return 0;
}
