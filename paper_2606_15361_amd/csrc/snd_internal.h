// Internal declarations shared by the plan builder, the C ABI and the HIP kernels.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "snd.h"

namespace snd {

// Dispersion constant in MHz^2 ms per (pc cm^-3) (Methods, "Incoherent dedispersion").
constexpr double kDM = 4.148808e6;
// Deepest sub-tree one kernel stage evaluates in registers.
constexpr int kMaxDepth = 16;
// Source rows addressable by a table entry (low 24 bits of Entry::rowc).
constexpr uint32_t kRowMask = 0x00FFFFFFu;

// One input of a stage output row: source row (low 24 bits), the number of sub-tree levels
// that complete after this input (high 8 bits), and the time offset into the source row.
struct Entry {
    uint32_t rowc;
    int32_t off;
};

// Kernel stage: every output row is the value of one tree node's neuron (or, in the final
// stage, of the root for one DM), computed from rows of a lower materialised level (or the
// input channels) by evaluating the sub-tree between them in registers.
struct Stage {
    int src_level = -1;      // -1 = input channels
    int dst_level = 0;       // tree level computed by this stage
    int depth = 1;           // dst_level - src_level
    bool final_stage = false;
    int64_t rows = 0;
    int64_t max_len = 0;     // longest output row (samples)
    int64_t pitch = 0;       // output pitch in elements (non-final stages)
    int src_dtype = 0, dst_dtype = 0;
    int64_t src_rows = 0;
    std::vector<uint32_t> row_ptr;  // rows + 1
    std::vector<int32_t> row_len;   // samples computed per output row
    std::vector<Entry> ent;
    int64_t off_row_ptr = 0, off_row_len = 0, off_ent = 0;  // byte offsets in the table image
    int64_t ws_off = 0;            // byte offset of the output plane in the workspace
    int64_t alg_bytes = 0;

    // Kernel chosen for the stage.
    int kernel = 0;  // kKernelGeneric, kKernelGroupLds or kKernelAnchored

    // kKernelGroupLds: rows in groups of kGroupRows sharing LDS-staged source windows.
    int64_t ngroups = 0;
    int32_t n_entries = 0;          // entries per row (identical for every row)
    int32_t lds_bytes = 0;          // dynamic LDS per workgroup
    int32_t lds_buf_elems = 0;      // elements per LDS buffer (group kernel)
    int32_t group_f1 = 0;           // inputs per level-1 node when regular (specialised kernel), else 0
    int32_t group_tile = 0;         // time samples per workgroup
    int32_t xcd_chunk = 1;          // DM groups of one time tile dealt to each XCD in turn
    int32_t group_rpw = 1;          // rows per wave (kFastRows for the specialised kernel)
    std::vector<int32_t> grp_rows;  // [ngroups * kGroupRows * rows per wave], -1 = padding
    std::vector<int32_t> batch_ptr; // [ngroups + 1] into batches
    std::vector<int32_t> batches;   // 4 ints per batch: entry begin, entry end, window begin, window end
    std::vector<int32_t> slots;     // 4 ints per staged window: source row, start offset, span, LDS element
                                    // offset (host only: plan statistics)
    std::vector<int32_t> instrs;    // 4 ints per staged window, as copied: source row, element offset of
                                    // its 16-byte aligned footprint, LDS byte offset of the footprint,
                                    // head + span (elements from the footprint start, tile excluded)
    std::vector<uint32_t> ldsb;     // [ngroups][kGroupRows][n_entries][rows per wave]: LDS element offset |
                                    // closes << 24 (general kernel) or LDS byte offset (specialised kernel)
    std::vector<int32_t> node_closes;  // specialised kernel: levels completed by each level-1 node
    // Linear kernel (float mode: the final stage is one sum over its inputs, no activation).  Per
    // (global batch index, wave): kLinWords offset words, one per lane: words
    // q * n .. q * n + n - 1 are the LDS byte offsets of the first samples of the n inputs of the
    // wave's row q (16-bit rows: those that start a dword first, each part in plan order); and
    // kLinSmemWords words read as scalars: the number of copy chunks of the wave, then for its
    // chunks (global -> LDS copies of up to 64 16-byte units, see kLinMaxChunks) three words each,
    // then (16-bit rows) the count of each
    // row's inputs that start a dword (4 bits per row), and last n.  The packed kernel keeps its
    // tables (kPackWords and kPackSmemWords per batch and wave) in the same two vectors.
    bool group_lin = false;
    int32_t lin_blocks = 0;  // f32 rows: blocks of a tile, or kLinDwords (0 on 16-bit rows)
    bool group_pack = false;
    // packed kernel, two-row shapes: the super nodes' level and largest number of inputs, and that of
    // the nodes one level below
    int32_t wide_level = 0, wide_inputs = 0, wide_sub = 0;
    bool pack_idle = false;  // packed kernel, in a launch of its own: fewer workgroups than it pays for
    std::vector<uint32_t> lin;
    std::vector<uint32_t> lin_smem;
    int64_t off_grp_rows = 0, off_batch_ptr = 0, off_batches = 0, off_instrs = 0, off_ldsb = 0;
    int64_t off_node_closes = 0, off_lin = 0, off_lin_smem = 0;

    // kKernelAnchored: one workgroup per (node, window of anchor_tile reference samples).
    std::vector<int32_t> nodes;     // 6 ints per node: row begin, row end, channel begin, channel end, rho max,
                                    // reach of its rows past n_out
    std::vector<int32_t> tiles;     // 2 ints per workgroup: node index, window start
    std::vector<int32_t> row_lo;    // [rows]
    // 8 ints per row of a one-level stage (not on bit rows): row_lo, row_len, inputs (channel within the
    // node << 24 | offset past row_lo; the first four), first entry, entries
    std::vector<int32_t> leaf;
    int32_t anchor_tile = 0;        // reference samples per workgroup window
    int32_t spread = 0;             // largest delay difference between the inputs of a row
    int64_t off_nodes = 0, off_tiles = 0, off_row_lo = 0, off_leaf = 0;
    int64_t ntiles = 0;
};

constexpr int kKernelGeneric = 0;
constexpr int kKernelGroupLds = 1;
constexpr int kKernelAnchored = 2;
constexpr int kGroupRows = 16;       // rows (waves) per LDS-group workgroup
constexpr int kGroupTile = 256;      // time samples per LDS-group workgroup
constexpr int kGroupLdsBytes = 20480;  // per LDS buffer
constexpr int kGroupBuffers = 3;       // batches b, b+1, b+2 in LDS at once
// Specialised group kernel: regular level-1 nodes of f1 inputs, compile-time depth; each wave
// computes kFastRows DM rows of 64 * kFastV samples, so a workgroup covers kGroupRows *
// kFastRows rows (more rows share each staged window) and a tile of kGroupTileFast samples.
constexpr int kFastRows = 2;
// FDMT: neighbouring delay rows a workgroup forms together (two workgroups' LDS on a CU), and the most
// iterations of a pass.
constexpr int kFdmtRun = 28;
constexpr int kFdmtMaxIters = 5;
constexpr int kFastV = 8;
constexpr int kGroupTileFast = 64 * kFastV;
constexpr int kFastBuffers = 2;           // batch b + 1 lands while b is read
constexpr int kGroupFastLdsBytes = 81920; // per buffer (two fill the 160 KB of LDS)
constexpr int kGroupTileBits = 2048;  // bit rows: 32 samples (one word) per lane
// Linear kernel shape per row storage: four rows per wave (64-row groups share the staged windows).  f32
// rows: tiles of 4 x 252 samples, read by 16-byte units that run up to four samples past the tile, or other
// shapes (lin_blocks).
// 16-bit rows: tiles of 1024 samples, lane i owning the sample pairs 2 i + 128 v (v = 0 .. 7); an input
// that starts in the upper half of a dword reads one dword past the tile, so those windows stage one
// 16-byte unit more.
constexpr int kLinBlock = 4 * 63;
constexpr int kLinDwords = 8;   // (in place of the blocks of a tile) eight rows per wave, 512 samples by dwords
constexpr int64_t kLinMinBlocks = 128, kLinRound = 256;
constexpr int lin_rows(int src_dtype, int blocks = 4) { return src_dtype == SND_DT_F32 && blocks == kLinDwords ? 8 : 4; }
constexpr int lin_tile(int src_dtype, int blocks = 4)
{
    return src_dtype != SND_DT_F32 ? 1024 : blocks == kLinDwords ? 512 : blocks * kLinBlock;
}
constexpr int lin_cover(int src_dtype, int blocks = 4)
{
    return lin_tile(src_dtype, blocks) + (src_dtype != SND_DT_F32 ? 8 : blocks == kLinDwords ? 0 : 4);
}
// Blocks of a tile on f32 rows.  Two where the rows are one group and tiles of four would give fewer
// workgroups than half the CUs (final stage of 1024 channels, 24 DMs x 30,014 samples: 214 us in tiles of four,
// 151 of two; 64 x 2514 221 and 158; 300 channels, 16 x 9017: 66 and 48).  Else four, or eight rows by dwords
// where that takes so many fewer rounds of a workgroup on every CU that they make up for its longer ones (320
// against 290 us a round at 1024 channels x 4096 DMs): rows of 2^k samples divide into its tiles alone.  1024
// channels x 4096 DMs x 8192 samples 782 us by four blocks, 639 by dwords; 16,384 1376 and 1265; 256 x 2000 x
// 8192 159 and 108; but 8064 samples 583 and 690, 16,128 1154 and 1331, 65,536 4906 and 5122.
inline int lin_blocks(int64_t rows, int64_t n_out)
{
    auto wgs = [&](int b) {
        const int64_t gr = kGroupRows * lin_rows(SND_DT_F32, b), tile = lin_tile(SND_DT_F32, b);
        return ((rows + gr - 1) / gr) * ((n_out + tile - 1) / tile);
    };
    auto rounds = [&](int b) { return (wgs(b) + kLinRound - 1) / kLinRound; };
    if (rows <= kGroupRows * lin_rows(SND_DT_F32) && wgs(4) < kLinMinBlocks) return 2;
    return 32 * rounds(kLinDwords) < 29 * rounds(4) ? kLinDwords : 4;
}
// inputs per row and batch: the wave's offset words fit 64 lanes, and the 16-bit kernels pack
// each row's count of inputs of one dword phase in 4 bits
constexpr int lin_max_batch_entries(int src_dtype, int blocks = 4)
{
    return 64 / lin_rows(src_dtype, blocks) < 15 ? 64 / lin_rows(src_dtype, blocks) : 15;
}
constexpr int kLinWords = 64;                  // offset words per (batch, wave), at most
// Copy chunks of a wave and batch: up to 64 consecutive 16-byte units of the LDS buffer each, from one
// window or the end of one and the start of the next (windows are laid out one after the other, and a
// window's last chunk alone would leave most lanes idle: u8 windows of 65 or 66 units took two chunks
// each, and 112 chunks, not the LDS, ended a batch; 4096 graded DMs now take 2278 batches instead of 3050,
// and their final stage 4.5 ms instead of 4.9).
constexpr int kLinMaxChunks = 7;
constexpr int kLinSmemWords = 24;              // chunk count, 7 x 3 chunk words, counts, n
// Chunk words: the first lane's source unit; the source unit of the lane where the second window
// starts, less that lane's index (both plus kChunkBias); LDS unit | that lane << 16 | lanes << 24.
constexpr int kChunkBias = 64;
constexpr int64_t kChunkReach = int64_t(1) << 26;  // source units between a chunk's two windows
constexpr int kLinBuffers = 2;                 // batch b + 1 lands while b is read
constexpr int kLinLdsBytes = 163840 / kLinBuffers;  // window bytes per buffer
// Packed kernel (graded mode on u8 rows): the staging and copy tables of the linear kernel.  Each
// wave computes pack_rows DM rows over tiles of pack_tile samples: two rows where the open level sums
// of the shape fit the registers (regular level-1 nodes of four inputs and depth <= 4, or any nodes
// of depth <= kPackAnyDepth: f1 0; 32-row groups), four rows over 512 samples otherwise (64-row
// groups).  Windows stage one 16-byte unit beyond the tile's reach, since an input's first samples may
// start anywhere in a dword.
// Two-row shapes sum the inputs of whole nodes as bytes (the wide path, chosen per launch when the
// input plane's bound allows it): the super nodes, of the highest level whose nodes have at most
// kPackWideInputs inputs.  Its lanes own 63 dwords of samples and the 64th only feeds its neighbour, so
// those tiles are 4 x 252 samples.
// Offset words: lane i, component q of a 16-byte word holds input i of row q, in the tree's order;
// two-row shapes keep in components 2 and 3 the inputs of rows 0 and 1 grouped by byte phase within
// each part (a batch's share of one super node): the byte offset of the dword that holds the first
// sample, and in its low two bits by how many bytes the phase drops from the input before.
// Scalar words: the chunk words of the linear kernel; the levels each level-1 node (f1 0: each input)
// of the batch completes, 4 bits each; the parts, 16 bits each (inputs, levels completed from the super
// node on (0: it goes on in the next batch), last phase of rows 0 and 1); their number; the inputs.
constexpr int kPackAnyDepth = 4;
constexpr int kPackWideInputs = 16;
constexpr int kPackWideTile = 4 * 4 * 63;
constexpr int kPackMaxParts = 8;
constexpr int pack_rows(int f1, int depth) { return f1 == 0 || (f1 == 4 && depth <= 4) ? 2 : 4; }
constexpr int pack_tile(int f1, int depth) { return pack_rows(f1, depth) == 2 ? kPackWideTile : 512; }
constexpr int kPackReach = 1024 + 16;          // samples a two-row window holds beyond its span
// Irregular nodes, and regular ones whose windows nearly fill a buffer (more than kPackRoom bytes for one
// node: a batch is then one node), take the packed kernel only in launches of at least this many
// workgroups, about half the CUs: its groups are wider and its tiles longer than the other row-group
// kernels', which leaves CUs idle on smaller grids.  (Streaming plans below that keep both: the
// beams of a batched push share one grid.)  Final stage of 1000 channels, against the general kernel: 100 DMs x 9042
// samples (36 workgroups) 84 us, packed 185; 64 DMs x 30,014 (60) 99 and 155; 300 x 9042 (90) 142 and 150;
// 100 x 30,042 (120) 188 and 186; 600 x 9042 (171) 233 and 138.  Of 256 channels, regular, DMs 1.3 apart,
// against the specialised kernel: 600 x 2640 (57) 40 and 51; 200 x 30,047 (210) 76 and 52.
constexpr int kPackRoom = 59 * 1024;
constexpr int64_t kPackMinBlocks = 128;
constexpr int kPackRowsMax = 4;
constexpr int kPackMaxBatchEntries = 64;
constexpr int kPackWords = 256;                // offset words per (batch, wave), at most
constexpr int kPackCloses = 22, kPackParts = kPackCloses + kPackMaxBatchEntries / 8;  // first words
constexpr int kPackSmemWords = kPackParts + kPackMaxParts / 2 + 2;
// The device image holds the offset words without the unused ones, group by group and in each wave by
// wave: lin_input_words per input of the row, batch after batch.  A wave's lanes may read up to kPackWords
// words on from a batch's first.  (1024 channels x 4096 DMs: 49 MB of tables graded and 44 in f32 with them,
// 20 and 21.)  Four-row packed shapes keep them, kPackWords a batch and wave: their scalar registers are
// full, and a running address cost the kernel 10 % (1024 channels by eights x 1000 DMs, 0.48 -> 0.53 ms).
constexpr bool lin_compact(bool pack, int rows) { return !(pack && rows == 4); }
constexpr int lin_input_words(bool pack, int rows) { return pack ? 4 : rows; }
constexpr int kPackLdsBytes = 163840 / 2;
inline bool group_fast_types(int mode, int src_dt, int dst_dt)
{
    if (mode == SND_MODE_BINARY) return (src_dt == SND_DT_U8 || src_dt == SND_DT_BITS) && dst_dt == SND_DT_U8;
    if (mode == SND_MODE_GRADED) return src_dt == dst_dt && (src_dt == SND_DT_U8 || src_dt == SND_DT_U16);
    return dst_dt == SND_DT_F32;
}
inline bool group_fast_supported(int f1, int depth)
{
    return (f1 == 2 && depth >= 1 && depth <= 8) || (f1 == 4 && depth >= 1 && depth <= 5) ||
           (f1 == 8 && depth >= 1 && depth <= 4);
}
constexpr int kGroupMaxSpan = 256;   // offset spread of one staged window (window <= span + tile)
constexpr int kGroupSlotsPerWave = 8;  // staged windows per wave per batch
constexpr int kAnchorTile = 512;     // reference samples per anchored sub-tile (8 per lane)
constexpr int kAnchorMaxTile = 2048;  // largest anchored window per workgroup
constexpr int kAnchorWaves = 16;     // waves per anchored workgroup
constexpr int kAnchorLdsBytes = 65536;
constexpr int kAnchorLdsTarget = 40960;  // larger windows only while four workgroups fit a CU
constexpr int kAnchorBitsW = 4;                         // bit input: words per lane
constexpr int kAnchorTileBits = 64 * 32 * kAnchorBitsW;  // bit input: samples per workgroup
// words of one staged channel window on bit input: the tile, the largest offset, one more word
// for the funnel shift
inline int64_t anchor_bits_words(int32_t rho_max) { return 64 * kAnchorBitsW + (rho_max >> 5) + 1; }

struct Level {
    int nnodes = 0;
    std::vector<int32_t> chlo, chhi, kidlo, kidhi, ref;
    std::vector<int32_t> nid;       // [nnodes][ndm]: neuron (within the node) serving each DM
    std::vector<int32_t> nneu;      // [nnodes]
    std::vector<int64_t> row_base;  // [nnodes]: first row of the node within the level
    std::vector<int32_t> rep;       // [rows]: one DM served by the row's neuron
    std::vector<int32_t> lo, hi;    // [rows]: range of the node reference delay over its DMs
    std::vector<int32_t> node_of;   // [rows]
    int64_t rows = 0;
    int64_t synapses = 0;
};

struct PlanImpl {
    snd_plan_desc desc{};
    std::vector<double> freq, dm;
    int nchan = 0, ndm = 0;
    int64_t nsamp = 0, n_out = 0, max_delay = 0;
    double fref = 0.0;
    std::vector<int32_t> delay;  // [ndm][nchan]
    std::vector<Level> lev;
    std::vector<Stage> stages;
    std::vector<Stage> direct;   // at most one: the whole tree from the input, for plain executions
    std::vector<Stage> alone;    // at most one: the final stage for launches of this plan alone, where
                                 // stages.back() is for grids shared by several beams (kPackMinBlocks)
    std::vector<uint8_t> table;  // host image of the device tables
    int64_t workspace_bytes = 0;
    // graded plans of an input-anchored leaf stage and a packed final stage: workspace offset of
    // the leaf stage's per-workgroup bound words and their count (bound word after them); -1: none
    int64_t bound_off = -1;
    int64_t bound_n = 0;
    int out_dtype = SND_DT_F32;
    void *d_table = nullptr;
    snd_plan_info info{};
};

int dtype_size(int dt);
int64_t dtype_bytes(int dt, int64_t elems);  // storage bytes of elems elements (bit rows: rounded up)

// One execution of a plan: n_run <= n_out output samples from a source window of src_len
// samples per channel; the input rows are rings of ring_len samples whose window starts at
// column ring_start when ring_len > 0 (streaming), plain rows otherwise.
struct Run {
    int64_t n_run;
    int64_t src_len;
    int64_t ring_len;
    int64_t ring_start;
};
inline Run full_run(const PlanImpl &p) { return Run{p.n_out, p.nsamp, 0, 0}; }
// Enqueue stage si of one run (defined with the C ABI), the final one from PlanImpl::alone where there is
// one; kDirectStage: the stage in PlanImpl::direct.
constexpr size_t kDirectStage = ~size_t(0), kAloneStage = kDirectStage - 1;
snd_status run_stage(PlanImpl &P, size_t si, const Run &run, const void *d_in, int64_t in_pitch, void *d_out,
                     int64_t out_pitch, void *d_workspace, void *stream);
// Enqueue a plain execution of the whole block (snd_execute past its argument checks): the stage in
// PlanImpl::direct where there is one and the buffers allow it, else the stages in order.
snd_status run_block(PlanImpl &P, const void *d_in, int64_t in_pitch, void *d_out, int64_t out_pitch,
                     void *d_workspace, void *stream);
// Whether the byte ranges [a, a + na) and [b, b + nb) share memory.
inline bool ranges_overlap(const void *a, int64_t na, const void *b, int64_t nb)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}
// Depth classes of the kernels whose open-level stack is sized at compile time.
inline int depth_bucket(int d) { return d <= 1 ? 1 : d <= 2 ? 2 : d <= 4 ? 4 : d <= 8 ? 8 : 16; }
void set_error(const std::string &msg);
// Builds the whole plan; returns SND_OK or an error with a message in `err`.
snd_status build_plan(const snd_plan_desc &d, PlanImpl &p, std::string &err);

// ---- device launchers (kernels.hip) ----

// Several stage launches of one kernel class in a single grid: record r (an argument struct of
// the kernel in device memory) owns the workgroups [prefix[r], prefix[r + 1]).  n == 0 means a
// plain launch whose arguments are passed by value.
struct Multi {
    const void *recs;
    const int32_t *prefix;
    int32_t n;
};
struct StageArgs {
    const void *src;
    int64_t src_pitch;
    void *dst;
    int64_t dst_pitch;
    const uint32_t *row_ptr;
    const int32_t *row_len;
    const Entry *ent;
    int32_t rows;
    int32_t n_ttiles;
    int32_t n_rgroups;
    int32_t depth;
    int32_t src_is_input;
    int32_t k_leaf, k_int, cap;
    float scale;
    int32_t len_cut;  // samples dropped from the end of every row (runs with fewer outputs than n_out)
};

// Workgroups of one generic stage launch; fills a.n_ttiles and a.n_rgroups.
int64_t stage_blocks(StageArgs &a, int64_t max_len);
// Enqueue one stage; returns 0 or a HIP error code.  With m.n > 0 the arguments come from the
// records of m and the grid has `nblocks` workgroups (a is only used to choose the instance).
int launch_stage(int mode, int src_dtype, int dst_dtype, const StageArgs &a, int64_t max_len, void *stream,
                 const Multi &m = Multi{nullptr, nullptr, 0}, int64_t nblocks = 0);

struct GroupArgs {
    const void *src;
    int64_t src_pitch;
    void *dst;
    int64_t dst_pitch;
    const int32_t *grp_rows;
    const int32_t *batch_ptr;
    const int32_t *batches;  // 4 ints per batch
    const int32_t *instrs;   // 4 ints per staged window (copy descriptor)
    const uint32_t *ldsb;
    const int32_t *node_closes;  // specialised kernel only
    const uint32_t *lin_smem;    // linear kernel only
    const uint32_t *lin;
    int32_t lin_kernel;          // 1: linear kernel, 2: packed kernel
    int32_t lin_blocks;          // linear kernel on f32 rows: blocks of a tile, or kLinDwords
    int32_t xcd_chunk;           // DM groups of one time tile dealt to each XCD in turn
    int32_t ngroups;
    int32_t n_entries;
    int32_t buf_elems;
    int32_t f1;  // > 0: specialised kernel with level-1 nodes of f1 inputs
    int32_t n_out;
    int32_t depth;
    int32_t src_is_input;
    int32_t k_leaf, k_int, cap;
    float scale;
    int32_t wide_level, wide_inputs, wide_sub;  // packed graded kernel (see Stage); 0: no wide path
    // packed graded kernel: the largest value of its input plane, written by the stage that
    // produced it (k_bound_reduce); nullptr: no bound known, the kernel takes its general path
    const uint32_t *bound;
};
int launch_group(int mode, int src_dtype, int dst_dtype, const GroupArgs &a, int64_t n_out, int lds_bytes, void *stream,
                 const Multi &m = Multi{nullptr, nullptr, 0}, int64_t nblocks = 0);

struct AnchorArgs {
    const void *src;
    int64_t src_pitch;
    int64_t src_len;     // valid samples per source row, counted from the window start
    int64_t ring_len;    // > 0: source rows are rings of this many samples
    int64_t ring_start;  // ring column of the window start (0 when not a ring)
    void *dst;
    int64_t dst_pitch;
    const uint32_t *row_ptr;
    const int32_t *row_len;
    const Entry *ent;
    const int32_t *nodes;
    const int32_t *tiles;    // 2 ints per workgroup
    const int32_t *row_lo;
    const int32_t *leaf;     // one-level stages, not on bit rows (see Stage)
    int32_t depth;
    int32_t k_leaf, k_int, cap;
    float scale;
    int32_t n_run;    // output samples of this run (<= n_out)
    int32_t len_cut;  // n_out - n_run: samples dropped from the end of every row
    int32_t tile;     // reference samples per workgroup window (a multiple of kAnchorTile)
    int32_t spread;   // largest delay difference inside a row (see Stage)
    int32_t node_rows;  // rows of a node, on average
    // graded u8 output: one word per workgroup receives the largest value it computed, and
    // the word after the last the largest of them all (k_bound_reduce); nullptr: not tracked
    uint32_t *bound_slots;
};
int launch_anchored(int mode, int src_dtype, int dst_dtype, const AnchorArgs &a, int64_t ntiles, int lds_bytes,
                    void *stream, const Multi &m = Multi{nullptr, nullptr, 0});
// max of the n per-workgroup words at slots into slots[n] (one workgroup)
int launch_bound_reduce(uint32_t *slots, int64_t n, void *stream);
// the same for every record of a batched leaf grid that tracks its words (one workgroup each)
int launch_bound_reduce_records(const Multi &m, void *stream);
int launch_encode(const float *z, int64_t z_pitch, int time_major, int nchan, int64_t nsamp, const float *thr,
                  int nthr, uint8_t *out, int64_t out_pitch, void *stream);
int launch_encode_bits(const float *z, int64_t z_pitch, int time_major, int nchan, int64_t nsamp, float thr,
                       uint32_t *out, int64_t out_words, void *stream);
int launch_chanstats(const float *p, int64_t p_pitch, int nchan, int64_t n, double clip, double *stats, void *stream);
int launch_zero_dm(float *z, int64_t zp, int nchan, int64_t n, double gamma, int32_t *count, void *stream);
int launch_flag_channels(float *z, int64_t zp, int nchan, int64_t n, int64_t w, double k, double *sigma,
                         uint8_t *flags, int64_t fp, void *stream);
int launch_normalize(const float *p, int64_t p_pitch, int nchan, int64_t n, const double *stats, float *z,
                     int64_t z_pitch, void *stream);
int launch_cast(const float *src, int64_t src_pitch, int64_t rows, int64_t cols, void *dst, int64_t dst_pitch,
                int dst_dtype, void *stream);
// Bit rows: copy L bits of each of nchan chunk rows (from bit 0) into a ring of R bits per row
// (R a multiple of 32) at ring bit position pos, wrapping at R; the ring's other bits keep.
int launch_ring_put_bits(const uint32_t *chunk, int64_t chunk_words, uint32_t *ring, int64_t ring_words, int64_t R,
                         int64_t pos, int64_t L, int nchan, void *stream);

// Compile-time shape of the kernel instance that runs stage S: the depth class, or, for the
// specialised row-group kernel, 1000 * (inputs per level-1 node) + depth; -1 for the linear
// kernel, -2 with short tiles; minus the specialised shape for the packed kernel (irregular nodes: its depth and the
// levels above its super nodes).
inline int stage_shape(const Stage &S)
{
    if (S.kernel == kKernelGroupLds && S.group_lin) return S.lin_blocks ? -S.lin_blocks : -1;
    if (S.kernel == kKernelGroupLds && S.group_pack)
        return -(S.group_f1 ? 1000 * S.group_f1 + S.depth : 16000 + 10 * (S.depth - S.wide_level) + S.depth);
    if (S.kernel == kKernelGroupLds && S.group_f1 > 0) return 1000 * S.group_f1 + S.depth;
    return depth_bucket(S.depth);
}

// One stage launch with its arguments filled in, ready to run alone or as one record of a
// batched launch.  Launches may share a grid when kind, mode, dtypes and shape agree.
struct Prepared {
    int kind, mode, src_dt, dst_dt;
    int shape;   // compile-time shape of the instance: depth class, or 1000 * f1 + depth
    int lds;     // dynamic LDS bytes
    int64_t nblocks;
    int64_t n_run;    // LDS row groups: output samples of the run
    int64_t max_len;  // generic: longest row of the run
    bool bad_pitch;   // LDS row groups: source pitch the kernel cannot address
    StageArgs st;
    GroupArgs gr;
    AnchorArgs an;
};
// bound: track the leaf plane's largest value for the packed graded final stage (a batched leaf
// grid is followed by launch_bound_reduce_records, a single leaf launch by launch_bound_reduce)
Prepared prepare_stage(const PlanImpl &P, size_t si, const Run &run, const void *d_in, int64_t in_pitch, void *d_out,
                       int64_t out_pitch, void *d_workspace, bool bound = false);
snd_status launch_prepared(const Prepared &pr, void *stream, const Multi &m, int64_t nblocks);

// One beam of a batched execution: its plan, run and buffers.
struct Job {
    const PlanImpl *P;
    Run run;
    const void *in;
    int64_t in_pitch;
    void *out;
    int64_t out_pitch;
    void *ws;
};
// Device record bytes a batch of these plans needs, and the number of grids it launches.
int64_t batch_record_bytes(const std::vector<const PlanImpl *> &plans, int *n_launches);
// Every stage of every job, one grid per (stage wave, kernel class); records in d_records.
snd_status run_batch(const std::vector<Job> &jobs, void *d_records, int64_t records_bytes, void *stream,
                     int *n_launches);

}  // namespace snd

struct snd_plan_s {
    snd::PlanImpl impl;
};
