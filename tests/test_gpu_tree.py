"""GPU parity of the SND tree (libsnd through its C ABI) against the CPU oracle.

Integer modes must be bit-exact; float32 within rel-RMS 1e-5 of the FP64 oracle (bit-exact on
small-integer inputs); BF16/FP16 storage within rel-RMS 1e-2 of the FP64 oracle on the
original float32 input.
"""

import sys

import numpy as np
import pytest

import synth
from bitrows import pack_bits

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

STAGE_NONE = 0x80000000
FP32_TOL = 1e-5
REDUCED_TOL = 1e-2


@pytest.fixture(scope="module")
def snd():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_2606_15361_amd as m
    return m


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def to_np(y):
    if y.dtype == torch.uint16:
        y = y.view(torch.int16).to(torch.int32) & 0xFFFF
    elif y.dtype in (torch.bfloat16, torch.float16):
        y = y.float()
    return y.cpu().numpy()


def gpu_run(plan, x, stage_by_stage=False):
    xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    if stage_by_stage:
        out = plan.empty_output(xt.device)
        for s in range(plan.info["n_stages"]):
            plan.execute(xt, out=out, stage=s)
        y = out
    else:
        y = plan.execute(xt)
    torch.cuda.synchronize()
    return to_np(y)


def rel_rms(a, b):
    return float(np.sqrt(np.mean((a - b) ** 2)) / max(np.sqrt(np.mean(b ** 2)), 1e-300))


def _inputs(rng, mode, nchan, nsamp):
    if mode == "binary":
        return synth.random_spikes(rng, nchan, nsamp, 0.3)
    if mode == "graded":
        return synth.random_levels(rng, nchan, nsamp, 4)
    return synth.noise_filterbank(rng, nchan, nsamp)


def _case(nchan, ndm, seed, extra=1037):
    rng = synth.make_rng(seed)
    f = synth.channel_freqs(nchan)
    dms = rng.uniform(0, 40.0, ndm)
    dms[-1] = dms[0]
    dms[0] = 0.0
    return rng, f, dms, extra


SHAPES = [(64, 4, 2), (37, 3, 3), (24, 5, 4), (16, 1, 2), (9, 4, 8), (3, 4, 2), (1, 1, 2)]


@pytest.mark.parametrize("nchan,C_,B", SHAPES)
@pytest.mark.parametrize("mode,kw", [("binary", dict(k_leaf=2, k_int=2)), ("binary", dict(k_leaf=1, k_int=2)),
                                     ("graded", dict(cap=255)), ("graded", dict(cap=7)), ("float", {})])
def test_parity_small(snd, orc, nchan, C_, B, mode, kw):
    rng, f, dms, extra = _case(nchan, 33, nchan * 31 + B)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + extra
    x = _inputs(rng, mode, nchan, nsamp)
    want, _ = orc.snd_dedup(x, f, d, mode=mode, cluster=C_, branching=B, **kw)
    ys = []
    nlev = len(orc.tree_shape(f, C_, B))
    variants = [(0, False, None), (0, True, None), (STAGE_NONE, False, None)]
    if mode == "binary":
        variants.append((0, False, "u8"))  # byte rows next to the default bit rows
    if nlev > 2:
        variants += [((1 << (nlev - 1)) - 1, False, None), ((1 << (nlev - 1)) - 1, True, None)]
    for sl, generic, node in variants:
        _say(f"case nchan={nchan} C={C_} B={B} mode={mode} {kw} stage_levels={sl:#x} generic={generic} node={node}")
        p = snd.Plan(f, dms, 0.138e-3, nsamp, mode=mode, cluster=C_, branching=B, stage_levels=sl,
                     generic_kernels=generic, node_dtype=node, **kw)
        if not generic and sl == 0 and nlev > 1:
            assert p.info["stage_kernel"][0] == "anchored", p.info["stage_kernel"]
            assert p.info["stage_kernel"][1] in ("group_lds", "group_fast", "group_bits", "group_lin"), \
                p.info["stage_kernel"]
        y = gpu_run(p, x, stage_by_stage=(sl == 0))
        assert y.shape == want.shape
        if mode == "float":
            assert rel_rms(y, want) <= FP32_TOL
        else:
            assert np.array_equal(y, want.astype(y.dtype))
        ys.append(y)
    if mode == "binary":
        # bit input (rows of bits straight from the encoder) where the tree takes bit rows
        try:
            pb = snd.Plan(f, dms, 0.138e-3, nsamp, mode=mode, cluster=C_, branching=B, in_dtype="bits", **kw)
        except snd.SndError as e:
            assert e.status == -2 and snd.Plan(f, dms, 0.138e-3, nsamp, mode=mode, cluster=C_, branching=B,
                                              **kw).node_dtype == "u8"
        else:
            _say(f"case nchan={nchan} C={C_} B={B} mode={mode} {kw} bit input")
            if nlev > 1:
                assert pb.info["stage_kernel"] == ["anchored_bits", "group_bits"], pb.info["stage_kernel"]
            y = gpu_run(pb, pack_bits(x), stage_by_stage=True)
            assert np.array_equal(y, want.astype(y.dtype))
            ys.append(y)
    for y in ys[1:]:
        if mode == "float":
            # float mode fixes no FP32 summation order: each schedule's plane is within the float
            # tolerance of the others (every one already is of the FP64 oracle)
            assert rel_rms(y, ys[0]) <= FP32_TOL
        else:
            assert np.array_equal(y, ys[0])  # identical whatever levels are materialised


def test_float_small_integer_input_is_exact(snd, orc):
    rng, f, dms, extra = _case(48, 40, 7)
    d = orc.delays(f, dms, 0.138e-3)
    x = synth.random_levels(rng, 48, int(d.max()) + extra, 3).astype(np.float32)
    want, _ = orc.snd_dedup(x, f, d, mode="float", cluster=4, branching=4)
    p = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="float", branching=4)
    assert np.array_equal(gpu_run(p, x), want.astype(np.float32))
    pn = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="float", branching=4, root_norm=True)
    wn, _ = orc.snd_dedup(x, f, d, mode="float", cluster=4, branching=4, root_norm=True)
    assert rel_rms(gpu_run(pn, x), wn) <= FP32_TOL


@pytest.mark.parametrize("node,B", [("f32", 4), ("bf16", 4), ("f16", 4), ("bf16", 8), ("f16", 3)])
def test_float_storage_small_integers_exact(snd, orc, node, B):
    """Small-integer float input (levels -3..4): leaf sums (|v| <= 16) are exact in bf16 and f16
    and the roots exact in FP32, so every storage type must reproduce the FP64 oracle bit for bit.  300 DMs
    fill five 64-row groups of the one-sum final stage (the last one partly), and 2600 output
    samples make two full 1024-sample tiles and a ragged one; random DMs give inputs of both
    dword phases on 16-bit rows."""
    rng, f, dms, _ = _case(96, 300, 11 + B)
    d = orc.delays(f, dms, 0.138e-3)
    x = (synth.random_levels(rng, 96, int(d.max()) + 2600, 7).astype(np.float32) - 3.0)
    want, _ = orc.snd_dedup(x, f, d, mode="float", cluster=4, branching=B)
    p = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="float", branching=B, node_dtype=node)
    assert p.info["stage_kernel"] == ["anchored", "group_lin"], p.info["stage_kernel"]
    _say(f"small integers node={node} B={B} n_out={p.n_out}")
    assert p.n_out == x.shape[1] - int(d.max())
    y = gpu_run(p, x)
    assert np.array_equal(y, want.astype(np.float32))
    # the same leaf plane through the generic kernels
    pg = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="float", branching=B, node_dtype=node, generic_kernels=True)
    assert np.array_equal(gpu_run(pg, x), y)


@pytest.mark.parametrize("node", ["f32", "bf16", "f16"])
def test_float_rows_sum_error_bound(snd, orc, node):
    """Element-wise bound on the final stage's FP32 arithmetic.  One channel of every cluster of
    four carries values +-m 2^e (m < 256, e in -10..7), the others zero, so every leaf is exact in
    bf16 and f16 storage while the 128-input roots span 2^29 in magnitude and round.  Whatever the
    association, n roundings of at most one unit in the last place (round to nearest: half of
    one; the bf16 kernel's paired dots: one) keep |y - exact| <= n 2^-23 sum|x| with n = 128
    inputs per root; a dropped or foreign sample, or a non-sample half in a dot, breaks it.  300
    DMs and 2600 output samples: five 64-row groups, two full 1024-sample tiles and a ragged one."""
    rng, f, dms, _ = _case(512, 300, 71)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + 2600
    m = rng.integers(1, 256, (512, nsamp)).astype(np.float64)
    e = rng.integers(-10, 8, (512, nsamp)).astype(np.float64)
    x = (np.where(rng.random((512, nsamp)) < 0.5, -1.0, 1.0) * m * np.exp2(e)).astype(np.float32)
    x[np.arange(512) % 4 != 0] = 0.0
    want, _ = orc.snd_dedup(x, f, d, mode="float", cluster=4, branching=4)
    absum, _ = orc.snd_dedup(np.abs(x), f, d, mode="float", cluster=4, branching=4)
    p = snd.Plan(f, dms, 0.138e-3, nsamp, mode="float", branching=4, node_dtype=node)
    assert p.info["stage_kernel"] == ["anchored", "group_lin"], p.info["stage_kernel"]
    _say(f"float rows error bound node={node} n_out={p.n_out}")
    y = gpu_run(p, x).astype(np.float64)
    err = np.abs(y - want)
    bound = 128 * 2.0 ** -23 * absum
    assert np.all(np.isfinite(y))
    assert np.all(err <= bound), (float(np.max(err / np.maximum(bound, 1e-300))), np.argwhere(err > bound)[:5])
    assert np.any(err > 0)  # the roots do round


@pytest.mark.parametrize("nchan,B,cap,levels", [(1024, 4, 255, 4), (1024, 4, 3, 4), (256, 8, 255, 4),
                                                (512, 8, 7, 6), (64, 4, 2, 2), (4096, 4, 15, 4),
                                                (4096, 8, 255, 4)])
def test_graded_packed_levels_exact(snd, orc, nchan, B, cap, levels):
    """Graded u8 rows with level-1 nodes of 4 or 8 inputs run the packed kernel (two 16-bit
    counts per dword); small caps clip at every level.  Bit-exact against the oracle and the
    generic kernels, over 300 DMs (32-row groups over 1024-sample tiles at four inputs per node
    and depth <= 4, else 64-row groups over 512 samples; the last group partial in both) and
    2600 output samples (a ragged last tile in both)."""
    rng, f, dms, _ = _case(nchan, 300, 17 + B + cap)
    d = orc.delays(f, dms, 0.138e-3)
    x = synth.random_levels(rng, nchan, int(d.max()) + 2600, levels)
    want, _ = orc.snd_dedup(x, f, d, mode="graded", cluster=4, branching=B, cap=cap)
    p = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="graded", branching=B, cap=cap)
    assert p.info["stage_kernel"] == ["anchored", "group_pack"], p.info["stage_kernel"]
    _say(f"packed graded nchan={nchan} B={B} cap={cap} n_out={p.n_out}")
    y = gpu_run(p, x)
    assert np.array_equal(y, want.astype(y.dtype))
    pg = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="graded", branching=B, cap=cap, generic_kernels=True)
    assert np.array_equal(gpu_run(pg, x), y)


@pytest.mark.parametrize("B,top,cap", [(4, 63, 255), (4, 64, 255), (4, 63, 100), (8, 31, 255), (8, 32, 60)])
def test_graded_packed_byte_sums_at_the_bound(snd, orc, B, top, cap):
    """The packed kernel adds a level-1 node's inputs as four bytes per dword when the leaf
    stage's largest value m has F1 m < 256 (F1 = B here), and as 16-bit counts otherwise.  The
    first F1 clusters carry leaves of exactly `top` over most of the block, so their level-1 node
    reaches F1 top: 252 or 248 on the byte path, 256 on the other.  The workspace starts filled
    with 0xFF, so row padding past the valid length holds the largest bytes.  Bit-exact against
    the oracle and the generic kernels, with a ragged last tile."""
    rng, f, dms, _ = _case(256, 300, 29 + B + top)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + 2600
    hi = (top - 3) // 4 if B == 4 else (top - 3) // 4 // 2 * 2
    x = synth.random_levels(rng, 256, nsamp, min(hi, 15))
    q, r = divmod(top, 4)  # channel values of one cluster summing to top
    per_cluster = [q + (1 if k < r else 0) for k in range(4)]
    for c in range(4 * B):
        x[c, 50:nsamp - 50] = per_cluster[c % 4]
    want, _ = orc.snd_dedup(x, f, d, mode="graded", cluster=4, branching=B, cap=cap)
    p = snd.Plan(f, dms, 0.138e-3, nsamp, mode="graded", branching=B, cap=cap)
    assert p.info["stage_kernel"] == ["anchored", "group_pack"], p.info["stage_kernel"]
    _say(f"packed byte sums B={B} top={top} cap={cap} n_out={p.n_out}")
    xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ws = p.workspace(xt.device)
    ws.fill_(255)
    out = p.empty_output(xt.device)
    p.execute(xt, out=out, workspace=ws)
    torch.cuda.synchronize()
    y = to_np(out)
    assert np.array_equal(y, want.astype(y.dtype))
    pg = snd.Plan(f, dms, 0.138e-3, nsamp, mode="graded", branching=B, cap=cap, generic_kernels=True)
    assert np.array_equal(gpu_run(pg, x), y)


@pytest.mark.parametrize("nchan,B,top,cap", [
    (256, 4, 15, 255), (256, 4, 16, 255),              # regular nodes: 16 inputs of at most 15, or 16
    (64, 4, 15, 255), (1024, 4, 9, 255),               # no level, two levels above the super nodes
    (256, 4, 15, 60), (256, 4, 15, 59),                # the sums one level below reach the cap, or pass it
    (250, 4, 15, 255), (250, 4, 16, 255), (999, 4, 15, 255), (999, 4, 40, 200),  # ragged levels, both paths
    (97, 3, 28, 255), (97, 3, 29, 255),                # super nodes of nine inputs
    (203, 5, 30, 255), (500, 8, 31, 90), (500, 8, 32, 255), (255, 16, 15, 255), (255, 16, 17, 255),
    (5, 4, 60, 255), (3, 4, 60, 40), (17, 2, 40, 255),  # trees of one to four levels
])
def test_graded_packed_wide_sums_at_the_bound(snd, orc, nchan, B, top, cap):
    """The packed kernel adds whole super nodes (up to 16 inputs) as bytes when no sum inside one can
    pass a byte and no clip inside it can act, for regular and ragged trees, and forms every level on
    16-bit counts otherwise.  Most of the block carries leaves of exactly `top` in the first sixteen
    clusters, whose super node reaches the largest sum; the DM grid shifts inputs through every byte
    phase; rows end inside a tile and inside a lane's samples; the workspace starts filled with 0xFF.
    Bit-exact against the oracle and the generic kernels."""
    rng, f, dms, _ = _case(nchan, 150, 31 + nchan + B + top)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + 2 * 1008 + 253
    x = synth.random_levels(rng, nchan, nsamp, max(1, min(top // 4, 4)))
    q, r = divmod(top, 4)
    for c in range(min(nchan // 4 * 4, 64)):  # channel values of one cluster summing to top
        x[c, 50:nsamp - 50] = q + (1 if c % 4 < r else 0)
    want, _ = orc.snd_dedup(x, f, d, mode="graded", cluster=4, branching=B, cap=cap)
    p = snd.Plan(f, dms, 0.138e-3, nsamp, mode="graded", branching=B, cap=cap)
    _say(f"packed wide sums nchan={nchan} B={B} top={top} cap={cap} n_out={p.n_out} {p.info['stage_kernel']}")
    xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ws = p.workspace(xt.device)
    ws.fill_(255)
    out = p.empty_output(xt.device)
    p.execute(xt, out=out, workspace=ws)
    torch.cuda.synchronize()
    y = to_np(out)
    assert np.array_equal(y, want.astype(y.dtype))
    pg = snd.Plan(f, dms, 0.138e-3, nsamp, mode="graded", branching=B, cap=cap, generic_kernels=True)
    assert np.array_equal(gpu_run(pg, x), y)


@pytest.mark.parametrize("nchan,n_out,cap,top", [(64, 1, 255, 255), (64, 511, 200, 255), (64, 512, 7, 255),
                                                 (64, 513, 255, 40), (66, 2051, 255, 63), (64, 2045, 255, 255),
                                                 (7, 1027, 255, 255), (256, 4100, 255, 255), (600, 700, 90, 200)])
def test_graded_leaf_rows_as_dwords(snd, orc, nchan, n_out, cap, top):
    """Leaf rows of four u8 inputs are summed as dwords inside a row and sample by sample at its ends:
    every byte phase of the inputs, levels up to 255 (sums past the cap and past a byte), rows shorter
    than, equal to and just past a 512-sample sub-tile, clusters of fewer channels at a ragged end, and
    one leaf node of 600 channels.  Bit-exact against the oracle and the generic kernels."""
    rng, f, dms, _ = _case(nchan, 90, 41 + nchan + n_out + cap)
    d = orc.delays(f, dms, 0.138e-3)
    cluster = 600 if nchan == 600 else 4
    x = rng.integers(0, top + 1, size=(nchan, int(d.max()) + n_out), dtype=np.uint8)
    want, _ = orc.snd_dedup(x, f, d, mode="graded", cluster=cluster, branching=4, cap=cap)
    p = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="graded", cluster=cluster, branching=4, cap=cap)
    _say(f"leaf dwords nchan={nchan} n_out={n_out} cap={cap} {p.info['stage_kernel']}")
    y = gpu_run(p, x)
    assert np.array_equal(y, want.astype(y.dtype))
    pg = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode="graded", cluster=cluster, branching=4, cap=cap,
                  generic_kernels=True)
    assert np.array_equal(gpu_run(pg, x), y)


@pytest.mark.parametrize("mode", ["float", "graded"])
@pytest.mark.parametrize("nchan,B,ndm,n_out", [(64, 4, 200, 512), (64, 4, 65, 513), (64, 8, 63, 511), (64, 2, 130, 1),
                                               (16, 4, 300, 1500), (128, 2, 64, 3000), (32, 8, 1, 100)])
def test_sparse_dms_from_the_input(snd, orc, mode, nchan, B, ndm, n_out):
    """DMs in equal ratios hardly share leaf rows, and a plain execution then takes the whole tree from
    the input in one stage where its rows start on 16 bytes; from any other start the leaf plane is
    written as before.  Both, and the generic kernels, give the same bits; the oracle's sums within the
    FP32 tolerance (exactly, graded).  Groups and tiles that are partial, whole and just past whole."""
    rng, f, _, _ = _case(nchan, 2, 51 + ndm)
    dms = np.geomspace(2.0, 400.0, ndm)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + n_out
    x = rng.standard_normal((nchan, nsamp)).astype(np.float32) if mode == "float" else \
        rng.integers(0, 90, (nchan, nsamp), dtype=np.uint8)
    kw = dict(mode=mode, branching=B, cap=200)
    want, _ = orc.snd_dedup(x, f, d, cluster=4, **kw)
    p = snd.Plan(f, dms, 0.138e-3, nsamp, **kw)
    _say(f"sparse DMs mode={mode} nchan={nchan} B={B} ndm={ndm} n_out={n_out} {p.info['stage_kernel']}")
    ys = []
    for first, pitch in ((0, (nsamp + 31) // 16 * 16), (1, (nsamp + 31) // 16 * 16), (0, nsamp | 1)):
        block = torch.zeros(nchan * pitch + 16, dtype=torch.from_numpy(x).dtype, device="cuda")
        view = block[first:first + nchan * pitch].view(nchan, pitch)[:, :nsamp]
        view.copy_(torch.from_numpy(x))
        ys.append(to_np(p.execute(view)))
    assert np.array_equal(ys[0], ys[1]) and np.array_equal(ys[0], ys[2])
    pg = snd.Plan(f, dms, 0.138e-3, nsamp, generic_kernels=True, **kw)
    if mode == "graded":
        assert np.array_equal(ys[0], want.astype(ys[0].dtype)) and np.array_equal(gpu_run(pg, x), ys[0])
    else:
        assert rel_rms(ys[0], want) <= FP32_TOL and rel_rms(gpu_run(pg, x), ys[0]) <= FP32_TOL


@pytest.mark.parametrize("mode,node", [("float", "f32"), ("float", "bf16"), ("graded", "u8"), ("binary", "bits"),
                                       ("binary", "u8")])
def test_tune_variants_identical(snd, orc, mode, node):
    """Every launch shape of snd_plan_desc.tune (leaf window, XCD dealing, LDS batch budget)
    computes the same plane bit for bit, equal to the oracle's (float: within FP32 tolerance; f32
    rows bit for bit while the final stage keeps its kernel)."""
    rng, f, dms, _ = _case(256, 300, 23)
    d = orc.delays(f, dms, 0.138e-3)
    x = _inputs(rng, mode, 256, int(d.max()) + 3000)
    kw = dict(k_leaf=2, k_int=1) if mode == "binary" else {}
    want, _ = orc.snd_dedup(x, f, d, mode=mode, cluster=4, branching=4, **kw)
    tw = snd.tune_word
    base = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode=mode, branching=4, node_dtype=node, **kw)
    y0 = gpu_run(base, x)
    if mode == "float":
        assert rel_rms(y0, want) <= (FP32_TOL if node == "f32" else REDUCED_TOL)
    else:
        assert np.array_equal(y0, want.astype(y0.dtype))
    for t in (tw(xcd_groups=1), tw(xcd_groups=2), tw(xcd_groups=16), tw(lds_quarters_off=1), tw(lds_quarters_off=3),
              tw(leaf_window=512), tw(leaf_window=1024), tw(leaf_window=2048, xcd_groups=4, lds_quarters_off=2)):
        _say(f"tune mode={mode} node={node} tune={t:#x}")
        p = snd.Plan(f, dms, 0.138e-3, x.shape[1], mode=mode, branching=4, node_dtype=node, tune=t, **kw)
        y = gpu_run(p, x)
        if mode == "float" and (node != "f32" or p.info["stage_kernel"] != base.info["stage_kernel"]):
            # the one-sum kernel on 16-bit rows adds each batch's inputs grouped by dword phase,
            # so other batch boundaries associate differently; and a budget too small for its
            # batches moves the stage to a kernel that sums in the tree's association: the same
            # plane within FP32 rounding
            assert rel_rms(y, y0) <= FP32_TOL, snd.tune_fields(t)
        else:
            assert np.array_equal(y, y0), snd.tune_fields(t)


def test_encoder_parity(snd, orc):
    spec = synth.workload(1)
    z = spec.filterbank()
    zt = torch.from_numpy(z).cuda()
    for thr in ([2.0], [1.0, 2.0, 3.0, 4.0], [0.75]):
        _say(f"encode thresholds={thr}")
        a = to_np(snd.encode(zt, thr))
        b = to_np(snd.encode(zt.t().contiguous(), thr, time_major=True))
        want = orc.encode(z, thr)
        assert np.array_equal(a, want) and np.array_equal(b, want)


def test_encoder_bits_parity(snd, orc):
    spec = synth.workload(1)
    z = spec.filterbank()
    zt = torch.from_numpy(z).cuda()
    for thr, n in ((2.0, z.shape[1]), (0.75, z.shape[1]), (1.0, 1000), (1.5, 1)):
        _say(f"encode_bits threshold={thr} nsamp={n}")
        want = pack_bits(orc.encode(z[:, :n], [thr]))
        a = snd.encode_bits(zt[:, :n], thr).cpu().numpy()
        b = snd.encode_bits(zt[:, :n].t().contiguous(), thr, time_major=True).cpu().numpy()
        assert np.array_equal(a, want) and np.array_equal(b, want)


def test_encoders_at_exact_thresholds(snd, orc):
    # samples exactly at a threshold do not fire (x = 1[z > theta]); the float just above does
    rng = synth.make_rng(77)
    thr = [0.75, 1.5, 2.0, 3.0]
    t32 = np.array(thr, dtype=np.float32)
    vals = np.concatenate([t32, np.nextafter(t32, np.float32(np.inf)), np.nextafter(t32, np.float32(-np.inf))])
    z = rng.choice(vals, size=(5, 4100)).astype(np.float32)
    zt = torch.from_numpy(z).cuda()
    for th in ([2.0], [1.0, 2.0, 3.0, 4.0], [0.75, 1.5]):
        _say(f"encode at exact thresholds {th}")
        want = orc.encode(z, th)
        assert np.array_equal(to_np(snd.encode(zt, th)), want)
        assert np.array_equal(to_np(snd.encode(zt.t().contiguous(), th, time_major=True)), want)
    for th in thr:
        want = pack_bits(orc.encode(z, [th]))
        assert np.array_equal(snd.encode_bits(zt, th).cpu().numpy(), want)
        assert np.array_equal(snd.encode_bits(zt.t().contiguous(), th, time_major=True).cpu().numpy(), want)


@pytest.mark.parametrize("kl,ki", [(2, 2), (2, 1)])
def test_config1_binary_exact(snd, orc, kl, ki):
    spec = synth.workload(1)
    z = spec.filterbank()
    x = to_np(snd.encode(torch.from_numpy(z).cuda(), list(spec.enc_thresholds)))
    d = orc.delays(spec.freqs, spec.dms, spec.tsamp_s)
    want, counts = orc.snd_dedup(x, spec.freqs, d, mode="binary", cluster=4, branching=2, k_leaf=kl, k_int=ki)
    p = snd.Plan(spec.freqs, spec.dms, spec.tsamp_s, spec.nsamp, mode="binary", branching=2, k_leaf=kl, k_int=ki)
    assert p.info["n_neurons"] == sum(c[0] for c in counts) == 1984
    assert p.node_dtype == "bits" and p.info["stage_kernel"] == ["anchored", "group_bits"]
    assert np.array_equal(gpu_run(p, x), want.astype(np.uint8))
    pb = snd.Plan(spec.freqs, spec.dms, spec.tsamp_s, spec.nsamp, mode="binary", branching=2, k_leaf=kl, k_int=ki,
                  node_dtype="u8")
    assert pb.info["stage_kernel"] == ["anchored", "group_fast"]
    assert np.array_equal(gpu_run(pb, x), want.astype(np.uint8))
    if len(spec.enc_thresholds) == 1:  # bit input from the bit encoder
        xb = snd.encode_bits(torch.from_numpy(z).cuda(), spec.enc_thresholds[0])
        pi = snd.Plan(spec.freqs, spec.dms, spec.tsamp_s, spec.nsamp, mode="binary", branching=2, k_leaf=kl,
                      k_int=ki, in_dtype="bits")
        assert pi.info["stage_kernel"] == ["anchored_bits", "group_bits"]
        y = pi.execute(xb)
        torch.cuda.synchronize()
        assert np.array_equal(to_np(y), want.astype(np.uint8))


@pytest.mark.parametrize("B", [2, 4, 8])
@pytest.mark.parametrize("mode", ["binary", "graded", "float"])
def test_config3_modes_exact(snd, orc, B, mode):
    # the 64-channel geometric 3000-trial grid, n_out shortened to keep the oracle fast
    spec = synth.workload(3, mode=mode, branching=B)
    d = orc.delays(spec.freqs, spec.dms, spec.tsamp_s)
    nsamp = int(d.max()) + 1500
    z = spec.filterbank(nsamp)
    if mode == "float":
        x = z
    else:
        x = orc.encode(z, list(spec.enc_thresholds))
    kw = dict(k_leaf=spec.k_leaf, k_int=spec.k_int) if mode == "binary" else {}
    for cap in ((255, 15) if mode == "graded" else (255,)):
        _say(f"config3 mode={mode} B={B} cap={cap}")
        want, _ = orc.snd_dedup(x, spec.freqs, d, mode=mode, cluster=4, branching=B, cap=cap, **kw)
        p = snd.Plan(spec.freqs, spec.dms, spec.tsamp_s, nsamp, mode=mode, branching=B, cap=cap, **kw)
        y = gpu_run(p, x)
        if mode == "float":
            assert rel_rms(y, want) <= FP32_TOL
        else:
            assert np.array_equal(y, want.astype(y.dtype))


@pytest.mark.parametrize("node,inp", [("bf16", "f32"), ("f16", "f32"), ("bf16", "bf16"), ("f16", "f16")])
def test_reduced_precision_storage(snd, orc, node, inp):
    rng, f, dms, extra = _case(64, 50, 99)
    d = orc.delays(f, dms, 0.138e-3)
    z = synth.noise_filterbank(rng, 64, int(d.max()) + extra)
    want, _ = orc.snd_dedup(z, f, d, mode="float", cluster=4, branching=4)
    p = snd.Plan(f, dms, 0.138e-3, z.shape[1], mode="float", branching=4, in_dtype=inp, node_dtype=node)
    zt = torch.from_numpy(z).cuda()
    xin = zt if inp == "f32" else snd.cast(zt, inp)
    if inp != "f32":
        ref = xin.float().cpu() if inp == "bf16" else xin.float().cpu()
        cpu_cast = zt.cpu().to(torch.bfloat16 if inp == "bf16" else torch.float16).float()
        assert torch.equal(ref, cpu_cast)  # round-to-nearest-even like torch's own cast
    y = p.execute(xin)
    torch.cuda.synchronize()
    err = rel_rms(to_np(y), want)
    _say(f"storage node={node} in={inp} rel_rms={err:.3e}")
    assert err <= REDUCED_TOL


def test_edge_cases(snd, orc):
    f = synth.channel_freqs(40)
    rng = synth.make_rng(5)
    # all-zero DM grid: no delay, n_out = nsamp; duplicate rows identical
    x = synth.random_levels(rng, 40, 300, 4)
    p = snd.Plan(f, [0.0, 0.0, 0.0], 0.138e-3, 300, mode="graded", branching=2, cap=6)
    y = gpu_run(p, x)
    assert y.shape == (3, 300)
    assert np.array_equal(y[0], np.minimum(x.sum(0), 6)) and np.array_equal(y[0], y[2])
    # single DM, single channel
    p1 = snd.Plan([400.0], [100.0], 0.138e-3, 70, mode="float", branching=2, cluster=1)
    x1 = rng.standard_normal((1, 70)).astype(np.float32)
    assert np.array_equal(gpu_run(p1, x1), x1[:, :70])
    # unsorted DMs: rows follow the caller's order
    dms = np.array([30.0, 0.0, 15.0, 30.0])
    d = orc.delays(f, dms, 0.138e-3)
    x2 = synth.random_spikes(rng, 40, int(d.max()) + 600, 0.4)
    p2 = snd.Plan(f, dms, 0.138e-3, x2.shape[1], mode="binary", branching=3, k_leaf=1, k_int=2)
    want, _ = orc.snd_dedup(x2, f, d, mode="binary", cluster=4, branching=3, k_leaf=1, k_int=2)
    y2 = gpu_run(p2, x2)
    assert np.array_equal(y2, want.astype(np.uint8)) and np.array_equal(y2[0], y2[3])
    # a pitched input (extra columns) gives the same answer
    xt = torch.zeros((40, x2.shape[1] + 77), dtype=torch.uint8, device="cuda")
    xt[:, : x2.shape[1]] = torch.from_numpy(x2).cuda()
    y3 = to_np(p2.execute(xt))
    assert np.array_equal(y3, y2)


def test_bad_arguments_raise(snd):
    p = snd.Plan(synth.channel_freqs(8), [0.0, 2.0], 0.138e-3, 200, mode="float", branching=2)
    with pytest.raises(ValueError):
        p.execute(torch.zeros((8, 100), device="cuda"))
    with pytest.raises(TypeError):
        p.execute(torch.zeros((8, 200), dtype=torch.uint8, device="cuda"))


def test_determinism(snd):
    rng, f, dms, extra = _case(128, 64, 3)
    p = snd.Plan(f, dms, 0.138e-3, 4000, mode="float", branching=4)
    z = synth.noise_filterbank(rng, 128, 4000)
    a = gpu_run(p, z)
    b = gpu_run(p, z)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("mode", ["float", "graded", "binary", "binary-bits"])
def test_config2_full_size_sampled(snd, orc, mode):
    # The benchmarked workload (1024 ch, 4096 DM, 2^17 samples, B = 4) at full size, checked
    # on sampled outputs against the oracle's per-point recursion.
    spec = synth.workload(2)
    _say(f"config2 full size mode={mode}: generating input")
    z = spec.filterbank()
    d = orc.delays(spec.freqs, spec.dms, spec.tsamp_s)
    zt = torch.from_numpy(z).cuda()
    bit_input = mode == "binary-bits"
    mode = "binary" if bit_input else mode
    if mode == "float":
        x, xin = z, zt
    else:
        xin = snd.encode(zt, [1.0, 2.0, 3.0, 4.0] if mode == "graded" else [2.0])
        x = to_np(xin)
    if bit_input:
        xin = snd.encode_bits(zt, 2.0)
        assert np.array_equal(xin[:, :64].cpu().numpy(), pack_bits(x[:, :2048]))
    p = snd.Plan(spec.freqs, spec.dms, spec.tsamp_s, spec.nsamp, mode=mode, branching=4,
                 in_dtype="bits" if bit_input else None)
    if mode == "binary":
        assert p.info["stage_kernel"] == ["anchored_bits" if bit_input else "anchored", "group_bits"]
    _say(f"config2 mode={mode}: executing on the GPU")
    y = p.execute(xin)
    torch.cuda.synchronize()
    rng = synth.make_rng(77)
    n = 3000
    ks = rng.integers(0, spec.dms.size, n)
    ts = rng.integers(0, p.n_out, n)
    ks[:4] = [0, spec.dms.size - 1, 0, spec.dms.size - 1]
    ts[:4] = [0, 0, p.n_out - 1, p.n_out - 1]
    got = to_np(y[torch.from_numpy(ks).cuda(), torch.from_numpy(ts).cuda()])
    want = orc.snd_points(x, spec.freqs, d, ks, ts, mode=mode, cluster=4, branching=4)
    if mode == "float":
        assert rel_rms(got, want) <= FP32_TOL
    else:
        assert np.array_equal(got, want.astype(got.dtype))
    # DM 0 row is the plain channel sum
    if mode == "graded":
        row0 = to_np(y[0, :2000])
        assert np.array_equal(row0, np.minimum(x[:, :2000].astype(np.int64).sum(0), 255))


@pytest.mark.parametrize("mode", ["float", "graded"])
def test_sparse_dms_plane_in_place_of_the_block(snd, mode):
    """A plane may take the memory of the block it comes from, over a sparse DM grid too, whose plain
    execution reads the input while it writes the plane (the workspace keeps its 0xFF fill): with shared
    memory the leaf plane is written first, as for any other grid, and the bits are the same."""
    nchan, ndm, n_out = 64, 700, 1500
    f = synth.channel_freqs(nchan)
    dms = np.geomspace(2.0, 400.0, ndm)
    nsamp = n_out + 16 * 400
    p = snd.Plan(f, dms, 0.138e-3, nsamp, mode=mode)
    gen = torch.Generator(device="cuda").manual_seed(5)
    dt = p.out_dtype  # input and output rows are of one type
    pitch = (nsamp + 63) // 64 * 64
    x = torch.randn((nchan, pitch), device="cuda", generator=gen) if mode == "float" else \
        torch.randint(0, 60, (nchan, pitch), dtype=torch.uint8, device="cuda", generator=gen)
    ws = p.workspace(x.device)
    ws.fill_(255)
    want = p.execute(x[:, :nsamp], workspace=ws)
    assert bool((ws == 255).all())
    mem = torch.zeros(ndm * pitch + 2 * nchan * pitch, dtype=dt, device="cuda")
    for at in (0, 300 * pitch + 64, ndm * pitch - 64):  # at the plane's start, inside it, across its end
        block = mem[at:at + nchan * pitch].view(nchan, pitch)
        block.copy_(x)
        out = mem[:ndm * pitch].view(ndm, pitch)[:, :p.n_out]
        p.execute(block[:, :nsamp], out=out, workspace=ws)
        assert torch.equal(out, want)


def test_tuner_times_the_schedule_that_executes(snd):
    """Over a sparse DM grid a plain execution of the default schedule takes the whole tree from the
    input, and so does the tuner's timing of that candidate (its workspace keeps the 0xFF fill); from rows
    that do not start on 16 bytes both write the leaf plane.  A candidate with a tune word is timed on its
    own stages."""
    import ctypes as C
    from paper_2606_15361_amd import _capi as capi
    from paper_2606_15361_amd.plan import make_desc
    nchan, ndm = 64, 700
    f, dms = synth.channel_freqs(nchan), np.geomspace(2.0, 400.0, ndm)
    nsamp = 8000
    d, _f, _d, _, _ = make_desc(f, dms, 0.138e-3, nsamp, mode="float")
    block = torch.randn((nchan, nsamp + 8), device="cuda")
    for tune, first, in_one in ((0, 0, True), (0, 1, False), (16, 0, False)):
        p = snd.Plan(f, dms, 0.138e-3, nsamp, mode="float", tune=tune)
        x = block[:, first:first + nsamp]
        ws = torch.full_like(p.workspace(x.device), 255)
        tables = torch.empty(p.info["table_bytes"], dtype=torch.uint8, device="cuda")
        want = p.execute(x, workspace=ws)
        assert bool((ws == 255).all()) == in_one
        ws.fill_(255)
        out = torch.zeros_like(want)
        cand, best = (capi.TuneCandidate * 1)(), C.c_int32(-1)
        cand[0].tune = tune
        capi.check(capi.lib().snd_autotune(C.byref(d), cand, 1, C.c_void_p(x.data_ptr()), x.stride(0),
                                           C.c_void_p(out.data_ptr()), out.stride(0), C.c_void_p(ws.data_ptr()),
                                           ws.numel(), C.c_void_p(tables.data_ptr()), tables.numel(), 2,
                                           C.byref(best), None))
        torch.cuda.synchronize()
        assert best.value == 0 and cand[0].ms > 0
        assert bool((ws == 255).all()) == in_one
        assert torch.equal(out, want)


@pytest.mark.parametrize("nchan,B,top,cap", [
    (250, 4, 15, 255), (250, 4, 16, 255), (999, 4, 15, 255), (999, 4, 40, 200),  # ragged levels, both paths
    (97, 3, 28, 255), (97, 3, 29, 255),                # super nodes of nine inputs
    (203, 5, 30, 255), (500, 8, 31, 90), (500, 8, 32, 255), (255, 16, 15, 255), (255, 16, 17, 255),
    (5, 4, 60, 255), (3, 4, 60, 40), (17, 2, 40, 255),  # trees of one to four levels
])
def test_graded_ragged_packed_grid(snd, orc, nchan, B, top, cap):
    """Irregular nodes take the packed kernel only in grids that fill half the chip: 470 DMs over nine
    tiles and a partial one, with leaves at the bound of its byte sums and past it, as in the bound test
    above; and in a run of its own of the same tree's small grid, which takes the general kernel, the same
    rows.  Bit-exact against the oracle."""
    rng, f, _, _ = _case(nchan, 2, 61 + nchan + B + top)
    dms = np.linspace(0.0, 40.0, 470)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + 9 * 1008 + 253
    x = synth.random_levels(rng, nchan, nsamp, max(1, min(top // 4, 4)))
    q, r = divmod(top, 4)
    for c in range(min(nchan // 4 * 4, 64)):
        x[c, 50:nsamp - 50] = q + (1 if c % 4 < r else 0)
    want, _ = orc.snd_dedup(x, f, d, mode="graded", cluster=4, branching=B, cap=cap)
    xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    for step in (1, 9):
        p = snd.Plan(f, dms[::step], 0.138e-3, nsamp, mode="graded", branching=B, cap=cap)
        _say(f"ragged packed grid nchan={nchan} B={B} top={top} cap={cap} ndm={p.ndm} n_out={p.n_out}")
        ws = p.workspace(xt.device)
        ws.fill_(255)
        y = to_np(p.execute(xt, workspace=ws))
        assert np.array_equal(y[:, :want.shape[1]], want[::step].astype(y.dtype))


@pytest.mark.parametrize("n_out", [1, 503, 504, 505, 1008, 1009, 2600])
def test_float_rows_of_few_dms_in_short_tiles(snd, orc, n_out):
    """Up to 64 DMs of f32 rows take tiles of 504 samples: the same bits as the 1008-sample tiles that one
    DM more brings, on output rows that start on any element, and the oracle's sums of integer samples
    exactly."""
    nchan = 96
    f = synth.channel_freqs(nchan)
    dms = np.sort(synth.make_rng(n_out).uniform(0.0, 3.0, 65))
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + n_out
    rng = synth.make_rng(n_out + 1)
    for x in (rng.standard_normal((nchan, nsamp)).astype(np.float32), rng.integers(-9, 10, (nchan, nsamp)).astype(np.float32)):
        xt = torch.from_numpy(x).cuda()
        p = snd.Plan(f, dms, 0.138e-3, nsamp)
        assert p.info["stage_kernel"] == ["anchored", "group_lin"] and p.n_out == n_out
        long = to_np(p.execute(xt))
        for drop in (1, 40, 64):  # leading DMs left out: the last one, of the largest delay, stays
            q = snd.Plan(f, dms[drop:], 0.138e-3, nsamp)
            assert q.info["stage_kernel"] == ["anchored", "group_lin"] and q.n_out == n_out
            out = torch.full((q.ndm, n_out + 5), -3.0, device="cuda")
            q.execute(xt, out=out[:, 3:3 + n_out])
            y = out.cpu().numpy()
            assert np.array_equal(y[:, 3:3 + n_out], long[drop:])
            assert np.all(y[:, :3] == -3.0) and np.all(y[:, 3 + n_out:] == -3.0)
    want, _ = orc.snd_dedup(x, f, d, mode="float", cluster=4, branching=4)
    assert np.array_equal(long, want.astype(np.float32))


@pytest.mark.parametrize("mode,nchan,B,ndm,top,n_out,direct", [
    ("float", 64, 4, 600, 400.0, 2200, True), ("float", 64, 4, 600, 800.0, 2049, True),
    ("float", 64, 8, 700, 800.0, 1537, True), ("float", 100, 4, 600, 800.0, 2050, True),
    ("float", 37, 2, 600, 800.0, 2049, True), ("float", 16, 4, 1000, 800.0, 1100, True),
    ("float", 7, 3, 1300, 400.0, 1025, True), ("float", 100, 2, 600, 800.0, 2100, True),
    ("float", 128, 2, 400, 800.0, 3073, True), ("graded", 64, 4, 600, 400.0, 2200, True),
    ("graded", 64, 2, 650, 800.0, 2047, True), ("graded", 64, 8, 1000, 800.0, 1030, True),
    ("graded", 128, 4, 600, 800.0, 6001, True), ("graded", 16, 2, 1100, 400.0, 1024, True),
    ("graded", 128, 2, 600, 800.0, 2000, False), ("graded", 100, 2, 600, 800.0, 2000, False),
    ("float", 128, 3, 400, 800.0, 3000, False), ("float", 64, 2, 600, 800.0, 2000, False),
])
def test_sparse_dms_every_form_of_the_one_stage_schedule(snd, orc, mode, nchan, B, ndm, top, n_out, direct):
    """DM grids in equal ratios, large enough for the one-stage schedule: regular and ragged trees, the
    specialised and the general row-group kernel, whole and partial groups and tiles; and the shapes that
    stay on the leaf plane.  A plain execution that takes the tree from the input leaves the workspace's
    0xFF fill as it is; the same call on rows off 16 bytes and the stages in order give the same bits, the
    generic kernels the same sums, and the oracle's sums at 500 cells (exactly, graded)."""
    f = synth.channel_freqs(nchan)
    dms = np.geomspace(2.0, top, ndm)
    d = orc.delays(f, dms, 0.138e-3)
    nsamp = int(d.max()) + n_out
    rng = synth.make_rng(nchan * 31 + ndm + B)
    x = rng.standard_normal((nchan, nsamp)).astype(np.float32) if mode == "float" else \
        rng.integers(0, 90, (nchan, nsamp), dtype=np.uint8)
    kw = dict(mode=mode, branching=B, cap=200)
    p = snd.Plan(f, dms, 0.138e-3, nsamp, **kw)
    _say(f"one-stage schedule mode={mode} nchan={nchan} B={B} ndm={ndm} n_out={n_out} {p.info['stage_kernel']}")
    pitch = (nsamp + 31) // 16 * 16
    ws = p.workspace(torch.device("cuda"))
    ys = []
    for first, row in ((0, pitch), (1, pitch), (0, pitch + 1)):
        block = torch.zeros(nchan * row + 16, dtype=torch.from_numpy(x).dtype, device="cuda")
        view = block[first:first + nchan * row].view(nchan, row)[:, :nsamp]
        view.copy_(torch.from_numpy(x))
        ws.fill_(255)
        ys.append(to_np(p.execute(view, workspace=ws)))
        assert bool((ws == 255).all()) == (direct and first == 0 and row == pitch)
    ys.append(gpu_run(p, x, stage_by_stage=True))
    for y in ys[1:]:
        assert np.array_equal(ys[0], y)
    ks, ts = rng.integers(0, ndm, 500), rng.integers(0, p.n_out, 500)
    ks[:2], ts[:2] = (0, ndm - 1), (0, p.n_out - 1)
    want = orc.snd_points(x, f, d, ks, ts, cluster=4, **kw)
    if mode == "graded":
        assert np.array_equal(ys[0][ks, ts], want.astype(ys[0].dtype))
    else:
        assert rel_rms(ys[0][ks, ts], want) <= FP32_TOL
    pg = snd.Plan(f, dms, 0.138e-3, nsamp, generic_kernels=True, **kw)
    y = gpu_run(pg, x)
    assert np.array_equal(y, ys[0]) if mode == "graded" else rel_rms(y, ys[0]) <= FP32_TOL


@pytest.mark.parametrize("mode,nchan,dmax,around", [
    ("f32", 64, 1500.0, 18000), ("f32", 30, 700.0, 18000), ("f16", 64, 1500.0, 28000), ("u16", 64, 1500.0, 28000),
    ("u16", 512, 900.0, 28000)])
def test_leaf_rows_by_records_and_by_tables(snd, orc, mode, nchan, dmax, around):
    """Widely spread leaf rows on both sides of the length from which their words are read from the row and
    entry tables, ragged and unaligned: whole numbers, whose sums are exact in each type, so the planes equal
    the generic kernels' bit for bit, and the first samples those of the shorter block."""
    f = synth.channel_freqs(nchan)
    dms = np.linspace(0.0, dmax, 210 if nchan < 512 else 600)
    dmaxd = int(orc.delays(f, dms, 0.138e-3).max())
    rng = synth.make_rng(nchan + around)
    n = dmaxd + around + 1
    hi = 3 if mode == "f16" else 12
    x = rng.integers(0, hi, (nchan, n + 7))
    x = x.astype(np.uint8) if mode == "u16" else x.astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    if mode == "f16":
        xt = xt.half()
    kw = dict(mode="graded", cap=700, node_dtype="u16") if mode == "u16" else \
        dict(mode="float", in_dtype=mode, node_dtype=mode)
    first = None
    for n_out in (around - 1, around, around + 1):
        nsamp = dmaxd + n_out
        p = snd.Plan(f, dms, 0.138e-3, nsamp, **kw)
        pg = snd.Plan(f, dms, 0.138e-3, nsamp, generic_kernels=True, **kw)
        assert p.info["stage_kernel"][0] == "anchored" and p.n_out == n_out
        for off in (0, 3):
            _say(f"leaf rows mode={mode} nchan={nchan} n_out={n_out} off={off}")
            view = xt[:, off:off + nsamp]
            y = to_np(p.execute(view))
            assert np.array_equal(y, to_np(pg.execute(view)))
            if off == 0:
                first = y if first is None else first
                assert np.array_equal(y[:, :around - 1], first)


@pytest.mark.parametrize("top,cap", [(63, 255), (64, 255), (40, 100)])
def test_graded_packed_trees_of_one_level(snd, orc, top, cap):
    """Sixteen channels in fours: one level of four leaves in the packed kernel, as bytes up to four times 63
    and as 16-bit counts past it, under a cap that acts and one that does not, with a ragged last tile."""
    f = synth.channel_freqs(16)
    dms = np.linspace(0.0, 3.0, 300)
    d = orc.delays(f, dms, 0.138e-3)
    n_out = 16 * 1008 + 77
    nsamp = int(d.max()) + n_out
    rng = synth.make_rng(16 + top)
    x = rng.integers(0, top // 4, (16, nsamp), dtype=np.uint8)
    x[:, 500:900] = top // 4
    x[::4, 500:900] += top % 4
    p = snd.Plan(f, dms, 0.138e-3, nsamp, mode="graded", branching=4, cap=cap)
    assert p.info["stage_kernel"] == ["anchored", "group_pack"]
    xt = torch.from_numpy(x).cuda()
    ws = p.workspace(xt.device)
    ws.fill_(255)
    y = to_np(p.execute(xt, workspace=ws))
    want, _ = orc.snd_dedup(x, f, d, mode="graded", cluster=4, branching=4, cap=cap)
    assert np.array_equal(y, want.astype(y.dtype))


def test_float_final_stage_shapes_agree(snd, orc):
    """Grids whose f32 final stage takes eight rows by dwords (8065 to 8192 samples of these DMs) or tiles of
    four blocks, the last of them summed as one, two or four: the same sums in the same order, bit for bit,
    from unaligned output rows too, and the FP64 oracle's within the tolerance."""
    f = synth.channel_freqs(64)
    dms = np.linspace(0.0, 60.0, 2000)
    d = orc.delays(f, dms, 0.138e-3)
    top = 9072
    x = synth.make_rng(8192).standard_normal((64, int(d.max()) + top)).astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    planes = {}
    for n_out in (8064, 8065, 8100, 8192, 8193, 8064 + 253, 8064 + 505, top):
        p = snd.Plan(f, dms, 0.138e-3, int(d.max()) + n_out, mode="float")
        assert p.info["stage_kernel"] == ["anchored", "group_lin"] and p.n_out == n_out
        out = torch.full((p.ndm, n_out + 5), -3.0, device="cuda")
        p.execute(xt, out=out[:, 3:3 + n_out])
        y = out.cpu().numpy()
        assert np.all(y[:, :3] == -3.0) and np.all(y[:, 3 + n_out:] == -3.0)
        planes[n_out] = (y[:, 3:3 + n_out], p.info["stage_batches"][1])
    few = planes[8192][1]
    for n_out, (y, batches) in planes.items():
        assert (batches == few) == (8064 < n_out <= 8192)  # groups of 128 rows, not of 64
        assert np.array_equal(y, planes[top][0][:, :n_out]), n_out
    rng = synth.make_rng(5)
    ks, ts = rng.integers(0, 2000, 500), rng.integers(0, top, 500)
    want = orc.snd_points(x, f, d, ks, ts, mode="float", cluster=4, branching=4)
    assert rel_rms(planes[top][0][ks, ts], want) <= FP32_TOL
