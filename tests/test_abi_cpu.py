"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header declares,
and rejects bad arguments before touching a device (no compute call is made here)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "scan2d.h")
LIB = os.path.join(ROOT, "paper_2412_00678_amd", "libscan2d.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} not built: run `python -m paper_2412_00678_amd.build` first")
    from paper_2412_00678_amd import scan2d
    return scan2d


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(scan2d_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_the_expected_entry_points():
    assert declared_functions() == sorted(
        ["scan2d_fwd", "scan2d_fwd_softplus", "scan2d_fwd_softplus_gated", "scan2d_bwd", "scan2d_bwd_softplus",
         "scan2d_bwd_softplus_gated", "scan2d_workspace_bytes", "scan2d_describe_plan", "scan2d_strerror",
         "scan2d_version", "scan2d_debug_force_variant", "scan2d_bwd_static_scratch", "scan2d_fwd_variants", "scan2d_bwd_variants",
         "scan2d_block_conv_silu", "scan2d_block_xproj", "scan2d_saved_bytes", "scan2d_fwd_saving", "scan2d_bwd_saved",
         "scan2d_block_attn_pool", "scan2d_block_linear", "scan2d_block_norm"])


def test_library_exports_every_declared_symbol(lib):
    raw = ctypes.CDLL(LIB)
    for name in declared_functions():
        assert hasattr(raw, name), name
    assert sorted(lib.EXPORTS) == declared_functions()
    assert lib.version() >= 100


def test_error_strings_are_distinct_and_static(lib):
    seen = {lib.strerror(c) for c in range(0, -10, -1)}
    assert len(seen) == 10
    assert "unknown" in lib.strerror(-99)


def test_descriptor_validation_needs_no_device(lib):
    D = lib.Desc
    call = lambda d: lib.lib.scan2d_fwd(ctypes.byref(d), *([None] * 8), None, 0, None)
    assert call(D(0, 1, 1, 1, 1, 0, 0)) == -2
    assert call(D(1, 1, 1, 1, 65, 0, 0)) == -2
    assert call(D(1, 1, 1, -3, 4, 0, 0)) == -2
    assert call(D(1, 1, 4096, 4096, 16, 0, 0)) == -2          # N*H*W >= 2^27
    assert call(D(1, 1, 8, 8, 4, 7, 0)) == -3
    assert call(D(1, 1, 8, 8, 4, 0, 4)) == -4                    # an unknown flag bit
    assert call(D(1, 1, 8, 8, 4, 0, 3)) != -4                    # SCAN2D_FLAG_IDENTITY_CELLS | SCAN2D_FLAG_COLUMNS_FIRST
    assert call(D(1, 1, 8, 8, 4, 0, 0)) == -1                  # NULL tensors
    assert lib.lib.scan2d_fwd(None, *([None] * 8), None, 0, None) == -1
    bwd = lambda d: lib.lib.scan2d_bwd(ctypes.byref(d), *([None] * 14), None, 0, None)
    assert bwd(D(1, 0, 1, 1, 1, 0, 0)) == -2
    assert bwd(D(1, 1, 8, 8, 4, 1, 0)) == -1


def test_misaligned_pointers_are_rejected_before_any_launch(lib):
    d = lib.Desc(1, 1, 8, 8, 4, 0, 0)
    ok, bad = 4096, 4100                                       # fake addresses: never dereferenced
    args = [ok] * 5 + [None, None, ok]
    for k in (0, 1, 2, 3, 4, 7):                               # exactly one misaligned pointer each time
        a = list(args)
        a[k] = bad
        assert lib.lib.scan2d_fwd(ctypes.byref(d), *a, None, 0, None) == -6
    # the gated forward: x, delta_raw, delta_bias, A, Bm, Cm, Dskip, mask, z, y_scan, y, workspace; y_scan wanted and not
    gated = lambda a: lib.lib.scan2d_fwd_softplus_gated(ctypes.byref(d), *a, 0, None)
    for k in (0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11):
        a = [ok] * 11 + [None]
        a[k] = bad
        assert gated(a) == -6, k
        if k not in (9, 11):
            a[9] = None
            assert gated(a) == -6, k


def test_workspace_query(lib):
    small = lib.Desc(1, 16, 16, 16, 4, 0, 0)
    assert lib.workspace_bytes(small, lib.PASS_FWD) == 0       # one panel: no carry buffer
    wide = lib.Desc(1, 2, 8, 3000, 4, 0, 0)
    assert lib.workspace_bytes(wide, lib.PASS_FWD) == 1 * 2 * 4 * 8 * 4
    assert lib.workspace_bytes(lib.Desc(0, 1, 1, 1, 1, 0, 0), lib.PASS_FWD) == 0
    assert lib.workspace_bytes(small, 9) == 0                 # an unknown pass
    # the gated backward adds one map-sized buffer (dy * SiLU(z), storage type), rounded up to 256 bytes
    for dt, eb in ((0, 4), (1, 2)):
        d = lib.Desc(2, 8, 20, 40, 16, dt, 0)
        assert lib.workspace_bytes(d, lib.PASS_BWD_GATED) == lib.workspace_bytes(d, lib.PASS_BWD_SOFTPLUS) + ((2 * 8 * 20 * 40 * eb + 255) // 256) * 256
        # the shared-producer sweeps (16 states here) apply the softplus themselves: no step buffer
        assert lib.workspace_bytes(d, lib.PASS_BWD_SOFTPLUS) == lib.workspace_bytes(d, lib.PASS_BWD)
        # the plain sweeps keep the step in the workspace (one fp32 map-sized buffer)
        d5 = lib.Desc(2, 8, 20, 40, 5, dt, 0)
        extra = ((2 * 8 * 20 * 40 * 4 + 255) // 256) * 256 + 256      # and room behind it for reads past the last row
        assert lib.workspace_bytes(d5, lib.PASS_BWD_SOFTPLUS) == lib.workspace_bytes(d5, lib.PASS_BWD) + extra
    assert lib.workspace_bytes(lib.Desc(1, 2, 8, 3000, 4, 0, 0), lib.PASS_BWD_GATED) > 0       # wide maps: column panels
    # columns first inside the kernels (a shared-producer tiling takes the shape): the workspace of the plain call;
    # through transposes otherwise (here: 5 states): the transposed copies (x, delta, y; Bm, Cm; mask) behind the
    # workspace of the swapped shape; identity cells: one more copy of the step
    r256 = lambda v: (v + 255) // 256 * 256
    d = lib.Desc(2, 8, 20, 40, 16, 0, lib.FLAG_COLUMNS_FIRST)
    assert lib.workspace_bytes(d, lib.PASS_FWD) == 0
    assert lib.describe_plan(d, lib.PASS_FWD).startswith("columns-first(in-kernel) fwd form=shared")
    assert lib.describe_plan(d, lib.PASS_BWD).startswith("columns-first(in-kernel) bwd form=banded-shared")
    assert lib.workspace_bytes(d, lib.PASS_BWD) == lib.workspace_bytes(lib.Desc(2, 8, 20, 40, 16, 0, 0), lib.PASS_BWD)
    d = lib.Desc(2, 8, 20, 40, 5, 0, lib.FLAG_COLUMNS_FIRST)
    assert lib.describe_plan(d, lib.PASS_FWD).startswith("columns-first(transposed) fwd")
    assert lib.workspace_bytes(d, lib.PASS_FWD) == 3 * r256(2 * 8 * 800 * 4) + 2 * r256(2 * 5 * 800 * 4) + r256(2 * 800)
    # the two timed configurations run columns first inside the kernels, forward and backward
    for shape in ((1, 256, 256, 256, 16, 1), (8, 256, 128, 192, 16, 0)):
        d = lib.Desc(*shape, lib.FLAG_COLUMNS_FIRST)
        assert lib.describe_plan(d, lib.PASS_FWD).startswith("columns-first(in-kernel)")
    assert lib.describe_plan(lib.Desc(8, 256, 128, 192, 16, 0, lib.FLAG_COLUMNS_FIRST), lib.PASS_BWD).startswith("columns-first(in-kernel)")
    assert lib.workspace_bytes(lib.Desc(2, 8, 20, 40, 16, 1, lib.FLAG_IDENTITY_CELLS), lib.PASS_FWD) == r256(2 * 8 * 800 * 2)
    assert lib.workspace_bytes(lib.Desc(1, 2, 3000, 8, 4, 0, lib.FLAG_COLUMNS_FIRST), lib.PASS_BWD) > 0    # 3000 columns after the swap


# ------------------------------------------------------------------ host logic: variant choice and launch plans

def plan(lib, d, which):
    fields = {}
    for tok in lib.describe_plan(d, which).split()[1:]:
        k, v = tok.split("=")
        fields[k] = v if k == "form" else int(v)
    return fields


SWEEP_W = [1, 2, 3, 7, 13, 14, 15, 16, 17, 20, 28, 30, 31, 32, 33, 56, 60, 63, 64, 65, 100, 127, 128, 129, 132, 190, 192,
           193, 200, 250, 255, 256, 257, 300, 500, 512, 513, 777, 1000, 1024, 1025, 3000]
SWEEP_N = [1, 3, 4, 5, 8, 15, 16, 17, 24, 40, 63, 64]


def test_row_segments_keep_their_sums_inside_one_checkpoint_row(lib):
    """Each segment of the backward leaves N + 2 sums in the checkpoints' row of a map's first band, N * W floats at least."""
    most = 0
    for W in range(1, 40):
        for H in (17, 64, 300, 1000):
            for maps in ((1, 1), (1, 8), (1, 64), (3, 20)):
                segments = plan(lib, lib.Desc(*maps, H, W, 16, 0, 0), lib.PASS_BWD).get("segments", 1)
                assert segments == 1 or 18 * segments <= 16 * W, (maps, H, W, segments)
                most = max(most, segments)
    assert most == 15


@pytest.mark.parametrize("variant,shape", [("16,4,4,16,1,2", (1, 16, 8, 64)), ("16,4,4,12,1,8", (1, 16, 32, 64))])
def test_forced_segments_that_do_not_fit_are_ignored(lib, variant, shape):
    """Segments of fewer rows than hold what enters the channels of a job: the call takes the plan without them."""
    Bt, Dc, H, W = shape
    d = lib.Desc(Bt, Dc, H, W, 16, 0, 0)
    with lib.forced_variant(lib.TUNE_BWD, variant.rsplit(",", 1)[0]):
        one = plan(lib, d, lib.PASS_BWD)
    with lib.forced_variant(lib.TUNE_BWD, variant):
        assert plan(lib, d, lib.PASS_BWD) == one
    assert one["GS"] == int(variant.split(",")[3]) and one["segments"] == 1


def test_every_shape_has_a_forward_plan_within_the_hardware_limits(lib):
    for dtype in (0, 1):
        for W in SWEEP_W:
            for N in SWEEP_N:
                for (Bt, Dc, H) in ((1, 1, 1), (2, 7, 9), (4, 256, 64)):
                    d = lib.Desc(Bt, Dc, H, W, N, dtype, 0)
                    f = plan(lib, d, lib.PASS_FWD)
                    where = f"dtype {dtype} W {W} N {N} Bt {Bt} Dc {Dc} H {H}: {f}"
                    assert f["lds"] <= 160 * 1024, where
                    assert f["waves"] in (4, 8, 16), where
                    if f["form"] == "tile16":                 # few tiny maps: one workgroup per map
                        assert W <= 16 and H <= 16 and N <= 16 and Bt * Dc <= 1024, where
                        assert f["wgs"] == Bt * Dc and f["workspace"] == 0, where
                    elif f["form"] == "small":
                        assert W <= 16 * f["K"] and 4 * f["NW"] >= N, where
                        assert f["wgs"] == -(-Bt * Dc // 4), where
                    else:
                        assert f["NG"] * f["NW"] >= N and f["NG"] <= f["waves"] * 64 // f["LG"], where
                        assert f["panels"] * f["LG"] * f["K"] >= W, where
                        assert f["wgs"] * f["MPW"] >= Bt * Dc, where
                        assert (f["workspace"] > 0) == (f["panels"] > 1), where
                        assert f["fast"] == (f["panels"] == 1), where      # unguarded loads whenever one panel covers the row
                        if f["exact"]:
                            assert N % f["NW"] == 0, where
                    assert f["workspace"] == lib.workspace_bytes(d, lib.PASS_FWD), where


def test_tall_narrow_maps_have_a_forward_plan(lib):
    """Up to the limit of N * H * W < 2^27, beyond what the 32-bit lane offsets of the wider tilings span."""
    for dtype in (0, 1):
        for maps in ((1, 1), (1, 8), (3, 300)):
            for W in range(1, 33):
                for N in (1, 5, 9, 12, 15, 16, 17, 33, 64):
                    for part in (0.24, 0.5, 0.81, 1.0):
                        d = lib.Desc(*maps, max(1, int(part * 134217727) // (N * W)), W, N, dtype, 0)
                        f = plan(lib, d, lib.PASS_FWD)
                        assert f["form"] != "small" or (W <= 16 * f["K"] and 4 * f["NW"] >= N and f["wgs"] == -(-maps[0] * maps[1] // 4)), (maps, W, N, f)


def test_backward_plans_cover_every_shape_the_forward_accepts(lib):
    for dtype in (0, 1):
        for W in SWEEP_W:
            for N in SWEEP_N:
                for (Bt, Dc, H) in ((1, 1, 1), (2, 7, 9), (4, 512, 128)):
                    d = lib.Desc(Bt, Dc, H, W, N, dtype, 0)
                    f = plan(lib, d, lib.PASS_BWD)            # every width and state count the forward accepts
                    where = f"dtype {dtype} W {W} N {N} Bt {Bt} Dc {Dc} H {H}: {f}"
                    assert f["lds"] <= 160 * 1024, where
                    assert f["workspace"] == lib.workspace_bytes(d, lib.PASS_BWD), where
                    assert 1 <= f["GS"] <= 8 and f["CG"] == -(-Dc // f["GS"]), where
                    if f["form"] == "small":
                        assert W <= 16 and H <= 16 and N <= 16 and 4 * f["NW"] >= N, where
                    else:
                        assert f["LG"] * f["K"] * f["panels"] >= W, where
                        assert f["panels"] == 1 or (f["LG"] * f["K"] == 256 and f["panels"] == -(-W // 256)), where
                        assert f["bands"] == -(-H // f["RB"]), where
                        # checkpoints + partial sums over channel groups + partial sums over batch items
                        ck = Bt * Dc * f["bands"] * N * W * 4
                        part = 2 * Bt * f["CG"] * N * H * W * 4 if f["CG"] > 1 else 0
                        assert f["workspace"] >= ck + part, where
                        # ... + the padded copies of the tensors' last rows
                        tail = (W + 16) * (5 * (4 if dtype == 0 else 2) + 1)
                        # ... + the carries between column panels (row-end states per border, a*q twice)
                        carries = (f["panels"] + 1) * (Bt * Dc * N * H * 4 + 256) if f["panels"] > 1 else 0
                        # (checkpoint rows of the shared-producer sweeps are padded to the lane grid LG * K)
                        wide = max(W, f["LG"] * f["K"]) if f["form"] == "banded-shared" else W
                        ck_max = Bt * Dc * f["bands"] * N * wide * 4
                        part_max = 2 * Bt * f["CG"] * N * H * wide * 4 if f["CG"] > 1 else 0
                        assert f["workspace"] <= ck_max + part_max + Bt * Dc * (N + 2) * 4 + tail + carries + 7 * 256, where


@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_saved_buffer_covers_every_checkpoint_read(lib, dtype):
    """The backward's lanes read whole groups of K columns of a checkpoint row; rows by column are W floats apart, so the
    lane across the end of the very last row reads up to K - 1 floats behind it."""
    seen = set()
    for Bt, Dc, H in ((2, 5, 37), (1, 2, 64), (1, 1, 9)):
        for W in range(1, 193):
            d = lib.Desc(Bt, Dc, H, W, 16, dtype, 0)
            have = lib.saved_bytes(d)
            if have == 0:
                continue
            f = plan(lib, d, lib.PASS_BWD)
            K, rows = f["K"], Bt * Dc * f["bands"] * 16
            padded = -(-(rows * f["LG"] * K * 4) // 256) * 256
            if have >= padded:                                 # rows in lane order: LG * K floats each
                continue
            last = (rows - 1) * W + (W - 1) // K * K + K       # floats up to the end of the last read
            assert have >= 4 * last, (dtype, Bt, Dc, H, W, f)
            seen.add(K)
    assert seen == {4, 8, 12}


def test_benchmark_configurations_take_the_intended_forms(lib):
    f = plan(lib, lib.Desc(1, 256, 256, 256, 16, 1, 0), lib.PASS_FWD)
    # one map per compute unit: one state per lane on 16 wavefronts (four per SIMD); with more maps than compute units
    # two states per lane on 8 wavefronts, two workgroups per compute unit
    assert (f["form"], f["LG"], f["K"], f["NW"], f["waves"]) == ("shared", 64, 4, 1, 16) and f["fast"] and f["wgs"] == 256
    f = plan(lib, lib.Desc(2, 256, 256, 256, 16, 1, 0), lib.PASS_FWD)
    assert (f["form"], f["LG"], f["K"], f["NW"], f["waves"]) == ("shared", 64, 4, 2, 8) and f["wgs"] == 512
    f = plan(lib, lib.Desc(32, 192, 56, 56, 16, 1, 0), lib.PASS_FWD)
    # 24 maps per compute unit: eight channels per workgroup, two wavefronts of four 7-column blocks
    assert (f["form"], f["K"], f["waves"], f["wgs"]) == ("quads", 7, 4, 768) and f["fast"]
    assert (f["NG"], f["MPW"], f["panels"]) == (4, 8, 1)     # four state groups, eight maps per workgroup, one panel
    f = plan(lib, lib.Desc(1, 256, 64, 64, 16, 0, 0), lib.PASS_FWD)
    assert (f["form"], f["LG"], f["K"], f["NW"]) == ("shared", 16, 4, 1)
    f = plan(lib, lib.Desc(1, 16, 16, 16, 4, 0, 0), lib.PASS_FWD)
    assert f["form"] == "tile16" and f["wgs"] == 16          # few tiny maps: rows and columns as parallel scans
    f = plan(lib, lib.Desc(8, 128, 14, 14, 16, 0, 0), lib.PASS_FWD)
    assert f["form"] == "tile16" and f["wgs"] == 1024
    f = plan(lib, lib.Desc(64, 128, 14, 14, 16, 0, 0), lib.PASS_FWD)
    assert (f["form"], f["K"]) == ("quads", 4)               # many of them
    f = plan(lib, lib.Desc(64, 128, 12, 14, 16, 0, 0), lib.PASS_FWD)
    assert f["form"] == "small"                              # with few rows: four maps per workgroup, row by row
    b = plan(lib, lib.Desc(4, 512, 128, 192, 16, 0, 0), lib.PASS_BWD)
    assert (b["form"], b["LG"], b["K"], b["NW"]) == ("banded-shared", 16, 12, 1) and b["wgs"] * b["GS"] >= 4 * 512 // 1


@pytest.mark.parametrize("H,rows", [(1, 4), (9, 4), (12, 4), (17, 4), (26, 4), (35, 4), (23, 8), (32, 8), (47, 8), (64, 8)])
def test_rows_per_batch_follow_the_height(lib, H, rows):
    """Whole batches run: eight rows per batch only where that many rows are there."""
    f = plan(lib, lib.Desc(1, 256, H, 60, 16, 0, 0), lib.PASS_FWD)
    assert (f["form"], f["LG"], f["NW"], f["RPB"]) == ("shared", 16, 1, rows), f


@pytest.mark.parametrize("maps,H,W,N,dtype,form", [
    ((1, 256), 20, 19, 9, 0, "general"), ((1, 300), 20, 19, 9, 0, "small"), ((1, 300), 9, 19, 9, 0, "general"), ((1, 300), 9, 19, 9, 1, "small"),
    ((4, 160), 30, 30, 12, 0, "small"), ((4, 256), 30, 30, 15, 1, "small"), ((4, 160), 20, 18, 10, 0, "general"), ((5, 256), 20, 18, 12, 0, "general"),
    ((12, 256), 25, 25, 15, 1, "small"), ((12, 256), 25, 25, 15, 0, "general"), ((4, 160), 30, 28, 12, 0, "general"), ((4, 160), 30, 30, 16, 0, "shared")])
def test_narrow_maps_of_nine_to_fifteen_states(lib, maps, H, W, N, dtype, form):
    f = plan(lib, lib.Desc(*maps, H, W, N, dtype, 0), lib.PASS_FWD)
    assert f["form"] == form and (form != "small" or (f["K"], f["NW"]) == (2, 4)), f


@pytest.mark.parametrize("maps,channels", [((8, 128), 1), ((9, 192), 1), ((8, 256), 2), ((12, 192), 3), ((3, 700), 3), ((9, 256), 2), ((12, 256), 4),
                                           ((14, 256), 3), ((16, 256), 4), ((17, 256), 4)])
def test_tiny_maps_channels_per_workgroup(lib, maps, channels):
    """As many as keep 1024 workgroups, one more where a compute unit then has fewer channels to do."""
    f = plan(lib, lib.Desc(*maps, 14, 14, 16, 0, 0), lib.PASS_FWD)
    assert (f["form"], f["MPW"]) == ("tile16", channels) and f["wgs"] == maps[0] * -(-maps[1] // channels), f


@pytest.mark.parametrize("maps,H,W,N,form", [((8, 512), 14, 16, 4, "small"), ((32, 192), 13, 16, 8, "small"), ((8, 256), 14, 16, 16, "small"),
                                              ((8, 256), 16, 16, 16, "tile16"), ((6, 256), 13, 16, 3, "tile16"), ((24, 256), 13, 16, 12, "tile16"), ((8, 512), 14, 15, 4, "tile16")])
def test_many_maps_of_whole_16_column_rows(lib, maps, H, W, N, form):
    assert plan(lib, lib.Desc(*maps, H, W, N, 0, 0), lib.PASS_FWD)["form"] == form


def test_wide_grids_take_the_shared_producer_forms(lib):
    # 257 to 1024 columns, 16 states, one map per compute unit: wave-wide groups with 8, 12 or 16 columns per lane
    for W, K in ((300, 8), (400, 8), (512, 8), (513, 12), (600, 12), (768, 12), (769, 16), (1000, 16), (1024, 16)):
        for dtype in (0, 1):
            f = plan(lib, lib.Desc(1, 256, 200, W, 16, dtype, 0), lib.PASS_FWD)
            assert (f["form"], f["LG"], f["K"], f["panels"]) == ("shared", 64, K, 1) and f["workspace"] == 0, (W, dtype, f)
    f = plan(lib, lib.Desc(1, 256, 200, 1025, 16, 1, 0), lib.PASS_FWD)
    assert f["form"] == "general" and f["panels"] > 1
    # their backward: panels of 256 columns; with 16 states the shared-producer main sweep, two states per lane
    b = plan(lib, lib.Desc(1, 256, 400, 400, 16, 1, 0), lib.PASS_BWD)
    assert (b["form"], b["LG"], b["K"], b["NW"], b["waves"], b["panels"]) == ("banded-shared", 64, 4, 2, 8, 2)
    b = plan(lib, lib.Desc(1, 256, 400, 400, 8, 1, 0), lib.PASS_BWD)
    assert (b["form"], b["LG"], b["K"], b["panels"]) == ("banded", 64, 4, 2)


# The kernel for many maps: one shape on each side of every line of its rule; `wgs` batch items of eight channels are as many workgroups.
# K = 0: another form.  waves: two per column of wavefronts.
MANY_MAPS = [
    # 13 to 16 columns: 576 workgroups, 13 rows
    ("both", 576, 13, 13, 4, 2), ("both", 575, 13, 13, 0, 0), ("both", 576, 12, 16, 0, 0), ("both", 576, 13, 16, 4, 2), ("both", 4096, 48, 12, 0, 0),
    # from 17 columns on nine rows; to 20 columns 288 workgroups, to 24 columns 384
    ("both", 288, 9, 17, 5, 2), ("both", 288, 8, 17, 0, 0), ("both", 287, 48, 17, 0, 0), ("both", 288, 48, 20, 5, 2), ("both", 383, 48, 21, 0, 0),
    ("both", 384, 48, 21, 6, 2), ("both", 384, 9, 24, 6, 2),
    # to 32 columns: two columns of wavefronts from 384 workgroups and 24 rows on, one from 512 workgroups on
    ("both", 383, 48, 25, 0, 0), ("both", 384, 24, 25, 4, 4), ("both", 384, 23, 25, 0, 0), ("both", 511, 24, 32, 4, 4), ("both", 512, 23, 32, 8, 2),
    ("both", 512, 48, 25, 7, 2),
    # 33 to 48 columns: 641 workgroups, or 432 up to 48 columns in bf16, 40 in fp32 and 36 with the softplus step
    ("both", 431, 48, 33, 0, 0), ("both", 432, 48, 33, 5, 4), ("both", 432, 48, 36, 5, 4), ("sp", 640, 48, 37, 0, 0), ("bf16", 432, 48, 37, 5, 4),
    ("f32", 432, 48, 40, 5, 4), ("f32", 640, 48, 41, 0, 0), ("f32", 641, 48, 41, 11, 2), ("bf16", 432, 48, 48, 6, 4), ("bf16", 512, 48, 49, 0, 0),
    # one column of wavefronts: in fp32 from 513 workgroups on, in bf16 where the last round of four workgroups per compute unit is more than three
    # quarters full
    ("f32 sp", 641, 48, 48, 12, 2), ("f32", 641, 48, 48, 12, 2), ("f32", 640, 48, 40, 10, 2), ("f32 sp", 513, 48, 36, 9, 2), ("f32", 512, 48, 40, 5, 4),
    ("bf16 sp", 641, 48, 48, 6, 4), ("bf16 sp", 768, 48, 45, 6, 4),
    ("bf16 sp", 769, 48, 45, 12, 2), ("bf16", 768, 48, 45, 6, 4), ("bf16", 769, 48, 45, 12, 2), ("bf16", 1024, 48, 33, 9, 2), ("bf16", 1025, 48, 33, 5, 4),
    # 49 to 64 columns: 641 workgroups, 513 for the plain scan in bf16 up to 56 columns
    ("bf16", 513, 48, 49, 7, 4), ("bf16", 513, 48, 56, 7, 4), ("bf16", 513, 48, 57, 0, 0), ("bf16", 640, 48, 64, 0, 0), ("bf16", 641, 48, 57, 8, 4),
    ("f32", 640, 48, 49, 0, 0), ("f32", 1025, 48, 49, 7, 4), ("sp", 640, 48, 49, 0, 0), ("bf16 sp", 641, 48, 56, 7, 4),
    # with the softplus step in bf16 beyond 56 columns: whole blocks or a last round that is nearly full
    ("bf16 sp", 896, 48, 57, 0, 0), ("bf16 sp", 897, 48, 57, 15, 2), ("bf16 sp", 1024, 48, 63, 16, 2), ("bf16 sp", 1025, 48, 63, 0, 0),
    ("bf16 sp", 641, 48, 64, 8, 4), ("bf16 sp", 1025, 48, 64, 8, 4),
    # one column of wavefronts: the last round of four more than three quarters full; in fp32 up to 60 columns with the step always,
    # without it also where a last round of three is more than two thirds full
    ("both", 1024, 48, 64, 16, 2), ("bf16", 768, 48, 60, 8, 4), ("bf16", 832, 48, 60, 0, 0), ("bf16", 833, 48, 60, 15, 2), ("f32 sp", 1025, 48, 60, 15, 2), ("f32 sp", 1025, 48, 61, 8, 4),
    ("f32", 768, 48, 60, 15, 2), ("f32", 768, 48, 61, 8, 4), ("f32", 1281, 48, 60, 15, 2), ("f32", 1280, 48, 60, 8, 4), ("both", 4096, 48, 65, 0, 0),
    # two columns of wavefronts from 49 columns on: 21 rows, or 9, 13 and 17
    ("bf16", 641, 21, 57, 8, 4), ("bf16", 641, 20, 57, 0, 0), ("bf16 sp", 641, 18, 49, 0, 0), ("both", 1025, 17, 64, 8, 4), ("both", 1025, 16, 64, 0, 0),
    ("both", 1025, 13, 64, 8, 4), ("f32", 1281, 12, 61, 0, 0), ("f32", 1281, 9, 61, 8, 4), ("bf16", 641, 12, 48, 6, 4), ("f32 sp", 641, 12, 60, 15, 2),
    ("both", 1024, 10, 64, 16, 2),
    # bf16 from 49 columns on: not just past three workgroups per compute unit
    ("bf16", 768, 48, 49, 7, 4), ("bf16", 769, 48, 49, 0, 0), ("bf16 sp", 768, 48, 64, 8, 4), ("bf16 sp", 769, 48, 64, 0, 0), ("bf16 sp", 832, 48, 56, 0, 0),
    ("bf16 sp", 833, 48, 56, 14, 2), ("bf16", 1800, 48, 56, 14, 2), ("f32", 769, 48, 60, 15, 2), ("bf16", 769, 48, 48, 12, 2),
]


@pytest.mark.parametrize("which,wgs,H,W,K,waves", MANY_MAPS, ids=["-".join(map(str, c[:4])) for c in MANY_MAPS])
def test_many_maps_take_eight_channels_per_workgroup(lib, which, wgs, H, W, K, waves):
    ways = [(dt, sp) for dt in (0, 1) for sp in (False, True)]
    if which != "both":
        dts = [0] if "f32" in which else [1] if "bf16" in which else [0, 1]
        ways = [(dt, "sp" in which) for dt in dts]
    for dt, sp in ways:
        f = plan(lib, lib.Desc(wgs, 8, H, W, 16, dt, 0), lib.PASS_FWD_SOFTPLUS if sp else lib.PASS_FWD)
        if K:
            assert (f["form"], f["K"], f["waves"], f["wgs"]) == ("quads", K, waves, -(-wgs // 8) * 8), (dt, sp, f)
            assert (f["NG"], f["MPW"], f["panels"], f["workspace"]) == (4, 8, 1, 0)
            assert waves // 2 * 4 * (K - 1) < W <= waves // 2 * 4 * K
        else:
            assert f["form"] != "quads", (dt, sp, f)


def test_many_maps_need_sixteen_states_and_few_idle_channels(lib):
    form = lambda Bt, Dc, N=16, flags=0: plan(lib, lib.Desc(Bt, Dc, 28, 28, N, 1, flags), lib.PASS_FWD)["form"]
    assert form(48, 96) == "quads" and form(48, 96, 15) != "quads" and form(48, 96, 17) != "quads"
    # at most one channel in nine is idle
    assert form(512, 15) == "quads" and form(512, 14) != "quads" and form(512, 9) != "quads" and form(1024, 7) != "quads" and form(300, 22) == "quads"
    assert form(48, 96, 16, lib.FLAG_IDENTITY_CELLS) == "quads"


def test_plans_with_and_without_the_softplus_step_are_told_apart(lib):
    """The forms are ranked for each of them."""
    d = lib.Desc(720, 8, 48, 60, 16, 1, 0)
    assert plan(lib, d, lib.PASS_FWD)["form"] == "quads" and plan(lib, d, lib.PASS_FWD_SOFTPLUS)["form"] == "shared"
    assert lib.workspace_bytes(d, lib.PASS_FWD_SOFTPLUS) == lib.workspace_bytes(d, lib.PASS_FWD)
    assert lib.describe_plan(lib.Desc(2, 8, 20, 40, 16, 0, lib.FLAG_COLUMNS_FIRST), lib.PASS_FWD_SOFTPLUS).startswith("columns-first(in-kernel) fwd form=shared")
    assert lib.describe_plan(lib.Desc(2, 8, 20, 40, 5, 0, lib.FLAG_COLUMNS_FIRST), lib.PASS_FWD_SOFTPLUS).startswith("columns-first(transposed) fwd")
