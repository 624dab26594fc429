"""GPU parity tests: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Tolerances (per output tensor): max|gpu - ref| / max|ref| <= 1e-4 for fp32
storage and <= 2e-2 for bf16 storage; mask and indexing properties are bit-exact."""
import os

import numpy as np
import pytest

import oracle
from paper_2412_00678_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = {wl.F32: 1e-4, wl.BF16: 2e-2}


@pytest.fixture(scope="module")
def s2d():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2412_00678_amd import scan2d          # raises if the library is not built
    return scan2d


def rel_err(got, ref):
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    denom = max(np.abs(ref).max(), 1e-30)
    return float(np.abs(got - ref).max() / denom)


def run_fwd(s2d, inp, dtype, variant=None):
    import torch
    d = s2d.to_device(inp, dtype)
    kind = s2d.TUNE_FWD
    if variant is not None and variant.startswith("shared:"):
        kind, variant = s2d.TUNE_FWD_SHARED, variant[len("shared:"):]
    with s2d.forced_variant(kind, variant):
        if kind == s2d.TUNE_FWD_SHARED:                   # the forced form must be the one that runs
            plan = s2d.describe_plan(s2d.make_desc(d["x"], d["A"]), s2d.PASS_FWD)
            LG, K, NW, waves, rpb, *skew = (int(t) for t in variant.split(","))
            form = "skew" if skew and skew[0] else "shared"
            assert f"form={form} LG={LG} K={K} NW={NW} waves={waves} RPB={rpb} " in plan, plan
        y = s2d.scan2d_fwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
        torch.cuda.synchronize()
    return s2d.to_host(y)


def oracle_fwd(inp, dtype):
    return oracle.scan2d_fwd(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"],
                             inp["mask"], dtype=dtype)


def check_fwd(s2d, w, seed=0, variant=None, tol=None):
    inp = wl.make_inputs(w, seed=seed)
    print(f"fwd case {w.name} Bt={w.Bt} Dc={w.Dc} N={w.N} H={w.H} W={w.W} dtype={w.dtype} variant={variant}", flush=True)
    y = run_fwd(s2d, inp, w.dtype, variant)
    ref = oracle_fwd(inp, w.dtype)
    err = rel_err(wl.to_float(y, w.dtype), wl.to_float(ref, w.dtype))
    assert np.isfinite(wl.to_float(y, w.dtype)).all()
    assert err <= (tol or TOL[w.dtype]), f"{w.name}: rel err {err:.3e}"
    return err


# ------------------------------------------------------------------ the benchmark configurations

@pytest.mark.parametrize("idx", [0, 1, 2, 3, 4])
def test_forward_matches_oracle_on_benchmark_configs(s2d, idx):
    check_fwd(s2d, wl.CONFIGS[idx])


# ------------------------------------------------------------------ shapes, tails, degenerate cases

SHAPES = [
    # Bt, Dc, N, H, W, dtype, mask
    (1, 3, 4, 1, 1, wl.F32, 0.0),          # single cell
    (2, 3, 4, 1, 37, wl.F32, 0.3),         # H = 1: the 1D scan
    (2, 3, 4, 29, 1, wl.BF16, 0.3),        # W = 1
    (1, 5, 16, 14, 14, wl.BF16, 0.0),      # the paper's typical small map: ragged lanes
    (3, 7, 16, 56, 56, wl.F32, 0.0),
    (1, 2, 16, 200, 200, wl.BF16, 0.4),    # the paper's largest timed map
    (1, 3, 5, 23, 45, wl.F32, 0.2),        # N not divisible by the states per lane
    (1, 2, 64, 17, 33, wl.BF16, 0.2),      # maximum N
    (1, 2, 1, 19, 64, wl.F32, 0.0),        # N = 1
    (2, 2, 8, 9, 260, wl.F32, 0.3),        # one column past a 256-wide panel
    (1, 2, 4, 5, 1100, wl.BF16, 0.3),      # several panels
    (1, 1, 16, 300, 12, wl.F32, 0.5),      # tall and narrow
    (5, 1, 16, 20, 24, wl.BF16, 0.3),      # one channel: every map is another batch item
    (1, 40, 16, 16, 128, wl.F32, 0.0),
    (1, 9, 16, 33, 192, wl.F32, 0.3),
    # narrow maps: one wavefront per map
    (2, 9, 16, 14, 14, wl.F32, 0.2),       # 14 of 16 lanes
    (1, 7, 16, 7, 7, wl.BF16, 0.2),
    (2, 5, 16, 28, 28, wl.BF16, 0.3),      # two columns per lane
    (1, 6, 16, 11, 31, wl.F32, 0.3),       # odd width: the last lane holds one column
    (1, 3, 16, 40, 17, wl.BF16, 0.0),      # odd rows of bf16 start on a 2-byte boundary
    (1, 5, 4, 9, 16, wl.F32, 0.3),         # one state per lane group
    (1, 5, 3, 9, 13, wl.F32, 0.3),         # fewer states than lane groups
    (1, 3, 5, 9, 20, wl.BF16, 0.3),        # N not a multiple of the states per lane
    (1, 3, 30, 6, 15, wl.F32, 0.2),        # eight states per lane, last group ragged
    (1, 2, 64, 5, 32, wl.F32, 0.2),        # sixteen states per lane, two columns
    (3, 1, 16, 14, 14, wl.F32, 0.0),       # a partly filled last workgroup
    (9, 128, 16, 14, 14, wl.F32, 0.2),     # more than 1024 tiny maps: four per workgroup, row by row
    # at most 1024 maps of at most 16 x 16 positions and 16 states: one workgroup per map, rows and columns as parallel scans
    (1, 4, 5, 16, 16, wl.F32, 0.3),        # a full tile, states not a multiple of 4
    (2, 3, 13, 15, 9, wl.BF16, 0.4),       # ragged in both directions
    (8, 128, 16, 14, 14, wl.F32, 0.0),     # the paper's 14 x 14 grid at 128 channels, batch 8
    (1, 2, 1, 16, 1, wl.F32, 0.3),         # one column, one state
    # widths that are not a multiple of the columns per lane: the last lane reads across the row end
    (2, 5, 16, 19, 57, wl.F32, 0.3),       # mask rows off the 4-byte boundaries
    (2, 5, 16, 19, 58, wl.BF16, 0.3),      # bf16, even width: rows on 4-byte boundaries, mask rows not
    (1, 6, 16, 11, 201, wl.F32, 0.4),
    (1, 6, 16, 11, 250, wl.BF16, 0.4),
    (1, 3, 16, 9, 55, wl.BF16, 0.3),       # bf16, odd width: every other row starts on an odd 2-byte boundary
    (3, 5, 16, 21, 57, wl.BF16, 0.4),      # odd width and odd H*W: maps alternate their alignment too
    (2, 3, 16, 10, 201, wl.BF16, 0.3),     # the same with wave-wide lane groups
    (1, 7, 5, 13, 99, wl.BF16, 0.3),       # ragged last lane group
    (2, 4, 16, 12, 255, wl.BF16, 0.0),     # no mask
    (1, 2, 16, 1, 63, wl.BF16, 0.3),       # a single row
    (1, 4, 16, 13, 101, wl.F32, 0.0),      # no mask
    (1, 2, 5, 7, 150, wl.F32, 0.3),        # ragged states and a ragged last lane
    (1, 1, 16, 3, 255, wl.F32, 0.5),       # the last lane of the last row of the last map reads past the tensor
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_forward_edge_shapes(s2d, shape):
    Bt, Dc, N, H, W, dtype, mf = shape
    check_fwd(s2d, wl.Workload("edge", Bt, Dc, N, H, W, dtype, mask_frac=mf), seed=3)


VARIANT_CASES = [
    # (LG, K, NW) forced on a shape it fits: W multiple of K, N multiple of NW
    ("16,4,1", (1, 6, 4, 21, 64)), ("16,4,2", (1, 6, 4, 21, 48)), ("16,4,4", (2, 5, 16, 21, 56)),
    ("16,4,8", (1, 6, 16, 21, 64)), ("16,4,16", (1, 9, 16, 21, 60)),
    ("16,8,1", (1, 6, 2, 21, 128)), ("16,8,2", (1, 6, 4, 21, 120)), ("16,8,4", (1, 6, 16, 21, 128)),
    ("16,8,8", (1, 6, 16, 21, 96)),
    ("16,12,1", (1, 6, 2, 13, 192)), ("16,12,2", (1, 6, 4, 13, 180)), ("16,12,4", (1, 6, 16, 13, 192)),
    ("16,16,1", (1, 6, 2, 13, 256)), ("16,16,2", (1, 6, 4, 13, 240)), ("16,16,4", (1, 6, 16, 13, 256)),
    ("64,4,1", (1, 6, 4, 13, 256)), ("64,4,2", (1, 6, 4, 13, 200)), ("64,4,4", (1, 6, 16, 13, 256)),
    ("64,4,8", (1, 6, 16, 13, 252)), ("64,4,16", (1, 6, 32, 13, 256)),
    ("64,8,1", (1, 6, 2, 13, 512)), ("64,8,2", (1, 6, 4, 13, 504)), ("64,8,4", (1, 6, 16, 13, 512)),
    ("64,8,8", (1, 6, 16, 13, 400)),
    ("64,16,1", (1, 6, 2, 9, 1024)), ("64,16,2", (1, 6, 4, 9, 1008)), ("64,16,4", (1, 6, 16, 9, 1024)),
    # 8 and 16 waves per workgroup (the states of one map spread over more wavefronts)
    ("64,4,1,8", (1, 3, 8, 13, 256)), ("64,4,2,8", (1, 3, 16, 13, 256)), ("64,8,1,8", (1, 3, 8, 13, 512)),
    ("64,8,2,8", (1, 3, 16, 13, 512)), ("64,16,1,8", (1, 3, 8, 9, 1024)),
    ("64,4,1,16", (2, 3, 16, 13, 256)), ("64,8,1,16", (1, 3, 16, 13, 480)),
    ("64,4,1,16", (1, 3, 16, 9, 203)), ("64,4,1,16", (1, 2, 16, 5, 777)), ("64,4,2,8", (1, 2, 16, 5, 515)),
    ("64,4,1,8", (1, 5, 4, 9, 101)),
    # half-wave lane groups
    ("32,4,1,8", (1, 3, 16, 13, 128)), ("32,4,2,4", (1, 5, 16, 13, 124)), ("32,4,4,4", (1, 5, 16, 13, 128)),
    ("32,8,1,8", (1, 3, 16, 13, 256)), ("32,8,2,4", (1, 3, 16, 13, 248)), ("32,8,2,8", (1, 5, 16, 13, 256)),
    ("32,8,4,4", (1, 5, 16, 13, 200)),
    # rows between two barriers forced to 1, 2, 4, 8 (H = 13, 21, 3: short last batch)
    ("32,8,1,8,1", (1, 3, 16, 13, 256)), ("64,4,2,8,2", (1, 3, 16, 13, 256)), ("16,4,4,4,4", (2, 5, 16, 21, 56)),
    ("16,12,2,4,2", (1, 6, 4, 13, 180)), ("64,4,2,8,4", (1, 3, 16, 2, 256)), ("64,4,1,16,4", (1, 2, 16, 7, 600)),
    ("64,4,2,8,8", (1, 3, 16, 21, 256)), ("16,4,1,4,8", (1, 3, 16, 8, 64)), ("16,4,1,4,8", (2, 2, 16, 3, 60)),   # and 8
    # guarded (ragged W) and multi-panel forms of the K = 4 variants
    ("16,4,4", (1, 6, 16, 9, 61)), ("64,4,4", (1, 6, 16, 9, 203)), ("64,4,2", (1, 3, 4, 7, 777)),
    ("16,4,4", (1, 3, 16, 7, 150)), ("16,4,4", (1, 3, 10, 7, 150)), ("16,8,4", (1, 3, 10, 7, 128)),
    # narrow-map kernel with two columns per lane forced on a map that one column per lane would cover
    ("16,2", (1, 5, 16, 9, 14)), ("16,1", (2, 3, 8, 9, 16)), ("16,2", (2, 5, 20, 9, 29)), ("16,2", (1, 3, 64, 7, 30)),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("variant,shape", VARIANT_CASES, ids=[f"{v}-{s[4]}-{s[2]}" for v, s in VARIANT_CASES])
def test_every_kernel_variant(s2d, variant, shape, dtype):
    Bt, Dc, N, H, W = shape
    check_fwd(s2d, wl.Workload("var", Bt, Dc, N, H, W, dtype, mask_frac=0.25), seed=5, variant=variant)


@pytest.mark.parametrize("dtype,shape", [(wl.F32, (1, 2, 9, 200000, 18)), (wl.BF16, (1, 1, 15, 100000, 30))], ids=["f32", "bf16"])
def test_tall_narrow_maps(s2d, shape, dtype):
    """Maps whose states the 32-bit lane offsets of the wider tilings do not span run in the narrow-map kernel."""
    Bt, Dc, N, H, W = shape
    plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, N, dtype, 0), s2d.PASS_FWD)
    assert "form=small LG=16 K=2 " in plan, plan
    check_fwd(s2d, wl.Workload("tall", Bt, Dc, N, H, W, dtype, mask_frac=0.25), seed=6)


# The form whose lane groups share the per-position work through LDS: LG,K,NW,WAVES,RPB forced on shapes with
# N = NG * NW; odd widths, heights off the batch grid, map counts off the workgroup grid (idle lane groups).
SHARED_CASES = [
    ("64,4,2,8,4", (1, 3, 16, 13, 256)), ("64,4,2,8,4", (1, 2, 16, 9, 203)), ("64,4,2,8,8", (1, 3, 16, 21, 250)),
    ("64,4,1,16,4", (2, 3, 16, 13, 256)), ("64,4,1,16,4", (1, 2, 16, 6, 131)),
    ("16,12,1,4,4", (1, 5, 16, 13, 192)), ("16,12,1,4,4", (1, 3, 16, 7, 181)), ("16,12,2,4,2", (1, 5, 16, 13, 190)),
    ("16,8,1,4,4", (1, 3, 16, 9, 128)), ("16,8,2,4,2", (2, 3, 16, 9, 121)),
    ("16,4,1,4,4", (1, 3, 16, 11, 64)), ("16,4,2,4,4", (1, 5, 16, 11, 57)), ("16,4,4,4,4", (1, 7, 16, 11, 56)),
    ("16,4,8,4,4", (1, 11, 16, 11, 50)), ("16,4,8,4,4", (3, 64, 16, 5, 33)),
    # 257 to 1024 columns: 8, 12 and 16 columns per lane of a wave-wide group
    ("64,8,1,16,2", (1, 2, 16, 9, 512)), ("64,8,1,16,2", (1, 3, 16, 5, 301)), ("64,8,2,8,2", (2, 2, 16, 7, 334)),
    ("64,12,2,8,2", (1, 2, 16, 5, 768)), ("64,12,2,8,2", (1, 2, 16, 6, 601)), ("64,16,2,8,2", (1, 2, 16, 5, 1024)),
    ("64,16,2,8,2", (1, 2, 16, 3, 903)),
    # N = 8, 4, 32, 64
    ("64,4,1,8,4", (1, 3, 8, 13, 256)), ("16,4,1,4,4", (1, 3, 8, 9, 60)), ("16,4,2,4,4", (1, 7, 8, 9, 61)),
    ("16,8,1,4,4", (1, 3, 8, 9, 100)), ("16,12,1,4,4", (1, 3, 8, 9, 180)),
    ("64,4,1,4,4", (1, 3, 4, 9, 250)), ("16,4,1,4,4", (1, 6, 4, 9, 64)), ("16,8,1,4,4", (1, 5, 4, 9, 127)),
    ("64,4,2,16,4", (1, 2, 32, 9, 256)), ("64,4,4,8,4", (1, 2, 32, 9, 240)), ("16,4,2,4,4", (1, 2, 32, 9, 64)),
    ("16,8,2,4,4", (1, 2, 32, 9, 128)), ("16,4,4,4,4", (1, 3, 32, 9, 63)),
    ("64,4,4,16,4", (1, 2, 64, 5, 256)), ("16,4,4,4,4", (1, 2, 64, 5, 64)), ("16,8,4,4,2", (1, 2, 64, 5, 100)),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("variant,shape", SHARED_CASES, ids=[f"shared-{v}-{s[4]}-{s[2]}" for v, s in SHARED_CASES])
def test_every_shared_producer_variant(s2d, variant, shape, dtype):
    Bt, Dc, N, H, W = shape
    check_fwd(s2d, wl.Workload("shared", Bt, Dc, N, H, W, dtype, mask_frac=0.25), seed=6, variant="shared:" + variant)


# The same kernel with skewed rows (lane l of a group works on row t - l, no scan across the lanes; a measured
# alternative that only the override selects): LG,K,NW,WAVES,RPB,1.  Maps shorter than the skew, heights off the
# batch grid, even widths below the panel (bf16 rows of odd width are refused: the override is then ignored).
SKEW_CASES = [
    ("16,16,1,4,4,1", (1, 3, 16, 37, 256)), ("16,16,1,4,4,1", (2, 2, 16, 5, 250)), ("16,16,1,4,4,1", (1, 2, 16, 70, 202)),
    ("16,8,1,4,4,1", (2, 3, 16, 19, 100)), ("16,8,1,4,4,1", (1, 1, 16, 3, 8)), ("16,8,1,4,4,1", (1, 2, 16, 1, 66)),
    ("64,4,1,16,4,1", (1, 2, 16, 37, 256)), ("64,4,1,16,4,1", (1, 2, 16, 5, 202)), ("64,4,1,16,4,1", (1, 3, 16, 130, 130)),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("variant,shape", SKEW_CASES, ids=[f"skew-{v}-{s[3]}x{s[4]}" for v, s in SKEW_CASES])
def test_skewed_row_variants(s2d, variant, shape, dtype):
    Bt, Dc, N, H, W = shape
    check_fwd(s2d, wl.Workload("skew", Bt, Dc, N, H, W, dtype, mask_frac=0.25), seed=8, variant="shared:" + variant)


# A grid wider than 256 columns at full size, as bench-like launches see it (one map per compute unit, 256 maps): the
# oracle computes three of the 256 channels, the tiling must be the shared-producer one with 8 or 12 columns per lane.
@pytest.mark.parametrize("H,W,K", [(400, 400, 8), (150, 600, 12)])
def test_wide_grid_at_full_size_on_sampled_channels(s2d, H, W, K):
    import torch
    w = wl.Workload("wide_full", 1, 256, 16, H, W, wl.BF16, mask_frac=0.5)
    inp = wl.make_inputs(w, seed=12)
    print(f"wide grid Bt=1 Dc=256 N=16 H={H} W={W} bf16", flush=True)
    d = s2d.to_device(inp, w.dtype)
    plan = s2d.describe_plan(s2d.make_desc(d["x"], d["A"]), s2d.PASS_FWD)
    assert f"form=shared LG=64 K={K} " in plan, plan
    y = s2d.scan2d_fwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    torch.cuda.synchronize()
    got = s2d.to_host(y)
    for c in (0, 131, 255):
        ref = oracle.scan2d_fwd(inp["x"][:, c:c + 1], inp["delta"][:, c:c + 1], inp["A"][c:c + 1], inp["Bm"], inp["Cm"],
                                inp["Dskip"][c:c + 1], inp["mask"], dtype=w.dtype)
        err = rel_err(wl.to_float(got[:, c:c + 1], w.dtype), wl.to_float(ref, w.dtype))
        assert err <= TOL[w.dtype], f"channel {c}: rel err {err:.3e}"


# ------------------------------------------------------------------ mask / indexing: bit-exact

@pytest.mark.parametrize("H,W", [(40, 72), (19, 57), (9, 55), (7, 33), (5, 250)])   # also mask and bf16 tensors that end inside a dword
def test_mask_is_bit_identical_to_prezeroed_x_and_blocks_garbage(s2d, H, W):
    for dtype in (wl.F32, wl.BF16):
        w = wl.Workload("mask", 2, 6, 16, H, W, dtype, mask_frac=0.4)
        inp = wl.make_inputs(w, seed=7)
        y_mask = run_fwd(s2d, inp, dtype)
        nomask = dict(inp, mask=None)                     # x is already +0 under the mask
        assert np.array_equal(y_mask, run_fwd(s2d, nomask, dtype))
        for poison in (np.nan, np.inf, 1e30):
            p = wl.make_inputs(w, seed=7, poison_under_mask=poison)
            assert np.array_equal(y_mask, run_fwd(s2d, p, dtype)), poison
        full = dict(inp, mask=np.ones_like(inp["mask"]))
        assert not wl.to_float(run_fwd(s2d, full, dtype), dtype).any()


def test_causality_is_bit_exact(s2d):
    w = wl.Workload("causal", 1, 4, 16, 48, 80, wl.F32, mask_frac=0.2)
    inp = wl.make_inputs(w, seed=9)
    y0 = run_fwd(s2d, inp, wl.F32)
    i0, j0 = 20, 41
    rng = np.random.default_rng(1)
    alt = {k: (None if v is None else v.copy()) for k, v in inp.items()}
    for k in ("x", "delta", "Bm", "Cm"):
        alt[k][..., i0 + 1:, :] = np.abs(rng.standard_normal(alt[k][..., i0 + 1:, :].shape)).astype(np.float32)
        alt[k][..., :, j0 + 1:] = np.abs(rng.standard_normal(alt[k][..., :, j0 + 1:].shape)).astype(np.float32)
    alt["mask"][..., i0 + 1:, :] = 0
    alt["mask"][..., :, j0 + 1:] = 0
    y1 = run_fwd(s2d, alt, wl.F32)
    assert np.array_equal(y0[..., :i0 + 1, :j0 + 1], y1[..., :i0 + 1, :j0 + 1])
    assert not np.array_equal(y0, y1)


def test_each_map_lands_at_its_own_index_and_runs_are_reproducible(s2d):
    w = wl.Workload("perm", 3, 10, 16, 24, 56, wl.BF16, mask_frac=0.3)
    inp = wl.make_inputs(w, seed=11)
    y = run_fwd(s2d, inp, wl.BF16)
    assert np.array_equal(y, run_fwd(s2d, inp, wl.BF16))          # same bits on a second run
    perm_c = np.random.default_rng(2).permutation(w.Dc)
    perm_b = np.array([2, 0, 1])
    q = dict(inp)
    q["x"] = inp["x"][perm_b][:, perm_c].copy()
    q["delta"] = inp["delta"][perm_b][:, perm_c].copy()
    q["A"] = inp["A"][perm_c].copy()
    q["Dskip"] = inp["Dskip"][perm_c].copy()
    q["Bm"], q["Cm"], q["mask"] = inp["Bm"][perm_b].copy(), inp["Cm"][perm_b].copy(), inp["mask"][perm_b].copy()
    assert np.array_equal(run_fwd(s2d, q, wl.BF16), y[perm_b][:, perm_c])


def test_no_skip_term_and_no_mask(s2d):
    w = wl.Workload("plain", 1, 6, 16, 30, 64, wl.F32)
    inp = wl.make_inputs(w, seed=13)
    inp["Dskip"] = None
    y = run_fwd(s2d, inp, wl.F32)
    assert rel_err(y, oracle_fwd(inp, wl.F32)) <= 1e-4


def test_unit_decay_and_strong_decay(s2d):
    """A = 0 (summed-area table, sums grow with H*W) and very negative A (a underflows to 0)."""
    w = wl.Workload("decay", 1, 4, 4, 64, 64, wl.F32)
    inp = wl.make_inputs(w, seed=15)
    inp["A"] = np.zeros_like(inp["A"])
    assert rel_err(run_fwd(s2d, inp, wl.F32), oracle_fwd(inp, wl.F32)) <= 1e-4
    inp["A"] = np.full_like(inp["A"], -3000.0)
    assert rel_err(run_fwd(s2d, inp, wl.F32), oracle_fwd(inp, wl.F32)) <= 1e-4


# ====================================================================== backward

GRADS = ("dx", "ddelta", "dA", "dBm", "dCm", "dDskip")


def run_bwd(s2d, inp, dtype, variant=None):
    import torch
    d = s2d.to_device(inp, dtype)
    with s2d.forced_variant(s2d.TUNE_BWD, variant):
        out = s2d.scan2d_bwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"])
        torch.cuda.synchronize()
    return [None if t is None else s2d.to_host(t) for t in out]


def oracle_bwd(inp, dtype):
    return oracle.scan2d_bwd(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"],
                             inp["mask"], inp["dy"], dtype=dtype)


def check_bwd(s2d, w, seed=0, variant=None):
    inp = wl.make_inputs(w, seed=seed)
    print(f"bwd case {w.name} Bt={w.Bt} Dc={w.Dc} N={w.N} H={w.H} W={w.W} dtype={w.dtype} variant={variant}", flush=True)
    got = run_bwd(s2d, inp, w.dtype, variant)
    ref = oracle_bwd(inp, w.dtype)
    errs = {}
    for k, (name, g, r) in enumerate(zip(GRADS, got, ref)):
        if r is None:
            assert g is None
            continue
        gv = wl.to_float(g, w.dtype) if k < 2 else g.astype(np.float64)
        rv = wl.to_float(r, w.dtype) if k < 2 else r.astype(np.float64)
        assert np.isfinite(gv).all(), name
        errs[name] = rel_err(gv, rv)
        tol = TOL[w.dtype] if k < 2 else (1e-4 if w.dtype == wl.F32 else 2e-2)
        assert errs[name] <= tol, f"{w.name} {name}: rel err {errs[name]:.3e}"
    if inp["mask"] is not None:                       # dx under the mask is exactly +0
        m = np.broadcast_to(inp["mask"][:, None] != 0, got[0].shape)
        assert not got[0].view(np.uint32 if w.dtype == wl.F32 else np.uint16)[m].any()
    return errs


def test_backward_matches_oracle_on_the_training_config(s2d):
    check_bwd(s2d, wl.CONFIGS[4])


BWD_SHAPES = [
    # Bt, Dc, N, H, W, dtype, mask
    (1, 3, 4, 1, 1, wl.F32, 0.0),
    (2, 3, 4, 1, 37, wl.F32, 0.3),         # H = 1
    (2, 3, 4, 29, 1, wl.F32, 0.3),         # W = 1
    (1, 5, 16, 14, 14, wl.F32, 0.0),
    (2, 7, 16, 56, 56, wl.F32, 0.2),
    (1, 6, 16, 23, 100, wl.F32, 0.3),      # 8 columns per lane
    (1, 5, 16, 9, 200, wl.F32, 0.4),       # wave-wide lane groups
    (1, 3, 5, 11, 45, wl.F32, 0.2),        # N below a full set of lane groups
    (1, 2, 40, 7, 33, wl.F32, 0.2),        # N > 16: four states per lane
    (1, 2, 1, 19, 64, wl.F32, 0.0),
    (1, 9, 16, 6, 300, wl.F32, 0.3),
    (1, 4, 8, 5, 1000, wl.F32, 0.3),
    (3, 5, 16, 13, 24, wl.BF16, 0.3),      # bf16 storage
    (1, 3, 16, 10, 130, wl.BF16, 0.3),
    (4, 1, 16, 10, 24, wl.F32, 0.3),       # one channel per batch item
    (2, 21, 16, 10, 40, wl.F32, 0.3),      # ragged last channel group
    (1, 5, 16, 10, 68, wl.F32, 0.3),       # one lane past a 64-column boundary
    (1, 5, 16, 9, 129, wl.F32, 0.3),       # ragged width, odd
    (1, 6, 16, 9, 256, wl.F32, 0.3),       # widest map of the 16-lane groups
    (1, 6, 16, 9, 255, wl.BF16, 0.3),
    (1, 3, 24, 7, 132, wl.F32, 0.3),       # four states per lane, 12 columns per lane
    (1, 3, 40, 6, 250, wl.BF16, 0.2),
    # small maps: one wavefront per map, the whole map in registers
    (3, 5, 16, 14, 14, wl.F32, 0.3),
    (2, 7, 16, 7, 7, wl.BF16, 0.3),
    (1, 6, 4, 16, 16, wl.F32, 0.2),        # one state per lane group, all 16 rows and columns
    (2, 3, 8, 14, 14, wl.BF16, 0.0),       # two states per lane group
    (1, 4, 5, 9, 13, wl.F32, 0.3),         # N not a multiple of the states per lane
    (1, 4, 3, 16, 1, wl.F32, 0.3),         # W = 1, fewer states than lane groups
    (5, 1, 16, 14, 14, wl.F32, 0.3),       # one channel: no partial sums over channels
    (1, 2, 16, 17, 14, wl.F32, 0.3),       # one row too many for the small-map kernel
    (1, 2, 24, 14, 14, wl.F32, 0.3),       # too many states for it
    (1, 2, 64, 5, 256, wl.F32, 0.2),       # widest map with more than 16 states
    # widths that are not a multiple of the columns per lane: the last lane reads into the next row
    (2, 5, 16, 12, 57, wl.BF16, 0.3),      # rows on odd 2-byte boundaries
    (1, 4, 16, 9, 191, wl.BF16, 0.3),
    (1, 3, 16, 1, 190, wl.F32, 0.3),       # a single row: nothing may be read past its end
    (1, 4, 16, 2, 61, wl.F32, 0.3),
    (2, 3, 16, 33, 333, wl.F32, 0.3),
    (1, 2, 32, 9, 250, wl.F32, 0.3),
]


@pytest.mark.parametrize("shape", BWD_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_backward_edge_shapes(s2d, shape):
    Bt, Dc, N, H, W, dtype, mf = shape
    check_bwd(s2d, wl.Workload("bedge", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True), seed=4)


@pytest.mark.parametrize("variant,W", [("16,4", 60), ("16,8", 60), ("16,12", 190), ("16,16", 250),
                                       ("64,4", 250), ("64,4,8", 250), ("64,8", 260), ("64,16", 60),
                                       # LG,K,WAVES,GS,shared: the plain main sweep where the shared-producer one is the default
                                       ("16,4,4,0,0", 60), ("16,8,4,0,0", 121), ("16,12,4,0,0", 190)])
def test_backward_variants(s2d, variant, W):
    check_bwd(s2d, wl.Workload("bvar", 2, 6, 16, 11, W, wl.F32, mask_frac=0.3, backward=True), seed=6, variant=variant)


# The main sweep whose lane groups share the per-position work through LDS, every compiled tiling (LG,K,WAVES,GS,1):
# widths on and off the lane grid, heights off the band grid, channel counts off the channel-group grid.
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("variant,shape", [
    ("16,4,4,0,1", (2, 7, 16, 11, 64)), ("16,4,4,3,1", (1, 10, 16, 9, 57)), ("16,8,4,0,1", (2, 5, 16, 10, 128)),
    ("16,8,4,2,1", (1, 7, 16, 13, 99)), ("16,12,4,0,1", (1, 9, 16, 6, 192)), ("16,12,4,4,1", (2, 6, 16, 11, 185)),
    ("32,6,8,0,1", (1, 5, 16, 9, 192)), ("32,6,8,2,1", (2, 3, 16, 7, 187)), ("32,4,8,0,1", (1, 5, 16, 9, 128)),
    ("32,4,8,0,1", (2, 3, 16, 6, 101)), ("64,4,16,0,1", (1, 5, 16, 9, 256)), ("64,4,16,0,1", (1, 3, 16, 5, 203)),
], ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_backward_shared_producer_variants(s2d, variant, shape, dtype):
    Bt, Dc, N, H, W = shape
    w = wl.Workload("bshared", Bt, Dc, N, H, W, dtype, mask_frac=0.3, backward=True)
    import torch
    with s2d.forced_variant(s2d.TUNE_BWD, variant):
        plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, N, dtype, 0), s2d.PASS_BWD)
    assert "form=banded-shared" in plan, plan
    check_bwd(s2d, w, seed=12, variant=variant)


# Sums over batch items, eight requested at a time: below, at and past a multiple of eight, small and banded sweeps.
@pytest.mark.parametrize("Bt,Dc,H,W", [(7, 3, 14, 14), (8, 2, 7, 9), (9, 3, 14, 14), (17, 3, 10, 20), (25, 2, 6, 70)])
def test_backward_sums_over_batch_items(s2d, Bt, Dc, H, W):
    check_bwd(s2d, wl.Workload("bsum", Bt, Dc, 16, H, W, wl.F32, mask_frac=0.3, backward=True), seed=Bt)


# Maps wider than one lane-group panel (and, beyond 16 states, wider than 256 columns) are swept in panels of 256
# columns with the row recurrences carried across the panel borders in both directions.
@pytest.mark.parametrize("shape", [(1, 3, 16, 7, 1500, wl.F32, 0.3), (1, 2, 64, 6, 600, wl.BF16, 0.3), (2, 3, 32, 9, 300, wl.F32, 0.2),
                                   (1, 2, 16, 3, 1027, wl.BF16, 0.0), (1, 2, 24, 1, 513, wl.F32, 0.3), (1, 5, 16, 5, 2049, wl.F32, 0.3),
                                   # 16 states: the shared-producer main sweep, several bands, softplus-free plain step
                                   (2, 3, 16, 21, 520, wl.BF16, 0.3), (1, 9, 16, 13, 400, wl.F32, 0.4), (1, 2, 16, 9, 777, wl.BF16, 0.2)],
                         ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_backward_of_wide_maps_in_column_panels(s2d, shape):
    Bt, Dc, N, H, W, dtype, mf = shape
    plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, N, dtype, 0), s2d.PASS_BWD)
    assert f"panels={-(-W // 256)} " in plan, plan
    assert ("form=banded-shared" in plan) == (N == 16), plan
    check_bwd(s2d, wl.Workload("bwide", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True), seed=14)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("Bt,Dc,H,W", [(3, 5, 5, 17), (1, 9, 4, 64), (2, 3, 9, 65), (1, 7, 3, 128), (2, 2, 8, 131), (1, 11, 13, 189),
                                       (1, 3, 1, 192), (2, 3, 6, 193), (1, 2, 7, 259)])
def test_backward_sweeps_at_the_edges_of_bands_and_tiles(s2d, Bt, Dc, H, W, dtype):
    """Rows that fill a band exactly, leave one over or fall short of one; first and last widths of the lane tilings."""
    check_bwd(s2d, wl.Workload("edge", Bt, Dc, 16, H, W, dtype, mask_frac=0.3, backward=True), seed=3)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("Bt,Dc,H,W", [(2, 3, 1, 257), (1, 5, 2, 264), (2, 2, 3, 265), (1, 3, 6, 510), (1, 2, 5, 511), (2, 2, 4, 512), (1, 2, 5, 513)])
def test_backward_of_two_column_panels_checkpointed_in_one_sweep(s2d, Bt, Dc, H, W, dtype):
    """First and last widths, rows that fill a band of two or leave one over, with and without the softplus step; 513: three panels."""
    check_bwd(s2d, wl.Workload("wide", Bt, Dc, 16, H, W, dtype, mask_frac=0.3, backward=True), seed=6)
    test_backward_with_softplus_step_matches_oracle(s2d, (Bt, Dc, 16, H, W, dtype, 0.3), True)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("H,W,N", [(1, 17, 5), (20, 20, 8), (31, 264, 16), (32, 256, 8), (33, 257, 16)])
def test_softplus_chain_rule_outside_the_sweeps(s2d, H, W, N, dtype):
    """Maps below, at and above the size from which a map gets 16 wavefronts, with 0 to 3 elements behind the last four."""
    test_backward_with_softplus_step_matches_oracle(s2d, (2, 3, N, H, W, dtype, 0.3), True)


@pytest.mark.parametrize("W", [72, 75, 190])
def test_backward_is_reproducible_and_ignores_garbage_under_the_mask(s2d, W):
    w = wl.Workload("brep", 2, 12, 16, 20, W, wl.F32, mask_frac=0.4, backward=True)
    inp = wl.make_inputs(w, seed=8)
    a = run_bwd(s2d, inp, wl.F32)
    b = run_bwd(s2d, inp, wl.F32)
    for u, v in zip(a, b):
        assert np.array_equal(u, v)
    p = wl.make_inputs(w, seed=8, poison_under_mask=np.nan)
    for u, v in zip(a, run_bwd(s2d, p, wl.F32)):
        assert np.array_equal(u, v)


def test_backward_without_skip_term(s2d):
    w = wl.Workload("bnoskip", 1, 6, 16, 12, 64, wl.F32, backward=True)
    inp = wl.make_inputs(w, seed=10)
    inp["Dskip"] = None
    got, ref = run_bwd(s2d, inp, wl.F32), oracle_bwd(inp, wl.F32)
    assert got[5] is None and ref[5] is None
    for g, r in zip(got[:5], ref[:5]):
        assert rel_err(g, r) <= 1e-4


# ====================================================================== error paths on the device

def test_workspace_too_small_and_unsupported_shapes_are_reported(s2d):
    import ctypes
    import torch
    w = wl.Workload("err", 1, 2, 4, 6, 1500, wl.F32, backward=True)       # several panels: forward needs a carry buffer
    d = s2d.to_device(wl.make_inputs(w, seed=1), wl.F32)
    desc = s2d.make_desc(d["x"], d["A"])
    need = s2d.workspace_bytes(desc, s2d.PASS_FWD)
    assert need == 1 * 2 * 4 * 6 * 4
    y = torch.full_like(d["x"], 7.0)
    small = torch.empty(16, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(s2d.Scan2dError) as e:
        s2d.scan2d_fwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], None, y=y, workspace=small)
    assert e.value.code == -5
    torch.cuda.synchronize()
    assert bool((y == 7.0).all())                                          # nothing was written
    # backward of maps wider than 1024 columns: column panels, hence a workspace for the carries too
    assert s2d.workspace_bytes(desc, s2d.PASS_BWD) > 0
    # a backward workspace that is too small
    w2 = wl.Workload("err2", 2, 8, 16, 12, 40, wl.F32, backward=True)
    d2 = s2d.to_device(wl.make_inputs(w2, seed=1), wl.F32)
    assert s2d.workspace_bytes(s2d.make_desc(d2["x"], d2["A"]), s2d.PASS_BWD) > 0
    with pytest.raises(s2d.Scan2dError) as e:
        s2d.scan2d_bwd(d2["x"], d2["delta"], d2["A"], d2["Bm"], d2["Cm"], d2["Dskip"], None, d2["dy"], workspace=small)
    assert e.value.code == -5
    # Dskip / dDskip must match: checked by the C ABI itself
    rc = s2d.lib.scan2d_bwd(ctypes.byref(s2d.make_desc(d2["x"], d2["A"])), d2["x"].data_ptr(), d2["delta"].data_ptr(),
                            d2["A"].data_ptr(), d2["Bm"].data_ptr(), d2["Cm"].data_ptr(), d2["Dskip"].data_ptr(), None,
                            d2["dy"].data_ptr(), d2["x"].data_ptr(), d2["x"].data_ptr(), d2["A"].data_ptr(),
                            d2["Bm"].data_ptr(), d2["Cm"].data_ptr(), None, None, 0, None)
    assert rc == -1


def test_runs_on_a_side_stream(s2d):
    import torch
    w = wl.Workload("stream", 1, 8, 16, 32, 64, wl.BF16, mask_frac=0.3)
    inp = wl.make_inputs(w, seed=2)
    d = s2d.to_device(inp, wl.BF16)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        y = s2d.scan2d_fwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    st.synchronize()
    ref = oracle_fwd(inp, wl.BF16)
    assert rel_err(wl.to_float(s2d.to_host(y), wl.BF16), wl.to_float(ref, wl.BF16)) <= 2e-2


# ------------------------------------------------------------------ step computed in the kernels

def _softplus_inputs(w, seed):
    """The workload's tensors with `delta` replaced by a raw projection spread over both tails of the
    softplus (its stored values are rounded to the storage type once) and a per-channel bias."""
    inp = wl.make_inputs(w, seed=seed)
    r = np.random.default_rng(500 + seed)
    raw = r.normal(-2.0, 2.5, (w.Bt, w.Dc, w.H, w.W))
    raw.reshape(-1)[:: 97] = 30.0                      # far right tail: softplus(t) = t
    raw.reshape(-1)[5:: 101] = -40.0                   # far left tail: softplus(t) = exp(t)
    raw = raw.astype(np.float32)
    inp["delta"] = wl.f32_to_bf16_bits(raw) if w.dtype == wl.BF16 else raw
    inp["delta_bias"] = r.normal(0.0, 0.5, w.Dc).astype(np.float32)
    return inp


SOFTPLUS_SHAPES = [
    (1, 6, 16, 21, 64, wl.F32, 0.3), (2, 5, 16, 14, 14, wl.BF16, 0.2), (1, 3, 16, 9, 200, wl.BF16, 0.3),
    (1, 4, 5, 7, 45, wl.F32, 0.2), (1, 3, 16, 13, 192, wl.F32, 0.0), (1, 2, 8, 5, 600, wl.F32, 0.3),
    (1, 16, 16, 64, 256, wl.BF16, 0.5), (3, 2, 4, 6, 30, wl.F32, 0.3), (1, 4, 6, 12, 16, wl.F32, 0.3),
    (1, 5, 16, 9, 57, wl.F32, 0.3), (1, 5, 16, 9, 58, wl.BF16, 0.3),   # widths off the lane and mask boundaries
    (2, 5, 16, 11, 55, wl.BF16, 0.3), (1, 3, 16, 7, 201, wl.BF16, 0.0),  # bf16 rows on odd 2-byte boundaries
]


@pytest.mark.parametrize("shape", SOFTPLUS_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
@pytest.mark.parametrize("with_bias", [True, False], ids=["bias", "nobias"])
def test_forward_with_softplus_step_matches_oracle(s2d, shape, with_bias):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("sp", Bt, Dc, N, H, W, dtype, mask_frac=mf)
    inp = _softplus_inputs(w, seed=9)
    bias = inp["delta_bias"] if with_bias else None
    print(f"softplus fwd case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype} bias={with_bias}", flush=True)
    d = s2d.to_device(inp, dtype)
    db = torch.from_numpy(bias).cuda() if with_bias else None
    y = s2d.scan2d_fwd_softplus(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    torch.cuda.synchronize()
    ref = oracle.scan2d_fwd_softplus(inp["x"], inp["delta"], bias, inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"],
                                     inp["mask"], dtype=dtype)
    got = wl.to_float(s2d.to_host(y), dtype)
    assert np.isfinite(got).all()
    assert rel_err(got, wl.to_float(ref, dtype)) <= TOL[dtype]
    # the plain entry point on the step computed by a library routine gives the same result to rounding
    if dtype == wl.F32:
        t = inp["delta"].astype(np.float64) + (0.0 if bias is None else bias[None, :, None, None])
        inp2 = dict(inp)
        inp2["delta"] = np.logaddexp(0.0, t).astype(np.float32)
        y2 = run_fwd(s2d, inp2, dtype)
        assert rel_err(got, y2) <= 1e-5


SOFTPLUS_BWD_SHAPES = [
    (2, 5, 16, 14, 14, wl.F32, 0.2), (1, 6, 16, 21, 64, wl.F32, 0.3), (2, 3, 16, 9, 128, wl.BF16, 0.3),
    (1, 9, 16, 13, 192, wl.F32, 0.3), (1, 3, 16, 6, 250, wl.F32, 0.0), (1, 2, 8, 5, 600, wl.F32, 0.3),
    (3, 2, 40, 6, 30, wl.F32, 0.3), (1, 4, 5, 9, 13, wl.BF16, 0.3),
    # softplus, chain rule and bias gradient inside the shared-producer sweeps: several bands and channels per workgroup,
    # batch items (bias partials), a ragged 12-column width; and column panels (16 states), which keep the step kernel
    (3, 20, 16, 23, 190, wl.F32, 0.3), (2, 9, 16, 11, 256, wl.BF16, 0.4), (1, 3, 16, 9, 520, wl.F32, 0.3),
]


@pytest.mark.parametrize("shape", SOFTPLUS_BWD_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
@pytest.mark.parametrize("with_bias", [True, False], ids=["bias", "nobias"])
def test_backward_with_softplus_step_matches_oracle(s2d, shape, with_bias):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("spb", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True)
    inp = _softplus_inputs(w, seed=10)
    bias = inp["delta_bias"] if with_bias else None
    print(f"softplus bwd case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype} bias={with_bias}", flush=True)
    d = s2d.to_device(inp, dtype)
    db = torch.from_numpy(bias).cuda() if with_bias else None
    got = s2d.scan2d_bwd_softplus(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"])
    torch.cuda.synchronize()
    ref = oracle.scan2d_bwd_softplus(inp["x"], inp["delta"], bias, inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"],
                                     inp["mask"], inp["dy"], dtype=dtype)
    names = ("dx", "ddelta_raw", "ddelta_bias", "dA", "dBm", "dCm", "dDskip")
    for k, (name, g, r) in enumerate(zip(names, got, ref)):
        if r is None:
            assert g is None, name
            continue
        g = s2d.to_host(g)
        gv = wl.to_float(g, dtype) if k < 2 else g.astype(np.float64)
        rv = wl.to_float(r, dtype) if k < 2 else r.astype(np.float64)
        assert np.isfinite(gv).all(), name
        tol = TOL[dtype] if k < 2 else (1e-4 if dtype == wl.F32 else 2e-2)
        assert rel_err(gv, rv) <= tol, f"{name}: rel err {rel_err(gv, rv):.3e}"
    # every other gradient is that of the plain entry point on the step a library routine computes
    if dtype == wl.F32:
        t = inp["delta"].astype(np.float64) + (0.0 if bias is None else bias[None, :, None, None])
        inp2 = dict(inp)
        inp2["delta"] = np.logaddexp(0.0, t).astype(np.float32)
        plain = run_bwd(s2d, inp2, dtype)
        for k, j in ((0, 0), (3, 2), (4, 3), (5, 4), (6, 5)):
            assert rel_err(s2d.to_host(got[k]).astype(np.float64), plain[j].astype(np.float64)) <= 2e-5, names[k]


@pytest.mark.parametrize("gated", [False, True], ids=["softplus", "gated"])
@pytest.mark.parametrize("Dc,H,W", [(2, 9, 14), (4, 10, 56), (32, 9, 121), (3, 7, 190), (3, 6, 256), (2, 9, 300), (2, 5, 600)])
def test_softplus_derivative_of_small_steps(s2d, Dc, H, W, gated):
    """The derivative of the softplus where the step is small (raw projections around -4 to -8), element by element.  With every
    decay exp(-1e6 * step) = 0 (steps of 2e-4 and more) the gradient of the step is x * dy * sum_n B C, so that of the raw
    projection is known in 64 bits.
    Bound: the positive 16-term sums, their factors and x, at most 24 roundings of 2^-24; the exponential's argument, up to 16
    after the change of base, is rounded to 2^-21 (3.3e-7), the exponential, the sum and the reciprocal to an ulp or two
    each (4e-7)."""
    import torch
    r = np.random.default_rng(17)
    N, shape, states = 16, (1, Dc, H, W), (1, 16, H, W)
    pos = lambda s: r.uniform(0.5, 2.0, s).astype(np.float32)
    x, dy, Bm, Cm = pos(shape), pos(shape), pos(states), pos(states)
    raw = r.uniform(-8.0, -3.0, shape).astype(np.float32)
    bias = r.uniform(-0.5, 0.5, Dc).astype(np.float32)
    A, skip = np.full((Dc, N), -1e6, np.float32), np.zeros(Dc, np.float32)
    a = [torch.from_numpy(v).cuda() for v in (x, raw, bias, A, Bm, Cm, skip)]
    t = (raw + bias[None, :, None, None]).astype(np.float64)                # one fp32 sum, as in the kernels
    want = x.astype(np.float64) * dy * (Bm.astype(np.float64) * Cm).sum(1, keepdims=True) / (1.0 + np.exp(-t))
    if gated:                                                              # z = 32: SiLU(z) = 32 to the last bit
        z = torch.full(shape, 32.0, device="cuda:0")
        got = s2d.scan2d_bwd_softplus_gated(*a, None, z, z, torch.from_numpy(dy).cuda())
        want *= 32.0
    else:
        got = s2d.scan2d_bwd_softplus(*a, None, torch.from_numpy(dy).cuda())
    bound = 24 * 2.0 ** -24 + 3.3e-7 + 4e-7
    err = np.abs(s2d.to_host(got[1]).astype(np.float64) - want) / want
    assert err.max() <= bound, f"ddelta_raw: {err.max():.2e}"
    sums = want.sum((0, 2, 3))
    assert (np.abs(s2d.to_host(got[2]).astype(np.float64) - sums) / sums).max() <= bound + H * W * 2.0 ** -24


# ------------------------------------------------------------------ output gate of the block

def _gated_inputs(w, seed):
    """The softplus inputs plus a gate branch z spread over both tails of SiLU."""
    inp = _softplus_inputs(w, seed)
    r = np.random.default_rng(700 + seed)
    z = r.normal(0.0, 2.0, (w.Bt, w.Dc, w.H, w.W))
    z.reshape(-1)[3:: 89] = 25.0                       # SiLU(z) = z
    z.reshape(-1)[7:: 103] = -30.0                     # SiLU(z) = z exp(z)
    z.reshape(-1)[11:: 107] = 0.0
    z = z.astype(np.float32)
    inp["z"] = wl.f32_to_bf16_bits(z) if w.dtype == wl.BF16 else z
    return inp


GATED_SHAPES = [
    (1, 6, 16, 21, 64, wl.F32, 0.3),       # one lane group per state, 16-lane groups
    (2, 5, 16, 14, 14, wl.BF16, 0.2),      # narrow-map kernel
    (1, 3, 16, 9, 200, wl.BF16, 0.3),      # wave-wide lane groups
    (1, 4, 5, 7, 45, wl.F32, 0.2),         # ragged last lane group, mask rows off 4-byte boundaries
    (1, 3, 16, 13, 192, wl.F32, 0.0),
    (1, 2, 8, 5, 600, wl.F32, 0.3),        # wider than one panel
    (1, 3, 16, 9, 400, wl.BF16, 0.3),      # wave-wide groups with 8 columns per lane, gate inside the kernel
    (1, 16, 16, 64, 256, wl.BF16, 0.5),    # one map per workgroup, 4 rows per barrier
    (3, 2, 4, 6, 30, wl.F32, 0.3),
    (2, 3, 64, 11, 40, wl.F32, 0.3),       # all states in one lane: the lane that owns the columns applies the gate
    (1, 3, 64, 7, 57, wl.BF16, 0.3),
    (1, 2, 2, 10, 100, wl.F32, 0.3),       # fewer lane groups than columns per lane: several columns per summing thread
    (1, 5, 16, 9, 58, wl.BF16, 0.3),
    (4, 3, 16, 23, 28, wl.F32, 0.3),
]


@pytest.mark.parametrize("shape", GATED_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_gated_forward_matches_oracle(s2d, shape):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("gate", Bt, Dc, N, H, W, dtype, mask_frac=mf)
    inp = _gated_inputs(w, seed=13)
    print(f"gated fwd case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype}", flush=True)
    d = s2d.to_device(inp, dtype)
    db = torch.from_numpy(inp["delta_bias"]).cuda()
    ys, y = s2d.scan2d_fwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"])
    _, y_only = s2d.scan2d_fwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"],
                                              want_y_scan=False)
    plain = s2d.scan2d_fwd_softplus(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    torch.cuda.synchronize()
    rys, ry = oracle.scan2d_fwd_softplus_gated(inp["x"], inp["delta"], inp["delta_bias"], inp["A"], inp["Bm"], inp["Cm"],
                                               inp["Dskip"], inp["mask"], inp["z"], dtype=dtype)
    gy, gys = wl.to_float(s2d.to_host(y), dtype), wl.to_float(s2d.to_host(ys), dtype)
    assert np.isfinite(gy).all() and np.isfinite(gys).all()
    assert rel_err(gys, wl.to_float(rys, dtype)) <= TOL[dtype]
    assert rel_err(gy, wl.to_float(ry, dtype)) <= TOL[dtype]
    # the ungated output is bit for bit that of the ungated entry point; leaving it out changes nothing
    assert np.array_equal(s2d.to_host(ys), s2d.to_host(plain))
    assert np.array_equal(s2d.to_host(y), s2d.to_host(y_only))
    # z = 0 closes the gate exactly
    zero = torch.zeros_like(d["z"])
    _, y0 = s2d.scan2d_fwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], zero)
    assert not wl.to_float(s2d.to_host(y0), dtype).any()


GATED_BWD_SHAPES = [
    (2, 5, 16, 14, 14, wl.F32, 0.2), (1, 6, 16, 21, 64, wl.F32, 0.3), (2, 3, 16, 9, 128, wl.BF16, 0.3),
    (1, 9, 16, 13, 190, wl.F32, 0.3), (1, 3, 16, 6, 251, wl.F32, 0.0), (3, 2, 40, 6, 30, wl.F32, 0.3),
    (1, 4, 5, 9, 13, wl.BF16, 0.3), (1, 1, 16, 3, 5, wl.F32, 0.0),
    # the gate's backward inside the shared-producer sweeps: 12-column and wave-wide tilings, several bands, batch items;
    # and column panels, which keep the element-wise gate kernel
    (2, 11, 16, 22, 192, wl.F32, 0.3), (2, 5, 16, 9, 250, wl.BF16, 0.3), (1, 3, 16, 7, 400, wl.F32, 0.2),
]


@pytest.mark.parametrize("shape", GATED_BWD_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_gated_backward_matches_oracle(s2d, shape):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("gateb", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True)
    inp = _gated_inputs(w, seed=14)
    print(f"gated bwd case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype}", flush=True)
    d = s2d.to_device(inp, dtype)
    db = torch.from_numpy(inp["delta_bias"]).cuda()
    ys, _ = s2d.scan2d_fwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"])
    got = s2d.scan2d_bwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"], ys, d["dy"])
    torch.cuda.synchronize()
    ref = oracle.scan2d_bwd_softplus_gated(inp["x"], inp["delta"], inp["delta_bias"], inp["A"], inp["Bm"], inp["Cm"],
                                           inp["Dskip"], inp["mask"], inp["z"], inp["dy"], dtype=dtype)
    names = ("dx", "ddelta_raw", "ddelta_bias", "dA", "dBm", "dCm", "dDskip", "dz")
    for k, (name, g, r) in enumerate(zip(names, got, ref)):
        g = s2d.to_host(g)
        stored = k < 2 or k == 7
        gv = wl.to_float(g, dtype) if stored else g.astype(np.float64)
        rv = wl.to_float(r, dtype) if stored else r.astype(np.float64)
        assert np.isfinite(gv).all(), name
        tol = TOL[dtype] if stored else (1e-4 if dtype == wl.F32 else 2e-2)
        assert rel_err(gv, rv) <= tol, f"{name}: rel err {rel_err(gv, rv):.3e}"


def test_gated_backward_reports_a_short_workspace(s2d):
    import torch
    w = wl.Workload("gatews", 1, 4, 16, 20, 40, wl.F32, mask_frac=0.2, backward=True)
    inp = _gated_inputs(w, seed=15)
    d = s2d.to_device(inp, wl.F32)
    desc = s2d.make_desc(d["x"], d["A"])
    plain, gated = s2d.workspace_bytes(desc, s2d.PASS_BWD_SOFTPLUS), s2d.workspace_bytes(desc, s2d.PASS_BWD_GATED)
    assert gated >= plain + d["x"].numel() * 4
    ws = torch.empty(plain, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(s2d.Scan2dError) as e:
        s2d.scan2d_bwd_softplus_gated(d["x"], d["delta"], None, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"],
                                      d["x"], d["dy"], workspace=ws)
    assert e.value.code == -5


# ------------------------------------------------------------------ identity cells (skip mask mode)

SKIP_SHAPES = [
    (2, 5, 16, 21, 64, wl.F32, 0.4), (2, 5, 16, 14, 14, wl.BF16, 0.3), (1, 3, 16, 9, 200, wl.BF16, 0.5),
    (1, 4, 5, 7, 45, wl.F32, 0.3), (1, 3, 16, 13, 190, wl.F32, 0.3), (1, 2, 8, 5, 600, wl.F32, 0.3),
    (1, 4, 40, 6, 30, wl.F32, 0.3), (1, 3, 16, 9, 57, wl.BF16, 0.6), (3, 2, 4, 16, 16, wl.F32, 0.3),
]


@pytest.mark.parametrize("shape", SKIP_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_identity_cells_forward_and_backward_match_oracle(s2d, shape):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("skip", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True)
    inp = wl.make_inputs(w, seed=21, poison_under_mask=np.nan)      # nothing stored under the mask may matter
    print(f"identity cells case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype}", flush=True)
    d = s2d.to_device(inp, dtype)
    args = (d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    y = s2d.scan2d_fwd(*args, flags=s2d.FLAG_IDENTITY_CELLS)
    y_plain = s2d.scan2d_fwd(*args)
    torch.cuda.synchronize()
    clean = wl.make_inputs(w, seed=21)
    ref = oracle.scan2d_fwd_skip(clean["x"], clean["delta"], clean["A"], clean["Bm"], clean["Cm"], clean["Dskip"], clean["mask"], dtype=dtype)
    got = wl.to_float(s2d.to_host(y), dtype)
    assert np.isfinite(got).all()
    assert rel_err(got, wl.to_float(ref, dtype)) <= TOL[dtype]
    assert not np.array_equal(s2d.to_host(y), s2d.to_host(y_plain))         # the mode does change the result
    if True:
        grads = s2d.scan2d_bwd(*args, d["dy"], flags=s2d.FLAG_IDENTITY_CELLS)
        torch.cuda.synchronize()
        refs = oracle.scan2d_bwd_skip(clean["x"], clean["delta"], clean["A"], clean["Bm"], clean["Cm"], clean["Dskip"],
                                      clean["mask"], clean["dy"], dtype=dtype)
        m4 = np.broadcast_to(clean["mask"][:, None] != 0, got.shape)
        for k, (name, g, r) in enumerate(zip(GRADS, grads, refs)):
            g = s2d.to_host(g)
            gv = wl.to_float(g, dtype) if k < 2 else g.astype(np.float64)
            rv = wl.to_float(r, dtype) if k < 2 else r.astype(np.float64)
            assert np.isfinite(gv).all(), name
            tol = TOL[dtype] if k < 2 else (1e-4 if dtype == wl.F32 else 2e-2)
            assert rel_err(gv, rv) <= tol, f"{name}: rel err {rel_err(gv, rv):.3e}"
            if k < 2:
                assert not gv[m4].any(), name                                # dx and ddelta are exactly 0 under the mask


def test_identity_cells_with_softplus_step(s2d):
    import torch
    w = wl.Workload("skipsp", 2, 6, 16, 18, 75, wl.F32, mask_frac=0.4, backward=True)
    inp = _softplus_inputs(w, seed=22)
    d = s2d.to_device(inp, wl.F32)
    db = torch.from_numpy(inp["delta_bias"]).cuda()
    y = s2d.scan2d_fwd_softplus(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], flags=s2d.FLAG_IDENTITY_CELLS)
    g = s2d.scan2d_bwd_softplus(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"], flags=s2d.FLAG_IDENTITY_CELLS)
    torch.cuda.synchronize()
    step = np.logaddexp(0.0, inp["delta"].astype(np.float64) + inp["delta_bias"][None, :, None, None])
    ref = oracle.scan2d_fwd_skip(inp["x"].astype(np.float64), step, inp["A"], inp["Bm"].astype(np.float64), inp["Cm"].astype(np.float64),
                                 inp["Dskip"], inp["mask"], dtype=oracle.F64)
    assert rel_err(s2d.to_host(y), ref) <= 1e-4
    m4 = np.broadcast_to(inp["mask"][:, None] != 0, ref.shape)
    assert not s2d.to_host(g[1])[m4].any()                                   # ddelta_raw under the mask
    refs = oracle.scan2d_bwd_skip(inp["x"].astype(np.float64), step, inp["A"], inp["Bm"].astype(np.float64), inp["Cm"].astype(np.float64),
                                  inp["Dskip"], inp["mask"], inp["dy"].astype(np.float64), dtype=oracle.F64)
    from scipy.special import expit
    t = inp["delta"].astype(np.float64) + inp["delta_bias"][None, :, None, None]
    assert rel_err(s2d.to_host(g[0]), refs[0]) <= 1e-4
    assert rel_err(s2d.to_host(g[1]), refs[1] * expit(t)) <= 1e-4
    assert rel_err(s2d.to_host(g[3]), refs[2]) <= 1e-4


# ------------------------------------------------------------------ columns first (scan order ablation)

CF_SHAPES = [
    (2, 5, 16, 21, 64, wl.F32, 0.3), (2, 5, 16, 14, 9, wl.BF16, 0.3), (1, 3, 16, 70, 33, wl.BF16, 0.4),
    (1, 4, 5, 45, 7, wl.F32, 0.0), (1, 3, 16, 130, 190, wl.F32, 0.3), (3, 2, 4, 1, 50, wl.F32, 0.3), (1, 2, 8, 37, 1, wl.F32, 0.3),
    # in-kernel form: wave-wide forward tiling on odd bf16 rows with the ragged 12-column backward, 32 and 64 states,
    # several maps per workgroup, a width whose backward needs column panels (transposed form; the forward stays in-kernel)
    (1, 2, 16, 33, 191, wl.BF16, 0.3), (2, 3, 16, 37, 50, wl.F32, 0.5), (1, 2, 32, 20, 40, wl.F32, 0.3), (1, 2, 64, 9, 30, wl.BF16, 0.3),
    (3, 7, 16, 56, 56, wl.BF16, 0.2), (1, 2, 16, 12, 300, wl.F32, 0.3),
    # the tilings of 8 and of 12 columns per lane, whose rows are scanned one by one: whole and ragged
    (2, 3, 16, 9, 104, wl.F32, 0.3), (1, 3, 16, 13, 121, wl.BF16, 0.3), (1, 5, 16, 10, 192, wl.BF16, 0.3), (2, 3, 16, 11, 147, wl.F32, 0.2),
]


@pytest.mark.parametrize("shape", CF_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_columns_first_forward_and_backward_match_oracle(s2d, shape):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("cf", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True)
    inp = wl.make_inputs(w, seed=31)
    print(f"columns first case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype}", flush=True)
    d = s2d.to_device(inp, dtype)
    args = (d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    y = s2d.scan2d_fwd(*args, flags=s2d.FLAG_COLUMNS_FIRST)
    torch.cuda.synchronize()
    ref = oracle.scan2d_fwd_columns_first(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"], dtype=dtype)
    got = wl.to_float(s2d.to_host(y), dtype)
    assert np.isfinite(got).all()
    assert rel_err(got, wl.to_float(ref, dtype)) <= TOL[dtype]
    grads = s2d.scan2d_bwd(*args, d["dy"], flags=s2d.FLAG_COLUMNS_FIRST)
    torch.cuda.synchronize()
    refs = oracle.scan2d_bwd_columns_first(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"],
                                           inp["dy"], dtype=dtype)
    for k, (name, g, r) in enumerate(zip(GRADS, grads, refs)):
        if r is None:
            assert g is None
            continue
        g = s2d.to_host(g)
        gv = wl.to_float(g, dtype) if k < 2 else g.astype(np.float64)
        rv = wl.to_float(r, dtype) if k < 2 else r.astype(np.float64)
        assert np.isfinite(gv).all(), name
        tol = TOL[dtype] if k < 2 else (1e-4 if dtype == wl.F32 else 2e-2)
        assert rel_err(gv, rv) <= tol, f"{name}: rel err {rel_err(gv, rv):.3e}"


@pytest.mark.parametrize("H,W", [(9, 37), (9, 104), (13, 121), (10, 192), (11, 147)])
def test_columns_first_backward_with_softplus_step_is_the_transposed_one(s2d, H, W):
    import torch
    inp = wl.make_inputs(wl.Workload("cfsp", 2, 3, 16, H, W, wl.F32, mask_frac=0.3, backward=True), seed=33)
    d = s2d.to_device(inp, wl.F32)
    bias = torch.linspace(-0.2, 0.2, 3, device="cuda:0")
    tr = lambda t: t.transpose(-1, -2).contiguous()
    got = s2d.scan2d_bwd_softplus(d["x"], d["delta"], bias, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"], flags=s2d.FLAG_COLUMNS_FIRST)
    want = s2d.scan2d_bwd_softplus(tr(d["x"]), tr(d["delta"]), bias, d["A"], tr(d["Bm"]), tr(d["Cm"]), d["Dskip"], tr(d["mask"]), tr(d["dy"]))
    for name, g, w in zip(("dx", "ddelta", "dbias", "dA", "dBm", "dCm", "dDskip"), got, want):
        w = tr(w) if w.dim() == 4 else w
        assert rel_err(s2d.to_host(g), s2d.to_host(w)) <= 1e-4, name           # two orders of fp32 sums


def test_columns_first_with_identity_cells_softplus_and_gate(s2d):
    """All the options at once against the oracle's compositions: columns first = the transposed problem."""
    import torch
    w = wl.Workload("cfall", 2, 4, 16, 19, 42, wl.F32, mask_frac=0.4, backward=True)
    inp = _gated_inputs(w, seed=32)
    d = s2d.to_device(inp, wl.F32)
    db = torch.from_numpy(inp["delta_bias"]).cuda()
    fl = s2d.FLAG_COLUMNS_FIRST | s2d.FLAG_IDENTITY_CELLS
    ys, y = s2d.scan2d_fwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"], flags=fl)
    g = s2d.scan2d_bwd_softplus_gated(d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["z"], ys, d["dy"], flags=fl)
    torch.cuda.synchronize()
    tr = lambda a: None if a is None else np.ascontiguousarray(np.swapaxes(a, -1, -2))
    m4 = np.broadcast_to(inp["mask"][:, None] != 0, inp["x"].shape)
    raw = inp["delta"].astype(np.float64).copy()
    step = np.logaddexp(0.0, raw + inp["delta_bias"][None, :, None, None])
    step[m4] = 0.0
    f64 = lambda a: a.astype(np.float64)
    y_scan = tr(oracle.scan2d_fwd(tr(f64(inp["x"])), tr(step), inp["A"], tr(f64(inp["Bm"])), tr(f64(inp["Cm"])), inp["Dskip"], tr(inp["mask"]),
                                  dtype=oracle.F64))
    z = f64(inp["z"])
    sg = 1.0 / (1.0 + np.exp(-z))
    assert rel_err(s2d.to_host(ys), y_scan) <= 1e-4
    assert rel_err(s2d.to_host(y), y_scan * z * sg) <= 1e-4
    dyg = f64(inp["dy"]) * z * sg
    refs = oracle.scan2d_bwd(tr(f64(inp["x"])), tr(step), inp["A"], tr(f64(inp["Bm"])), tr(f64(inp["Cm"])), inp["Dskip"], tr(inp["mask"]),
                             tr(dyg), dtype=oracle.F64)
    from scipy.special import expit
    draw = tr(refs[1]) * expit(raw + inp["delta_bias"][None, :, None, None])
    draw[m4] = 0.0
    assert rel_err(s2d.to_host(g[0]), tr(refs[0])) <= 1e-4                   # dx
    assert rel_err(s2d.to_host(g[1]), draw) <= 1e-4                          # ddelta_raw
    assert not s2d.to_host(g[1])[m4].any()
    assert rel_err(s2d.to_host(g[2]), draw.sum(axis=(0, 2, 3))) <= 1e-4      # ddelta_bias
    assert rel_err(s2d.to_host(g[3]), refs[2]) <= 1e-4                       # dA
    assert rel_err(s2d.to_host(g[4]), tr(refs[3])) <= 1e-4                   # dBm
    assert rel_err(s2d.to_host(g[5]), tr(refs[4])) <= 1e-4                   # dCm
    assert rel_err(s2d.to_host(g[7]), f64(inp["dy"]) * y_scan * sg * (1.0 + z * (1.0 - sg))) <= 1e-4   # dz


@pytest.mark.parametrize("shape", [(2, 12, 16, 40, 96, wl.F32), (1, 4, 16, 24, 256, wl.BF16), (1, 16, 16, 24, 190, wl.F32)],
                         ids=["40x96-f32", "24x256-bf16-large-lds-fwd", "24x190-f32-large-lds-bwd"])
def test_forward_and_backward_replay_from_a_hip_graph(s2d, shape):
    """The library only enqueues kernels on the caller's stream (no allocation, no memset, no
    synchronisation), so its calls can be captured; every replay must equal the eager result bit for
    bit, also after the inputs changed and eager work ran in between.  The second shape takes kernels that
    need more than 64 KB of dynamic LDS (the attribute is raised once per kernel, outside the capture)."""
    import torch
    Bt, Dc, N, H, W, dtype = shape
    w = wl.Workload("graph", Bt, Dc, N, H, W, dtype, mask_frac=0.3, backward=True)
    sets = [wl.make_inputs(w, seed=k) for k in (11, 12)]
    static = s2d.to_device(sets[0], dtype)
    desc = s2d.make_desc(static["x"], static["A"])
    lds = lambda which: int(s2d.describe_plan(desc, which).split(" lds=")[1].split()[0])
    if W == 256:
        assert lds(s2d.PASS_FWD) > 65536
    if W == 190:
        assert lds(s2d.PASS_BWD) > 65536
    y = torch.empty_like(static["x"])
    ws_f = torch.empty(max(16, s2d.workspace_bytes(desc, s2d.PASS_FWD)), dtype=torch.uint8, device="cuda:0")
    ws_b = torch.empty(max(16, s2d.workspace_bytes(desc, s2d.PASS_BWD)), dtype=torch.uint8, device="cuda:0")
    args = [static[k] for k in ("x", "delta", "A", "Bm", "Cm", "Dskip", "mask")]

    def eager():
        yy = s2d.scan2d_fwd(*args, workspace=ws_f)
        gg = s2d.scan2d_bwd(*args, static["dy"], workspace=ws_b)
        torch.cuda.synchronize()
        return [s2d.to_host(yy)] + [s2d.to_host(t) for t in gg]

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                       # warm-up outside the capture
        s2d.scan2d_fwd(*args, y=y, workspace=ws_f)
        s2d.scan2d_bwd(*args, static["dy"], workspace=ws_b)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s2d.scan2d_fwd(*args, y=y, workspace=ws_f)
        grads = s2d.scan2d_bwd(*args, static["dy"], workspace=ws_b)
    for k in (0, 1, 0):
        new = s2d.to_device(sets[k], dtype)
        for name in ("x", "delta", "A", "Bm", "Cm", "Dskip", "mask", "dy"):
            static[name].copy_(new[name])
        y.fill_(float("nan"))
        for t in grads:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [s2d.to_host(y)] + [s2d.to_host(t) for t in grads]
        ref = eager()                                   # eager work between the replays
        for a, b in zip(got, ref):
            assert np.array_equal(a, b)
    yo = oracle_fwd(sets[0], dtype)
    assert rel_err(wl.to_float(got[0], dtype), wl.to_float(yo, dtype)) <= TOL[dtype]


# ------------------------------------------------------------------ shapes nobody chose by hand

def _random_shape(seed, backward):
    r = np.random.default_rng(1000 + seed)
    N = int(r.choice([1, 2, 3, 4, 5, 8, 12, 16, 16, 16, 17, 24, 32, 64]))
    W = int(r.choice([r.integers(1, 17), r.integers(17, 65), r.integers(65, 257), r.integers(257, 700)]))
    H = int(r.integers(1, 24))
    Bt, Dc = int(r.integers(1, 4)), int(r.integers(1, 10))
    dtype = int(r.integers(0, 2))
    mf = float(r.choice([0.0, 0.3]))
    return Bt, Dc, N, H, W, dtype, mf


@pytest.mark.parametrize("seed", range(24))
def test_forward_random_shapes(s2d, seed):
    Bt, Dc, N, H, W, dtype, mf = _random_shape(seed, False)
    check_fwd(s2d, wl.Workload(f"rand{seed}", Bt, Dc, N, H, W, dtype, mask_frac=mf), seed=seed)


@pytest.mark.parametrize("seed", range(24))
def test_backward_random_shapes(s2d, seed):
    Bt, Dc, N, H, W, dtype, mf = _random_shape(seed, True)
    check_bwd(s2d, wl.Workload(f"brand{seed}", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True), seed=seed)


# ------------------------------------------------------------------ the ablated variants: padding token, own vertical decay

def _variant_inputs(w, seed):
    inp = wl.make_inputs(w, seed=seed)
    r = np.random.default_rng(seed + 100)
    inp["A_v"] = (-np.exp(r.normal(0.3, 0.5, (w.Dc, w.N)))).astype(np.float32)
    inp["pad"] = r.standard_normal(w.Dc).astype(np.float32)
    return inp


VARIANT_SHAPES = [(2, 5, 16, 13, 70, wl.F32, 0.3), (1, 7, 16, 9, 57, wl.BF16, 0.4), (1, 3, 5, 6, 300, wl.F32, 0.3),
                  (2, 3, 24, 5, 130, wl.BF16, 0.2), (1, 4, 16, 14, 14, wl.F32, 0.3), (1, 2, 16, 3, 520, wl.BF16, 0.3)]


@pytest.mark.parametrize("use_av,use_pad", [(True, True), (True, False), (False, True), (False, False)], ids=["av+pad", "av", "pad", "plain"])
@pytest.mark.parametrize("shape", VARIANT_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_padding_token_and_independent_vertical_decay_match_the_oracle(s2d, shape, use_av, use_pad):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("variants", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True)
    inp = _variant_inputs(w, seed=31)
    print(f"variants case Bt={Bt} Dc={Dc} N={N} H={H} W={W} dtype={dtype} A_v={use_av} pad={use_pad}", flush=True)
    d = s2d.to_device(inp, dtype)
    A_v = torch.from_numpy(inp["A_v"]).cuda() if use_av else None
    pad = torch.from_numpy(inp["pad"]).cuda() if use_pad else None
    oa, op = (inp["A_v"] if use_av else None), (inp["pad"] if use_pad else None)
    y = s2d.scan2d_fwd_variants(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], A_v=A_v, pad=pad)
    grads = s2d.scan2d_bwd_variants(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"], A_v=A_v, pad=pad)
    torch.cuda.synchronize()
    ry = oracle.scan2d_fwd_variants(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"], A_v=oa, pad=op, dtype=dtype)
    rg = oracle.scan2d_bwd_variants(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"], inp["dy"],
                                    A_v=oa, pad=op, dtype=dtype)
    assert rel_err(wl.to_float(s2d.to_host(y), dtype), wl.to_float(ry, dtype)) <= TOL[dtype]
    names = ("dx", "ddelta", "dA", "dA_v", "dBm", "dCm", "dDskip", "dpad")
    for k, (name, g, r) in enumerate(zip(names, grads, rg)):
        if r is None:
            assert g is None, name
            continue
        g = s2d.to_host(g)
        gv = wl.to_float(g, dtype) if k < 2 else g.astype(np.float64)
        rv = wl.to_float(r, dtype) if k < 2 else r.astype(np.float64)
        assert np.isfinite(gv).all(), name
        tol = TOL[dtype] if k < 2 else (1e-4 if dtype == wl.F32 else 2e-2)
        assert rel_err(gv, rv) <= tol, f"{name}: rel err {rel_err(gv, rv):.3e}"
    m = np.broadcast_to(inp["mask"][:, None] != 0, grads[0].shape)          # dx under the mask is exactly +0
    assert not s2d.to_host(grads[0]).view(np.uint32 if dtype == wl.F32 else np.uint16)[m].any()
    if not use_av and not use_pad:            # no variant: bit for bit the plain entry points
        assert np.array_equal(s2d.to_host(y), run_fwd(s2d, inp, dtype))
        for g, r in zip((grads[0], grads[1], grads[2], grads[4], grads[5], grads[6]), run_bwd(s2d, inp, dtype)):
            assert np.array_equal(s2d.to_host(g), r)


def test_variants_reject_flags_and_mismatched_gradient_pointers(s2d):
    import ctypes
    import torch
    w = wl.Workload("verr", 1, 4, 16, 8, 40, wl.F32, mask_frac=0.3, backward=True)
    inp = _variant_inputs(w, seed=3)
    d = s2d.to_device(inp, wl.F32)
    desc = s2d.make_desc(d["x"], d["A"], s2d.FLAG_IDENTITY_CELLS)
    y = torch.full_like(d["x"], 7.0)
    ws = torch.empty(max(16, s2d.workspace_bytes(s2d.make_desc(d["x"], d["A"]), s2d.PASS_BWD_VARIANTS)), dtype=torch.uint8, device="cuda:0")
    p = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())
    v = s2d.Variants(None, p(torch.from_numpy(inp["pad"]).cuda()), None, None)
    rc = s2d.lib.scan2d_fwd_variants(ctypes.byref(desc), p(d["x"]), p(d["delta"]), p(d["A"]), p(d["Bm"]), p(d["Cm"]), p(d["Dskip"]),
                                     p(d["mask"]), ctypes.byref(v), p(y), p(ws), ws.numel(), None)
    assert rc == -4                                           # flags do not combine with the variants
    desc = s2d.make_desc(d["x"], d["A"])
    outs = [torch.empty_like(d["x"]), torch.empty_like(d["x"]), torch.empty_like(d["A"]),
            torch.empty(d["Bm"].shape, device="cuda:0"), torch.empty(d["Bm"].shape, device="cuda:0"), torch.empty_like(d["Dskip"])]
    rc = s2d.lib.scan2d_bwd_variants(ctypes.byref(desc), p(d["x"]), p(d["delta"]), p(d["A"]), p(d["Bm"]), p(d["Cm"]), p(d["Dskip"]),
                                     p(d["mask"]), ctypes.byref(v), p(d["dy"]), *[p(t) for t in outs], p(ws), ws.numel(), None)
    assert rc == -1                                           # pad without dpad
    torch.cuda.synchronize()
    assert bool((y == 7.0).all())


# ------------------------------------------------------------------ tensors beyond 2^32 bytes

def test_maps_beyond_the_32_bit_byte_range_land_at_their_own_index(s2d):
    """x, step, y (and dy, dx, ddelta) of 4.4 GB each: the maps that straddle the 2^31- and 2^32-byte offsets, the
    first and the last map are checked against the oracle.  The maps are eight random ones repeated with a per-map
    scale, made on the GPU; the oracle gets the bits of the maps it checks."""
    import torch
    Dc, N, H, W = 4400, 4, 500, 500
    HW = H * W
    assert Dc * HW * 4 > 2 ** 32
    w8 = wl.Workload("big8", 1, 8, N, H, W, wl.F32, mask_frac=0.3, backward=True)
    inp = wl.make_inputs(w8, seed=41)
    dev = "cuda:0"
    scale = (1.0 + torch.arange(Dc, device=dev, dtype=torch.float32) / 8192.0)[None, :, None, None]
    rep = lambda a: torch.from_numpy(a).to(dev).repeat(1, Dc // 8, 1, 1)
    x, dy = rep(inp["x"]) * scale, rep(inp["dy"]) * scale
    delta = rep(inp["delta"])
    A = torch.from_numpy(np.tile(inp["A"], (Dc // 8, 1))).to(dev)
    Dskip = torch.from_numpy(np.tile(inp["Dskip"], Dc // 8)).to(dev)
    Bm, Cm, mask = (torch.from_numpy(inp[k]).to(dev) for k in ("Bm", "Cm", "mask"))
    print(f"large-offset case Dc={Dc} N={N} H={H} W={W}: {x.numel() * 4 / 2**30:.2f} GiB per tensor", flush=True)
    y = s2d.scan2d_fwd(x, delta, A, Bm, Cm, Dskip, mask)
    torch.cuda.synchronize()
    picks = sorted({0, 2 ** 31 // (HW * 4), 2 ** 31 // (HW * 4) + 1, 2 ** 32 // (HW * 4), 2 ** 32 // (HW * 4) + 1, Dc - 1})
    sub = lambda t: np.ascontiguousarray(t[:, picks].cpu().numpy())
    hA, hD = A[picks].cpu().numpy(), Dskip[picks].cpu().numpy()
    ref = oracle.scan2d_fwd(sub(x), sub(delta), hA, inp["Bm"], inp["Cm"], hD, inp["mask"], dtype=wl.F32)
    assert rel_err(sub(y), ref) <= 1e-4
    # every other map: y of map m is that of map m % 8 computed with its own scale (linear in x), within rounding
    probe = [7, 1234, 2146, 3333, 4295, 4398]
    ref8 = oracle.scan2d_fwd(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"], dtype=wl.F32)
    for m in probe:
        assert rel_err(y[0, m].cpu().numpy(), ref8[0, m % 8].astype(np.float64) * (1.0 + m / 8192.0)) <= 1e-4, m
    del y
    dx, ddelta, dA, dBm, dCm, dD = s2d.scan2d_bwd(x, delta, A, Bm, Cm, Dskip, mask, dy)
    torch.cuda.synchronize()
    rg = oracle.scan2d_bwd(sub(x), sub(delta), hA, inp["Bm"], inp["Cm"], hD, inp["mask"], sub(dy), dtype=wl.F32)
    assert rel_err(sub(dx), rg[0]) <= 1e-4
    assert rel_err(sub(ddelta), rg[1]) <= 1e-4
    assert rel_err(dA[picks].cpu().numpy(), rg[2]) <= 1e-4
    assert rel_err(dD[picks].cpu().numpy(), rg[5]) <= 1e-4
    assert bool(torch.isfinite(dBm).all()) and bool(torch.isfinite(dCm).all())


# ------------------------------------------------------------------ training pair: the forward leaves the band checkpoints

PAIR_SHAPES = [
    (2, 5, 16, 37, 50, wl.F32, 0.3), (1, 3, 16, 130, 190, wl.F32, 0.3), (2, 4, 16, 23, 101, wl.BF16, 0.4), (1, 6, 16, 56, 56, wl.BF16, 0.0),
    (1, 2, 16, 9, 128, wl.F32, 0.2),
    # no saving forward for these (8 states; 256 columns; one band; small maps): the pair is scan2d_fwd / scan2d_bwd
    (1, 3, 8, 20, 40, wl.F32, 0.3), (1, 2, 16, 12, 256, wl.BF16, 0.3), (1, 2, 16, 3, 40, wl.F32, 0.0), (2, 3, 16, 14, 14, wl.F32, 0.0),
]


@pytest.mark.parametrize("shape", PAIR_SHAPES, ids=lambda s: "x".join(map(str, s[:5])) + ("bf16" if s[5] else "f32"))
def test_training_pair_matches_oracle_and_the_plain_backward(s2d, shape):
    import torch
    Bt, Dc, N, H, W, dtype, mf = shape
    w = wl.Workload("pair", Bt, Dc, N, H, W, dtype, mask_frac=mf, backward=True)
    inp = wl.make_inputs(w, seed=51)
    d = s2d.to_device(inp, dtype)
    desc = s2d.make_desc(d["x"], d["A"])
    print(f"training pair case {shape}: saved bytes {s2d.saved_bytes(desc)}", flush=True)
    expect_saving = N == 16 and 16 < W <= 192 and H > 4
    assert (s2d.saved_bytes(desc) > 0) == expect_saving
    y = torch.empty_like(d["x"])
    out = (torch.empty_like(d["x"]), torch.empty_like(d["x"]), torch.empty_like(d["A"]), torch.empty(d["Bm"].shape, dtype=torch.float32, device="cuda"),
           torch.empty(d["Bm"].shape, dtype=torch.float32, device="cuda"), None if d["Dskip"] is None else torch.empty_like(d["Dskip"]))
    fwd, bwd, saved = s2d.prepare_training_pair(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], y, d["dy"], out)
    assert (saved is not None) == expect_saving
    fwd()
    bwd()
    torch.cuda.synchronize()
    ref = oracle.scan2d_fwd(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"], dtype=dtype)
    assert rel_err(wl.to_float(s2d.to_host(y), dtype), wl.to_float(ref, dtype)) <= TOL[dtype]
    plain = s2d.scan2d_bwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"])
    torch.cuda.synchronize()
    for name, g, p in zip(GRADS, out, plain):             # the same sweeps on the same checkpoints: bit for bit
        if p is None:
            assert g is None
            continue
        assert torch.equal(g.view(torch.uint8), p.view(torch.uint8)), name
    refs = oracle.scan2d_bwd(inp["x"], inp["delta"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"], inp["mask"], inp["dy"], dtype=dtype)
    for k, (name, g, r) in enumerate(zip(GRADS, out, refs)):
        if r is None:
            continue
        gv = wl.to_float(s2d.to_host(g), dtype) if k < 2 else s2d.to_host(g).astype(np.float64)
        rv = wl.to_float(r, dtype) if k < 2 else r.astype(np.float64)
        tol = TOL[dtype] if k < 2 else (1e-4 if dtype == wl.F32 else 2e-2)
        assert rel_err(gv, rv) <= tol, f"{name}: rel err {rel_err(gv, rv):.3e}"


def test_training_pair_rejects_flags_and_short_buffers(s2d):
    import ctypes
    import torch
    w = wl.Workload("pairerr", 1, 2, 16, 24, 64, wl.F32, backward=True)
    d = s2d.to_device(wl.make_inputs(w, seed=52), wl.F32)
    desc = s2d.make_desc(d["x"], d["A"])
    need = s2d.saved_bytes(desc)
    assert need > 0
    assert s2d.saved_bytes(s2d.make_desc(d["x"], d["A"], s2d.FLAG_COLUMNS_FIRST)) == 0
    y = torch.empty_like(d["x"])
    saved = torch.empty(need, dtype=torch.uint8, device="cuda")
    p = lambda t: None if t is None else t.data_ptr()
    args = (p(d["x"]), p(d["delta"]), p(d["A"]), p(d["Bm"]), p(d["Cm"]), p(d["Dskip"]), p(d["mask"]), p(y))
    rc = s2d.lib.scan2d_fwd_saving(ctypes.byref(desc), *args, p(saved), need - 1, None, 0, None)
    assert rc == -5
    flagged = s2d.make_desc(d["x"], d["A"], s2d.FLAG_IDENTITY_CELLS)
    assert s2d.lib.scan2d_fwd_saving(ctypes.byref(flagged), *args, p(saved), need, None, 0, None) == -4
    assert s2d.lib.scan2d_fwd_saving(ctypes.byref(desc), *args, None, need, None, 0, None) == -1


def test_threads_with_streams_of_their_own_and_more_shapes_than_plans_are_kept(s2d):
    """Each thread remembers its own launch plans, fewer than it is given shapes here, and calls run side by side."""
    import threading
    import torch
    dev, g = "cuda", torch.Generator(device="cuda").manual_seed(5)
    cases = []
    for k in range(24):
        H, W, N, Dc = 3 + 2 * k, 5 + 3 * k, (4, 16)[k % 2], 6
        dt = (torch.float32, torch.bfloat16)[k // 2 % 2]
        r = lambda *s: torch.randn(s, device=dev, generator=g)
        cases.append((r(1, Dc, H, W).to(dt), r(1, Dc, H, W).sub(2).exp().to(dt), -r(Dc, N).exp(), r(1, N, H, W).to(dt), r(1, N, H, W).to(dt), r(Dc), None,
                      r(1, Dc, H, W).to(dt)))
    both = lambda c: (s2d.scan2d_fwd(*c[:7]),) + tuple(s2d.scan2d_bwd(*c))
    want = [both(c) for c in cases]
    torch.cuda.synchronize()
    got, failed = [{} for _ in range(3)], []

    def work(t):
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                for k in range(2 * len(cases)):
                    k = (k * (1, 5, 7)[t] + t) % len(cases)
                    got[t][k] = both(cases[k])
            st.synchronize()
        except Exception as e:                             # noqa: BLE001 (reported below, in the test's own thread)
            failed.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    for outs in got:
        assert len(outs) == len(cases)
        for k, o in outs.items():
            assert all(torch.equal(a, b) for a, b in zip(o, want[k]))


@pytest.mark.parametrize("wrong", ["host", "strided", "dtype", "shape", "missing", "rank"])
def test_binding_refuses_what_does_not_fit(s2d, wrong):
    import torch
    x = torch.zeros((1, 4, 6, 8), device="cuda")
    A, B = torch.zeros((4, 2), device="cuda"), torch.zeros((1, 2, 6, 8), device="cuda")
    bad = {"host": x.cpu(), "strided": x.transpose(2, 3).contiguous().transpose(2, 3), "dtype": x.bfloat16(), "shape": x[:, :3].contiguous(),
           "missing": None, "rank": x[0]}[wrong]
    with pytest.raises(ValueError):
        s2d.scan2d_fwd(x, bad, A, B, B)
    if wrong == "rank":
        with pytest.raises(ValueError):
            s2d.scan2d_fwd(bad, bad, A, B, B)


@pytest.mark.parametrize("form", ["tuple", "list", "generator", "map"])
def test_backward_writes_into_the_tensors_of_any_iterable(s2d, form):
    """`out` may make its items as they are taken: nothing but the call itself then holds them."""
    import torch
    w = wl.Workload("out", 1, 3, 16, 9, 21, wl.F32, mask_frac=0.3, backward=True)
    d = s2d.to_device(wl.make_inputs(w, seed=3), wl.F32)
    args = (d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"])
    want = s2d.scan2d_bwd(*args)
    make = lambda: {"tuple": tuple(torch.empty_like(t) for t in want), "list": [torch.empty_like(t) for t in want],
                    "generator": (torch.empty_like(t) for t in want), "map": map(torch.empty_like, want)}[form]
    for _ in range(3):
        got = s2d.scan2d_bwd(*args, out=make())
        assert all(torch.equal(g, r) for g, r in zip(got, want))
    with pytest.raises(ValueError):
        s2d.scan2d_bwd(*args, out=(torch.empty_like(t) for t in want[:5]))


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("H,W", [(14, 14), (13, 16), (16, 9), (37, 56), (5, 128), (7, 192), (5, 256), (3, 260), (5, 512)])
def test_infinity_in_the_last_cell_of_a_map_stays_out_of_dA(s2d, H, W, dtype):
    """B of the last cell reaches the state of that cell only, behind which no decay is applied: dA does not depend on it,
    and only that cell's gradients of x and delta do.  (Rows that do not fill a band, lanes past the last column.)"""
    import torch
    w = wl.Workload("last", 2, 3, 16, H, W, dtype, backward=True)
    d = s2d.to_device(wl.make_inputs(w, seed=12), dtype)
    args = lambda: (d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"])
    want = s2d.scan2d_bwd(*args())
    d["Bm"][:, ::3, -1, -1] = float("inf")
    got = s2d.scan2d_bwd(*args())
    assert torch.equal(got[2], want[2])
    for k in (0, 1):
        assert torch.equal(got[k].flatten(2)[..., :-1], want[k].flatten(2)[..., :-1])


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("H,W", [(6, 300), (5, 512), (4, 530)])
def test_column_panels_beside_a_column_whose_state_overflows(s2d, H, W, dtype):
    """Columns 40, 43, 255 and 281 collect 3e38 per row and overflow; the decay of the column behind each is exp(-200) = 0,
    so nothing of it reaches the other columns: their gradients are those of ordinary inputs, to the bit."""
    import torch
    w = wl.Workload("over", 1, 2, 16, H, W, dtype, backward=True)
    d = s2d.to_device(wl.make_inputs(w, seed=13), dtype)
    cols = [40, 43, 255, 281]
    d["A"].fill_(-1.0)
    d["delta"].fill_(1e-3)
    d["delta"][..., [c + 1 for c in cols]] = 200.0
    d["Bm"][..., cols] = 3e21
    d["dy"].mul_(1e-3)                                   # the gradients themselves stay far from overflow
    out = []
    for big in (1.0, 1e20):
        d["x"][..., cols] = big
        out.append(s2d.scan2d_bwd(d["x"], d["delta"], d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"], d["dy"]))
    assert not bool(torch.isfinite(out[1][4][..., cols]).all())             # dC: the states did overflow
    others = [j for j in range(W) if j not in cols]
    assert bool(torch.isfinite(out[0][1]).all()) and torch.equal(out[1][0], out[0][0])
    assert torch.equal(out[1][1][..., others], out[0][1][..., others])


# Bt, Dc, N, H, W, channels per workgroup
SMALL_CHANNEL_GROUPS = [(8, 128, 16, 14, 14, 2), (9, 129, 16, 14, 14, 2), (13, 119, 16, 7, 7, 3), (16, 129, 8, 12, 16, 2), (32, 131, 4, 7, 9, 2)]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("form", ["plain", "softplus", "gated"])
@pytest.mark.parametrize("Bt,Dc,N,H,W,GS", SMALL_CHANNEL_GROUPS, ids=lambda v: str(v))
def test_backward_of_small_maps_with_several_channels_per_workgroup(s2d, Bt, Dc, N, H, W, GS, form, dtype):
    """A workgroup handles GS channels in turn (whole groups and a ragged last one), states on one, two and four wavefronts;
    the channel groups' partial sums are added by 16 threads per element."""
    plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, N, dtype, 0), s2d.PASS_BWD)
    assert "form=small " in plan and f" GS={GS} " in plan, plan
    if form == "plain":
        check_bwd(s2d, wl.Workload("small", Bt, Dc, N, H, W, dtype, mask_frac=0.3, backward=True), seed=16)
    elif form == "softplus":
        test_backward_with_softplus_step_matches_oracle(s2d, (Bt, Dc, N, H, W, dtype, 0.3), True)
    else:
        test_gated_backward_matches_oracle(s2d, (Bt, Dc, N, H, W, dtype, 0.3))


# Row segments of the banded backward: a segment starts its reverse column recurrence from what a pass in front of the sweep
# has formed with the sweep's own operations, so at the same channels per workgroup everything but the sums over a whole map
# (dA, dDskip, the bias gradient: another order) is bit for bit what one segment per map gives.
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("form", ["plain", "softplus", "gated"])
@pytest.mark.parametrize("variant,segments,shape", [
    ("16,4,4,2,1", 2, (1, 5, 16, 57)), ("16,4,4,3,1", 5, (2, 7, 18, 64)), ("16,8,4,1,1", 3, (1, 3, 41, 121)), ("16,12,4,2,1", 4, (2, 3, 30, 190)),
    ("16,4,4,2,1", 8, (2, 3, 64, 10)), ("16,4,4,2,1", 2, (1, 3, 64, 3)),      # as many as the checkpoints' row holds the sums of
    ("64,4,8,2,1", 3, (1, 3, 11, 255)), ("64,4,8,2,-1", 4, (2, 3, 23, 397)), ("64,4,8,1,-1", 2, (1, 2, 9, 777))],
    ids=lambda v: v if isinstance(v, str) else ("x".join(map(str, v)) if isinstance(v, tuple) else f"{v}seg"))
def test_backward_row_segments(s2d, variant, segments, shape, form, dtype):
    import torch
    Bt, Dc, H, W = shape
    d = s2d.to_device(wl.make_inputs(wl.Workload("bseg", Bt, Dc, 16, H, W, dtype, mask_frac=0.3, backward=True), seed=21), dtype)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    z = torch.randn(d["x"].shape, device="cuda:0", generator=g).to(d["x"].dtype)
    bias = torch.randn(Dc, device="cuda:0", generator=g) * 0.1

    def grads(seg):
        with s2d.forced_variant(s2d.TUNE_BWD, f"{variant},{seg}"):
            plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, 16, dtype, 0), s2d.PASS_BWD)
            assert f"segments={seg} " in plan, plan
            a = (d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
            if form == "plain":
                names, out = ("dx", "ddelta", "dA", "dBm", "dCm", "dDskip"), s2d.scan2d_bwd(d["x"], d["delta"], *a, d["dy"])
            elif form == "softplus":
                names, out = ("dx", "ddelta", "dbias", "dA", "dBm", "dCm", "dDskip"), s2d.scan2d_bwd_softplus(d["x"], d["delta"], bias, *a, d["dy"])
            else:
                names = ("dx", "ddelta", "dbias", "dA", "dBm", "dCm", "dDskip", "dz")
                out = s2d.scan2d_bwd_softplus_gated(d["x"], d["delta"], bias, *a, z, d["x"], d["dy"])
        torch.cuda.synchronize()
        return dict(zip(names, out))

    one, many = grads(1), grads(segments)
    for k, v in one.items():
        if k in ("dA", "dDskip", "dbias"):
            # fp32 sums of up to H * W terms in two orders: a few units in the last place of the sum of magnitudes, which
            # for these inputs is within 100 times the largest entry
            assert (many[k] - v).abs().max() <= 100 * 2.0 ** -23 * v.abs().max(), k
        else:
            assert torch.equal(many[k], v), k


# Forward forms for small and narrow maps: several channels of a batch item per workgroup (channels off the group grid), the
# gate inside, half-wave groups, eight rows per batch (heights off it), one and several maps of a batch item.
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("Bt,Dc,N,H,W,form", [
    (5, 411, 16, 13, 14, "tile16 "), (2, 1025, 7, 16, 16, "tile16 "), (300, 17, 4, 14, 3, "tile16 "), (3, 700, 16, 13, 14, "tile16 "), (3, 700, 16, 5, 9, "small "),
    (1, 7, 5, 9, 30, "small "), (2, 300, 13, 11, 19, "small LG=16 K=2 NW=4 "), (2, 3, 16, 33, 14, "small LG=16 K=1 "), (1, 5, 3, 15, 22, "small LG=16 K=2 "),
    (3, 700, 8, 12, 13, "small LG=16 K=1 "), (2, 3, 16, 5, 31, "shared LG=16 K=4 "), (1, 5, 16, 21, 64, "shared LG=16 K=4 "), (1, 3, 16, 8, 17, "shared LG=16 K=4 "),
    (2, 130, 16, 6, 65, "shared LG=32 K=4 "), (1, 260, 16, 9, 127, "shared LG=32 K=4 ")])
def test_forward_of_small_and_narrow_maps(s2d, Bt, Dc, N, H, W, form, dtype):
    import torch
    w = wl.Workload("narrow", Bt, Dc, N, H, W, dtype, mask_frac=0.3)
    inp = _gated_inputs(w, seed=31)
    plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, N, dtype, 0), s2d.PASS_FWD)
    assert f"form={form}" in plan, plan
    d = s2d.to_device(inp, dtype)
    db = torch.from_numpy(inp["delta_bias"]).cuda()
    a = (d["x"], d["delta"], db, d["A"], d["Bm"], d["Cm"], d["Dskip"], d["mask"])
    ys, y = s2d.scan2d_fwd_softplus_gated(*a, d["z"])
    _, y_only = s2d.scan2d_fwd_softplus_gated(*a, d["z"], want_y_scan=False)
    plain = s2d.scan2d_fwd_softplus(*a)
    torch.cuda.synchronize()
    rys, ry = oracle.scan2d_fwd_softplus_gated(inp["x"], inp["delta"], inp["delta_bias"], inp["A"], inp["Bm"], inp["Cm"], inp["Dskip"],
                                               inp["mask"], inp["z"], dtype=dtype)
    assert rel_err(wl.to_float(s2d.to_host(ys), dtype), wl.to_float(rys, dtype)) <= TOL[dtype]
    assert rel_err(wl.to_float(s2d.to_host(y), dtype), wl.to_float(ry, dtype)) <= TOL[dtype]
    assert torch.equal(ys, plain) and torch.equal(y, y_only)


# The forward kernel for many maps, eight channels per workgroup (blocks of K or K - 1 columns, four per wavefront): K and columns of
# wavefronts forced at both ends of their widths, channels off the eights, heights off the batches of four and below the skew.
QUADS_CASES = [(4, 1, (2, 9, 1, 13)), (4, 2, (1, 12, 9, 25)), (4, 4, (1, 7, 6, 64)), (5, 1, (3, 8, 5, 17)), (5, 3, (1, 5, 4, 59)), (6, 1, (2, 5, 3, 24)),
               (6, 2, (1, 16, 11, 41)), (7, 1, (2, 4, 14, 28)), (7, 2, (2, 13, 13, 49)), (7, 2, (1, 8, 21, 56)), (7, 4, (1, 3, 18, 109)), (8, 1, (1, 9, 7, 29)),
               (8, 2, (1, 8, 2, 64)), (8, 4, (1, 8, 17, 128)), (9, 1, (1, 8, 10, 33)), (10, 1, (2, 6, 9, 40)), (11, 1, (1, 8, 5, 43)), (12, 1, (1, 10, 13, 47)),
               (12, 4, (1, 5, 11, 189)), (13, 1, (1, 8, 6, 52)), (14, 1, (2, 3, 9, 55)), (15, 1, (1, 8, 9, 57)), (16, 1, (1, 11, 10, 64))]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("K,cols,shape", QUADS_CASES, ids=[f"{k}-{c}-" + "x".join(map(str, s)) for k, c, s in QUADS_CASES])
def test_forward_of_many_maps(s2d, K, cols, shape, dtype):
    Bt, Dc, H, W = shape
    with s2d.forced_variant(s2d.TUNE_FWD, f"4,{K},4,{cols}"):
        plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, 16, dtype, 0), s2d.PASS_FWD)
        assert f"form=quads LG=4 K={K} NW=4 waves={2 * cols} " in plan, plan
        for mask in (0.3, 0.0):
            check_fwd(s2d, wl.Workload("quads", Bt, Dc, 16, H, W, dtype, mask_frac=mask), seed=21)
        test_forward_with_softplus_step_matches_oracle(s2d, (Bt, Dc, 16, H, W, dtype, 0.3), True)
        test_gated_forward_matches_oracle(s2d, (Bt, Dc, 16, H, W, dtype, 0.3))
        test_mask_is_bit_identical_to_prezeroed_x_and_blocks_garbage(s2d, H, W)


# As the dispatcher takes it, on grids of many workgroups per compute unit, cell by cell against the general form (small grids of both are
# compared with the oracle where they are forced).  The lines of the rule are checked without a GPU; the rows here run what each of its
# branches launches.  K = 0: another form.
@pytest.mark.parametrize("Bt,Dc,H,W,dtype,sp,K,cols", [
    (48, 96, 13, 13, wl.F32, False, 4, 1), (47, 96, 13, 13, wl.F32, False, 0, 0), (48, 96, 12, 14, wl.BF16, False, 0, 0), (24, 96, 9, 17, wl.BF16, True, 5, 1),
    (32, 96, 9, 21, wl.F32, True, 6, 1), (32, 96, 24, 25, wl.BF16, False, 4, 2), (32, 96, 23, 25, wl.BF16, False, 0, 0), (43, 92, 9, 32, wl.F32, False, 8, 1),
    (36, 96, 9, 48, wl.BF16, False, 6, 2), (36, 96, 9, 40, wl.F32, False, 5, 2), (36, 96, 9, 36, wl.F32, True, 5, 2), (36, 96, 9, 37, wl.BF16, True, 0, 0),
    (54, 96, 9, 44, wl.F32, False, 11, 1), (86, 96, 9, 45, wl.BF16, True, 6, 2), (80, 96, 9, 45, wl.BF16, True, 12, 1), (80, 96, 9, 33, wl.BF16, False, 9, 1),
    (43, 96, 21, 56, wl.BF16, False, 7, 2), (70, 96, 21, 56, wl.BF16, False, 14, 1), (54, 96, 21, 53, wl.F32, True, 14, 1), (76, 96, 21, 59, wl.F32, True, 15, 1),
    (77, 96, 21, 61, wl.BF16, True, 16, 1), (86, 96, 22, 64, wl.BF16, True, 8, 2), (54, 96, 21, 64, wl.F32, False, 8, 2), (54, 97, 21, 64, wl.F32, False, 8, 2),
    (300, 9, 21, 64, wl.F32, False, 0, 0), (54, 96, 21, 65, wl.F32, False, 0, 0)])
def test_forward_of_many_maps_as_dispatched(s2d, Bt, Dc, H, W, dtype, sp, K, cols):
    import torch
    plan = s2d.describe_plan(s2d.Desc(Bt, Dc, H, W, 16, dtype, 0), s2d.PASS_FWD_SOFTPLUS if sp else s2d.PASS_FWD)
    assert (f"form=quads LG=4 K={K} NW=4 waves={2 * cols} " in plan) if K else ("form=quads" not in plan), plan
    g = torch.Generator(device="cuda:0").manual_seed(5)
    td = torch.float32 if dtype == wl.F32 else torch.bfloat16
    draw = lambda *s: torch.randn(s, device="cuda:0", generator=g)
    x, raw, z = (draw(Bt, Dc, H, W).to(td) for _ in range(3))
    Bm, Cm = (draw(Bt, 16, H, W).to(td) for _ in range(2))
    A, skip, bias = -(0.5 * draw(Dc, 16)).exp(), draw(Dc), draw(Dc)
    mask = (draw(Bt, H, W) > 0.5).to(torch.uint8)
    x.masked_fill_(mask.bool().unsqueeze(1), float("nan"))                      # nothing under the mask leaks
    most_gate = torch.nn.functional.silu(z.float()).abs().max()

    def run():
        if sp:
            return s2d.scan2d_fwd_softplus_gated(x, raw, bias, A, Bm, Cm, skip, mask, z)
        return (s2d.scan2d_fwd(x, torch.nn.functional.softplus(raw.float()).to(td), A, Bm, Cm, None, mask),)

    def compare(finite):
        got = run()
        with s2d.forced_variant(s2d.TUNE_FWD, "16,4,4,4"):
            want = run()
        torch.cuda.synchronize()
        # In both forms a value is 16 products in fp32, summed in another order: at most 16 roundings of sums that are at most 16 times
        # the largest value, and what the gate makes of that.  bf16 results round these to eight significant bits: neighbours, up to
        # 2^-7 of the value apart.  The general form gates the rounded y: half a unit of y, half a unit of each of the two results, 2^-8 of the value each.
        most = torch.nan_to_num(want[0].float(), posinf=0.0, neginf=0.0).abs().max()
        for k, (a, b) in enumerate(zip(got, want)):
            a, b = a.float(), b.float()
            assert torch.equal(torch.isfinite(a), torch.isfinite(b))
            assert torch.isfinite(b).all() or not finite
            a, b = torch.nan_to_num(a, posinf=0.0, neginf=0.0), torch.nan_to_num(b, posinf=0.0, neginf=0.0)
            unit = 0.0 if dtype == wl.F32 else 2.0 ** -7 if k == 0 else 3.1 * 2.0 ** -8
            room = 16 * 16 * 2.0 ** -24 * most * (1.0 if k == 0 else most_gate)
            far = (a - b).abs() - unit * torch.maximum(a.abs(), b.abs())
            assert far.max() <= room, (k, far.max().item(), room.item())
            # 2-norm: 16 roundings of the typical value; bf16, one value in 16 next to a rounding boundary, and gated twice rounded
            bound = 2.0 ** -20 if dtype == wl.F32 else 2.0 ** -10 if k == 0 else 2.0 ** -8
            dist = ((a - b).double().norm() / b.double().norm()).item()
            assert dist <= bound, (k, dist)

    compare(finite=True)                                                        # every cell
    Bm[-1, 3, H // 2, W // 2] = float("inf")                                    # beside an infinite input the same cells are not finite
    compare(finite=False)
