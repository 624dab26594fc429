"""The work that programs built on this library have it do, as cases that can be prepared, run and compared.

Three kinds of program use the operator:

* slide models: one grid of patch features per slide (batch 1, sometimes a few), any height and width, part of it
  background under a mask, 128 to 512 channels (the inner width of a block); inference runs the whole block and the
  attention pooling behind it, training runs the scan forward and backward;
* image models: square feature maps of a few to a hundred cells a side, batches of images, no mask;
* operator studies: the bare scan on ready-made steps, small grids and other state counts among them.

Kinds of case (`kind`), each ONE pass through the public entry points of `paper_2412_00678_amd.scan2d`:

  scan         scan2d_fwd                                                       inference with the bare operator
  train        scan2d_fwd_saving, scan2d_bwd_saved (prepare_training_pair)      a training step of the bare operator
  train_gated  scan2d_fwd_softplus_gated, scan2d_bwd_softplus_gated             a training step of the scan inside a block
  block        norm, two input projections, convolution, projections of step, B and C, gated scan, output projection
               with the skip connection                                         inference of one block
  slide        block, then attention pooling over the bag of positions          inference of a slide model

bf16 and fp32 are the two storage types.  Sizes are those of this repository's configurations, tests and benchmark, or
plain odd ones in between.
"""
import math

import torch

from paper_2412_00678_amd import scan2d as s2d

DEV = "cuda:0"


def _case(name, kind, Bt, Dc, H, W, dtype, mask=0.0, N=16, mu=-2.0):
    return {"name": name, "kind": kind, "Bt": Bt, "Dc": Dc, "H": H, "W": W, "N": N, "dtype": dtype, "mask": mask, "mu": mu}


def listed():
    return [
        # the smallest call: a 16 x 16 grid with 4 states; host work and launch latency are all there is
        _case("scan_16x16_fp32", "scan", 1, 16, 16, 16, "fp32", N=4),
        # a small slide grid
        _case("scan_64x64_fp32_mask", "scan", 1, 256, 64, 64, "fp32", mask=0.4),
        # a large slide grid, half of it background: the benchmark's default workload
        _case("scan_256x256_bf16_mask", "scan", 1, 256, 256, 256, "bf16", mask=0.5),
        # an image model's stage, batch 32
        _case("scan_56x56_bf16_b32", "scan", 32, 192, 56, 56, "bf16", mu=-3.0),
        # the smallest grid that the paper trains on, 128 channels, batch 8
        _case("train_14x14_fp32_b8", "train", 8, 128, 14, 14, "fp32"),
        # the training workload of the benchmark
        _case("train_128x192_fp32_mask", "train", 4, 512, 128, 192, "fp32", mask=0.3),
        # the image model's stage in training, step and gate inside the operator
        _case("train_gated_56x56_bf16_b32", "train_gated", 32, 192, 56, 56, "bf16", mu=-3.0),
        # a slide as it comes in training: odd sides, wider than 256 columns, background
        _case("train_gated_211x397_bf16_mask", "train_gated", 1, 256, 211, 397, "bf16", mask=0.4),
        # a small map through a whole block: seven short calls in a row
        _case("block_14x14_bf16_b8", "block", 8, 256, 14, 14, "bf16"),
        # inference of a large slide
        _case("slide_256x256_bf16_mask", "slide", 1, 256, 256, 256, "bf16", mask=0.5),
        # slides as they come: odd sides in both storage types
        _case("slide_57x83_bf16_mask", "slide", 1, 256, 57, 83, "bf16", mask=0.4),
        _case("slide_127x201_fp32_mask", "slide", 1, 512, 127, 201, "fp32", mask=0.3),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    """Slide grids of 20 to 400 cells a side or batches of 1 to 64 square maps of 7 to 112 cells a side."""
    kind = rng.choice(("scan", "train", "train_gated", "block", "slide"))
    dtype = rng.choice(("fp32", "bf16"))
    if kind == "slide" or (kind != "block" and rng.random() < 0.5):
        Bt, Dc = 1, rng.choice((128, 192, 256, 384, 512))
        H, W = _log_int(rng, 20, 400), _log_int(rng, 20, 400)
        mask, mu = round(rng.uniform(0.2, 0.6), 2), -2.0
    else:
        Bt, Dc = _log_int(rng, 1, 64), rng.choice((96, 128, 192, 256, 384))
        H = W = _log_int(rng, 7, 112)
        mask, mu = 0.0, -3.0
    N = rng.choice((4, 8, 16, 16, 16, 16, 32, 64)) if kind == "scan" else 16
    most = 800e6 if kind == "scan" else 300e6       # (position, channel, state) triples
    while Bt * Dc * H * W * N > most and Bt > 1:
        Bt -= 1
    while Bt * Dc * H * W * N > most:
        Dc //= 2
    c = _case("", kind, Bt, Dc, H, W, dtype, mask=mask, N=N, mu=mu)
    del c["name"]
    return c


def _blobs(g, Bt, H, W, frac):
    """Background in contiguous blobs: the share `frac` of a smooth random field's cells, its lowest."""
    coarse = torch.randn((Bt, 1, H // 12 + 2, W // 12 + 2), device=DEV, generator=g)
    field = torch.nn.functional.interpolate(coarse, size=(H, W), mode="bilinear", align_corners=True).reshape(Bt, H * W)
    k = max(1, int(round(frac * H * W)))
    level = field.kthvalue(k, dim=1, keepdim=True).values
    return (field <= level).to(torch.uint8).reshape(Bt, H, W).contiguous()


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    Bt, Dc, H, W, N, mu = (case[k] for k in ("Bt", "Dc", "H", "W", "N", "mu"))

    def normal(*shape, scale=1.0, mean=0.0, dtype=torch.float32):
        return torch.randn(shape, device=DEV, generator=g).mul_(scale).add_(mean).to(dtype)

    s = {"kind": case["kind"], "N": N}
    s["A"] = -normal(Dc, N, scale=0.5).exp()
    s["Dskip"] = normal(Dc)
    s["mask"] = _blobs(g, Bt, H, W, case["mask"]) if case["mask"] > 0 else None
    if case["kind"] in ("block", "slide"):
        Dm = Dc // 2
        R = max(1, (Dm + 15) // 16)
        s["t"] = normal(Bt, Dm, H, W, dtype=dt)
        s["gamma"], s["beta"] = normal(Dm, scale=0.1, mean=1.0), normal(Dm, scale=0.1)
        s["Win_x"], s["Win_z"] = (normal(Dc, Dm, scale=Dm ** -0.5, dtype=dt) for _ in range(2))
        s["w"], s["bias"] = normal(Dc, 3, 3, scale=1 / 3), normal(Dc, scale=0.1)
        s["Wx"], s["Wdt"] = normal(R + 2 * N, Dc, scale=Dc ** -0.5, dtype=dt), normal(Dc, R, scale=R ** -0.5)
        s["delta_bias"] = normal(Dc, scale=0.5, mean=mu)
        s["Wout"] = normal(Dm, Dc, scale=Dc ** -0.5, dtype=dt)
        if case["kind"] == "slide":
            s["V"], s["pool_w"] = normal(128, Dm, scale=Dm ** -0.5, dtype=dt), normal(128)
        return s
    x = normal(Bt, Dc, H, W)
    s["x"] = (x if s["mask"] is None else x.mul_(1 - s["mask"].unsqueeze(1))).to(dt)
    raw = normal(Bt, Dc, H, W, scale=0.5, mean=mu)
    s["Bm"], s["Cm"] = normal(Bt, N, H, W, dtype=dt), normal(Bt, N, H, W, dtype=dt)
    if case["kind"] == "train_gated":
        s["raw"], s["delta_bias"], s["z"] = raw.to(dt), normal(Dc, scale=0.1), normal(Bt, Dc, H, W, dtype=dt)
    else:
        s["delta"] = torch.nn.functional.softplus(raw).to(dt)
    if case["kind"] != "scan":
        s["dy"] = normal(Bt, Dc, H, W, dtype=dt)
    if case["kind"] == "train":
        # a training loop over fixed activation buffers keeps its prepared pair of calls and what they write
        s["y"] = torch.empty_like(s["x"])
        s["grads"] = (torch.empty_like(s["x"]), torch.empty_like(s["x"]), torch.empty_like(s["A"]),
                      torch.empty(s["Bm"].shape, device=DEV), torch.empty(s["Bm"].shape, device=DEV), torch.empty_like(s["Dskip"]))
        s["fwd"], s["bwd"], _ = s2d.prepare_training_pair(s["x"], s["delta"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["mask"], s["y"],
                                                          s["dy"], s["grads"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "scan":
        return s2d.scan2d_fwd(s["x"], s["delta"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["mask"])
    if kind == "train":
        s["fwd"]()
        s["bwd"]()
        return (s["y"],) + s["grads"]
    if kind == "train_gated":
        y_scan, y = s2d.scan2d_fwd_softplus_gated(s["x"], s["raw"], s["delta_bias"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["mask"], s["z"])
        grads = s2d.scan2d_bwd_softplus_gated(s["x"], s["raw"], s["delta_bias"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["mask"], s["z"],
                                              y_scan, s["dy"])
        return (y,) + grads
    tn = s2d.block_norm(s["t"], s["gamma"], s["beta"])
    u = s2d.block_linear(tn, s["Win_x"])
    z = s2d.block_linear(tn, s["Win_z"])
    x = s2d.block_conv_silu(u, s["w"], s["bias"])
    raw, Bm, Cm = s2d.block_xproj(x, s["Wx"], s["Wdt"], s["N"])
    _, y = s2d.scan2d_fwd_softplus_gated(x, raw, s["delta_bias"], s["A"], Bm, Cm, s["Dskip"], s["mask"], z, want_y_scan=False)
    t = s2d.block_linear(y, s["Wout"], None, s["t"])
    if kind == "block":
        return t
    pooled, attn = s2d.block_attn_pool(t, s["V"], s["pool_w"], s["mask"])
    return t, pooled, attn


def work(case):
    """Bytes: the tensors that go into and come out of each entry point of the pass, once each for the whole of a
    training step and once per call along a block (whose calls hand tensors to each other).  Flops: 9 per (position,
    channel, state) forward (exp, two products, three multiply-adds), 32 backward; 2 per multiply-add of a layer."""
    e = 2 if case["dtype"] == "bf16" else 4
    Bt, Dc, N, kind = case["Bt"], case["Dc"], case["N"], case["kind"]
    P = Bt * case["H"] * case["W"]
    M, S, units = P * Dc, P * N, P * Dc * N
    m = P if case["mask"] > 0 else 0
    params = (Dc * N + Dc) * 4
    if kind == "scan":
        return {"bytes": (3 * M + 2 * S) * e + m + params, "flops": 9.0 * units}
    if kind == "train":            # x, step, dy in; y and their two gradients out
        return {"bytes": (6 * M + 2 * S) * e + 2 * S * 4 + m + 2 * params, "flops": 41.0 * units}
    if kind == "train_gated":      # x, raw step, z, dy in; y and three gradients out
        return {"bytes": (8 * M + 2 * S) * e + 2 * S * 4 + m + 2 * (params + Dc * 4), "flops": 41.0 * units}
    Dm = Dc // 2
    R = max(1, (Dm + 15) // 16)
    T = P * Dm
    byts = 2 * T * e + 2 * (T + M) * e + 2 * M * e + (2 * M + 2 * S) * e + (4 * M + 2 * S) * e + m + (M + 2 * T) * e
    byts += (3 * Dc * Dm + (R + 2 * N) * Dc) * e + params + Dc * (R + 11) * 4
    flops = 3 * 2.0 * M * Dm + 2.0 * 9 * M + 2.0 * (R + 2 * N) * M + 2.0 * R * M + 9.0 * units
    if kind == "slide":
        byts += T * e + m + P * 4 + Dm * 4 + 128 * (Dm * e + 4)
        flops += 2.0 * 128 * T + 2.0 * T
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """fp32: the order of fp32 sums over the states, the map and the channels.  bf16: results are rounded once, and where
    two calls of a pass hand a bf16 tensor over, a value next to a rounding boundary may come out one unit apart."""
    return {"rel": 2e-5} if case["dtype"] == "fp32" else {"rel": 1e-2}
