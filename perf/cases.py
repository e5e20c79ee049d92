"""The work this library is used for, as timed cases with their inputs and
64-bit results.

A heightmap viewer reconstructs and refines tiles (one at a time as they come
into view, the tiles near the viewpoint first, whole regions in a batch) and
splats full-resolution points into their textures; a training run builds
ground-truth textures from dense points and runs the network forward and
backward.  Each listed case is one such call through the package's functions;
`draw` gives others of the same kinds and ranges.  Inputs come from a seeded
torch generator: value-noise terrain, uniform points with per-tile counts
whose distribution is fixed by the case (the seed permutes the counts and
places the points), smooth height and colour maps for the network alone.
"""
import math

import numpy as np
import torch

import paper_2509_20198_amd as ls
from paper_2509_20198_amd import train as ls_train

# (Cin, Cout) of the U-Net's 3x3 layers in storage order
UNET = [(8, 16), (16, 16), (16, 32), (32, 32), (32, 64), (64, 64), (96, 32), (32, 32), (48, 16), (16, 16), (24, 4)]
INPUTS = {"all": ls.IN_ALL, "hm": ls.IN_HM_ONLY, "nn": ls.IN_NN_ONLY, "lin": ls.IN_LIN_ONLY}


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one tile with 400 sparse points comes into view: reconstruction and BF16 network, latency counts
        _serve("serve_one_tile", 1, 1, 1, "uniform", 400, 400),
        # the 256 tiles nearest to the viewer of a 128 x 128 region with long-tailed point counts: the first picture
        _serve("serve_nearest_256", 128, 128, 256, "pareto", 20, 5000),
        # a 32 x 32 batch at once, 50-2000 points per tile, no priority among the tiles
        _recon("recon_batch_1024", 32, 32, "loguniform", 50, 2000, order="longest"),
        # the whole 128 x 128 region in viewing order, long-tailed point counts
        _recon("recon_stream_16384", 128, 128, "pareto", 20, 5000, order="list"),
        # the network on a batch of reconstructed tiles, BF16, as the viewer runs it
        _refine("refine_bf16_1024", "bf16", 1024),
        # the same in FP32 (the accuracy reference of every BF16 run), an uneven batch
        _refine("refine_fp32_99", "fp32", 99),
        # the paper's larger network, BF16, an uneven batch
        _lsnet("lsnet_bf16_333", "bf16", 333, "all"),
        # one training step's forward, loss and backward as the trainer runs it
        _train("train_bf16_256", "bf16", 256, "mse", save=True, grad_x=False),
        # FP32 gradients of weights and inputs, activations recomputed (gradient checks, large-batch training)
        _train("train_fp32_24", "fp32", 24, "l1", save=False, grad_x=True),
        # full-resolution points of a close-up into the textures of 64 x 64 tiles
        _points("splat_100m", "splat", 100_000_000, 64, 64),
        # ground truth of 16 tiles from 2 M dense points each: sums and mean texture
        _points("mean_32m", "mean", 32_000_000, 4, 4),
        # the point renderer on the close-up's points, one 1920 x 1080 frame
        _points("raster_100m", "raster", 100_000_000, 64, 64, width=1920, height=1080, above=0.3),
    ]


def _named(name, case):
    return dict(case, name=name) if name else case


def _serve(name, tx, ty, tiles, counts, lo, hi, cell=1000, pad=16):
    return _named(name, {"kind": "serve", "tiles_x": tx, "tiles_y": ty, "tiles": tiles, "counts": counts, "lo": lo,
                         "hi": hi, "cell": cell, "pad": pad, "order": "list"})


def _recon(name, tx, ty, counts, lo, hi, order, cell=1000, pad=16):
    return _named(name, {"kind": "recon", "tiles_x": tx, "tiles_y": ty, "tiles": tx * ty, "counts": counts, "lo": lo,
                         "hi": hi, "cell": cell, "pad": pad, "order": order})


def _refine(name, dtype, tiles, pad=16):
    return _named(name, {"kind": "refine", "dtype": dtype, "tiles": tiles, "pad": pad})


def _lsnet(name, dtype, tiles, inputs, pad=16):
    return _named(name, {"kind": "lsnet", "dtype": dtype, "tiles": tiles, "inputs": inputs, "pad": pad})


def _train(name, dtype, tiles, loss, save, grad_x, pad=16):
    return _named(name, {"kind": "train", "dtype": dtype, "tiles": tiles, "loss": loss, "save": save,
                         "grad_x": grad_x, "pad": pad})


def _points(name, kind, n, tx, ty, mapped=1.0, **view):
    return _named(name, {"kind": kind, "points": n, "tiles_x": tx, "tiles_y": ty, "mapped": mapped, **view})


def _log(rng, lo, hi):
    return min(hi, int(lo * ((hi + 1) / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["serve", "recon", "recon", "refine", "refine", "lsnet", "train", "train", "splat", "mean",
                       "raster"])
    if kind in ("serve", "recon"):
        tx, ty = _log(rng, 1, 128), _log(rng, 1, 128)
        # 1 to 40 m texels; most data is at 10 m
        cell = rng.choice([100, 250, 500, 1000, 1000, 1000, 1000, 2000, 4000])
        pad = rng.choice([16, 16, 16, 16, 4, 0])
        counts = rng.choice(["loguniform", "pareto", "uniform"])
        lo, hi = {"loguniform": (50, 2000), "pareto": (20, 5000), "uniform": (200, 800)}[counts]
        if tx * ty <= 8 and counts == "uniform":  # a few densely scanned tiles
            hi = lo = _log(rng, 100, 16000)
        if kind == "serve":
            return _serve(None, tx, ty, min(tx * ty, _log(rng, 1, 512)), counts, lo, hi, cell, pad)
        if tx * ty > 1024 and counts != "pareto":
            counts, lo, hi = "pareto", 20, 5000
        return _recon(None, tx, ty, counts, lo, hi, rng.choice(["list", "longest"]), cell, pad)
    pad = rng.choice([16, 16, 16, 16, 0])
    dtype = rng.choice(["bf16", "fp32"])
    if kind == "refine":
        return _refine(None, dtype, _log(rng, 1, 1024 if dtype == "bf16" else 128), pad)
    if kind == "lsnet":
        return _lsnet(None, dtype, _log(rng, 1, 512 if dtype == "bf16" else 64),
                      rng.choice(["all", "all", "hm", "nn", "lin"]), pad)
    if kind == "train":
        return _train(None, dtype, _log(rng, 1, 256 if dtype == "bf16" else 32), rng.choice(["mse", "l1"]),
                      rng.random() < 0.7, rng.random() < 0.3, rng.choice([16, 16, 16, 4, 0]))
    n = _log(rng, 50_000, 100_000_000)
    side = max(1, min(64, int(math.sqrt(n / 4096 / math.exp(rng.uniform(math.log(2.0), math.log(500.0)))))))
    tx, ty = side, max(1, min(64, side + rng.randint(-side // 2, side // 2)))
    if kind == "raster":
        w, h = rng.choice([(1920, 1080), (1280, 720), (641, 479), (3840, 2160)])
        return _points(None, kind, n, tx, ty, width=w, height=h, above=rng.uniform(0.07, 0.6))
    return _points(None, kind, n, tx, ty, rng.choice([1.0, 1.0, 0.75]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _terrain(x, y, seed):
    """Four octaves of value noise (wavelengths 200 m to 25 m, amplitude about 50 m) in metres, float32."""
    g = _gen(seed ^ 0x7E22A1)
    total = torch.zeros(x.shape, dtype=torch.float32, device=x.device)
    for o in range(4):
        table = torch.rand(512 * 512, device=x.device, generator=g) * 2 - 1
        lam = 20000 >> o
        i, j = torch.div(x, lam, rounding_mode="floor"), torch.div(y, lam, rounding_mode="floor")
        fx, fy = (x - i * lam).float() / lam, (y - j * lam).float() / lam
        fx, fy = fx * fx * (3 - 2 * fx), fy * fy * (3 - 2 * fy)
        at = lambda a, b: table[((b & 511) << 9) | (a & 511)]  # noqa: E731
        lower, upper = torch.lerp(at(i, j), at(i + 1, j), fx), torch.lerp(at(i, j + 1), at(i + 1, j + 1), fx)
        total += 0.5 ** o * torch.lerp(lower, upper, fy)
    return total * (50.0 / 1.875)


def _colour(zm):
    """16-bit height ramp [n, 3] as int16 bit patterns."""
    v = ((zm + 50.0) * 2.55).round().clamp(0, 255).to(torch.int32)
    return (torch.stack([v, 255 - v, torch.full_like(v, 128)], dim=1) * 257).to(torch.int16).contiguous()


def _counts(case):
    """Sparse points per tile: the quantiles of the case's distribution (the seed permutes them over the tiles)."""
    n = case["tiles_x"] * case["tiles_y"]
    u = (np.arange(n) + 0.5) / n
    lo, hi = case["lo"], case["hi"]
    if case["counts"] == "loguniform":
        c = lo * (hi / lo) ** u
    elif case["counts"] == "pareto":
        c = np.minimum(hi, lo * (1 - u) ** (-1 / 1.5))
    else:
        c = lo + u * (hi - lo)
    return c.astype(np.int64)


def _grid(case):
    return ls.Grid(tile_size=64 * case.get("cell", 1000), pad=case.get("pad", 16), tiles_x=case.get("tiles_x", 1),
                   tiles_y=case.get("tiles_y", 1))


def _sparse(case, seed):
    """Uniform points in every tile of the region in shuffled order, and the tile list by distance to a viewpoint."""
    grid, g = _grid(case), _gen(seed)
    counts = torch.from_numpy(_counts(case)).cuda()
    nt = counts.numel()
    counts = counts[torch.randperm(nt, device="cuda", generator=g)]
    owner = torch.repeat_interleave(torch.arange(nt, device="cuda"), counts)
    owner = owner[torch.randperm(owner.numel(), device="cuda", generator=g)]
    S, n = grid.tile_size, owner.numel()
    x = (owner % grid.tiles_x * S + torch.randint(0, S, (n,), device="cuda", generator=g)).to(torch.int32)
    y = (owner // grid.tiles_x * S + torch.randint(0, S, (n,), device="cuda", generator=g)).to(torch.int32)
    zm = _terrain(x, y, seed)
    eye = torch.rand(2, device="cuda", generator=g) * torch.tensor([grid.tiles_x, grid.tiles_y], device="cuda")
    t = torch.arange(nt, device="cuda")
    away = (t % grid.tiles_x + 0.5 - eye[0]) ** 2 + (t // grid.tiles_x + 0.5 - eye[1]) ** 2
    tiles = torch.argsort(away, stable=True)[:case["tiles"]].to(torch.int32)
    return grid, x, y, (zm * 100).round().to(torch.int32), _colour(zm), tiles


def _maps(n, grid, seed):
    """Network inputs like reconstructed tiles: smooth heights (about 20 m of 480 m) and colours, and their blocky
    nearest-point versions, [n, R, R, 8]; centre heights [n]."""
    g, R = _gen(seed), grid.R
    noise = lambda c, k: torch.randn((n, c, k, k), device="cuda", generator=g)  # noqa: E731
    up = lambda t, mode: torch.nn.functional.interpolate(t, size=(R, R), mode=mode)  # noqa: E731
    h = sum(0.04 * 0.5 ** o * up(noise(1, 4 << o), "bilinear") for o in range(4))
    c = (0.5 + 4 * h + 0.1 * up(noise(3, 12), "bilinear")).clamp(0, 1)
    blocky = up(torch.nn.functional.avg_pool2d(torch.cat([h, c], 1), 4), "nearest")
    x = torch.cat([h, blocky[:, :1], c, blocky[:, 1:]], 1).permute(0, 2, 3, 1).contiguous()
    return x, torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * 1000


def _kaiming(shapes, seed, last_std):
    """Flat weights: Kaiming-normal layers [(outputs, fan-in)], a small last layer, small biases."""
    g, parts = _gen(seed ^ 0x3EED), []
    for k, (out, fan) in enumerate(shapes):
        std = last_std if k == len(shapes) - 1 else math.sqrt(2.0 / fan)
        parts += [torch.randn(out * fan, device="cuda", generator=g) * std,
                  torch.randn(out, device="cuda", generator=g) * 0.02 * min(1.0, std * 10)]
    return torch.cat(parts)


def _unet_weights(seed):
    return _kaiming([(co, 9 * ci) for ci, co in UNET], seed, 0.01 / math.sqrt(216))


def _lsnet_layers(R):
    """[(kind, inputs, outputs)] in weight order."""
    feat = (R // 16) ** 2 * 32
    enc = [("conv", a, b) for c in (1, 1, 3, 3) for a, b in ((c, 16), (16, 32), (32, 32), (32, 32))]
    fc = [("fc", 2 * feat, 256), ("fc", 2 * feat, 256), ("fc", 512, feat), ("fc", 512, feat)]
    dec = [("conv", a, b) for _ in range(2) for a, b in ((32, 32), (32, 32), (32, 16), (16, 16))]
    return enc + fc + dec + [("conv", 40, 32), ("conv", 32, 32), ("conv", 32, 4)]


def _lsnet_weights(seed, R):
    return _kaiming([(co, ci if k == "fc" else 9 * ci) for k, ci, co in _lsnet_layers(R)], seed, 0.01 / math.sqrt(288))


def _dense(case, seed):
    """Full-resolution points, uniform over the region, in Morton order of the 10 m cell; 0.1 m height noise."""
    g, n = _gen(seed), case["points"]
    w, h = case["tiles_x"] * 64, case["tiles_y"] * 64

    def spread(v):
        for s, m in ((8, 0x00FF00FF), (4, 0x0F0F0F0F), (2, 0x33333333), (1, 0x55555555)):
            v = (v | (v << s)) & m
        return v

    def gather(v):
        v = v & 0x55555555
        for s, m in ((1, 0x33333333), (2, 0x0F0F0F0F), (4, 0x00FF00FF), (8, 0x0000FFFF)):
            v = (v | (v >> s)) & m
        return v

    code = spread(torch.randint(0, w, (n,), device="cuda", generator=g, dtype=torch.int32))
    code |= spread(torch.randint(0, h, (n,), device="cuda", generator=g, dtype=torch.int32)) << 1
    code = torch.sort(code)[0]
    x, y, z = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3))
    rgb = torch.empty((n, 3), dtype=torch.int16, device="cuda")
    for a in range(0, n, 1 << 24):
        c = code[a:a + (1 << 24)]
        at = slice(a, a + c.numel())
        jit = torch.randint(0, 1000, (2, c.numel()), device="cuda", generator=g, dtype=torch.int32)
        x[at], y[at] = gather(c) * 1000 + jit[0], gather(c >> 1) * 1000 + jit[1]
        zm = _terrain(x[at], y[at], seed) + 0.1 * torch.randn(c.numel(), device="cuda", generator=g)
        z[at] = (zm * 100).round().to(torch.int32)
        rgb[at] = _colour(zm)
    return x, y, z, rgb


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind in ("recon", "serve"):
        s["grid"], *s["points"], s["tiles"] = _sparse(case, seed)
        g, nt = s["grid"], case["tiles"]
        new = lambda *shape, dtype=torch.float32: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
        s["order"] = ls.ORDER_LONGEST_FIRST if case["order"] == "longest" else ls.ORDER_LIST
        s["x"], s["cz"] = new(nt, g.R, g.R, 8), new(nt, dtype=torch.float64)
        s["status"] = new(nt, dtype=torch.int32)
        s["ws"] = ls.alloc_workspace(ls.workspace_bytes(ls.OP_RECON, g, nt, s["points"][0].numel()))
        if kind == "serve":
            s["w"] = _unet_weights(seed)
            s["wb"] = ls.pack_weights_bf16(s["w"])
            s["net_ws"] = ls.alloc_workspace(ls.workspace_bytes(ls.OP_REFINE, g, nt, 0, ls.BF16))
            s["tex"] = new(nt, g.res, g.res, 4)
    elif kind in ("refine", "lsnet", "train"):
        g = s["grid"] = _grid(case)
        s["precision"] = ls.BF16 if case["dtype"] == "bf16" else ls.FP32
        s["x"], s["cz"] = _maps(case["tiles"], g, seed)
        if kind == "lsnet":
            s["w"] = _lsnet_weights(seed, g.R)
            s["ws"] = ls.alloc_workspace(ls.workspace_bytes(ls.OP_REFINE_LSNET, g, case["tiles"], 0, s["precision"]))
        else:
            s["w"] = _unet_weights(seed)
        if kind == "refine":
            s["wb"] = ls.pack_weights_bf16(s["w"]) if s["precision"] == ls.BF16 else None
            s["ws"] = ls.alloc_workspace(ls.workspace_bytes(ls.OP_REFINE, g, case["tiles"], 0, s["precision"]))
        if kind == "train":
            s["w"].requires_grad_(True)
            s["x"].requires_grad_(case["grad_x"])
            s["target"] = _target(s, g, seed)
            s["loss"] = ls.LOSS_L1 if case["loss"] == "l1" else ls.LOSS_CLIPPED_MSE
    else:
        s["points"] = _dense(case, seed)
        nt = case["tiles_x"] * case["tiles_y"]
        s["grid"] = ls.Grid(tiles_x=case["tiles_x"], tiles_y=case["tiles_y"])
        if kind == "raster":
            # a perspective view straight down at the region's centre, from `above` of its side up
            side = 640.0 * max(case["tiles_x"], case["tiles_y"])
            f, a = 1.2, case["width"] / case["height"]
            m = [f, 0, 0, -f * 320.0 * case["tiles_x"], 0, f * a, 0, -f * a * 320.0 * case["tiles_y"],
                 0, 0, 0, 0, 0, 0, -1, 100.0 + case["above"] * side]
            s["view"] = ls.View(m=tuple(v / (side * 0.5) for v in m), width=case["width"], height=case["height"])
        else:
            slots = max(1, int(nt * case["mapped"]))
            order = torch.randperm(nt, device="cuda", generator=_gen(seed ^ 0x510))
            s["slots"], s["slot"] = slots, torch.full((nt,), -1, dtype=torch.int32, device="cuda")
            s["slot"][order[:slots]] = torch.arange(slots, dtype=torch.int32, device="cuda")
            if kind == "splat":
                s["tex"] = torch.rand((slots, 64, 64, 4), device="cuda", generator=_gen(seed ^ 0x7E))
    return s


def _target(s, g, seed):
    """Target textures near the input's linear maps, in metres and [0, 1], 3 % of the texels without a point."""
    r = _gen(seed ^ 0x7A6)
    c = s["x"].detach()[:, g.pad:g.pad + g.res, g.pad:g.pad + g.res][..., [0, 2, 3, 4]]
    t = c + 0.01 * torch.randn(c.shape, device="cuda", generator=r)
    radius = (g.tile_size / 2 + g.pad * (g.tile_size // g.res)) * g.scale_xy
    t[..., 0] = t[..., 0] * radius + s["cz"].float()[:, None, None]
    t[..., 1:].clamp_(0, 1)
    t[torch.rand(t.shape[:3], device="cuda", generator=r) < 0.03] = float("nan")
    return t.contiguous()


def run(s):
    case, g = s["case"], s["grid"]
    kind = case["kind"]
    if kind in ("recon", "serve"):
        x, cz, status = ls.recon_tiles(g, *s["points"], s["tiles"], order=s["order"], x_out=s["x"], cz_out=s["cz"],
                                       status=s["status"], ws=s["ws"])
        out = {"x": x, "cz": cz, "status": status}
        if kind == "serve":
            _, out["tex"] = ls.refine_tiles(s["w"], x, cz, g, ls.BF16, w_bf16=s["wb"], tex_out=s["tex"], want_y=False,
                                            ws=s["net_ws"])
        return out
    if kind == "refine":
        y, tex = ls.refine_tiles(s["w"], s["x"], s["cz"], g, s["precision"], w_bf16=s["wb"], ws=s["ws"])
        return {"y": y, "tex": tex}
    if kind == "lsnet":
        y, tex = ls.lsnet_refine_tiles(s["w"], s["x"], s["cz"], g, s["precision"], inputs=INPUTS[case["inputs"]],
                                       ws=s["ws"])
        return {"y": y, "tex": tex}
    if kind == "train":
        y = ls.RefineFn.apply(s["x"], s["w"], g, s["precision"], case["save"])
        loss = ls_train.TargetLossFn.apply(y, s["target"], s["cz"], g, s["loss"])
        grads = torch.autograd.grad(loss, [s["w"], s["x"]] if case["grad_x"] else [s["w"]])
        return {"y": y.detach(), "loss": loss.detach(), "grads": list(grads)}
    if kind == "splat":
        keys, dropped = ls.splat_points(g, *s["points"], s["slot"], s["slots"], tex_inout=s["tex"])
        return {"keys": keys, "dropped": dropped, "tex": s["tex"]}
    if kind == "mean":
        acc, dropped = ls.splat_mean(g, *s["points"], s["slot"], s["slots"])
        return {"acc": acc, "dropped": dropped, "tex": ls.resolve_mean(g, acc)}
    fb, drawn = ls.raster_points(s["view"], *s["points"])
    return {"fb": fb, "drawn": drawn, "rgba": ls.raster_resolve(fb)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _unet_flops(res, pad):
    """Multiply-adds x 2 of one tile's forward; the last level only near the crop, where the output reads it."""
    R = res + 2 * pad
    side = [R, R, R // 2, R // 2, R // 4, R // 4, R // 2, R // 2, min(R, res + 4), min(R, res + 2), res]
    return sum(18.0 * n * n * ci * co for n, (ci, co) in zip(side, UNET))


def _lsnet_flops(res, pad):
    R, f = res + 2 * pad, 0.0
    w = [min(R, res + 2 * h) for h in (3, 2, 1, 0)]
    side = [R, R // 2, R // 4, R // 8] * 4 + [0] * 4 + [R // 8, R // 4, R // 2, w[0]] * 2 + w[1:]
    for (k, ci, co), n in zip(_lsnet_layers(R), side):
        f += 2.0 * ci * co * (1 if k == "fc" else 9 * n * n)
    return f


def work(case):
    kind = case["kind"]
    if kind in ("serve", "recon", "refine", "lsnet", "train"):
        g, nt = _grid(case), case["tiles"]
        x, crop = 32.0 * g.R * g.R * nt, 16.0 * g.res * g.res * nt
        weights = 4.0 * sum(co * (9 * ci + 1) for ci, co in UNET)
    if kind in ("serve", "recon"):
        b = 18.0 * float(_counts(case).sum()) + 4 * nt + x + 12 * nt
        if kind == "recon":
            return {"bytes": b, "flops": 0.0}
        return {"bytes": b + weights / 2 + crop, "flops": _unet_flops(g.res, g.pad) * nt}
    if kind == "refine":
        return {"bytes": x + weights + 2 * crop + 8 * nt, "flops": _unet_flops(g.res, g.pad) * nt}
    if kind == "lsnet":
        p = sum(co * ((ci if k == "fc" else 9 * ci) + 1) for k, ci, co in _lsnet_layers(g.R))
        return {"bytes": x + 4.0 * p + 2 * crop + 8 * nt, "flops": _lsnet_flops(g.res, g.pad) * nt}
    if kind == "train":
        return {"bytes": x * (2 if case["grad_x"] else 1) + 2 * weights + 2 * crop + 8 * nt,
                "flops": 3 * _unet_flops(g.res, g.pad) * nt}
    n, texels = case["points"], max(1, int(case["tiles_x"] * case["tiles_y"] * case["mapped"])) * 4096.0
    if kind == "splat":
        return {"bytes": 18.0 * n + 24 * texels, "flops": 0.0}
    if kind == "mean":
        return {"bytes": 18.0 * n + 56 * texels, "flops": 0.0}
    return {"bytes": 18.0 * n + 12.0 * case["width"] * case["height"], "flops": 0.0}


# ---------------------------------------------------------------------------
# results in 64 bits
# ---------------------------------------------------------------------------
def _conv(x, w, b):
    """3x3 convolution, zero padding, NHWC, as one matrix product."""
    n, h, k, c = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    cols = torch.cat([p[:, i:i + h, j:j + k] for i in range(3) for j in range(3)], 3)
    return (cols.reshape(-1, 9 * c) @ w.reshape(w.shape[0], -1).T + b).reshape(n, h, k, -1)


def _pool(x):
    n, h, w, c = x.shape
    return x.reshape(n, h // 2, 2, w // 2, 2, c).mean((2, 4))


def _up(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2)


def _split(w, shapes):
    """The flat weights as (matrix, bias) per layer."""
    out, at = [], 0
    for co, fan in shapes:
        out.append((w[at:at + co * fan].reshape(co, fan), w[at + co * fan:at + co * fan + co]))
        at += co * fan + co
    return out


def _crop(x, g):
    return x[:, g.pad:g.pad + g.res, g.pad:g.pad + g.res]


def _unet64(x, w, g):
    """The U-Net's normalised output in 64 bits."""
    p = iter(_split(w, [(co, 9 * ci) for ci, co in UNET]))
    layer = lambda t: torch.relu(_conv(t, *next(p)))  # noqa: E731
    a2 = layer(layer(x))
    a4 = layer(layer(_pool(a2)))
    a6 = layer(layer(_pool(a4)))
    a8 = layer(layer(torch.cat([_up(a6), a4], 3)))
    a10 = layer(layer(torch.cat([_up(a8), a2], 3)))
    return _crop(x, g)[..., [0, 2, 3, 4]] + _crop(_conv(torch.cat([a10, x], 3), *next(p)), g)


def _lsnet64(x, w, g, inputs):
    """The paper's network in 64 bits; absent inputs read as zero."""
    keep = torch.tensor([inputs & b != 0 for b in (1, 2, 4, 4, 4, 8, 8, 8)], device=x.device)
    x = x * keep
    n, p = x.shape[0], iter(_split(w, [(co, ci if k == "fc" else 9 * ci) for k, ci, co in _lsnet_layers(g.R)]))
    feats = []
    for sel in (slice(0, 1), slice(1, 2), slice(2, 5), slice(5, 8)):
        f = x[..., sel]
        for _ in range(4):
            f = _pool(torch.relu(_conv(f, *next(p))))
        feats.append(f.reshape(n, -1))
    fc = lambda t, q: torch.relu(t @ q[0].T + q[1])  # noqa: E731
    merged = torch.cat([fc(torch.cat(feats[:2], 1), next(p)), fc(torch.cat(feats[2:], 1), next(p))], 1)
    heads, side = [fc(merged, next(p)) for _ in range(2)], g.R // 16
    for k in range(2):
        d = heads[k].reshape(n, side, side, 32)
        for _ in range(4):
            d = torch.relu(_conv(_up(d), *next(p)))
        heads[k] = d
    f = torch.relu(_conv(torch.cat([heads[0], heads[1], x], 3), *next(p)))
    f = _conv(torch.relu(_conv(f, *next(p))), *next(p))
    return _crop(x, g)[..., [0, 2, 3, 4]] + _crop(f, g)


def _texture64(y, cz, g):
    r = (g.tile_size / 2 + g.pad * (g.tile_size // g.res)) * g.scale_xy
    return torch.cat([cz[:, None, None, None] + r * y[..., :1], y[..., 1:].clamp(0, 1)], 3)


def _tile64(g, u, v, z, rgb):
    """One window's maps in 64 bits: per texel the nearest point, and the Delaunay interpolant as the linear program
    it is (the convex weights of points that reach the texel with the least sum of squares), by the simplex method."""
    dev = u.device
    key = torch.stack([v, u, -z, -rgb[:, 0], -rgb[:, 1], -rgb[:, 2]], 1)
    key = torch.unique(key, dim=0)  # by (v, u), the largest (z, R, G, B) of a position first
    first = torch.ones(key.shape[0], dtype=torch.bool, device=dev)
    first[1:] = (key[1:, :2] != key[:-1, :2]).any(1)
    key = key[first]
    m, C, R = key.shape[0], g.tile_size // g.res, g.R
    H = g.tile_size // 2 + g.pad * C
    P = torch.cat([key[:, 1:2], key[:, :1]], 1).double()
    val = torch.cat([-key[:, 2:3].double() * g.scale_z + g.offset_z, -key[:, 3:].double() / 65535], 1)
    ax = -H + C // 2 + C * torch.arange(R, device=dev)
    q = torch.stack([ax.repeat(R), ax.repeat_interleave(R)], 1)
    near = torch.cat([(((a[:, None].double() - P) ** 2).sum(2).long() * (1 << 17) + torch.arange(m, device=dev)).min(1)
                      .values & ((1 << 17) - 1) for a in q.split(2048)])
    q = q.double()
    # three far artificial points of a prohibitive cost start the program; a texel that keeps one is outside the hull
    far = torch.tensor([[-4.0, -3.0], [4.0, -3.0], [0.0, 5.0]], device=dev, dtype=torch.float64) * H
    A = torch.cat([torch.cat([P, far]), torch.ones((m + 3, 1), device=dev, dtype=torch.float64)], 1)
    cost = torch.cat([(P ** 2).sum(1), torch.full((3,), 1e15, device=dev, dtype=torch.float64)])
    basis = torch.arange(m, m + 3, device=dev).repeat(R * R, 1)
    one = torch.cat([q, torch.ones((R * R, 1), device=dev, dtype=torch.float64)], 1)
    todo = torch.arange(R * R, device=dev)

    def solve(b, rhs):  # barycentric coordinates of rhs [k, 2] in the triangles b [k, 3]
        p0, p1, p2 = (A[b[:, i], :2] for i in range(3))
        cr = lambda s, t: s[:, 0] * t[:, 1] - s[:, 1] * t[:, 0]  # noqa: E731
        area = cr(p1 - p0, p2 - p0)
        return torch.stack([cr(p1 - rhs, p2 - rhs), cr(p2 - rhs, p0 - rhs), cr(p0 - rhs, p1 - rhs)], 1) / area[:, None]

    for _ in range(400):
        b = basis[todo]
        p0, d1, d2 = A[b[:, 0], :2], A[b[:, 1], :2] - A[b[:, 0], :2], A[b[:, 2], :2] - A[b[:, 0], :2]
        c1, c2 = cost[b[:, 1]] - cost[b[:, 0]], cost[b[:, 2]] - cost[b[:, 0]]
        det = d1[:, 0] * d2[:, 1] - d1[:, 1] * d2[:, 0]
        gx, gy = (c1 * d2[:, 1] - c2 * d1[:, 1]) / det, (c2 * d1[:, 0] - c1 * d2[:, 0]) / det
        plane = torch.stack([gx, gy, cost[b[:, 0]] - gx * p0[:, 0] - gy * p0[:, 1]], 1)
        red = cost[None, :m] - plane @ A[:m].T
        red.scatter_(1, b.clamp(max=m - 1), torch.where(b < m, 0.0, red.gather(1, b.clamp(max=m - 1))))
        best, j = red.min(1)
        more = best < -1e-3
        if not bool(more.any()):
            break
        todo, b, j = todo[more], b[more], j[more]
        lam, d = solve(b, q[todo]), solve(b, A[j, :2])
        ratio = torch.where(d > 1e-13, lam.clamp(min=0) / d, float("inf"))
        b[torch.arange(b.shape[0], device=dev), ratio.argmin(1)] = j
        basis[todo] = b
    lam = solve(basis, q)
    inside = ((basis < m) | (lam.abs() < 1e-12)).all(1)
    lin = (val[basis.clamp(max=m - 1)] * lam[:, :, None]).sum(1)
    lin = torch.where(inside[:, None], lin, val[near])
    cz = lin[(R // 2) * R + R // 2, 0]
    r = H * g.scale_xy
    maps = torch.cat([(lin[:, :1] - cz) / r, (val[near][:, :1] - cz) / r, lin[:, 1:], val[near][:, 1:]], 1)
    return maps.reshape(R, R, 8), cz


def _recon64(case, seed):
    g, x, y, z, rgb, tiles = _sparse(case, seed)
    rgb, S = rgb.int() & 0xFFFF, g.tile_size
    H = S // 2 + g.pad * (S // g.res)
    out = torch.empty((len(tiles), g.R, g.R, 8), dtype=torch.float64, device="cuda")
    czs = torch.empty(len(tiles), dtype=torch.float64, device="cuda")
    for k, t in enumerate(tiles.tolist()):
        u, v = x - (t % g.tiles_x * S + S // 2), y - (t // g.tiles_x * S + S // 2)
        w = torch.nonzero((u >= -H) & (u < H) & (v >= -H) & (v < H))[:, 0]
        out[k], czs[k] = _tile64(g, u[w].long(), v[w].long(), z[w].long(), rgb[w].long())
    return g, out, czs


def _loss64(y, s, g):
    r = (g.tile_size / 2 + g.pad * (g.tile_size // g.res)) * g.scale_xy
    t = s["target"].double()
    t = torch.cat([(t[..., :1] - s["cz"][:, None, None, None]) / r, t[..., 1:]], 3)
    d = torch.where(torch.isnan(t), 0.0, y - torch.nan_to_num(t))
    e = d.abs() if s["loss"] == ls.LOSS_L1 else torch.where(d.detach() ** 2 <= 1, d ** 2, torch.ones_like(d))
    return e[..., 0].sum(), e[..., 1:].sum()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("recon", "serve"):
        per_tile = float(_counts(case).mean()) * (1 + 2 * case["pad"] / 64) ** 2
        if case["tiles"] > 300 or case["tiles"] * per_tile > 150_000:
            return None
        g, x, cz = _recon64(case, seed)
        out = {"x": x, "cz": cz, "status": None}
        if kind == "serve":
            w = _unet_weights(seed).double()
            y = torch.cat([_unet64(x[a:a + 16], w, g) for a in range(0, len(x), 16)])
            out["tex"] = _texture64(y, cz, g)
        return out
    if kind in ("refine", "lsnet"):
        s = prepare(case, seed)
        g, w = s["grid"], s["w"].double()
        net = (lambda t: _unet64(t, w, g)) if kind == "refine" else \
            (lambda t: _lsnet64(t, w, g, INPUTS[case["inputs"]]))
        y = torch.cat([net(t.double()) for t in s["x"].split(16)])
        return {"y": y, "tex": _texture64(y, s["cz"], g)}
    if kind == "train":
        s = prepare(case, seed)
        g, w = s["grid"], s["w"].detach().double().requires_grad_(True)
        nh = case["tiles"] * g.res * g.res
        ys, loss, gw, gx = [], 0.0, torch.zeros_like(w), []
        for a in range(0, case["tiles"], 8):
            x = s["x"].detach()[a:a + 8].double().requires_grad_(case["grad_x"])
            part = {"target": s["target"][a:a + 8], "cz": s["cz"][a:a + 8], "loss": s["loss"]}
            y = _unet64(x, w, g)
            eh, ec = _loss64(y, part, g)
            e = (eh / nh + ec / (3 * nh)) / 2
            grads = torch.autograd.grad(e, [w, x] if case["grad_x"] else [w])
            gw += grads[0]
            gx += list(grads[1:])
            ys.append(y.detach())
            loss += float(e)
        # BF16 gradients differ from these by the rounded network's flipped ReLU units: held to the start's alone
        bf = case["dtype"] == "bf16"
        grads = [None if bf else gw] + ([None if bf else torch.cat(gx)] if case["grad_x"] else [])
        return {"y": torch.cat(ys), "loss": loss, "grads": grads}
    if kind == "splat":
        s = prepare(case, seed)
        cell, ok = _cells(s, case)
        z, c = s["points"][2].long(), (s["points"][3].int() & 0xFFFF) >> 8
        key = (z << 32) | (c[:, 0] << 24 | c[:, 1] << 16 | c[:, 2] << 8 | 0xFF).long() & 0xFFFFFFFF
        top = torch.full((s["slots"] * 4096,), -(1 << 62), dtype=torch.int64, device="cuda")
        top.scatter_reduce_(0, cell[ok], key[ok], "amax")
        g = s["grid"]
        tex = torch.stack([(top >> 32).double() * g.scale_z + g.offset_z] +
                          [((top >> b) & 255).double() / 255 for b in (24, 16, 8)], 1)
        tex = torch.where((top > -(1 << 62))[:, None], tex, s["tex"].reshape(-1, 4).double())
        return {"keys": None, "dropped": None, "tex": tex.reshape(s["tex"].shape)}
    if kind == "mean":
        s = prepare(case, seed)
        cell, ok = _cells(s, case)
        g, k = s["grid"], s["slots"] * 4096
        n = torch.bincount(cell[ok], minlength=k).double()
        cols = [s["points"][2].double()] + [(s["points"][3][:, i].int() & 0xFFFF).double() for i in range(3)]
        sums = [torch.zeros(k, dtype=torch.float64, device="cuda").index_add_(0, cell[ok], v[ok]) / n for v in cols]
        tex = torch.stack([sums[0] * g.scale_z + g.offset_z] + [v / 65535 for v in sums[1:]], 1)
        return {"acc": None, "dropped": None, "tex": tex.reshape(s["slots"], 64, 64, 4)}
    return None  # the point renderer's outputs are whole numbers


def _cells(s, case):
    """Texel index [slot][row][column] of every point, and whether its tile has a slot."""
    x, y = (torch.div(v, 1000, rounding_mode="floor").long() for v in s["points"][:2])
    slot = s["slot"][(y // 64) * case["tiles_x"] + x // 64].long()
    return slot * 4096 + (y % 64) * 64 + x % 64, slot >= 0
