"""Cases the framework's speed is measured on: calls of its public entry points over the sizes they are used at.

A case names an entry point, a problem shape, the band operators and the head allocation (a text with one hexadecimal
band mask per head, or the timestep `t` that the router gets).  Inputs follow the synthetic recipe of the benchmark
(low-frequency fields plus noise); sizes are the repository's own workloads and generic ones around them.
"""
import math

import numpy as np
import torch

from paper_2604_22808_amd import binding as B
from paper_2604_22808_amd import workloads as WL

SOFT = dict(low_num=1, low_den=4, mid_num=1, mid_den=2, mid_block0=1, softmax_scale=0.0)


def _case(name, entry, dtype, batch, heads, d, grid, band, alloc="", t=0.0, d_model=0, haar=False, bands=3):
    c = dict(name=name, entry=entry, dtype=dtype, batch=batch, heads=heads, head_dim=d, T=grid[0], H=grid[1], W=grid[2],
             compress=band["low_compress"], block=band["mid_block"], diag=band["mid_diag"], stride=band["mid_stride"],
             window=band["high_window"], summary=band["n_summary"], alloc=alloc, t=t, d_model=d_model, haar=haar, bands=bands)
    if not name:
        del c["name"]
    return c


def _workload(name, wl, entry, alloc="", t=0.0, d_model=0, heads=None):
    w = WL.WORKLOADS[wl]
    return _case(name, entry, w.dtype, w.batch, heads or w.heads, w.head_dim, w.grid, w.band, alloc, t, d_model)


def _band(compress, block, diag, stride, window, summary):
    return dict(low_compress=compress, mid_block=block, mid_diag=diag, mid_stride=stride, high_window=window, n_summary=summary)


def listed():
    return [
        # smallest call: the fp32 configuration on a toy grid, where launches and host work are all there is
        _workload("f32_256_tokens", "tiny_f32", "forward", alloc="14"),
        # fp32 on a latent grid with odd axes: what a user runs who wants no fp16 range limit
        _case("f32_odd_grid", "forward", "f32", 1, 4, 64, (9, 30, 45), _band(4, 16, 1, 8, 128, 8), alloc="1244"),
        # bf16 on a grid the matrix-core path does not take (axes that are no multiples of 16), several bands per head
        _case("bf16_odd_grid", "forward", "bf16", 1, 6, 128, (7, 22, 40), _band(4, 64, 1, 8, 200, 16), alloc="122347"),
        # a short clip, allocation fixed: launch latency of the matrix-core path
        _workload("16k_fixed", "16k", "forward", alloc="11222444"),
        # a medium clip, router in the loop, early denoising (most heads low)
        _workload("64k_routed", "64k", "routed", t=0.9),
        # a batch of two on a grid of no powers of two, heads with one, several and no bands
        _case("ragged_batch2_mixed", "forward", "bf16", 2, 12, 128, (32, 48, 80), _band(4, 128, 2, 16, 333, 24), alloc="111222443670"),
        # four bands (second block-sparse band), one band per head
        _case("four_bands_64k", "forward", "bf16", 1, 12, 64, (16, 64, 64), _band(4, 64, 1, 16, 256, 16), alloc="111222888444", bands=4),
        # a long clip: early denoising through the router, late denoising (most heads high) with the allocation given
        _workload("256k_routed", "256k", "routed", t=0.9),
        _workload("256k_high_heavy", "256k", "forward", alloc="11" + "2" * 5 + "4" * 17),
        # the benchmark's own workload: a million tokens, router in the loop
        _workload("1m_routed", "1m", "routed", t=0.5),
        # the whole layer with its four projections folded in
        _workload("projected_256k", "256k", "projected", alloc="1" * 6 + "2" * 6 + "4" * 4, d_model=2048, heads=16),
        # the dense comparison, at a size a sweep would run it at
        _case("dense_32k", "dense", "bf16", 1, 8, 128, (32, 32, 32), WL.WORKLOADS["256k"].band),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _grid(rng, tokens):
    """A grid the matrix-core path takes, near `tokens` tokens."""
    axes = [tuple(16 * max(1, min(8, round(_log(rng, 0.7, 8.4)))) for _ in range(3)) for _ in range(60)]
    return min(axes, key=lambda g: abs(math.log(g[0] * g[1] * g[2] / tokens)))


def _masks(rng, heads, bands):
    """Most heads run one band, some several, a few none."""
    weight = [rng.uniform(0.2, 1.0) for _ in range(bands)]
    out = ""
    for _ in range(heads):
        u = rng.random()
        out += "%x" % (1 << rng.choices(range(bands), weight)[0] if u < 0.85 else rng.randrange(1 << bands))
    return out


def draw(rng):
    entry = rng.choice(["forward"] * 3 + ["routed"] * 3 + ["projected", "dense", "f32", "odd"])
    if entry in ("f32", "odd"):
        f32 = entry == "f32"
        grid = (rng.randint(3, 12), rng.randint(6, 32), rng.randint(6, 48))
        d, heads = rng.choice([32, 64, 128]), rng.randint(1, 6)
        band = _band(rng.choice([2, 4]), rng.choice([8, 16, 64]), 1, rng.randint(4, 12), rng.randint(16, 256), rng.randint(2, 16))
        return _case("", "forward", "f32" if f32 else "bf16", 1, heads, d, grid, band, alloc=_masks(rng, heads, 3))
    d, heads, batch = rng.choice([64, 128]), round(_log(rng, 3, 24)), rng.choice([1, 1, 1, 2])
    most = 2.0 ** (29 if entry == "projected" else 30)
    tokens = min(2 ** 20, max(8192, _log(rng, 2.0 ** 23, most) / (batch * heads * d)))
    if entry == "dense":
        tokens = _log(rng, 4096, min(49152, math.sqrt(4e12 / (4 * d * batch * heads))))
    grid = _grid(rng, tokens)
    n = grid[0] * grid[1] * grid[2]
    haar = all(a & (a - 1) == 0 for a in grid) and rng.random() < 0.3
    bands = 4 if entry == "forward" and rng.random() < 0.25 else 3
    block = rng.choice([64, 128])
    stride = max(4, round(n * 7 / 64 / block / rng.uniform(12, 32)))   # 12 to 32 strided key blocks per query block
    band = _band(rng.choice([2, 4, 8]), block, rng.randint(1, 2), stride, rng.randint(100, 600), rng.choice([8, 16, 24, 32, 50, 64]))
    alloc = "" if entry in ("routed", "dense") else _masks(rng, heads, bands)
    t = round(rng.uniform(0.05, 0.95), 3) if entry == "routed" else 0.0
    d_model = 0
    if entry == "projected":
        batch, d_model = 1, 64 * max(1, round(heads * d / 64 * rng.uniform(0.5, 1.0)))
    return _case("", entry, "bf16", batch, heads, d, grid, band, alloc, t, d_model, haar, bands)


def _cfg(c):
    return B.make_cfg(**SOFT, low_compress=c["compress"], mid_block=c["block"], mid_diag=c["diag"], mid_stride=c["stride"],
                      high_window=c["window"], n_summary=c["summary"], transform=int(c["haar"]),
                      mid2_num=3 if c["bands"] == 4 else 0, mid2_den=4)


def _context(c, path=B.PATH_AUTO):
    return B.Context(c["batch"], c["heads"], c["head_dim"], (c["T"], c["H"], c["W"]), B.F32 if c["dtype"] == "f32" else B.BF16,
                     _cfg(c), path)


def prepare(case, seed):
    c = case
    wl = WL.Workload("", c["dtype"], c["batch"], c["heads"], c["head_dim"], (c["T"], c["H"], c["W"]), {}, {}, seed)
    s = {"entry": c["entry"], "ctx": _context(c), "alloc": np.array([int(m, 16) for m in c["alloc"]], np.int32), "t": c["t"]}
    if c["entry"] == "projected":
        dm, hd = c["d_model"], c["heads"] * c["head_dim"]
        import dataclasses
        x = WL.qkv_torch(dataclasses.replace(wl, heads=dm // 64, head_dim=64))[0]
        s["x"] = x.permute(0, 2, 1, 3).reshape(c["batch"], -1, dm).contiguous()
        gen = torch.Generator(device="cuda").manual_seed(seed)
        s["w"] = [(torch.randn(sh, device="cuda", generator=gen) / sh[0] ** 0.5).to(torch.bfloat16)
                  for sh in ((dm, hd), (dm, hd), (dm, hd), (hd, dm))]
        s["out"] = torch.empty_like(s["x"])
    else:
        s["q"], s["k"], s["v"] = WL.qkv_torch(wl)
        s["out"] = torch.empty_like(s["q"])
    if c["entry"] == "routed":
        s["router"] = WL.router_weights()
    return s


def run(s):
    ctx, entry = s["ctx"], s["entry"]
    if entry == "routed":
        alloc, pi = ctx.forward_routed(s["q"], s["k"], s["v"], s["t"], *s["router"], s["out"])
        return s["out"], alloc, pi
    if entry == "projected":
        return ctx.forward_projected(s["x"], *s["w"], s["alloc"], s["out"])
    if entry == "dense":
        return ctx.dense_forward(s["q"], s["k"], s["v"], s["out"])
    return ctx.forward(s["q"], s["k"], s["v"], s["alloc"], s["out"])


def _expected_masks(c, ctx):
    """The allocation the router gives a case in expectation: its statistics from the recipe's spectral variances."""
    var = WL.amplitude(c["T"], c["H"], c["W"]).reshape(-1) ** 2 + 0.01
    x = np.repeat([math.log(1e-6 + var[ctx.band_index(l)].mean()) for l in range(3)], 64)
    a = 1000.0 * c["t"] * 10000.0 ** (-2.0 * np.arange(32) / 64)
    w1, b1, w2, b2 = WL.router_weights()
    z = np.maximum(np.concatenate([x - x.mean(), np.sin(a), np.cos(a)]) @ w1 + b1, 0.0) @ w2 + b2
    z = np.exp(z + 1.5 * (2 * c["t"] - 1) * np.array([1.0, 0.0, -1.0]))
    share = z / z.sum() * (c["heads"] - 3)
    n = np.floor(share).astype(int)
    for l in np.argsort(-(share - n), kind="stable")[:c["heads"] - 3 - n.sum()]:
        n[l] += 1
    return [1] * (1 + n[0]) + [2] * (1 + n[1]) + [4] * (1 + n[2])


def work(case):
    c = case
    N, d, S = c["T"] * c["H"] * c["W"], c["head_dim"], c["batch"] * c["heads"]
    size = 4 if c["dtype"] == "f32" else 2
    if c["entry"] == "dense":
        return {"bytes": 4 * S * N * d * size, "flops": 4.0 * d * N * N * S}
    ctx = _context(c, B.PATH_TABLES_ONLY)
    n = ctx.band_sizes()
    masks = _expected_masks(c, ctx) if c["entry"] == "routed" else [int(m, 16) for m in c["alloc"]]

    def blocks(rp_ci, rows):
        rp, ci = rp_ci
        length = np.minimum(c["block"], rows - c["block"] * np.arange(len(rp) - 1)).astype(float)
        return float((np.repeat(length, np.diff(rp)) * length[ci]).sum())

    w = min(c["window"], n[2] - 1) if n[2] else 0
    pairs = [math.ceil(n[0] / c["compress"]) ** 2, blocks(ctx.mid_blocks(), n[1]), n[2] * (2 * w + 1) - w * (w + 1)]
    if c["bands"] == 4:
        pairs.append(blocks(ctx.mid2_blocks(), n[3]))
    m = [min(c["summary"], x) for x in n]
    flops = 0.0
    for mask in masks:   # the bands' operators and their exchange with the other bands' summary tokens
        for l in range(len(n)):
            if mask >> l & 1:
                flops += c["batch"] * 4.0 * d * (pairs[l] + n[l] * (sum(m) - m[l]))
    fast = 2.5 * N * math.log2(N)   # a fast transform of one channel
    if c["entry"] == "projected":
        dm = c["d_model"]
        flops += 2 * c["batch"] * dm * fast
        for l in range(len(n)):
            runs = sum(mask >> l & 1 for mask in masks)
            flops += c["batch"] * 2.0 * n[l] * dm * (4 * d * runs + (dm if runs < len(masks) else 0))
        return {"bytes": 2 * c["batch"] * N * dm * size + 4 * dm * c["heads"] * d * size, "flops": flops}
    return {"bytes": 4 * S * N * d * size, "flops": flops + 4 * S * d * fast}


def tolerance(case):
    # Measured: fp32 against 64 bits rel 2.4e-7, max 1.3e-6 on 12K tokens (sums grow with the axes and windows drawn);
    # bf16 results against 64 bits rel 1.8e-3, two paths' bf16 results one last place (2^-7) apart at most.
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1e-5}
    return {"rel": 7e-3, "max": 3e-2}
