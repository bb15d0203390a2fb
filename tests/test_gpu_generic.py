"""The generic fp32 kernels at the edges of their tiles, against the fp64 oracle on whole forwards.

Tolerance: 1e-5 (max-abs and relative L2) as for the fp32 configuration: sums of at most a few hundred terms of
magnitude 1 in fp32 stay below 1e-6, the exponentials below 2e-7 relative."""
import numpy as np
import pytest

from oracle import freqformer as O
from paper_2604_22808_amd import binding as B
from paper_2604_22808_amd import workloads as WL
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _check(grid, d, heads, alloc, dtype="f32", **band):
    rng = np.random.default_rng(5)
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, **band)
    N = int(np.prod(grid))
    q, k, v = (WL.round_to_io(0.7 * rng.standard_normal((1, heads, N, d)), dtype) for _ in range(3))
    ctx = B.Context(1, heads, d, grid, B.F32 if dtype == "f32" else B.BF16, B.make_cfg(**cfgd), path=B.PATH_GENERIC)
    got = U.run_forward(ctx, q, k, v, dtype, alloc)
    want = O.forward(q, k, v, grid, O.BandConfig(**cfgd), alloc)
    mx, rl = U.errors(got, want)
    print(f"generic {grid} d={d} {dtype} {band}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    tol = (1e-5, 1e-5) if dtype == "f32" else U.TOL["bf16"]
    assert mx <= tol[0] and rl <= tol[1], (mx, rl)


@pytest.mark.parametrize("d", [1, 30, 32, 64, 100, 128, 132, 256])
def test_generic_attention_head_dims(d):
    """Head dimensions below, at and above each channel tile, multiples of four and not (unaligned rows)."""
    _check((5, 9, 11), d, 2, (6, 7), mid_block=17, mid_stride=2, high_window=41, n_summary=5)


@pytest.mark.parametrize("block,window,c", [(1, 0, 1), (15, 15, 3), (16, 31, 4), (32, 32, 7), (33, 64, 2), (64, 5000, 5)])
def test_generic_attention_blocks_and_windows(block, window, c):
    """Block edges around the 16- and 32-row query tiles and the 32-key tiles, windows of nothing and of everything, on a
    grid large enough for the 32-row tiles (33 to 260 rows in the mid band, thousands in the high band)."""
    _check((7, 24, 26), 64, 2, (7, 7), mid_block=block, mid_stride=3, high_window=window, n_summary=9, low_compress=c)


@pytest.mark.parametrize("dtype,path,grid", [("f32", B.PATH_GENERIC, (7, 24, 26)), ("bf16", B.PATH_GENERIC, (5, 9, 11)),
                                             ("bf16", B.PATH_MFMA, (16, 32, 48))])
def test_windows_of_everything(dtype, path, grid):
    """Every window from one row short of the band's length up is the whole band, up to the longest that a configuration can hold."""
    rng = np.random.default_rng(8)
    N = int(np.prod(grid))
    x = [WL.round_to_io(0.7 * rng.standard_normal((1, 1, N, 64)), dtype) for _ in range(3)]
    cfgd = dict(WL.WORKLOADS["16k"].band)
    n = len(O.band_partition(*grid, O.BandConfig(**cfgd))[2])
    outs = []
    for window in (n - 1, n, n + 1, 2 ** 31 - n, 2 ** 31 - 2, 2 ** 31 - 1):
        ctx = B.Context(1, 1, 64, grid, B.F32 if dtype == "f32" else B.BF16, B.make_cfg(**dict(cfgd, high_window=window)), path=path)
        outs.append(U.run_forward(ctx, *x, dtype, (4,)))
        ctx.destroy()
        assert np.array_equal(outs[-1], outs[0]), window
    mx, rl = U.errors(outs[0], O.forward(*x, grid, O.BandConfig(**dict(cfgd, high_window=n)), (4,)))
    print(f"window of everything {dtype} {grid}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL[dtype][0] and rl <= U.TOL[dtype][1], (mx, rl)


@pytest.mark.parametrize("block,window", [(16, 48), (48, 100), (80, 17), (40, 16)])
def test_generic_attention_of_large_scores(block, window):
    """Scores of up to about +-40 before the softmax (rounded at 2^-24 of themselves: 2.4e-6 in a probability), block lists whose
    tiles follow one another and not, windows with and without tiles that need no mask."""
    _check((7, 24, 26), 64, 2, (6, 7), mid_block=block, mid_stride=2, high_window=window, n_summary=9, softmax_scale=2.0)


@pytest.mark.parametrize("block", [100, 1190, 1200, 100000, 2 ** 31 - 1])
def test_generic_attention_blocks_beyond_the_band(block):
    """Mid blocks of which the last is cut short by the band (1,199 rows), down to one block that holds all of it (a dense mid
    band) or is longer than it by any amount: the keys and query tiles end with the band."""
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, mid_block=block)
    assert len(O.band_partition(9, 26, 44, O.BandConfig(**cfgd))[1]) == 1199
    _check((9, 26, 44), 64, 2, (2, 6), mid_block=block, mid_diag=0, mid_stride=3, n_summary=5)


@pytest.mark.parametrize("grid,d,dtype", [((1, 15, 16), 4, "f32"), ((17, 3, 31), 6, "bf16"), ((2, 64, 65), 12, "f32"),
                                          ((130, 5, 4), 20, "bf16"), ((3, 4, 200), 33, "f32")])
def test_generic_axis_lengths(grid, d, dtype):
    """Axis lengths around the 16-row steps and the 64-row groups of an axis pass, beyond two groups, and head dimensions
    that are no multiple of the 4 (unaligned) or 64 (several slabs per wave) adjacent columns."""
    _check(grid, d, 3, (0, 5, 7), dtype, n_summary=3)


# T and H axes in one pass: T of one step of four rows with and without a remainder up to four, H of one to four tiles, the most rows that
# fit a workgroup and one too many; rows of whole 64-column groups, less than one, a remainder of no multiple of four
@pytest.mark.parametrize("grid,d,dtype", [((1, 2, 3), 64, "f32"), ((4, 16, 5), 32, "bf16"), ((5, 17, 3), 33, "f32"), ((16, 26, 2), 20, "bf16"),
                                          ((6, 64, 3), 12, "f32"), ((12, 34, 3), 36, "f32"), ((13, 34, 3), 36, "f32"), ((3, 49, 4), 6, "bf16")])
def test_generic_axes_in_pairs(grid, d, dtype):
    """Outputs against the oracle, and the same bits wherever the tensors start."""
    import torch
    rng = np.random.default_rng(9)
    N, alloc, tdt = int(np.prod(grid)), (1, 6, 4), torch.float32 if dtype == "f32" else torch.bfloat16
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, n_summary=3)
    ctx = B.Context(1, 3, d, grid, B.F32 if dtype == "f32" else B.BF16, B.make_cfg(**cfgd), path=B.PATH_GENERIC)
    host = [WL.round_to_io(0.7 * rng.standard_normal((1, 3, N, d)), dtype) for _ in range(3)]
    outs = []
    for skip in (0, 1):
        q, k, v, out = (torch.zeros(x.size + 8, dtype=tdt, device="cuda")[skip:skip + x.size].view(x.shape).copy_(torch.from_numpy(x))
                        for x in host + [np.zeros_like(host[0])])
        ctx.forward(q, k, v, alloc, out)
        outs.append(U.to_host64(out))
    assert np.array_equal(outs[0], outs[1])
    mx, rl = U.errors(outs[0], O.forward(*host, grid, O.BandConfig(**cfgd), alloc))
    print(f"generic pairs {grid} d={d} {dtype}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL[dtype][0] and rl <= U.TOL[dtype][1], (mx, rl)


@pytest.mark.parametrize("bands", [3, 4])
def test_generic_branches_in_launches_of_their_own(bands):
    """One launch per branch: the stages are the branches' own and the outputs the same bits as from one launch."""
    import torch
    grid, d, alloc = (9, 20, 24), 64, (1, 2, 4, 7 if bands == 3 else 14)
    gen = torch.Generator(device="cuda").manual_seed(15)
    q, k, v = (torch.randn((1, 4, int(np.prod(grid)), d), device="cuda", generator=gen) for _ in range(3))
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, high_window=50, **(dict(mid2_num=3, mid2_den=4) if bands == 4 else {}))
    ctx = B.Context(1, 4, d, grid, B.F32, B.make_cfg(**cfgd), path=B.PATH_GENERIC)
    outs, names = [], []
    for mode in (B.LAUNCH_FUSED, B.LAUNCH_SEPARATE):
        ctx.set_launch_mode(mode)
        ctx.set_stage_timing(True)
        outs.append(torch.empty_like(q))
        ctx.forward(q, k, v, alloc, outs[-1])
        torch.cuda.synchronize()
        names.append([n for n, _ in ctx.stage_times() if n.endswith("attention") or n.endswith("fused")])
    assert names == [["band_attention_fused"], ["low_attention", "mid_attention", "high_attention"]], names
    assert torch.equal(*outs)


@pytest.mark.parametrize("d,m,c", [(64, 1, 5), (30, 2, 3)])
def test_generic_pooling_of_long_chunks(d, m, c):
    """Summary chunks above 1 MB (10,000 rows and more of the high band) are pooled in parts; rows of 16 bytes and of single
    elements; a compression factor that leaves a shorter last group."""
    _check((9, 40, 50), d, 2, (1, 3), n_summary=m, low_compress=c, mid_block=64, mid_stride=16, high_window=4)


@pytest.mark.parametrize("alloc", [(1, 2), (5, 6)])
def test_matrix_core_pooling_of_long_chunks(alloc):
    """The same on fp16 rows: one summary token per band, 1.8 MB per high-band chunk at 16K tokens; the low band's outputs
    written to whole groups by the band operator, with and without the exchange inside its items."""
    wl = WL.WORKLOADS["16k"]
    q, k, v = (WL.round_to_io(x, wl.dtype) for x in WL.qkv_numpy(wl, heads=[0, 3]))
    ctx, band = U.make_ctx(wl, heads=2, n_summary=1, low_compress=7)
    got = U.run_forward(ctx, q, k, v, wl.dtype, alloc)
    mx, rl = U.errors(got, O.forward(q, k, v, wl.grid, U.oracle_cfg(band), alloc))
    print(f"16k m=1 c=7 {alloc}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= 2e-2 and rl <= 5e-3, (mx, rl)


@pytest.mark.parametrize("c", [16, 17, 2 ** 31 - 1])
@pytest.mark.parametrize("dtype,path,d", [("bf16", B.PATH_MFMA, 64), ("f32", B.PATH_GENERIC, 64), ("f32", B.PATH_GENERIC, 6)])
def test_long_low_band_groups(dtype, path, d, c):
    """Low-band groups whose rows the band operator writes itself (up to 16), the first longer one (the last group shorter
    still) and a group length far beyond the band; with and without the exchange inside the band items."""
    rng = np.random.default_rng(6)
    grid, alloc = (16, 16, 32), (1, 3)
    cfgd = dict(WL.WORKLOADS["16k"].band, low_compress=c)
    q, k, v = (WL.round_to_io(0.7 * rng.standard_normal((1, 2, int(np.prod(grid)), d)), dtype) for _ in range(3))
    ctx = B.Context(1, 2, d, grid, B.F32 if dtype == "f32" else B.BF16, B.make_cfg(**cfgd), path=path)
    mx, rl = U.errors(U.run_forward(ctx, q, k, v, dtype, alloc), O.forward(q, k, v, grid, O.BandConfig(**cfgd), alloc))
    print(f"low groups of {c} {dtype} d={d}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL[dtype][0] and rl <= U.TOL[dtype][1], (mx, rl)


@pytest.mark.parametrize("dtype,path,grid,skip", [("f32", B.PATH_GENERIC, (5, 9, 11), 1), ("bf16", B.PATH_GENERIC, (5, 9, 11), 1),
                                                  ("bf16", B.PATH_MFMA, (16, 32, 32), 2)])
def test_tensors_that_start_between_16_byte_pieces(dtype, path, grid, skip):
    """Contiguous views that start `skip` elements into their storage: no kernel may take their alignment for granted."""
    import torch
    rng = np.random.default_rng(7)
    N, d, alloc = int(np.prod(grid)), 64, (3, 4)
    cfgd = dict(WL.WORKLOADS["16k"].band)
    ctx = B.Context(1, 2, d, grid, B.F32 if dtype == "f32" else B.BF16, B.make_cfg(**cfgd), path=path)
    host = [WL.round_to_io(0.7 * rng.standard_normal((1, 2, N, d)), dtype) for _ in range(3)]

    def view(x):
        t = torch.zeros(x.size + 8, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        v = t[skip:skip + x.size].view(x.shape)
        return v.copy_(torch.from_numpy(x))
    q, k, v = (view(x) for x in host)
    out = view(np.zeros_like(host[0]))
    ctx.forward(q, k, v, alloc, out)
    mx, rl = U.errors(U.to_host64(out), O.forward(*host, grid, O.BandConfig(**cfgd), alloc))
    print(f"unaligned {dtype} {grid}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL[dtype][0] and rl <= U.TOL[dtype][1], (mx, rl)


@pytest.mark.parametrize("dtype,path,grid,d", [("f32", B.PATH_GENERIC, (3, 10, 12), 8), ("bf16", B.PATH_MFMA, (16, 16, 16), 64)])
def test_more_than_256_slices(dtype, path, grid, d):
    """Batch x heads beyond the 256 slices whose unused summary tokens are left out: every band is pooled behind the band
    operators."""
    import torch
    heads, batch, N = 130, 2, int(np.prod(grid))
    alloc = [h % 8 for h in range(heads)]
    cfgd = dict(WL.WORKLOADS["16k"].band)
    gen = torch.Generator(device="cuda").manual_seed(16)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v = ((0.7 * torch.randn((batch, heads, N, d), device="cuda", generator=gen)).to(t) for _ in range(3))
    ctx = B.Context(batch, heads, d, grid, B.F32 if dtype == "f32" else B.BF16, B.make_cfg(**cfgd), path=path)
    out = torch.empty_like(q)
    ctx.forward(q, k, v, alloc, out)
    pick = [0, 1, 2, 3, 4, 5, 6, 7, 122, 125, 129]
    got, qh, kh, vh = (U.to_host64(x[:, pick]) for x in (out, q, k, v))
    want = O.forward(qh, kh, vh, grid, O.BandConfig(**cfgd), [alloc[h] for h in pick])
    mx, rl = U.errors(got, want)
    print(f"{batch * heads} slices {dtype}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    # Summary tokens of white noise make outputs of up to 10, where a bf16 is rounded by up to 2^-8 of its value; the other tests'
    # bound is for values below 4, 2^-6 of it that rounding.
    assert mx <= U.TOL[dtype][0] + (2.0 ** -8 * np.abs(want).max() - 2.0 ** -6 if dtype == "bf16" else 0.0), mx
    assert rl <= U.TOL[dtype][1], rl


# every mask of a slice's bands beside slices that need everything: coefficients that are not made (boxes of one row too, Q~ and K~ of an
# idle slice) must not reach an output, whatever lies in the scratch and in LDS; grids whose T and H axes go in one pass and in two, axes of
# length one and H axes around the four rows that a product takes
@pytest.mark.parametrize("grid,d", [((9, 10, 13), 64), ((3, 4, 5), 250), ((5, 13, 24), 50), ((17, 6, 11), 64), ((2, 65, 13), 64), ((16, 1, 67), 64),
                                    ((3, 1, 400), 64), ((15, 2, 40), 64), ((7, 3, 61), 64), ((1, 9, 130), 64), ((8, 40, 1), 250)])
@pytest.mark.parametrize("bands", [3, 4])
def test_generic_boxes_of_all_masks(grid, d, bands):
    import torch
    rng = np.random.default_rng(10)
    N = int(np.prod(grid))
    alloc = tuple(range(1 << bands)) * -(-(1 << 19) // (N * d << bands))
    assert len(alloc) * N * d >= 1 << 19   # (below, everything is made)
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, n_summary=3, **(dict(mid2_num=3, mid2_den=4) if bands == 4 else {}))
    ctx = B.Context(1, len(alloc), d, grid, B.F32, B.make_cfg(**cfgd), path=B.PATH_GENERIC)
    q, k, v = (0.7 * rng.standard_normal((1, len(alloc), N, d)).astype(np.float32).astype(np.float64) for _ in range(3))
    nan = np.full_like(q, np.nan)
    U.run_forward(ctx, nan, nan, nan, "f32", (alloc[-1],) * len(alloc))   # (leaves NaN in all of the scratch, and where its last pass kept the tensor between T and H)
    got = U.run_forward(ctx, q, k, v, "f32", alloc)
    mx, rl = U.errors(got, O.forward(q, k, v, grid, U.oracle_cfg(cfgd), alloc))
    print(f"generic boxes {grid} d={d} bands={bands}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL["f32"][0] and rl <= U.TOL["f32"][1], (mx, rl)


@pytest.mark.parametrize("heads,bands", [(8, 3), (16, 4), (7, 3)])
def test_generic_coefficients_that_were_not_made_read_as_nan(heads, bands):
    """Q~ and K~ of the bands a slice runs, and those made along with them, are coefficients of this forward's inputs; of what was not made
    nothing is handed out that another call left behind.  Below 2^19 elements everything is made."""
    rng = np.random.default_rng(18)
    grid, d = (8, 9, 15), 64
    boxed = heads >= 8
    N = int(np.prod(grid))
    assert (heads * N * d >= 1 << 19) == boxed
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, n_summary=3, **(dict(mid2_num=3, mid2_den=4) if bands == 4 else {}))
    ctx = B.Context(1, heads, d, grid, B.F32, B.make_cfg(**cfgd), path=B.PATH_GENERIC)
    q, k, v = (0.7 * rng.standard_normal((1, heads, N, d)).astype(np.float32).astype(np.float64) for _ in range(3))
    U.run_forward(ctx, v, q, k, "f32", [(1 << bands) - 1] * heads)   # (other coefficients, in all of the scratch)
    alloc = [h % (1 << bands) for h in range(heads)]
    U.run_forward(ctx, q, k, v, "f32", alloc)
    want = [[O.spectral_forward(x[0, h].reshape(grid + (d,))).reshape(N, d) for h in range(heads)] for x in (q, k)]
    index = O.band_partition(*grid, U.oracle_cfg(cfgd))
    for which in range(2):
        for h in range(heads):
            for l in range(bands):
                got = ctx.read_spectral(which, h, l)
                if boxed and alloc[h] >> min(l, 2) == 0:
                    assert np.isnan(got).all(), (which, h, l)
                else:
                    assert U.errors(got, want[which][h][index[l]])[1] <= 1e-5, (which, h, l)


@pytest.mark.parametrize("d,block,window,c", [(64, 16, 32, 4), (30, 5, 7, 17), (128, 40, 300, 1), (256, 16, 20, 3)])
def test_generic_exchange_inside_the_band_launch(d, block, window, c):
    """Slices that run one band each have their exchange in the band's launch; beside a slice that runs two it is a launch of its own.
    The outputs are the oracle's, and those of a slice the same bits either way."""
    rng = np.random.default_rng(12)
    grid, alloc = (7, 12, 14), (1, 2, 4, 0)
    N = int(np.prod(grid))
    cfgd = dict(WL.WORKLOADS["tiny_f32"].band, mid_block=block, high_window=window, low_compress=c, n_summary=11)
    ctx = B.Context(1, 4, d, grid, B.F32, B.make_cfg(**cfgd), path=B.PATH_GENERIC)
    q, k, v = (0.7 * rng.standard_normal((1, 4, N, d)).astype(np.float32).astype(np.float64) for _ in range(3))
    inside, apart = (U.run_forward(ctx, q, k, v, "f32", a) for a in (alloc, alloc[:3] + (6,)))
    assert np.array_equal(inside[:, :3], apart[:, :3])
    mx, rl = U.errors(inside, O.forward(q, k, v, grid, U.oracle_cfg(cfgd), alloc))
    print(f"generic exchange d={d}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL["f32"][0] and rl <= U.TOL["f32"][1], (mx, rl)
