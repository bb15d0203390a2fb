"""Spectral coefficients of the matrix-core path at the edges of the transform passes' tiles, against scipy's orthonormal
DCT-II of the stored bf16 values.

Tolerance 2e-3 relative L2, the bound the other transform tests use: three axis passes whose fp16 matrices and fp16
intermediates each carry a relative rounding error of 2^-12 to 2^-11 (measured 4.6e-4)."""
import numpy as np
import pytest

from oracle import freqformer as O
from paper_2604_22808_amd import binding as B
from paper_2604_22808_amd import workloads as WL
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

ALLOC = (1, 2, 4, 6, 0)   # low box, low+mid box, whole grid (twice), nothing


# W of every number of 32-deep steps with and without a remainder and every number of workgroups per plane; H keeping one to
# four coefficient tiles on the low box, the low+mid box or the whole axis, and more (two passes); both head dimensions; more
# planes than workgroups and fewer
@pytest.mark.parametrize("grid,d", [((16, 16, 16), 64), ((16, 32, 48), 128), ((16, 48, 80), 64), ((32, 64, 112), 64),
                                    ((16, 16, 128), 128), ((16, 128, 32), 64), ((48, 64, 64), 64), ((16, 96, 96), 64),
                                    ((16, 80, 64), 128), ((64, 48, 16), 64), ((16, 32, 96), 64), ((16, 32, 112), 64), ((16, 32, 128), 128), ((16, 64, 96), 64),
                                    ((16, 128, 112), 64)])
def test_spectral_coefficients(grid, d):
    from scipy.fft import dctn
    rng = np.random.default_rng(11)
    N, heads = int(np.prod(grid)), len(ALLOC)
    q, k, v = (WL.round_to_io(rng.standard_normal((1, heads, N, d)), "bf16") for _ in range(3))
    band = WL.WORKLOADS["16k"].band
    ctx = B.Context(1, heads, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    U.run_forward(ctx, q, k, v, "bf16", ALLOC)
    index = O.band_partition(*grid, U.oracle_cfg(band))
    worst = 0.0
    for which, x in enumerate((q, k, v)):
        for h in range(heads):
            want = dctn(x[0, h].reshape(grid + (d,)), type=2, norm="ortho", axes=(0, 1, 2)).reshape(N, d)
            for l, idx in enumerate(index):
                if len(idx) == 0 or (which < 2 and not (ALLOC[h] >> l) & 1):
                    continue   # Q~ and K~ exist on the bands a head runs
                try:
                    got = ctx.read_spectral(which, h, l)
                except B.FreqAttnError as e:   # V~ of a slice without the high band may stop at the low+mid box
                    assert e.status == B.EUNSUPPORTED and which == 2 and l == 2
                    continue
                worst = max(worst, U.errors(got, want[idx])[1])
    print(f"spectral {grid} d={d}: rel-L2 {worst:.3e}", flush=True)
    assert worst <= 2e-3, worst


# whole planes of three and four tiles of H coefficients with one to eight workgroups on a plane, an odd number of them, and a last
# step of a row that is half empty; fewer planes than an XCD has workgroups
@pytest.mark.parametrize("grid,d", [((16, 64, 16), 128), ((16, 48, 48), 128), ((16, 48, 112), 128), ((16, 64, 112), 64), ((16, 64, 128), 64),
                                    ((16, 48, 128), 128)])
def test_spectral_coefficients_of_whole_planes(grid, d):
    test_spectral_coefficients(grid, d)


# a model width that is no power of two times 64: chunks of 64 channels in other places of the XCDs' lists
def test_projected_forward_of_a_model_of_192_channels():
    test_projected_forward_of_narrow_models(192)


# boxes of one and two 16-coefficient tiles per axis (n low and n low+mid heads: enough planes for the one-pass inverse), whole
# planes and parts of planes per workgroup, added to V and - where the box is the whole grid - not; an axis of 48, which is kept
# whole and takes the two passes
@pytest.mark.parametrize("grid,d,n", [((16, 16, 16), 64, 32), ((32, 64, 48), 64, 4), ((16, 64, 32), 128, 4), ((32, 32, 64), 64, 8),
                                      ((16, 128, 64), 64, 4), ((64, 32, 16), 128, 9)])
def test_outputs_of_boxed_inverse(grid, d, n):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(12)
    N, alloc = int(np.prod(grid)), [1] * n + [2] * n
    q, k, v = ((0.5 * torch.randn((1, 2 * n, N, d), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(3))
    band = WL.WORKLOADS["16k"].band
    ctx = B.Context(1, 2 * n, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    out = torch.empty_like(q)
    ctx.forward(q, k, v, alloc, out)
    heads = [0, n - 1, n, 2 * n - 1]
    got, qh, kh, vh = (U.to_host64(x[:, heads]) for x in (out, q, k, v))
    mx, rl = U.errors(got, O.forward(qh, kh, vh, grid, U.oracle_cfg(band), [alloc[h] for h in heads]))
    print(f"boxed inverse {grid} d={d}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= U.TOL["bf16"][0] and rl <= U.TOL["bf16"][1], (mx, rl)


# outputs from whole planes and from boxes through the pass that keeps the output in its accumulators: one to four tiles of rows per
# workgroup, rows in one and two parts (an odd number of tiles among them), every number of tiles of columns, an input row
# whose last step is half empty, fewer planes than an XCD has workgroups and more; and a plane that takes an axis at a time
@pytest.mark.parametrize("grid,d,n", [((16, 48, 80), 64, 1), ((32, 80, 48), 128, 1), ((16, 112, 16), 64, 2), ((16, 128, 64), 128, 1),
                                      ((16, 64, 112), 64, 1), ((48, 64, 64), 64, 3), ((16, 128, 128), 64, 2), ((32, 32, 96), 64, 1),
                                      ((16, 16, 128), 64, 1), ((16, 96, 96), 64, 1)])
def test_outputs_of_one_pass_inverse(grid, d, n):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(19)
    N, alloc = int(np.prod(grid)), [1] * n + [2] * n + [4] * n
    q, k, v = ((0.5 * torch.randn((1, 3 * n, N, d), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(3))
    band = dict(WL.WORKLOADS["16k"].band, n_summary=0, high_window=16)
    ctx = B.Context(1, 3 * n, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    out = torch.empty_like(q)
    ctx.forward(q, k, v, alloc, out)
    # The inverse alone: the band outputs and V~ as the library left them, through scipy's inverse transform.  Tolerance of the
    # other output tests: fp16 matrices and intermediates in three passes (5e-4 relative) and the bf16 rounding of the result.
    from scipy.fft import idctn
    index = O.band_partition(*grid, U.oracle_cfg(band))
    host_v = U.to_host64(v)
    for h in range(3 * n):
        spec = np.zeros((N, d))
        for l, idx in enumerate(index):
            if len(idx) and (alloc[h] >> l) & 1:
                spec[idx] = ctx.read_spectral(3, h, l)
                if alloc[h] != 4:
                    spec[idx] -= ctx.read_spectral(2, h, l)
            elif len(idx) and alloc[h] == 4:
                spec[idx] = ctx.read_spectral(2, h, l)
        want = idctn(spec.reshape(grid + (d,)), type=2, norm="ortho", axes=(0, 1, 2)).reshape(N, d)
        if alloc[h] != 4:
            want += host_v[0, h]
        mx, rl = U.errors(U.to_host64(out[0, h]), want)
        print(f"one-pass inverse {grid} d={d} head {h}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
        assert mx <= U.TOL["bf16"][0] and rl <= U.TOL["bf16"][1], (h, mx, rl)


# boxes of axes that are no powers of two, on every axis: one to three tiles of 32 rows kept of two, three and four, and back; edges at
# other fractions keep 48, 80 and 96 rows, also with more than 64 rows along H (an axis at a time)
@pytest.mark.parametrize("grid,low,mid", [((48, 48, 80), (1, 4), (1, 2)), ((80, 16, 48), (1, 4), (1, 2)), ((96, 96, 16), (1, 4), (1, 2)),
                                          ((112, 16, 112), (1, 4), (1, 2)), ((112, 16, 48), (1, 8), (3, 8)), ((96, 16, 80), (1, 6), (5, 6)),
                                          ((128, 16, 96), (1, 8), (5, 8)), ((128, 48, 16), (1, 2), (3, 4)), ((16, 112, 96), (1, 4), (5, 7)),
                                          ((16, 128, 80), (1, 8), (3, 4)), ((16, 80, 112), (1, 8), (3, 5))])
def test_boxes_of_axes_of_any_length(grid, low, mid):
    import torch
    from scipy.fft import dctn, idctn
    gen = torch.Generator(device="cuda").manual_seed(37)
    N, d, alloc = int(np.prod(grid)), 64, (1, 2, 4)
    q, k, v = ((0.5 * torch.randn((1, 3, N, d), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(3))
    band = dict(WL.WORKLOADS["16k"].band, n_summary=0, high_window=16, low_num=low[0], low_den=low[1], mid_num=mid[0], mid_den=mid[1])
    ctx = B.Context(1, 3, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    out = torch.empty_like(q)
    ctx.forward(q, k, v, alloc, out)
    index, worst = O.band_partition(*grid, U.oracle_cfg(band)), 0.0
    for h, l in enumerate((0, 1, 2)):   # the coefficients each head attends with
        for which, x in enumerate((q, k, v)):
            if len(index[l]):
                want = dctn(U.to_host64(x[0, h]).reshape(grid + (d,)), type=2, norm="ortho", axes=(0, 1, 2)).reshape(N, d)
                worst = max(worst, U.errors(ctx.read_spectral(which, h, l), want[index[l]])[1])
    assert worst <= 2e-3, worst
    for h, l in enumerate((0, 1)):      # the inverse alone, from the band outputs as the library left them
        spec = np.zeros((N, d))
        if len(index[l]):
            spec[index[l]] = ctx.read_spectral(3, h, l) - ctx.read_spectral(2, h, l)
        want = idctn(spec.reshape(grid + (d,)), type=2, norm="ortho", axes=(0, 1, 2)).reshape(N, d) + U.to_host64(v[0, h])
        mx, rl = U.errors(U.to_host64(out[0, h]), want)
        assert mx <= U.TOL["bf16"][0] and rl <= U.TOL["bf16"][1], (h, mx, rl)


# the same bits from the low box, the low+mid box and the whole grid, and after any guess, where axes of 48 to 112 are cut
@pytest.mark.parametrize("grid", [(48, 48, 80), (32, 96, 48), (16, 112, 112)])
def test_outputs_do_not_depend_on_the_box_of_axes_of_any_length(grid, monkeypatch):
    test_outputs_do_not_depend_on_the_box(grid, 1.0, "1", monkeypatch)


# classes of slices that keep different boxes and are small enough to share launches: boxes one, two and four tiles of 16 wide, one to
# four tiles of rows, T axes of which a class keeps a tile of 32 less than the one whose launch it joins, and reads less, a class that is missing
@pytest.mark.parametrize("grid,d,alloc", [((16, 32, 32), 64, (1, 2, 4)), ((16, 64, 64), 128, (1, 2, 4, 6, 0)), ((32, 16, 64), 64, (1, 1, 4)),
                                          ((64, 32, 16), 64, (2, 4, 2)), ((16, 128, 32), 64, (1, 2, 4)), ((16, 32, 128), 64, (1, 2, 4)),
                                          ((16, 48, 64), 64, (1, 2, 4)), ((32, 32, 32), 64, (1, 3, 5)), ((48, 16, 16), 64, (1, 2, 4)), ((80, 16, 32), 64, (1, 2, 2, 0)),
                                          ((112, 32, 16), 128, (1, 2, 4)), ((128, 16, 48), 64, (2, 1, 4)), ((96, 16, 16), 64, (1, 0, 4))])
def test_shared_launches_give_the_bits_of_launches_of_their_own(grid, d, alloc):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(23)
    N, n = int(np.prod(grid)), len(alloc)
    q, k, v = ((0.5 * torch.randn((1, n, N, d), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(3))
    # (no summaries: sums over tokens are split by the number of slices; fewer slices than the small-box inverse takes)
    cfg = B.make_cfg(**dict(WL.WORKLOADS["16k"].band, n_summary=0))
    ctx, one = B.Context(1, n, d, grid, B.BF16, cfg, path=B.PATH_MFMA), B.Context(1, 1, d, grid, B.BF16, cfg, path=B.PATH_MFMA)
    out, alone = torch.empty_like(q), torch.empty((1, 1, N, d), dtype=torch.bfloat16, device="cuda")
    ctx.forward(q, k, v, alloc, out)
    for h in range(n):
        one.forward(*(x[:, h:h + 1].contiguous() for x in (q, k, v)), alloc[h:h + 1], alone)
        torch.cuda.synchronize()
        assert torch.equal(out[0, h], alone[0, 0]), (h, float((out[0, h].float() - alone[0, 0].float()).abs().max()))


# low+mid boxes and whole grids of enough slices to fill the chip, which go through one launch: three and four tiles of rows, W with and
# without a remainder of a step, items that come out even and not
@pytest.mark.parametrize("grid,mid,high", [((16, 64, 64), 11, 2), ((16, 64, 48), 16, 3), ((16, 48, 80), 7, 2), ((16, 48, 96), 6, 3), ((16, 64, 112), 6, 1),
                                           ((32, 64, 128), 4, 2)])
def test_boxes_and_whole_grids_in_one_launch(grid, mid, high):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(37)
    N, d, n = int(np.prod(grid)), 64, mid + high
    alloc = (2,) * mid + (4,) * high
    q, k, v = ((0.5 * torch.randn((1, n, N, d), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(3))
    cfg = B.make_cfg(**dict(WL.WORKLOADS["16k"].band, n_summary=0))   # (sums over tokens are split by the number of slices)
    ctx, one = B.Context(1, n, d, grid, B.BF16, cfg, path=B.PATH_MFMA), B.Context(1, 1, d, grid, B.BF16, cfg, path=B.PATH_MFMA)
    out, alone = torch.empty_like(q), torch.empty((1, 1, N, d), dtype=torch.bfloat16, device="cuda")
    ctx.forward(q, k, v, alloc, out)
    for h in range(n):
        one.forward(*(x[:, h:h + 1].contiguous() for x in (q, k, v)), alloc[h:h + 1], alone)
        torch.cuda.synchronize()
        assert torch.equal(out[0, h], alone[0, 0]), (h, float((out[0, h].float() - alone[0, 0].float()).abs().max()))


@pytest.mark.parametrize("path", [B.PATH_MFMA, B.PATH_GENERIC])
def test_routing_leaves_the_band_outputs_readable(path, monkeypatch):
    """The transforms of a routing call that is no forward use scratch that is not the last forward's result."""
    monkeypatch.setenv("FREQATTN_V_BOX", "1")   # (Q, K and V on the same box also at this size: three tensors per launch)
    rng = np.random.default_rng(13)
    grid, d, alloc = (16, 16, 32), 64, (1, 2, 4)
    band = WL.WORKLOADS["16k"].band
    q, k, v = (WL.round_to_io(rng.standard_normal((1, 3, int(np.prod(grid)), d)), "bf16") for _ in range(3))
    ctx = B.Context(1, 3, d, grid, B.BF16, B.make_cfg(**band), path=path)
    U.run_forward(ctx, q, k, v, "bf16", alloc)
    before = [ctx.read_spectral(3, h, h) for h in range(3)]
    ctx.route_mlp(*(U.to_device(2.0 * x, "bf16") for x in (v, q, k)), 0.5, *WL.router_weights())
    for h in range(3):
        assert np.array_equal(ctx.read_spectral(3, h, h), before[h]), h


# T axes that the statistics of a short pass add up four rows at a time, with band edges at multiples of 4 and between them (5.33 and 10 of
# 16, 10.67 and 20 of 32), on the low+mid box and on the whole grid.  Tolerance as for the other statistics: 5e-3 on logarithms of energies of fp16 spectra.
@pytest.mark.parametrize("low,mid", [((1, 4), (1, 2)), ((1, 3), (5, 8)), ((1, 16), (7, 16))])
@pytest.mark.parametrize("grid,d", [((16, 16, 32), 64), ((16, 48, 32), 128), ((32, 32, 16), 64)])
def test_router_statistics_at_band_edges(grid, d, low, mid, monkeypatch):
    monkeypatch.setenv("FREQATTN_V_BOX", "1")
    rng = np.random.default_rng(29)
    q, k, v = (WL.round_to_io(rng.standard_normal((1, 3, int(np.prod(grid)), d)), "bf16") for _ in range(3))
    band = dict(WL.WORKLOADS["16k"].band, low_num=low[0], low_den=low[1], mid_num=mid[0], mid_den=mid[1])
    ctx = B.Context(1, 3, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    got = ctx.route_mlp(*(U.to_device(x, "bf16") for x in (q, k, v)), 0.5, *WL.router_weights())[2]
    assert np.abs(got - O.band_statistics(q, k, v, grid, O.BandConfig(**band))).max() < 5e-3


# A routed forward whose heads were guessed low, mid and high: the T passes with statistics of the box and of the whole grid share a launch, the box's
# with fewer rows than tiles.  The same output bits as with launches of a class each (no guess), probabilities to 2e-3 as elsewhere (5e-3 on the statistics).
@pytest.mark.parametrize("grid", [(48, 16, 16), (64, 16, 16), (80, 16, 32), (112, 16, 16)])
def test_statistics_of_unequal_boxes_in_one_launch(grid):
    import torch
    rng = np.random.default_rng(37)
    heads, d, t = 4, 64, 0.6
    q, k, v = (WL.round_to_io(rng.standard_normal((1, heads, int(np.prod(grid)), d)), "bf16") for _ in range(3))
    band, w = WL.WORKLOADS["16k"].band, WL.router_weights()
    ctx = B.Context(1, heads, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    x = [U.to_device(a, "bf16") for a in (q, k, v)]
    outs = []
    for guess in (False, True):
        ctx.set_alloc_prediction(guess)
        ctx.forward(*x, [1, 2, 4, 4], torch.empty_like(x[0]))
        out = torch.empty_like(x[0])
        alloc, pi = ctx.forward_routed(*x, t, *w, out)
        want_alloc, want_pi = O.route_mlp(q, k, v, grid, O.BandConfig(**band), t, *w)
        assert np.abs(pi - want_pi).max() < 2e-3 and np.array_equal(alloc, want_alloc)
        outs.append(out)
    assert torch.equal(*outs)


# High-band summaries from the untransformed V of slices that do not run it: one and two groups of 32 chunks.  Tolerance as for the other
# forwards (bf16 rounding of the output 1.6e-3, fp16 spectra 4.6e-4; relative L2 3e-3).
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("m", [1, 31, 32, 33, 64])
def test_summaries_of_bands_that_no_slice_runs(m, d, monkeypatch):
    monkeypatch.setenv("FREQATTN_V_BOX", "1")
    rng = np.random.default_rng(41)
    grid, alloc = (16, 16, 32), (1, 2, 3)
    q, k, v = (WL.round_to_io(rng.standard_normal((1, 3, int(np.prod(grid)), d)), "bf16") for _ in range(3))
    band = dict(WL.WORKLOADS["16k"].band, n_summary=m)
    ctx = B.Context(1, 3, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    got = U.run_forward(ctx, q, k, v, "bf16", alloc)
    assert U.errors(got, O.forward(q, k, v, grid, O.BandConfig(**band), alloc))[1] < 3e-3


# planes of which the boxes go through the one-pass kernel and the whole does not, with a narrow and a wide low+mid box; the last
# one goes through it whole
@pytest.mark.parametrize("grid", [(16, 128, 64), (16, 128, 96), (16, 64, 128), (16, 32, 128)])
@pytest.mark.parametrize("noise,vbox", [(1.0, "1"), (1e-3, "1"), (1e-3, "0")])   # (with little noise the high band's energy has to be taken again, on the whole grid)
def test_outputs_do_not_depend_on_the_box(grid, noise, vbox, monkeypatch):
    """The routed forward computes a head's coefficients on the low+mid box or the whole grid by what it guessed, and the forward
    with the allocation given on the low box where that is enough: the outputs are the same bits after right and wrong guesses."""
    import torch
    monkeypatch.setenv("FREQATTN_V_BOX", vbox)
    gen = torch.Generator(device="cuda").manual_seed(14)
    T, H, W = grid
    wave = [torch.cos(torch.arange(n, device="cuda") * (2.5 / n)) for n in grid]
    smooth = (wave[0][:, None, None] * wave[1][:, None] * wave[2]).reshape(-1, 1)
    q, k, v = ((smooth + noise * torch.randn((1, 6, T * H * W, 64), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(3))
    band = WL.WORKLOADS["64k"].band
    ctx, ref = (B.Context(1, 6, 64, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA) for _ in range(2))
    out, plain = torch.empty_like(q), torch.empty_like(q)
    seen = set()
    for t in (0.05, 0.05, 0.95, 0.95, 0.5, 0.05):   # nothing to guess from; then right and wrong guesses
        alloc, _ = ctx.forward_routed(q, k, v, t, *WL.router_weights(), out)
        ref.forward(q, k, v, alloc, plain)
        torch.cuda.synchronize()
        assert torch.equal(out, plain), (t, list(alloc), float((out.float() - plain.float()).abs().max()))
        seen.add(tuple(int(a) for a in alloc))
    assert len(seen) >= 2, seen   # the sequence really changes the allocation


@pytest.mark.parametrize("skip", [(0, 0, 1, 0), (1, 0, 0, 0), (2, 4, 6, 1)])   # elements in front of q, k, v and out
def test_outputs_do_not_depend_on_where_tensors_start(skip, monkeypatch):
    """Contiguous views that start between 16-byte pieces, some or all: the bits of aligned tensors, by either entry point."""
    import torch
    monkeypatch.setenv("FREQATTN_V_BOX", "1")
    gen = torch.Generator(device="cuda").manual_seed(31)
    grid, d = (16, 64, 64), 64
    shape = (1, 6, int(np.prod(grid)), d)

    def view(x, n):
        t = torch.zeros(x.numel() + 8, dtype=torch.bfloat16, device="cuda")
        return t[n:n + x.numel()].view(shape).copy_(x)
    aligned = [torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3)]
    views, out, want = [view(x, n) for x, n in zip(aligned, skip)], view(torch.zeros_like(aligned[0]), skip[3]), torch.empty_like(aligned[0])
    ctx, ref = (B.Context(1, 6, d, grid, B.BF16, B.make_cfg(**WL.WORKLOADS["64k"].band), path=B.PATH_MFMA) for _ in range(2))
    for t in (0.95, 0.95, 0.05):   # nothing to guess from, a right guess, a wrong one
        alloc, _ = ctx.forward_routed(*views, t, *WL.router_weights(), out)
        ref.forward(*aligned, alloc, want)
        torch.cuda.synchronize()
        assert 1 in alloc and torch.equal(out, want), ("routed", t, list(alloc), float((out.float() - want.float()).abs().max()))
        out.zero_()
        ref.forward(*views, alloc, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want), ("given", t, list(alloc), float((out.float() - want.float()).abs().max()))


@pytest.mark.parametrize("value", [65536.0, float("inf"), float("nan")])
def test_input_outside_fp16_is_reported(value):
    """One input value that fp16 cannot hold, in a plane that several workgroups share."""
    import torch
    ctx, _ = U.make_ctx(WL.WORKLOADS["16k"], path=B.PATH_MFMA)
    q = torch.zeros((1, 8, 16 * 32 * 32, 64), dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    v = q.clone()
    ctx.forward(q, q, v, [4] * 8, out)
    ctx.check_range()
    v[0, 3, 4321, 17] = value
    ctx.forward(q, q, v, [4] * 8, out)
    with pytest.raises(B.FreqAttnError) as e:
        ctx.check_range()
    assert e.value.status == B.ERANGE


@pytest.mark.parametrize("d_model", [64, 128])
def test_projected_forward_of_narrow_models(d_model):
    """A model width of 64 or 128 channels goes through the one-pass transform like a head does."""
    import torch
    rng = np.random.default_rng(17)
    grid, d, heads, alloc = (16, 32, 48), 64, 3, (1, 2, 4)
    N, hd = int(np.prod(grid)), heads * d
    x = WL.round_to_io(0.5 * rng.standard_normal((1, N, d_model)), "bf16")
    w = [WL.round_to_io(rng.standard_normal(s) / np.sqrt(s[0]), "bf16") for s in ((d_model, hd),) * 3 + ((hd, d_model),)]
    band = WL.WORKLOADS["16k"].band
    ctx = B.Context(1, heads, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    dx, *dw = (U.to_device(a, "bf16") for a in [x] + w)
    out = torch.empty_like(dx)
    ctx.forward_projected(dx, *dw, alloc, out)
    mx, rl = U.errors(U.to_host64(out), O.forward_projected(x, *w, grid, O.BandConfig(**band), alloc))
    print(f"projected d_model={d_model}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= 2e-2 and rl <= 5e-3, (mx, rl)


@pytest.mark.parametrize("d_model,heads,alloc", [(256, 4, (1, 2, 4, 0)), (320, 5, (1, 2, 4, 7, 4)), (448, 7, (2, 2, 1, 1, 4, 6, 7)),
                                                 (704, 11, (1, 2, 4) * 3 + (6, 7)), (768, 12, (1, 2, 4) * 4),
                                                 (832, 13, (1, 2, 4) * 4 + (0,))])
def test_projected_forward_of_products_in_wide_tiles(d_model, heads, alloc):
    """Products of 256 rows and columns and more: even and odd numbers of steps of 64, below 12 and from 12 on, one segment and several, tiles whose second
    half is cut short by the columns or the rows, and tiles that span several problems."""
    rng = np.random.default_rng(18)
    grid, d = (16, 32, 32), 64
    N, hd = int(np.prod(grid)), heads * d
    x = WL.round_to_io(0.5 * rng.standard_normal((1, N, d_model)), "bf16")
    w = [WL.round_to_io(rng.standard_normal(s) / np.sqrt(s[0]), "bf16") for s in ((d_model, hd),) * 3 + ((hd, d_model),)]
    band = WL.WORKLOADS["16k"].band
    ctx = B.Context(1, heads, d, grid, B.BF16, B.make_cfg(**band), path=B.PATH_MFMA)
    import torch
    dx, *dw = (U.to_device(a, "bf16") for a in [x] + w)
    out = torch.empty_like(dx)
    ctx.forward_projected(dx, *dw, alloc, out)
    mx, rl = U.errors(U.to_host64(out), O.forward_projected(x, *w, grid, O.BandConfig(**band), alloc))
    print(f"projected d_model={d_model}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= 2e-2 and rl <= 5e-3, (mx, rl)


def test_products_of_large_launches():
    """From four rounds of the chip on products of 12 steps copy as those of fewer do.  Heads that run no band: the layer is X W_V W_O.  Tolerance of the
    other outputs."""
    import torch
    grid, d, heads, d_model = (32, 64, 64), 64, 12, 768
    gen = torch.Generator(device="cuda").manual_seed(31)
    N = int(np.prod(grid))
    x = 0.5 * torch.randn((1, N, d_model), device="cuda", generator=gen, dtype=torch.bfloat16)
    wv, wo = (torch.randn((d_model, d_model), device="cuda", generator=gen, dtype=torch.bfloat16) / d_model ** 0.5 for _ in range(2))
    out = torch.empty_like(x)
    ctx = B.Context(1, heads, d, grid, B.BF16, B.make_cfg(**dict(WL.WORKLOADS["16k"].band, n_summary=0)), path=B.PATH_MFMA)
    ctx.forward_projected(x, wv, wv, wv, wo, [0] * heads, out)
    want = x[0].float() @ (wv.float() @ wo.float())
    mx, rl = U.errors(U.to_host64(out[0]), U.to_host64(want))
    print(f"large launches: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    assert mx <= 2e-2 and rl <= 5e-3, (mx, rl)


def test_projected_forward_of_a_model_of_8192_channels():
    """Rows of the transformed X 4 MB apart and more.  Heads that run no band: the layer is X W_V W_O.  Tolerance of the other outputs."""
    import torch
    grid, d, heads, d_model = (128, 16, 128), 128, 64, 8192
    gen = torch.Generator(device="cuda").manual_seed(29)
    N = int(np.prod(grid))
    x = 0.5 * torch.randn((1, N, d_model), device="cuda", generator=gen, dtype=torch.bfloat16)
    wv, wo = (torch.randn((d_model, d_model), device="cuda", generator=gen, dtype=torch.bfloat16) / d_model ** 0.5 for _ in range(2))
    ctx = B.Context(1, heads, d, grid, B.BF16, B.make_cfg(**WL.WORKLOADS["16k"].band), path=B.PATH_MFMA)
    out = torch.empty_like(x)
    ctx.forward_projected(x, wv, wv, wv, wo, [0] * heads, out)
    rows = torch.randperm(N, device="cuda", generator=gen)[:4096]
    mx, rl = U.errors(U.to_host64(out[0, rows]), U.to_host64(x[0, rows].float() @ (wv.float() @ wo.float())))
    print(f"projected d_model={d_model}: max-abs {mx:.3e} rel-L2 {rl:.3e}", flush=True)
    ctx.destroy()
    assert mx <= 2e-2 and rl <= 5e-3, (mx, rl)
