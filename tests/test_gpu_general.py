"""The general kernels on the GPU, at the sizes where their tiles, vectors and slices end and at every tile they dispatch,
against the fp64 oracle.

Tolerance: a sum of n products in fp32 (bf16 products are exact in fp32) is off by about sqrt(n) roundings of 2^-24
relative to its terms' norm; four times that."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro
from general_tiles import TILES

pytestmark = pytest.mark.gpu


def bar(n):
    return 4.0 * max(n, 16) ** 0.5 * 2.0 ** -24


def operand(a, dtype):
    """(device tensor in the operand type, the values it holds as fp32)."""
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    t = t.bfloat16() if dtype == lc.LC_BF16 else t
    return t, t.float().cpu().numpy()


def nan(*shape):
    return torch.full(shape, float("nan"), device="cuda")


# (B, H, W, C, R, S, F): patch rows of 4 to 7 values and of odd lengths, one vector per row, filters below a tile, at a
# tile's edge and one past it, one image, one image past a tile, contractions cut into slices, one field, gaps
SHAPES = [(1, 9, 11, 4, 1, 1, 3), (1, 7, 7, 5, 1, 2, 1), (17, 9, 14, 3, 2, 1, 17), (16, 12, 9, 7, 1, 1, 16), (33, 11, 13, 1, 5, 2, 33),
          (5, 31, 29, 3, 11, 4, 50), (2, 24, 27, 16, 13, 5, 60), (65, 10, 12, 3, 5, 3, 49), (130, 13, 11, 5, 3, 2, 19),
          (3, 20, 20, 8, 20, 1, 40), (7, 17, 23, 3, 3, 5, 11), (70, 19, 18, 5, 7, 2, 72), (48, 15, 17, 6, 4, 3, 65)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_forward(shape, dtype):
    print(f"case general forward {shape} {dtype}", flush=True)
    g = wl.LCGeom(*shape)
    G = lc.geom(*shape)
    x, w, _, bias = wl.lc_inputs(g, "gaussian", seed=1, with_bias=True)
    (xd, xv), (wd, wv) = operand(x, dtype), operand(w, dtype)
    y = nan(g.B, g.LH, g.LW, g.F)
    lc.lc_forward(G, xd, wd, torch.from_numpy(bias).cuda(), 0.75, y, dtype)
    ref = oracle.lc_forward(shape, xv, wv, bias, 0.75)
    assert rel_fro(y.cpu().numpy(), ref) <= bar(g.K)
    again = nan(g.B, g.LH, g.LW, g.F)
    lc.lc_forward(G, xd, wd, torch.from_numpy(bias).cuda(), 0.75, again, dtype)
    assert torch.equal(y, again)


@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_forward_infinities_stay_in_their_fields(dtype):
    """An infinite pixel makes the outputs of the fields that hold it infinite, NaN nowhere; a NaN between fields (stride
    beyond the field) reaches nothing."""
    print(f"case general forward infinities {dtype}", flush=True)
    shape = (3, 18, 20, 3, 3, 5, 11)
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=2)
    x[:, 3:5] = np.nan
    x[:, :, 3:5] = np.nan
    x[1, 6, 7, 2] = np.inf                       # last value of a patch row
    x[2, 10, 10, 0] = -np.inf                    # first value of a field
    (xd, xv), (wd, wv) = operand(x, dtype), operand(w, dtype)
    y = nan(g.B, g.LH, g.LW, g.F)
    lc.lc_forward(lc.geom(*shape), xd, wd, None, 1.0, y, dtype)
    ref = oracle.lc_forward(shape, xv, wv)
    y = y.cpu().numpy()
    assert np.isinf(ref).sum() == 2 * g.F and not np.isnan(ref).any()
    assert np.array_equal(np.isinf(y), np.isinf(ref)) and np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert rel_fro(y[m], ref[m]) <= bar(g.K)


# backward data: besides SHAPES, filters in vectors of eight with and without a shared last vector, one and few strides per
# block of values, an image border that cuts a block, and strides far beyond the image (on either side of the grid's limit)
DATA_SHAPES = SHAPES + [(20, 14, 15, 1, 4, 1, 8), (4, 13, 18, 2, 6, 2, 9), (33, 16, 13, 3, 8, 2, 24), (18, 25, 23, 3, 8, 4, 16),
                        (6, 12, 10, 1, 10, 1, 4), (50, 14, 22, 64, 4, 2, 20), (2, 26, 26, 1, 7, 3, 303),
                        (3, 9, 11, 4, 3, 1023, 41), (3, 9, 11, 1, 3, 2049, 41)]


@pytest.mark.parametrize("shape", DATA_SHAPES, ids=str)
@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_backward_data(shape, dtype):
    print(f"case general backward data {shape} {dtype}", flush=True)
    g = wl.LCGeom(*shape)
    G = lc.geom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=3)
    (yd, yv), (wd, wv) = operand(dy, dtype), operand(w, dtype)
    dx = nan(g.B, g.H, g.W, g.C)
    lc.lc_backward_data(G, yd, wd, dx, dtype)
    ref = oracle.lc_backward_data(shape, yv, wv)
    out = dx.cpu().numpy()
    assert rel_fro(out, ref) <= bar(g.F * (-(-g.R // g.S)) ** 2)
    assert np.all(out[ref == 0.0] == 0.0)
    again = nan(g.B, g.H, g.W, g.C)
    lc.lc_backward_data(G, yd, wd, again, dtype)
    assert torch.equal(dx, again)


@pytest.mark.parametrize("shape", [(3, 14, 15, 1, 4, 1, 12), (18, 17, 19, 3, 5, 3, 21)], ids=str)
@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_backward_data_infinities_stay_in_their_fields(shape, dtype):
    print(f"case general backward data infinities {shape} {dtype}", flush=True)
    g = wl.LCGeom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=4)
    dy[1, 1, 2, g.F - 1] = np.inf                # the last filter of one field, the first of another
    dy[2, g.LH - 1, 0, 0] = np.nan
    (yd, yv), (wd, wv) = operand(dy, dtype), operand(w, dtype)
    dx = nan(g.B, g.H, g.W, g.C)
    lc.lc_backward_data(lc.geom(*shape), yd, wd, dx, dtype)
    ref = oracle.lc_backward_data(shape, yv, wv)
    out = dx.cpu().numpy()
    assert np.isinf(ref).sum() == np.isnan(ref).sum() == g.K
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert rel_fro(out[m], ref[m]) <= bar(g.F * (-(-g.R // g.S)) ** 2)


# what a tile with a NaN is formed again from: tiles of several batch and value blocks, sliced contractions, both vector widths
NAN_SHAPES = [(40, 18, 19, 3, 5, 3, 21), (70, 20, 17, 4, 7, 4, 40), (9, 31, 29, 3, 11, 4, 50), (33, 12, 13, 1, 4, 1, 9), (5, 23, 25, 2, 7, 3, 130)]


@pytest.mark.parametrize("shape", NAN_SHAPES, ids=str)
@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_backward_data_of_images_without_a_finite_value(shape, dtype):
    """Positive weights: an image whose dy is infinite everywhere comes out infinite wherever a field reaches, one with
    infinities of both signs NaN where they meet; images around them stay what they are."""
    print(f"case general backward data infinite images {shape} {dtype}", flush=True)
    g = wl.LCGeom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=11)
    w = np.abs(w) + np.float32(2.0 ** -6)
    dy[1] = np.inf
    dy[2, g.LH // 2] = -np.inf
    dy[3, :, ::2] = np.inf
    dy[3, 0, :, g.F // 2] = -np.inf
    dy[4, g.LH - 1, g.LW - 1, g.F - 1] = np.nan
    (yd, yv), (wd, wv) = operand(dy, dtype), operand(w, dtype)
    dx = nan(g.B, g.H, g.W, g.C)
    lc.lc_backward_data(lc.geom(*shape), yd, wd, dx, dtype)
    ref = oracle.lc_backward_data(shape, yv, wv)
    out = dx.cpu().numpy()
    assert np.isinf(ref).any() and np.isnan(ref).any()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert rel_fro(out[m], ref[m]) <= bar(g.F * (-(-g.R // g.S)) ** 2)


@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_backward_data_takes_its_time_whatever_the_data(dtype):
    """Tiles are formed again at most once, by matrix instructions: infinite gradients cost a small multiple of finite ones."""
    shape = (32, 60, 60, 3, 11, 4, 96)
    print(f"case general backward data time {shape} {dtype}", flush=True)
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=12)
    wd, _ = operand(np.abs(w), dtype)
    dx = nan(g.B, g.H, g.W, g.C)

    def time(values):
        yd, _ = operand(values, dtype)
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            lc.lc_backward_data(G, yd, wd, dx, dtype)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    finite, infinite = time(dy), time(np.full_like(dy, np.inf))
    print(f"finite {1e3 * finite:.1f} us, infinite {1e3 * infinite:.1f} us", flush=True)
    # one of a task's eight waves forms its six tiles again (5 times the finite pass measured; value by value it was 110)
    assert torch.isinf(dx).any() and infinite <= 16 * finite


# weight gradient: besides SHAPES, batches around a step of four and of sixteen images, one slice and several
WEIGHT_SHAPES = SHAPES + [(4, 11, 12, 5, 3, 1, 30), (15, 12, 10, 3, 5, 1, 18), (31, 10, 11, 7, 2, 1, 6), (64, 9, 9, 3, 9, 1, 35),
                          (200, 8, 9, 3, 7, 1, 21), (3, 12, 14, 1, 4, 2, 2),
                          (1, 17, 15, 8, 4, 2, 40), (2, 20, 20, 3, 6, 2, 50), (9, 13, 14, 5, 3, 2, 19), (7, 9, 10, 9, 5, 1, 70)]


@pytest.mark.parametrize("shape", WEIGHT_SHAPES, ids=str)
@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_backward_weights(shape, dtype):
    print(f"case general backward weights {shape} {dtype}", flush=True)
    g = wl.LCGeom(*shape)
    G = lc.geom(*shape)
    x, _, dy = wl.lc_inputs(g, "gaussian", seed=5)
    (xd, xv), (yd, yv) = operand(x, dtype), operand(dy, dtype)
    dw = nan(g.LH, g.LW, g.K, g.F)
    lc.lc_backward_weights(G, xd, yd, 0.0, dw, dtype)
    ref = oracle.lc_backward_weights(shape, xv, yv)
    assert rel_fro(dw.cpu().numpy(), ref) <= bar(g.B)
    # accumulation: what vectors or runs share is added once
    prev = torch.from_numpy(np.random.default_rng(6).standard_normal(ref.shape).astype(np.float32)).cuda()
    acc = prev.clone()
    lc.lc_backward_weights(G, xd, yd, 1.0, acc, dtype)
    assert rel_fro(acc.cpu().numpy(), ref + prev.cpu().numpy().astype(np.float64)) <= bar(g.B)
    again = nan(g.LH, g.LW, g.K, g.F)
    lc.lc_backward_weights(G, xd, yd, 0.0, again, dtype)
    assert torch.equal(dw, again)


@pytest.mark.parametrize("shape", [(17, 9, 14, 3, 2, 3, 17), (5, 31, 29, 3, 11, 4, 50), (37, 17, 23, 3, 3, 5, 11)], ids=str)
@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16], ids=["f32", "bf16"])
def test_backward_weights_infinities_stay_in_their_rows(shape, dtype):
    """An infinite pixel reaches its weight rows alone, an infinite dy its filter's columns, in every batch position; a NaN
    that no field covers reaches nothing."""
    print(f"case general backward weights infinities {shape} {dtype}", flush=True)
    g = wl.LCGeom(*shape)
    x, _, dy = wl.lc_inputs(g, "gaussian", seed=14)
    if g.R < g.S:
        x[:, g.R:g.S] = np.nan
        x[:, :, g.R:g.S] = np.nan
    x[g.B - 1, 0, 0, g.C - 1] = np.inf                         # the last image of a partly filled step
    x[1, g.S + g.R - 1, g.R - 1, 0] = -np.inf                  # first vector of a patch row's last pixel
    dy[g.B - 2, g.LH - 1, g.LW - 1, g.F - 1] = np.inf          # the filter that the last run shares
    dy[0, g.LH - 1, 0, 0] = np.nan
    (xd, xv), (yd, yv) = operand(x, dtype), operand(dy, dtype)
    dw = nan(g.LH, g.LW, g.K, g.F)
    lc.lc_backward_weights(lc.geom(*shape), xd, yd, 0.0, dw, dtype)
    ref = oracle.lc_backward_weights(shape, xv, yv)
    out = dw.cpu().numpy()
    assert np.isinf(ref).any() and np.isnan(ref).any()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert rel_fro(out[m], ref[m]) <= bar(g.B)


@pytest.mark.parametrize("shape", [(6, 13, 14, 5, 3, 2, 19), (18, 17, 12, 3, 7, 3, 33), (2, 20, 20, 1, 6, 2, 50), (9, 13, 14, 5, 3, 2, 19),
                                   (2, 20, 20, 3, 6, 2, 50)], ids=str)
def test_sae_step_projects_with_shared_vectors(shape):
    """The row projection's sums of squares count every updated weight once."""
    print(f"case general sae_step projection {shape}", flush=True)
    g = wl.LCGeom(*shape)
    G = lc.geom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=7)
    b = np.zeros((g.H, g.W, g.C), dtype=np.float32)
    wd, bd = torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda()
    alpha, cost = torch.full((1,), 0.8, device="cuda"), nan(1)
    ws = torch.empty(lc.workspace_bytes(G, lc.LC_OP_SAE_STEP), dtype=torch.uint8, device="cuda")
    lc.sae_step(G, torch.from_numpy(x).cuda(), wd, bd, alpha, 0.1, 1e-6, 1e-2, lc.LC_SAE_PROJECT_ROWS, None, cost, ws)
    _, wo, _, _, _ = oracle.sae_step(shape, x, w, b, float(np.float32(0.8)), 0.1, 1e-6, 1e-2, 1)
    out = wd.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(np.linalg.norm(out, axis=2), 1.0, rtol=1e-6)
    assert rel_fro(out, wo) <= 1e-6


# Per-channel normalisation on maps large enough for the kernels that walk down the rows: windows of 3 to 9, channels that
# fill a chunk of 32, leave one partly filled or are no multiple of four, strips and segments that end off the grid
@pytest.mark.parametrize("shape,ks", [((40, 21, 26, 32), 5), ((3, 70, 75, 52), 5), ((9, 40, 37, 36), 3), ((24, 33, 18, 24), 7),
                                      ((6, 31, 130, 16), 9), ((130, 13, 12, 20), 9), ((64, 23, 29, 6), 5), ((2, 150, 170, 7), 3), ((150, 40, 11, 4), 7),
                                      ((300, 33, 12, 8), 5), ((300, 33, 13, 8), 5)], ids=str)
@pytest.mark.parametrize("flags", [1, 3, 5, 7])
def test_channel_normalisation_walks(shape, ks, flags):
    print(f"case channel normalisation {shape} {ks} {flags}", flush=True)
    rng = np.random.default_rng(8)
    x = (rng.standard_normal(shape) + 0.5).astype(np.float32)
    dy = rng.standard_normal(shape).astype(np.float32)
    xd, dyd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
    y, mu, rstd, dx = (nan(*shape) for _ in range(4))
    nbytes = lc.lcn_variant_workspace_bytes(shape, flags)
    ws = torch.full((nbytes // 4,), float("nan"), device="cuda").view(torch.uint8) if nbytes else None
    lc.lcn_variant_fwd(xd, y, mu, rstd, ks, 1.0, 1e-4, flags)
    lc.lcn_variant_bwd(xd, mu, rstd, dyd, dx, ks, 1.0, flags, ws)
    yo, muo, rso = oracle.lcn_var_fwd(x, ks, 1.0, 1e-4, flags)
    dxo = oracle.lcn_var_bwd(x, muo, rso, dy, ks, 1.0, flags)
    # window sums of ks*ks terms; the one-stage variance is a difference of two of them, a few times their size
    for got, ref in ((mu, muo), (rstd, rso), (y, yo), (dx, dxo)):
        assert rel_fro(got.cpu().numpy(), ref) <= 8 * bar(ks * ks)


# Normalisation with statistics pooled over channels that have no band kernel, or maps these do not take: tiles of every
# size the launcher halves down to, lanes per pixel that fill its vectors, leave some empty or take single channels, one
# vector per lane (four channels, and maps the caches do not hold)
@pytest.mark.parametrize("shape,ks", [((4, 33, 35, 96), 5), ((1, 12, 13, 40), 3), ((2, 20, 70, 384), 5), ((40, 17, 18, 24), 7),
                                      ((600, 5, 5, 72), 9), ((3, 30, 31, 7), 5), ((2, 16, 90, 64), 15), ((1, 3, 50, 12), 9),
                                      ((2, 40, 300, 4), 5), ((64, 110, 84, 44), 3)], ids=str)
@pytest.mark.parametrize("flags", [0, 2, 4, 6])
def test_pooled_normalisation_tiles(shape, ks, flags):
    print(f"case pooled normalisation {shape} {ks} {flags}", flush=True)
    rng = np.random.default_rng(9)
    x = (rng.standard_normal(shape) + 0.5).astype(np.float32)
    dy = rng.standard_normal(shape).astype(np.float32)
    xd, dyd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
    y, dx, mu, rstd = nan(*shape), nan(*shape), nan(*shape[:3]), nan(*shape[:3])
    nbytes = lc.lcn_variant_workspace_bytes(shape, flags)
    ws = torch.full((nbytes // 4,), float("nan"), device="cuda").view(torch.uint8) if nbytes else None
    lc.lcn_variant_fwd(xd, y, mu, rstd, ks, 1.0, 1e-4, flags)
    lc.lcn_variant_bwd(xd, mu, rstd, dyd, dx, ks, 1.0, flags, ws)
    yo, muo, rso = oracle.lcn_var_fwd(x, ks, 1.0, 1e-4, flags)
    dxo = oracle.lcn_var_bwd(x, muo, rso, dy, ks, 1.0, flags)
    # sums of ks*ks*C terms; the one-stage variance is a difference of two of them, a few times their size
    for got, ref in ((mu, muo), (rstd, rso), (y, yo), (dx, dxo)):
        assert rel_fro(got.cpu().numpy(), ref) <= 8 * bar(ks * ks * shape[3])


# one shape per kernel: the two walks (whole, part-filled and scalar chunks), the tiles, and the band kernel beside them
@pytest.mark.parametrize("shape,ks", [((40, 21, 26, 32), 5), ((3, 70, 75, 52), 5), ((64, 23, 29, 6), 5), ((6, 31, 130, 16), 9),
                                      ((4, 33, 35, 96), 5), ((3, 30, 31, 7), 5), ((2, 16, 90, 64), 3)], ids=str)
@pytest.mark.parametrize("flags", range(8))
def test_normalisation_keeps_a_nan_in_its_windows(shape, ks, flags):
    """A NaN in x (forward) or dy (gradient) makes NaN of what its windows reach, of its channel or of all, and changes no
    other value by a bit."""
    print(f"case normalisation with a NaN {shape} {ks} {flags}", flush=True)
    torch.manual_seed(15)
    stats = shape if flags & 1 else shape[:3]
    nbytes = lc.lcn_variant_workspace_bytes(shape, flags)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
    x, dy = torch.randn(*shape, device="cuda"), torch.randn(*shape, device="cuda")
    y, dx, mu, rstd = nan(*shape), nan(*shape), nan(*stats), nan(*stats)
    lc.lcn_variant_fwd(x, y, mu, rstd, ks, 1.0, 1e-4, flags)
    lc.lcn_variant_bwd(x, mu, rstd, dy, dx, ks, 1.0, flags, ws)
    reach = (ks - 1) // 2 * (2 if flags & 4 else 1)
    for b, i, j, c in ((0, 0, 0, 0), (shape[0] - 1, shape[1] - 1, shape[2] - 1, shape[3] - 1), (1, shape[1] // 2, shape[2] // 2, 3)):
        touched = torch.zeros(shape, dtype=torch.bool, device="cuda")
        touched[b, max(0, i - reach):i + reach + 1, max(0, j - reach):j + reach + 1, slice(c, c + 1) if flags & 1 else slice(None)] = True
        x1, dy1, y1, dx1, mu1, rstd1 = x.clone(), dy.clone(), nan(*shape), nan(*shape), nan(*stats), nan(*stats)
        x1[b, i, j, c] = dy1[b, i, j, c] = float("nan")
        lc.lcn_variant_fwd(x1, y1, mu1, rstd1, ks, 1.0, 1e-4, flags)
        lc.lcn_variant_bwd(x, mu, rstd, dy1, dx1, ks, 1.0, flags, ws)
        for got, clean in ((y1, y), (dx1, dx)):
            assert torch.equal(got.isnan(), touched) and torch.equal(got[~touched], clean[~touched])


# 3x3 stride-1 pooling gradient: the stream's segments and borders, the smallest map, and both sides of the tile kernel's sizes
@pytest.mark.parametrize("shape", [(1, 3, 3, 4), (2, 9, 7, 128), (3, 41, 35, 16), (1, 4, 100, 8), (5, 33, 34, 44), (2, 32, 33, 24),
                                   (2, 31, 40, 32), (1, 70, 5, 384), (127, 32, 32, 32), (128, 32, 32, 32), (160, 33, 40, 24), (2, 40, 300, 4)], ids=str)
def test_pool_gradient_streams(shape):
    print(f"case pool gradient {shape}", flush=True)
    rng = np.random.default_rng(10)
    x = rng.standard_normal(shape).astype(np.float32)
    y = oracle.l2pool_fwd(x, 3, 1, 1e-6).astype(np.float32)
    dy = rng.standard_normal(y.shape).astype(np.float32)
    dx = nan(*shape)
    lc.l2pool_bwd(*(torch.from_numpy(a).cuda() for a in (x, y, dy)), dx, 3, 1)
    # nine quotients and a product, each a rounding or two
    assert rel_fro(dx.cpu().numpy(), oracle.l2pool_bwd(x, y, dy, 3, 1)) <= bar(16)
    # behind the normalisation, which leaves dp / p in the scratch array
    n, mu, rstd = oracle.lcn_fwd(y, 3, 1.0, 1e-4)
    mu32, rs32 = mu.astype(np.float32), rstd.astype(np.float32)
    scratch, dx2 = nan(*y.shape), nan(*shape)
    lc.lcn_l2pool_bwd(*(torch.from_numpy(a).cuda() for a in (x, y, mu32, rs32, dy)), scratch, dx2, 3, 1, 3, 1.0)
    ref = oracle.l2pool_bwd(x, y, oracle.lcn_bwd(y, mu32, rs32, dy, 3, 1.0), 3, 1)
    assert rel_fro(dx2.cpu().numpy(), ref) <= 8 * bar(9 * shape[3])


def run_pass(op, shape, dt):
    """One pass over seeded operands: (result, fp64 oracle, products per result)."""
    G, g = lc.geom(*shape), wl.LCGeom(*shape)
    x, w, dy = wl.lc_inputs(g, "gaussian", seed=6)
    (xd, xv), (wd, wv), (dyd, dyv) = operand(x, dt), operand(w, dt), operand(dy, dt)
    if op == "forward":
        out, n = nan(g.B, g.LH, g.LW, g.F), g.K
        lc.lc_forward(G, xd, wd, None, 1.0, out, dt)
        ref = oracle.lc_forward(shape, xv, wv, None, 1.0)
    elif op == "backward_data":
        out, n = nan(g.B, g.H, g.W, g.C), g.F * (-(-g.R // g.S)) ** 2
        lc.lc_backward_data(G, dyd, wd, out, dt)
        ref = oracle.lc_backward_data(shape, dyv, wv)
    else:
        out, n = nan(g.LH, g.LW, g.K, g.F), g.B
        lc.lc_backward_weights(G, xd, dyd, 0.0, out, dt)
        ref = oracle.lc_backward_weights(shape, xv, dyv)
    return out.cpu().numpy(), ref, n


@pytest.mark.parametrize("op,dtype,shape", [(*k, s) for k, shapes in TILES.items() for s in shapes], ids=str)
def test_every_tile(op, dtype, shape):
    print(f"case tile {op} {dtype} {shape}", flush=True)
    out, ref, n = run_pass(op, shape, lc.LC_BF16 if dtype == "bf16" else lc.LC_F32)
    assert rel_fro(out, ref) <= bar(n)


@pytest.mark.parametrize("shape", [(2, 9, 7, 128), (3, 41, 35, 16), (5, 33, 34, 44), (2, 64, 64, 32), (32, 64, 64, 32), (1, 3, 3, 4)], ids=str)
def test_pool_gradient_keeps_a_nan_in_its_window(shape):
    print(f"case pool gradient with a NaN {shape}", flush=True)
    torch.manual_seed(16)
    B, H, W, C = shape
    x = torch.randn(*shape, device="cuda")
    y, dx = nan(B, H - 2, W - 2, C), nan(*shape)
    lc.l2pool_fwd(x, y, 3, 1, 1e-6)
    dy = torch.randn_like(y)
    lc.l2pool_bwd(x, y, dy, dx, 3, 1)
    for b, i, j, c in ((0, 0, 0, 0), (B - 1, H - 3, W - 3, C - 1), (B // 2, (H - 3) // 2, (W - 3) // 3, C // 2)):
        for value, quotient in ((float("nan"), None), (float("inf"), None), (0.0, 0.0)):
            dy1, y1, dx1 = dy.clone(), y.clone(), nan(*shape)
            dy1[b, i, j, c] = value
            if quotient is not None:
                y1[b, i, j, c] = quotient                      # 0 / 0
            lc.l2pool_bwd(x, y1, dy1, dx1, 3, 1)
            touched = torch.zeros(shape, dtype=torch.bool, device="cuda")
            touched[b, i:i + 3, j:j + 3, c] = True
            assert torch.equal(~dx1.isfinite(), touched) and torch.equal(dx1[~touched], dx[~touched])


# Aligned layers on both sides of the lines between the general kernels and the others: (op, dtype, shape, kernel).
ROUTES = [
    ("forward", "f32", (40, 20, 21, 16, 4, 2, 32), "lc_forward_general"),       # little overlap
    ("forward", "f32", (64, 56, 56, 8, 8, 2, 64), "lc_forward_general"),        # two batch tiles
    ("forward", "f32", (32, 80, 80, 8, 8, 2, 64), "lc_forward_fast"),           # one, overlap of four
    ("forward", "f32", (96, 18, 18, 16, 16, 1, 128), "lc_forward_wide"),        # 9 fields, long patches
    ("forward", "f32", (96, 19, 19, 16, 16, 1, 128), "lc_forward_general"),     # 16 fields
    ("forward", "f32", (96, 10, 10, 16, 8, 1, 128), "lc_forward_general"),      # 9 fields, short patches
    ("forward", "bf16", (64, 12, 12, 8, 4, 2, 32), "lc_forward_general"),       # K at the line
    ("forward", "bf16", (64, 19, 20, 16, 15, 1, 64), "lc_forward_general"),     # few workgroups in strips
    ("backward_data", "f32", (16, 72, 72, 32, 4, 4, 16), "lc_bwd_data_generic"),    # large cells, enough of them
    ("backward_data", "f32", (16, 40, 40, 32, 4, 4, 16), "lc_bwd_data_general"),    # too few
    ("backward_data", "f32", (15, 72, 72, 32, 4, 4, 40), "lc_bwd_data_general"),    # a batch below
    ("backward_data", "f32", (15, 72, 72, 32, 4, 4, 16), "lc_bwd_data_generic"),    # one short sum a value
    ("backward_data", "bf16", (16, 72, 72, 64, 4, 4, 13), "lc_bwd_data_generic"),
    ("backward_data", "f32", (64, 26, 26, 16, 6, 2, 32), "lc_bwd_data_direct"),     # full tiles
    ("backward_data", "f32", (40, 30, 32, 3, 10, 2, 64), "lc_bwd_data_general"),    # mostly padding
    ("backward_data", "bf16", (64, 26, 26, 16, 6, 2, 64), "lc_bwd_data_fast"),
    ("backward_data", "bf16", (64, 26, 26, 16, 6, 2, 96), "lc_bwd_data_general"),
    ("backward_data", "bf16", (32, 24, 24, 8, 8, 4, 128), "lc_bwd_data_general"),
    ("backward_weights", "f32", (100, 26, 38, 16, 4, 2, 48), "lc_bwd_weights_general"),
    ("backward_weights", "f32", (104, 20, 22, 16, 4, 2, 48), "lc_bwd_weights_fast"),        # one round of waves
    ("backward_weights", "f32", (96, 20, 22, 16, 4, 2, 48), "lc_bwd_weights_fast"),
    ("backward_weights", "f32", (1, 44, 49, 16, 20, 3, 31), "lc_bwd_weights_generic"),   # a gradient beyond 2^24 elements
    ("backward_weights", "f32", (1, 44, 49, 16, 20, 3, 33), "lc_bwd_weights_general"),
    ("backward_weights", "bf16", (1, 44, 49, 16, 20, 3, 31), "lc_bwd_weights_generic"),
    ("backward_weights", "bf16", (64, 20, 20, 4, 8, 2, 16), "lc_bwd_weights_general"),
    # 128-wide tiles: few and enough of them
    ("forward", "bf16", (96, 11, 11, 32, 4, 1, 128), "lc_forward_general"),             # 64 tiles
    ("forward", "bf16", (96, 11, 17, 32, 4, 1, 128), "lc_forward_bf16_tiled"),          # 112
    ("backward_data", "bf16", (96, 16, 16, 32, 6, 2, 64), "lc_bwd_data_general"),       # 64
    ("backward_data", "bf16", (96, 16, 18, 32, 6, 2, 64), "lc_bwd_data_bf16_tiled"),    # 72
    ("backward_weights", "bf16", (96, 7, 7, 32, 4, 1, 128), "lc_bwd_weights_general"),      # 16
    ("backward_weights", "bf16", (96, 7, 8, 32, 4, 1, 128), "lc_bwd_weights_bf16_tiled"),   # 20
    # patch rows and rows of dy that other kernels' staging does not hold
    ("forward", "f32", (70, 8, 8, 640, 4, 1, 128), "lc_forward_wide"),                      # 25 fields, rows of 2560 values
    ("forward", "bf16", (33, 50, 49, 64, 49, 1, 16), "lc_forward_fast"),                    # rows of 3136
    ("backward_data", "f32", (20, 42, 83, 8, 39, 1, 4), "lc_bwd_data_general"),
    ("backward_data", "bf16", (20, 42, 83, 8, 39, 1, 4), "lc_bwd_data_general"),
    ("backward_data", "bf16", (32, 62, 60, 64, 60, 1, 64), "lc_bwd_data_bf16_simple"),
    ("backward_data", "bf16", (128, 46, 50, 8, 46, 2, 832), "lc_bwd_data_bf16_simple"),
]
OPS = {"forward": 0, "backward_data": 1, "backward_weights": 2}


@pytest.mark.parametrize("op,dtype,shape,kernel", ROUTES, ids=str)
def test_routes(op, dtype, shape, kernel):
    print(f"case route {op} {dtype} {shape}", flush=True)
    dt = lc.LC_BF16 if dtype == "bf16" else lc.LC_F32
    assert kernel in [p["kernel"] for p in lc.plan_query(lc.geom(*shape), OPS[op], dt)]
    out, ref, n = run_pass(op, shape, dt)
    assert rel_fro(out, ref) <= bar(n)


# Images of 2^24 values and more (2^25 in bf16), beyond the general kernel's 32-bit offsets: the register-staged kernel keeps
# every aligned layer there, at tiles (MT, NT) that smaller images no longer reach.
LARGE_IMAGES = [("f32", (33, 8192, 1024, 2, 10, 26, 16), (4, 1)), ("f32", (33, 131072, 64, 2, 10, 28, 32), (4, 2)),
                ("f32", (33, 16384, 256, 4, 5, 42, 128), (4, 4)), ("f32", (33, 10952, 383, 4, 5, 14, 64), (4, 4)),
                ("f32", (33, 8192, 512, 4, 8, 39, 128), (4, 4)), ("f32", (65, 131072, 64, 2, 10, 12, 32), (8, 2)),
                ("f32", (65, 131072, 64, 2, 12, 12, 32), (8, 2)), ("bf16", (17, 262144, 64, 2, 10, 57, 32), (2, 2)),
                ("bf16", (17, 10181, 824, 4, 5, 63, 128), (2, 4)), ("bf16", (17, 65536, 256, 2, 10, 43, 64), (2, 4)),
                ("bf16", (33, 131072, 128, 2, 10, 27, 32), (4, 2)), ("bf16", (33, 16384, 512, 4, 5, 42, 128), (4, 4)),
                ("bf16", (33, 32768, 512, 2, 12, 23, 64), (4, 4)), ("bf16", (65, 262144, 64, 2, 10, 11, 32), (8, 2))]


@pytest.mark.parametrize("dtype,shape,tile", LARGE_IMAGES, ids=str)
def test_forward_of_large_images(dtype, shape, tile):
    print(f"case forward of large images {dtype} {shape}", flush=True)
    G, g = lc.geom(*shape), wl.LCGeom(*shape)
    dt, td = (lc.LC_BF16, torch.bfloat16) if dtype == "bf16" else (lc.LC_F32, torch.float32)
    plans = lc.plan_query(G, lc.LC_OP_FORWARD, dt)
    assert ("lc_forward_fast", tile) in [(p["kernel"], tuple(p["tparam"][:2])) for p in plans], plans
    torch.manual_seed(13)
    x = torch.randn(g.B, g.H, g.W, g.C, device="cuda", dtype=td)
    w = torch.randn(g.LH, g.LW, g.K, g.F, device="cuda", dtype=td)
    bias = torch.randn(g.LH, g.LW, g.F, device="cuda")
    y = nan(g.B, g.LH, g.LW, g.F)
    lc.lc_forward(G, x, w, bias, 0.75, y, dt)
    # fp64 products of all fields, some field rows at a time
    fields = x.unfold(1, g.R, g.S).unfold(2, g.R, g.S)         # [B, LH, LW, C, R, R]
    rows = max(1, 30_000_000 // (g.LW * g.K * max(g.B, g.F)))
    diff = norm = 0.0
    for i in range(0, g.LH, rows):
        n = min(rows, g.LH - i)
        a = fields[:, i:i + n].permute(1, 2, 0, 4, 5, 3).double().reshape(n * g.LW, g.B, g.K)
        ref = 0.75 * torch.bmm(a, w[i:i + n].double().reshape(n * g.LW, g.K, g.F)) + bias[i:i + n].double().reshape(-1, 1, g.F)
        got = y[:, i:i + n].permute(1, 2, 0, 3).double().reshape(n * g.LW, g.B, g.F)
        diff, norm = diff + (got - ref).square().sum(), norm + ref.square().sum()
    assert float((diff / norm).sqrt()) <= bar(g.K)
    del x, w, y, fields
    torch.cuda.empty_cache()
