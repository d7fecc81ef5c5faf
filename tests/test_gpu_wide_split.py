"""The workgroup-tiled kernels (few fields and long patches forwards, cells of 128 values and dense layers backwards), whose fp32
products are split into bf16 parts, against the fp64 oracle: every batch tile, patch rows in chunks of 32 and of 16 values with a
last step of one chunk, with and without the workspace that slices the contraction.  Tolerance as for the general kernels: four
times sqrt(n) roundings of 2^-24."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

# (units of 32 images per workgroup, chunk): layers
FORWARD = {(2, 32): [(300, 8, 8, 64, 8, 1, 128), (310, 17, 16, 16, 16, 1, 128)], (3, 32): [(70, 17, 16, 32, 16, 1, 128), (70, 23, 24, 20, 8, 1, 128)],
           (4, 32): [(128, 8, 8, 64, 8, 1, 128), (97, 18, 16, 18, 16, 2, 128)],
           (2, 16): [(300, 17, 17, 16, 17, 1, 128)], (3, 16): [(70, 17, 18, 16, 17, 1, 128), (96, 20, 22, 12, 20, 2, 128)],
           (4, 16): [(100, 17, 17, 16, 17, 1, 128), (256, 20, 20, 12, 20, 1, 128)]}


def bar(n):
    return 4.0 * max(n, 16) ** 0.5 * 2.0 ** -24


def forward(shape, x, w, b, alpha, sliced):
    G = lc.geom(*shape)
    y = torch.full((shape[0], *b.shape), float("nan"), device="cuda")
    n = lc.workspace_bytes(G, lc.LC_OP_FORWARD, lc.LC_F32)
    ws = torch.full((n // 4,), float("nan"), device="cuda").view(torch.uint8) if sliced and n else None
    lc.lc_forward(G, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda(), alpha, y, lc.LC_F32, ws)
    return y


@pytest.mark.parametrize("tile,shape", [(k, s) for k, v in FORWARD.items() for s in v], ids=str)
@pytest.mark.parametrize("sliced", [True, False])
def test_forward(tile, shape, sliced):
    print(f"case wide forward {tile} {shape} {sliced}", flush=True)
    g = wl.LCGeom(*shape)
    p = lc.plan_query(lc.geom(*shape), lc.LC_OP_FORWARD, lc.LC_F32)[0]
    assert (p["kernel"], p["tparam"][0], p["tparam"][2]) == ("lc_forward_wide", *tile)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=3)
    b = np.random.default_rng(2).standard_normal((g.LH, g.LW, g.F)).astype(np.float32)
    y = forward(shape, x, w, b, 0.75, sliced)
    assert rel_fro(y.cpu().numpy(), oracle.lc_forward(shape, x, w, b, 0.75)) <= bar(g.R * g.R * g.C)
    assert torch.equal(y, forward(shape, x, w, b, 0.75, sliced))


@pytest.mark.parametrize("shape", [FORWARD[2, 32][0], FORWARD[3, 16][0], FORWARD[4, 16][0]], ids=str)
@pytest.mark.parametrize("scale", [1.0, 1e-30, 2e38], ids=str)
def test_forward_infinities_and_ends_of_the_range(shape, scale):
    """Infinities and NaNs stay in the outputs that they reach; small and large values keep their precision (parts that overflow
    where fp32 does not: formed again in fp32)."""
    print(f"case wide forward range {shape} {scale}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=4)
    x = (x / np.abs(x).max() * scale).astype(np.float32)
    w = (w / np.abs(w).max() / (g.R * g.R * g.C)).astype(np.float32)
    if scale == 1.0:
        x[0, 0, 0, 0] = np.inf
        x[g.B - 1, g.H - 1, g.W - 1, g.C - 1] = -np.inf
        w[0, 0, -1, g.F // 2] = np.nan
    else:
        x[0, 0, 0, 0] = 1.69 * scale
    b = np.zeros((g.LH, g.LW, g.F), dtype=np.float32)
    ref, out = oracle.lc_forward(shape, x, w, b, 1.0), forward(shape, x, w, b, 1.0, True).cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert m.any() and rel_fro(out[m].astype(np.float64) / scale, ref[m] / scale) <= bar(g.R * g.R * g.C)


@pytest.mark.parametrize("sliced", [True, False])
@pytest.mark.parametrize("row", [3, -5], ids=["first", "last"])
@pytest.mark.parametrize("shape", [FORWARD[2, 32][0], FORWARD[2, 16][0], FORWARD[3, 16][0], FORWARD[3, 16][1], FORWARD[4, 16][0]], ids=str)
def test_forward_infinite_weights(shape, row, sliced):
    """An infinite weight among the first or last 16 of a patch makes its filter's outputs infinite (chunks of 16 and an odd number
    of them: the last step has 16 elements and no others), and no others anything but finite."""
    print(f"case wide forward infinite weights {shape} {row} {sliced}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=6)
    w[0, 0, row, g.F // 2] = np.inf
    w[-1, -1, row, 0] = -np.inf
    b = np.zeros((g.LH, g.LW, g.F), dtype=np.float32)
    ref, out = oracle.lc_forward(shape, x, w, b, 1.0), forward(shape, x, w, b, 1.0, sliced).cpu().numpy()
    assert np.isinf(ref).sum() == 2 * g.B and not np.isnan(ref).any()
    assert not np.isnan(out).any() and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert rel_fro(out[m], ref[m]) <= bar(g.R * g.R * g.C)


def test_forward_millions_of_filters():
    """Rows of filters 64 MB apart: offsets of more than 31 bits from a step's first row to a lane's last."""
    shape = (66, 1, 1, 32, 1, 1, 2 ** 24 + 128)
    print(f"case wide forward {shape}", flush=True)
    B, F = shape[0], shape[-1]
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn((B, 1, 1, 32), generator=gen, device="cuda")
    w = torch.randn((1, 1, 32, F), generator=gen, device="cuda")
    y = torch.full((B, 1, 1, F), float("nan"), device="cuda")
    lc.lc_forward(lc.geom(*shape), x, w, None, 1.0, y, lc.LC_F32, None)
    for f in (0, 2 ** 23 - 64, F - 256):
        ref = x.view(B, 32).double() @ w.view(32, F)[:, f:f + 256].double()
        assert rel_fro(y.view(B, F)[:, f:f + 256].cpu().numpy(), ref.cpu().numpy()) <= bar(32)
    assert not torch.isnan(y).any()


# (units of 32 images, dense): layers
BACKWARD = {(2, 0): [(300, 11, 13, 32, 4, 2, 32), (128, 14, 15, 32, 6, 2, 64)], (3, 0): [(80, 11, 13, 64, 4, 2, 64), (96, 21, 26, 8, 8, 4, 96)],
            (4, 0): [(128, 33, 36, 32, 4, 2, 32), (256, 16, 18, 128, 3, 1, 32)],
            (2, 1): [(300, 9, 9, 3, 9, 1, 64), (100, 12, 12, 5, 12, 1, 160)], (3, 1): [(70, 15, 15, 3, 15, 1, 96), (96, 7, 7, 2, 7, 1, 32)],
            (4, 1): [(128, 58, 58, 10, 58, 1, 32)]}


def backward(shape, dy, w):
    B, H, W, C = shape[:4]
    dx = torch.full((B, H, W, C), float("nan"), device="cuda")
    lc.lc_backward_data(lc.geom(*shape), torch.from_numpy(dy).cuda(), torch.from_numpy(w).cuda(), dx)
    return dx


@pytest.mark.parametrize("tile,shape", [(k, s) for k, v in BACKWARD.items() for s in v], ids=str)
def test_backward_data(tile, shape):
    print(f"case wide backward data {tile} {shape}", flush=True)
    g = wl.LCGeom(*shape)
    (p,) = lc.plan_query(lc.geom(*shape), lc.LC_OP_BACKWARD_DATA, lc.LC_F32)
    assert (p["kernel"], p["tparam"][0], p["tparam"][2]) == ("lc_bwd_data_wide", *tile)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=3)
    dx, ref = backward(shape, dy, w), oracle.lc_backward_data(shape, dy, w)
    out = dx.cpu().numpy()
    assert rel_fro(out, ref) <= bar(g.F * (-(-g.R // g.S)) ** 2)
    assert np.all(out[ref == 0.0] == 0.0)
    assert torch.equal(dx, backward(shape, dy, w))


@pytest.mark.parametrize("shape", [BACKWARD[2, 0][1], BACKWARD[3, 0][0], BACKWARD[3, 1][0], BACKWARD[2, 1][1]], ids=str)
@pytest.mark.parametrize("scale", [1.0, 1e-30, 2e38], ids=str)
def test_backward_data_infinities_and_ends_of_the_range(shape, scale):
    print(f"case wide backward data range {shape} {scale}", flush=True)
    g = wl.LCGeom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=4)
    dy = (dy / np.abs(dy).max() * scale).astype(np.float32)
    w = (w / np.abs(w).max() / 1024).astype(np.float32)
    if scale == 1.0:
        dy[0, 0, 0, g.F - 1] = np.inf
        dy[g.B - 1, g.LH - 1, g.LW - 1, 0] = -np.inf
        w[g.LH - 1, g.LW - 1, -1, g.F // 2] = np.nan
    else:
        dy[0, 0, 0, 0] = 1.69 * scale
    ref, out = oracle.lc_backward_data(shape, dy, w), backward(shape, dy, w).cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert m.any() and rel_fro(out[m].astype(np.float64) / scale, ref[m] / scale) <= bar(g.F * (-(-g.R // g.S)) ** 2)


@pytest.mark.parametrize("columns", ["all", "some"])
def test_not_a_number_in_the_first_weights(columns):
    """A diverged layer: NaN in every filter's first weights (the sums are all NaN), or in every second one's (the others are not)."""
    print(f"case wide NaN {columns}", flush=True)
    step = 1 if columns == "all" else 2
    shape = FORWARD[3, 16][0]
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=5)
    w[:, :, 3, ::step] = np.nan
    b = np.zeros((g.LH, g.LW, g.F), dtype=np.float32)
    ref, out = oracle.lc_forward(shape, x, w, b, 1.0), forward(shape, x, w, b, 1.0, True).cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.isnan(ref).all() == (step == 1)
    m = np.isfinite(ref)
    assert step == 1 or rel_fro(out[m], ref[m]) <= bar(g.R * g.R * g.C)
    for shape in (BACKWARD[3, 1][0], BACKWARD[2, 0][1]):
        g = wl.LCGeom(*shape)
        _, w, dy = wl.lc_inputs(g, "gaussian", seed=5)
        w[:, :, ::step, 1] = np.nan
        ref, out = oracle.lc_backward_data(shape, dy, w), backward(shape, dy, w).cpu().numpy()
        assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.isnan(ref[0, 0, 0]).all() == (step == 1)
        m = np.isfinite(ref)       # (pixels that no field covers among them)
        assert step == 1 or rel_fro(out[m], ref[m]) <= bar(g.F * (-(-g.R // g.S)) ** 2)


@pytest.mark.parametrize("shape", [BACKWARD[2, 0][1], BACKWARD[3, 0][0], BACKWARD[3, 1][0], BACKWARD[2, 1][1]], ids=str)
def test_backward_data_infinite_weights(shape):
    """An infinite weight of the first or last filter stays in the pixel that it reaches."""
    print(f"case wide backward data infinite weights {shape}", flush=True)
    g = wl.LCGeom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=9)
    w[0, 0, 1, 0], w[0, 0, g.K - 2, g.F - 1] = np.inf, -np.inf
    ref, out = oracle.lc_backward_data(shape, dy, w), backward(shape, dy, w).cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert np.isinf(ref).any() and rel_fro(out[m], ref[m]) <= bar(g.F * (-(-g.R // g.S)) ** 2)
