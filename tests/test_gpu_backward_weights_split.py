"""The weight-gradient kernel's tiles whose fp32 products are split into bf16 parts, against the fp64 oracle: batches of whole
steps of 32 images and with each kind of remainder, last blocks of a field with one to four groups of patch elements, and on
either side of the least batch and grid.  Tolerance as for the general kernels: four times sqrt(n) roundings of 2^-24."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

# {groups, patch vector, filter tiles, images in flight / 4}: layers
SHAPES = {(1, 4, 4, 4): [(64, 35, 36, 4, 4, 1, 64), (80, 20, 20, 8, 2, 1, 192), (128, 10, 4, 6, 2, 2, 64)],
          (1, 4, 4, 2): [(72, 4, 6, 16, 2, 2, 64), (88, 11, 10, 10, 6, 1, 192)],
          (1, 4, 4, 1): [(60, 15, 13, 8, 5, 2, 64), (92, 20, 14, 1, 8, 3, 192), (100, 14, 18, 4, 8, 2, 64)],
          (2, 4, 2, 4): [(64, 11, 15, 16, 5, 2, 32), (112, 17, 17, 8, 7, 2, 96)],
          (2, 4, 2, 1): [(68, 6, 12, 16, 2, 2, 32), (92, 17, 14, 12, 5, 3, 96)],
          (2, 2, 4, 4): [(96, 11, 20, 14, 5, 3, 64), (64, 9, 13, 10, 3, 2, 192)],
          (2, 2, 4, 2): [(120, 4, 4, 10, 3, 1, 64)],
          (4, 2, 2, 4): [(64, 13, 9, 2, 3, 2, 32), (80, 15, 15, 14, 5, 2, 96)],
          (4, 2, 2, 1): [(84, 6, 5, 1, 2, 1, 32), (76, 11, 17, 14, 5, 3, 96), (68, 8, 8, 6, 5, 1, 32)]}


def bar(n):
    return 4.0 * max(n, 16) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("tile,shape", [(k, s) for k, v in SHAPES.items() for s in v], ids=str)
def test_tiles(tile, shape):
    print(f"case split weight gradient {tile} {shape}", flush=True)
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    (p,) = lc.plan_query(G, lc.LC_OP_BACKWARD_WEIGHTS, lc.LC_F32)
    assert (p["kernel"], tuple(p["tparam"][:4])) == ("lc_bwd_weights_fast", tile)
    x, w, dy = wl.lc_inputs(g, "gaussian", seed=3)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
    dw = torch.full(w.shape, float("nan"), device="cuda")
    lc.lc_backward_weights(G, xd, yd, 0.0, dw)
    ref = oracle.lc_backward_weights(shape, x, dy)
    assert rel_fro(dw.cpu().numpy(), ref) <= bar(g.B)
    acc = torch.from_numpy(w).cuda()
    lc.lc_backward_weights(G, xd, yd, 1.0, acc)
    assert rel_fro(acc.cpu().numpy(), ref + w.astype(np.float64)) <= bar(g.B)
    again = torch.full_like(dw, float("nan"))
    lc.lc_backward_weights(G, xd, yd, 0.0, again)
    assert torch.equal(dw, again)


@pytest.mark.parametrize("shape", [SHAPES[1, 4, 4, 1][1], SHAPES[2, 4, 2, 1][0], SHAPES[2, 2, 4, 2][0], SHAPES[4, 2, 2, 1][2]], ids=str)
@pytest.mark.parametrize("scale", [1.0, 1e-30, 2e38], ids=str)
def test_infinities_and_ends_of_the_range(shape, scale):
    """Infinities and NaNs stay in the weights that they reach; small and large values keep their precision (parts that overflow
    where fp32 does not: formed again in fp32)."""
    print(f"case split weight gradient range {shape} {scale}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, dy = wl.lc_inputs(g, "gaussian", seed=4)
    dy = (dy / np.abs(dy).max() / 256).astype(np.float32)
    x = (x / np.abs(x).max() * scale).astype(np.float32)
    if scale == 1.0:
        x[0, 0, 0, 0] = np.inf
        x[g.B - 1, g.H - 1, g.W - 1, g.C - 1] = -np.inf
        dy[g.B // 2, g.LH // 2, g.LW // 2, g.F // 2] = np.nan
    else:
        x[0, 0, 0, 0] = 1.69 * scale
    dw = torch.full(w.shape, float("nan"), device="cuda")
    lc.lc_backward_weights(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda(), 0.0, dw)
    ref, out = oracle.lc_backward_weights(shape, x, dy), dw.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert m.any() and rel_fro(out[m].astype(np.float64) / scale, ref[m] / scale) <= bar(g.B)


@pytest.mark.parametrize("shape", [SHAPES[1, 4, 4, 2][0], SHAPES[2, 4, 2, 4][0], SHAPES[2, 2, 4, 4][0], SHAPES[4, 2, 2, 4][0]], ids=str)
def test_two_terms_and_row_norms(shape):
    """The training step's update: two pairs of operands into one gradient, and the squares that its row projection sums."""
    print(f"case split weight gradient sae_step {shape}", flush=True)
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=7)
    b = np.zeros((g.H, g.W, g.C), dtype=np.float32)
    wd, bd = torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda()
    alpha, cost = torch.full((1,), 0.8, device="cuda"), torch.full((1,), float("nan"), device="cuda")
    ws = torch.empty(lc.workspace_bytes(G, lc.LC_OP_SAE_STEP), dtype=torch.uint8, device="cuda")
    lc.sae_step(G, torch.from_numpy(x).cuda(), wd, bd, alpha, 0.1, 1e-6, 1e-2, lc.LC_SAE_PROJECT_ROWS, None, cost, ws)
    _, wo, _, _, _ = oracle.sae_step(shape, x, w, b, float(np.float32(0.8)), 0.1, 1e-6, 1e-2, 1)
    out = wd.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(np.linalg.norm(out, axis=2), 1.0, rtol=1e-6)
    assert rel_fro(out, wo) <= 1e-6


@pytest.mark.parametrize("step", [1, 2])
@pytest.mark.parametrize("shape", [SHAPES[1, 4, 4, 1][1], SHAPES[2, 2, 4, 4][0], SHAPES[4, 2, 2, 1][1]], ids=str)
def test_not_a_number_in_the_first_gradients(shape, step):
    """A diverged layer: NaN in every filter's first gradients (the sums are all NaN), or in every second one's."""
    print(f"case split weight gradient NaN {shape} {step}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, dy = wl.lc_inputs(g, "gaussian", seed=5)
    dy[2, :, :, ::step] = np.nan
    dw = torch.zeros(w.shape, device="cuda")
    lc.lc_backward_weights(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda(), 0.0, dw)
    ref, out = oracle.lc_backward_weights(shape, x, dy), dw.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.isnan(ref).all() == (step == 1)
    m = np.isfinite(ref)
    assert step == 1 or rel_fro(out[m], ref[m]) <= bar(g.B)


@pytest.mark.parametrize("image", [1, -1], ids=["first", "last"])
@pytest.mark.parametrize("shape", [SHAPES[1, 4, 4, 4][1], SHAPES[2, 4, 2, 1][0], SHAPES[2, 2, 4, 4][0], SHAPES[4, 2, 2, 1][0]], ids=str)
def test_not_a_number_in_one_filter(shape, image):
    """Among the first images a NaN sends a tile to the fp32 form at once, among the last ones after its split products: the filter's
    gradient is NaN, all others are what they are."""
    print(f"case split weight gradient NaN {shape} {image}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, dy = wl.lc_inputs(g, "gaussian", seed=6)
    dy[image, :, :, 0] = np.nan
    dw = torch.full(w.shape, float("nan"), device="cuda")
    lc.lc_backward_weights(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda(), 0.0, dw)
    ref, out = oracle.lc_backward_weights(shape, x, dy), dw.cpu().numpy()
    assert np.isnan(out[..., 0]).all() and np.isnan(ref[..., 0]).all()
    assert rel_fro(out[..., 1:], ref[..., 1:]) <= bar(g.B)


@pytest.mark.parametrize("shape", [SHAPES[1, 4, 4, 1][1], SHAPES[2, 4, 2, 1][0], SHAPES[2, 2, 4, 2][0], SHAPES[4, 2, 2, 1][2]], ids=str)
def test_infinite_gradients(shape):
    """An infinite gradient among the first or last images stays in its filter's weights."""
    print(f"case split weight gradient infinite gradients {shape}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, dy = wl.lc_inputs(g, "gaussian", seed=9)
    dy[0, 0, 0, 0], dy[g.B - 1, 0, 0, g.F - 1] = np.inf, -np.inf
    dw = torch.full(w.shape, float("nan"), device="cuda")
    lc.lc_backward_weights(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda(), 0.0, dw)
    ref, out = oracle.lc_backward_weights(shape, x, dy), dw.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert np.isinf(ref).any() and m.any() and rel_fro(out[m], ref[m]) <= bar(g.B)
