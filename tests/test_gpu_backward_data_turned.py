"""The backward-data kernel that turns its operands in LDS: one layer for every tile it is launched in, with and without masks
(the least work found among seeded layers that the plan gives that tile), against the fp64 oracle.  Tolerance as for the
general kernels: four times sqrt(n) roundings of 2^-24, which products split into bf16 parts meet as well."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

# (image tiles, value tiles, masks): layer
F32 = {(1, 1, 0): (2, 4, 2, 1, 2, 2, 64), (1, 1, 1): (1, 3, 10, 1, 2, 5, 64), (1, 2, 0): (1, 13, 39, 4, 8, 4, 64),
       (1, 2, 1): (1, 35, 19, 1, 6, 5, 127), (1, 3, 0): (1, 18, 14, 4, 9, 3, 96), (1, 3, 1): (1, 25, 14, 3, 7, 2, 26),
       (1, 4, 0): (1, 17, 20, 16, 8, 2, 32), (1, 4, 1): (1, 19, 21, 7, 5, 4, 131), (2, 1, 0): (17, 26, 17, 1, 2, 1, 32),
       (2, 1, 1): (17, 6, 15, 1, 2, 1, 57), (2, 2, 0): (17, 35, 19, 5, 8, 2, 16), (2, 2, 1): (17, 32, 38, 1, 12, 5, 53),
       (2, 3, 0): (49, 12, 45, 4, 9, 3, 96), (2, 3, 1): (17, 25, 39, 4, 7, 3, 57), (2, 4, 0): (17, 20, 41, 16, 12, 4, 96),
       (2, 4, 1): (17, 29, 42, 8, 9, 4, 65), (3, 1, 0): (33, 9, 15, 2, 3, 1, 112), (3, 1, 1): (33, 11, 27, 1, 3, 2, 65),
       (3, 2, 0): (33, 35, 31, 2, 12, 3, 48), (3, 2, 1): (33, 19, 46, 3, 8, 3, 65), (3, 3, 0): (70, 28, 41, 16, 3, 3, 80),
       (3, 3, 1): (130, 28, 33, 16, 2, 3, 16), (3, 4, 0): (33, 24, 38, 16, 6, 2, 96),
       (3, 4, 1): (130, 31, 42, 16, 2, 4, 16), (4, 1, 0): (49, 17, 18, 3, 8, 2, 32), (4, 1, 1): (49, 14, 16, 1, 3, 2, 127),
       (4, 2, 0): (128, 25, 30, 16, 3, 3, 16), (4, 2, 1): (97, 32, 40, 16, 2, 5, 40), (4, 3, 0): (97, 35, 39, 16, 5, 5, 16),
       (4, 3, 1): (128, 31, 40, 16, 2, 3, 32), (4, 4, 1): (97, 35, 47, 7, 9, 4, 53)}
BF16 = {(1, 1, 0): (2, 4, 2, 1, 2, 2, 64), (1, 1, 1): (1, 3, 10, 1, 2, 5, 64), (1, 2, 0): (1, 23, 36, 2, 3, 3, 32),
        (1, 2, 1): (1, 13, 11, 1, 6, 5, 64), (1, 3, 0): (1, 18, 17, 3, 12, 4, 96), (1, 3, 1): (1, 9, 34, 1, 5, 4, 57),
        (1, 4, 0): (1, 16, 16, 7, 9, 3, 32), (1, 4, 1): (1, 35, 12, 2, 6, 5, 57), (2, 1, 0): (130, 20, 5, 1, 2, 2, 32),
        (2, 1, 1): (31, 6, 21, 7, 2, 5, 32), (2, 2, 0): (17, 29, 17, 1, 10, 5, 64), (2, 2, 1): (17, 11, 18, 1, 6, 5, 127),
        (2, 3, 0): (17, 13, 22, 4, 12, 3, 64), (2, 3, 1): (17, 23, 38, 16, 2, 5, 32), (2, 4, 0): (17, 21, 20, 4, 10, 5, 64),
        (2, 4, 1): (17, 15, 14, 4, 6, 5, 131), (3, 1, 0): (70, 28, 13, 1, 2, 2, 32), (3, 1, 1): (33, 6, 16, 16, 2, 5, 32),
        (3, 2, 0): (33, 13, 21, 5, 12, 4, 96), (3, 2, 1): (130, 31, 17, 1, 2, 5, 104),
        (3, 3, 0): (33, 12, 26, 5, 12, 3, 64), (3, 3, 1): (33, 10, 35, 1, 5, 3, 131), (3, 4, 0): (47, 30, 17, 4, 12, 4, 96),
        (3, 4, 1): (33, 15, 31, 2, 7, 5, 127), (4, 1, 0): (128, 11, 33, 1, 2, 2, 32), (4, 1, 1): (49, 31, 6, 7, 2, 5, 104),
        (4, 2, 0): (49, 17, 30, 2, 12, 4, 96), (4, 2, 1): (49, 10, 20, 2, 5, 4, 127), (4, 3, 0): (49, 14, 24, 4, 9, 3, 96),
        (4, 3, 1): (97, 12, 16, 2, 4, 3, 131), (4, 4, 0): (49, 17, 22, 7, 12, 3, 96), (4, 4, 1): (49, 14, 25, 4, 6, 5, 127)}


def bar(n):
    return 4.0 * max(n, 16) ** 0.5 * 2.0 ** -24


def operand(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    t = t.bfloat16() if dtype == lc.LC_BF16 else t
    return t, t.float().cpu().numpy()


@pytest.mark.parametrize("tile,shape", [((0, *k), v) for k, v in F32.items()] + [((1, *k), v) for k, v in BF16.items()], ids=str)
def test_tiles(tile, shape):
    print(f"case turned backward data {tile} {shape}", flush=True)
    dtype, MT, NT, mask = tile
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    (p,) = lc.plan_query(G, lc.LC_OP_BACKWARD_DATA, dtype)
    whole = p["arg"][:2] == [g.S, g.S] and g.R % g.S == 0 and g.F % (32 if dtype else 16) == 0
    assert (p["kernel"], p["tparam"][0], p["tparam"][1], p["tparam"][7], int(not whole)) == ("lc_bwd_data_general", MT, NT, 1, mask)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=3)
    (yd, yv), (wd, wv) = operand(dy, dtype), operand(w, dtype)
    dx = torch.full((g.B, g.H, g.W, g.C), float("nan"), device="cuda")
    lc.lc_backward_data(G, yd, wd, dx, dtype)
    ref, out = oracle.lc_backward_data(shape, yv, wv), dx.cpu().numpy()
    assert rel_fro(out, ref) <= bar(g.F * (-(-g.R // g.S)) ** 2)
    assert np.all(out[ref == 0.0] == 0.0)
    again = torch.full_like(dx, float("nan"))
    lc.lc_backward_data(G, yd, wd, again, dtype)
    assert torch.equal(dx, again)


@pytest.mark.parametrize("shape", [F32[1, 1, 1], F32[1, 2, 1], F32[1, 4, 0], F32[1, 4, 1], F32[2, 2, 1], F32[3, 2, 1]], ids=str)
@pytest.mark.parametrize("scale", [1.0, 1e-30, 2e38], ids=str)
def test_infinities_and_ends_of_the_range(shape, scale):
    """Infinities and NaNs of a field stay in its pixels, as the sums of fp32 products have them; small and large values keep
    their precision (products split into bf16 parts overflow where fp32 does not: formed again)."""
    print(f"case turned backward data range {shape} {scale}", flush=True)
    g = wl.LCGeom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=4)
    dy = (dy / np.abs(dy).max() * scale).astype(np.float32)
    w = (w / np.abs(w).max() / 64).astype(np.float32)
    if scale == 1.0:
        dy[0, 0, 0, g.F - 1] = np.inf
        dy[g.B - 1, g.LH - 1, g.LW - 1, 0] = -np.inf
        dy[g.B // 2, g.LH // 2, g.LW // 2, g.F // 2] = np.nan
    else:
        dy[0, 0, 0, 0] = 1.69 * scale
    dx = torch.full((g.B, g.H, g.W, g.C), float("nan"), device="cuda")
    lc.lc_backward_data(lc.geom(*shape), torch.from_numpy(dy).cuda(), torch.from_numpy(w).cuda(), dx)
    ref, out = oracle.lc_backward_data(shape, dy, w), dx.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    if m.any():
        assert rel_fro(out[m].astype(np.float64) / scale, ref[m] / scale) <= bar(g.F * (-(-g.R // g.S)) ** 2)


@pytest.mark.parametrize("shape", [F32[1, 1, 1], F32[1, 2, 1], F32[1, 4, 0], F32[1, 4, 1], F32[2, 2, 1], F32[3, 2, 1]], ids=str)
def test_infinite_weights(shape):
    """An infinite weight stays in the pixel that it reaches."""
    print(f"case turned backward data infinite weights {shape}", flush=True)
    g = wl.LCGeom(*shape)
    _, w, dy = wl.lc_inputs(g, "gaussian", seed=9)
    w[0, 0, 0, 0], w[g.LH - 1, g.LW - 1, -1, g.F - 1] = np.inf, -np.inf
    dx = torch.full((g.B, g.H, g.W, g.C), float("nan"), device="cuda")
    lc.lc_backward_data(lc.geom(*shape), torch.from_numpy(dy).cuda(), torch.from_numpy(w).cuda(), dx)
    ref, out = oracle.lc_backward_data(shape, dy, w), dx.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert np.isinf(ref).any() and rel_fro(out[m], ref[m]) <= bar(g.F * (-(-g.R // g.S)) ** 2)
