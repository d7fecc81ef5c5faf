"""The forward kernel that turns its operands in LDS: one layer for every tile and form it is launched in (the least work found
among seeded layers that the plan gives that tile), against the fp64 oracle.  Tolerance as for the general kernels: four times
sqrt(n) roundings of 2^-24, which products split into bf16 parts meet as well."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

# (tile, form): layer; form 1: rows of whole 16-element blocks, 2: places from a table (ragged and whole vectors)
F32 = {(1, 1, 1): (1, 3, 6, 8, 2, 5, 24), (1, 1, 2): (65, 37, 34, 4, 11, 1, 8), (1, 2, 1): (1, 16, 39, 8, 2, 2, 150),
       (1, 2, 2): (17, 36, 42, 5, 10, 1, 24), (1, 3, 1): (1, 29, 43, 32, 4, 4, 40), (1, 3, 2): (17, 35, 51, 2, 11, 1, 40),
       (1, 4, 1): (1, 22, 37, 8, 2, 1, 163), (1, 4, 2): (17, 37, 38, 2, 11, 1, 64), (2, 1, 1): (17, 18, 41, 8, 2, 2, 80),
       (2, 1, 2): (49, 25, 44, 7, 10, 1, 8), (2, 2, 1): (63, 31, 34, 8, 2, 1, 24), (2, 2, 2): (49, 39, 43, 2, 12, 1, 24),
       (2, 3, 1): (63, 30, 38, 8, 2, 2, 80), (2, 3, 2): (17, 15, 48, 7, 11, 1, 72), (2, 4, 1): (49, 15, 20, 4, 4, 1, 112),
       (2, 4, 2): (17, 35, 46, 5, 9, 2, 104), (3, 1, 1): (33, 29, 34, 8, 2, 1, 8), (3, 1, 2): (33, 30, 51, 7, 11, 1, 8),
       (3, 2, 1): (33, 32, 17, 8, 2, 1, 150), (3, 2, 2): (33, 24, 35, 7, 10, 1, 24), (3, 3, 1): (33, 14, 42, 8, 2, 1, 72),
       (3, 3, 2): (33, 29, 15, 5, 11, 1, 129), (3, 4, 1): (33, 23, 37, 8, 2, 1, 104), (3, 4, 2): (33, 39, 32, 5, 11, 3, 163),
       (4, 1, 1): (97, 32, 36, 8, 4, 1, 8), (4, 1, 2): (97, 40, 39, 4, 10, 1, 8), (4, 2, 1): (49, 30, 19, 16, 8, 3, 150),
       (4, 2, 2): (49, 12, 43, 5, 11, 1, 150), (4, 3, 1): (49, 26, 35, 8, 2, 2, 163), (4, 3, 2): (49, 27, 13, 7, 11, 1, 129),
       (4, 4, 1): (49, 27, 23, 8, 2, 1, 104), (4, 4, 2): (49, 29, 32, 7, 7, 2, 104)}
BF16 = {(1, 1, 1): (1, 5, 15, 4, 4, 5, 8), (1, 2, 1): (1, 3, 29, 8, 2, 5, 24), (1, 2, 2): (33, 29, 46, 3, 11, 1, 24),
        (1, 4, 1): (1, 26, 6, 8, 2, 1, 163), (1, 4, 2): (17, 23, 26, 5, 9, 1, 104), (2, 1, 1): (97, 27, 32, 8, 2, 3, 8),
        (2, 1, 2): (17, 42, 51, 7, 12, 1, 16), (2, 2, 1): (49, 23, 7, 8, 2, 1, 40), (2, 2, 2): (17, 36, 42, 5, 10, 1, 24),
        (2, 4, 1): (49, 27, 17, 8, 2, 1, 104), (2, 4, 2): (17, 24, 41, 7, 11, 2, 131), (3, 1, 1): (33, 32, 33, 8, 2, 2, 8),
        (3, 1, 2): (33, 30, 51, 7, 11, 1, 8), (3, 2, 1): (33, 23, 25, 4, 4, 1, 40), (3, 2, 2): (33, 21, 38, 7, 11, 1, 32),
        (3, 4, 1): (33, 16, 41, 8, 2, 1, 129), (3, 4, 2): (33, 30, 36, 7, 12, 3, 129), (4, 1, 1): (97, 7, 39, 8, 2, 1, 8),
        (4, 1, 2): (97, 32, 34, 4, 11, 1, 8), (4, 2, 1): (97, 21, 28, 8, 2, 1, 40), (4, 2, 2): (49, 13, 44, 7, 11, 1, 72),
        (4, 4, 1): (63, 15, 37, 8, 2, 1, 72), (4, 4, 2): (49, 27, 13, 7, 11, 1, 129)}
# contractions in slices: number, form
SLICES = {(2, 1): (1, 15, 39, 8, 8, 4, 40), (8, 1): (1, 19, 8, 4, 8, 5, 8), (16, 1): (1, 15, 8, 8, 8, 5, 8), (2, 2): (49, 23, 47, 7, 11, 1, 8)}


def bar(n):
    return 4.0 * max(n, 16) ** 0.5 * 2.0 ** -24


def operand(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    t = t.bfloat16() if dtype == lc.LC_BF16 else t
    return t, t.float().cpu().numpy()


def compare(shape, dtype):
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    x, w, _, bias = wl.lc_inputs(g, "gaussian", seed=1, with_bias=True)
    (xd, xv), (wd, wv) = operand(x, dtype), operand(w, dtype)
    y = torch.full((g.B, g.LH, g.LW, g.F), float("nan"), device="cuda")
    lc.lc_forward(G, xd, wd, torch.from_numpy(bias).cuda(), 0.75, y, dtype)
    assert rel_fro(y.cpu().numpy(), oracle.lc_forward(shape, xv, wv, bias, 0.75)) <= bar(g.K)
    again = torch.full_like(y, float("nan"))
    lc.lc_forward(G, xd, wd, torch.from_numpy(bias).cuda(), 0.75, again, dtype)
    assert torch.equal(y, again)


@pytest.mark.parametrize("tile,shape", [((0, *k), v) for k, v in F32.items()] + [((1, *k), v) for k, v in BF16.items()], ids=str)
def test_tiles(tile, shape):
    print(f"case turned forward {tile} {shape}", flush=True)
    (p,) = lc.plan_query(lc.geom(*shape), lc.LC_OP_FORWARD, tile[0])
    assert (p["kernel"], p["tparam"][0], p["tparam"][1], p["tparam"][7]) == ("lc_forward_general", *tile[1:])
    compare(shape, tile[0])


@pytest.mark.parametrize("slices,shape", SLICES.items(), ids=str)
def test_slices(slices, shape):
    print(f"case turned forward slices {slices} {shape}", flush=True)
    (p,) = lc.plan_query(lc.geom(*shape), lc.LC_OP_FORWARD, lc.LC_F32)
    assert (p["tparam"][5], p["tparam"][7]) == slices
    compare(shape, lc.LC_F32)


@pytest.mark.parametrize("shape", [F32[1, 2, 1], F32[2, 3, 1], F32[4, 4, 1], F32[2, 3, 2], F32[1, 3, 2]], ids=str)
@pytest.mark.parametrize("scale", [1.0, 1e-30, 2e38], ids=str)
def test_infinities_and_ends_of_the_range(shape, scale):
    """Infinite pixels make the outputs of their fields infinite or NaN as the sums of fp32 products are, nothing else; small
    and large values keep their precision (products split into bf16 parts overflow where fp32 does not: formed again)."""
    print(f"case turned forward range {shape} {scale}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=2)
    x = (x / np.abs(x).max() * scale).astype(np.float32)
    w = (w / 64).astype(np.float32)
    if scale == 1.0:
        x[0, 1, 2, 0] = np.inf
        x[g.B - 1, g.H // 2, g.W // 2, g.C - 1] = -np.inf
    else:
        x[0, 0, 0, 0] = 1.69 * scale
    y = torch.full((g.B, g.LH, g.LW, g.F), float("nan"), device="cuda")
    lc.lc_forward(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None, 1.0, y)
    ref, y = oracle.lc_forward(shape, x, w), y.cpu().numpy()
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert m.mean() > 0.3 and rel_fro(y[m].astype(np.float64) / scale, ref[m] / scale) <= bar(g.K)


@pytest.mark.parametrize("shape", [(49, 27, 23, 8, 2, 1, 145), (49, 27, 23, 8, 2, 1, 193), (64, 30, 30, 16, 4, 2, 193)], ids=str)
def test_one_writer_for_every_filter(shape):
    """A last block of one filter: its wave also forms the two or three before it, which belong to the block before.  Formed again in
    fp32 for an infinite weight, it leaves those as they are, bit by bit; and so does the block before with the last one."""
    print(f"case turned forward last filters {shape}", flush=True)
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    (p,) = lc.plan_query(G, lc.LC_OP_FORWARD, lc.LC_F32)
    MT, NT = p["tparam"][:2]
    assert p["tparam"][7] and MT * NT >= 6 and g.F % (16 * NT) == 1
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=7)
    xd = torch.from_numpy(x).cuda()

    def forward(weights):
        y = torch.full((g.B, g.LH, g.LW, g.F), float("nan"), device="cuda")
        lc.lc_forward(G, xd, torch.from_numpy(weights).cuda(), None, 1.0, y)
        return y

    y = forward(w)
    assert rel_fro(y.cpu().numpy(), oracle.lc_forward(shape, x, w)) <= bar(g.K)
    last, before = w.copy(), w.copy()
    last[:, :, 1, g.F - 1], before[:, :, 1, g.F - 1 - 8 * NT] = np.inf, np.inf
    assert torch.equal(forward(last)[..., :-1], y[..., :-1])
    assert torch.equal(forward(before)[..., -1], y[..., -1])


@pytest.mark.parametrize("row", [1, -2], ids=["first", "last"])
@pytest.mark.parametrize("shape", [F32[2, 3, 1], F32[4, 4, 1], F32[2, 3, 2], F32[4, 2, 2]], ids=str)
def test_not_a_number_in_one_filter(shape, row):
    """Among the first weights a NaN sends a tile to the fp32 form at once, among the last ones after its split products: the filter's
    outputs are NaN, all others are what they are."""
    print(f"case turned forward NaN {shape} {row}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=8)
    w[:, :, row, 3] = np.nan
    y = torch.full((g.B, g.LH, g.LW, g.F), float("nan"), device="cuda")
    lc.lc_forward(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None, 1.0, y)
    ref, out = oracle.lc_forward(shape, x, w), y.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.isnan(ref[..., 3]).all()
    m = np.isfinite(ref)
    assert rel_fro(out[m], ref[m]) <= bar(g.K)


@pytest.mark.parametrize("shape", [F32[1, 2, 1], F32[2, 3, 1], F32[4, 4, 1], F32[2, 3, 2], F32[1, 3, 2]], ids=str)
def test_infinite_weights(shape):
    """An infinite weight, the first or last of a patch, makes its filter's outputs infinite and no others."""
    print(f"case turned forward infinite weights {shape}", flush=True)
    g = wl.LCGeom(*shape)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=9)
    w[0, 0, -1, g.F - 1], w[g.LH - 1, g.LW - 1, 0, 0] = np.inf, -np.inf
    y = torch.full((g.B, g.LH, g.LW, g.F), float("nan"), device="cuda")
    lc.lc_forward(lc.geom(*shape), torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None, 1.0, y)
    ref, out = oracle.lc_forward(shape, x, w), y.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(out[np.isinf(ref)], ref[np.isinf(ref)])
    m = np.isfinite(ref)
    assert np.isinf(ref).any() and rel_fro(out[m], ref[m]) <= bar(g.K)
