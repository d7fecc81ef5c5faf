"""fp32 products that are split into bf16 parts, where the parts are hardest to hold: operands down to subnormal values (a third
part would lie below what bf16 holds) against large ones, and sums of a single product.  Layers of each split kernel, against the
fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

# (pass, kernel): layers whose tiles are split
LAYERS = [("forward", "lc_forward_wide", (70, 17, 16, 32, 16, 1, 128)), ("forward", "lc_forward_wide", (70, 17, 18, 16, 17, 1, 128)),
          ("forward", "lc_forward_general", (49, 27, 23, 8, 2, 1, 104)), ("forward", "lc_forward_general", (17, 15, 48, 7, 11, 1, 72)),
          ("data", "lc_bwd_data_wide", (80, 11, 13, 64, 4, 2, 64)), ("data", "lc_bwd_data_wide", (70, 15, 15, 3, 15, 1, 96)),
          ("data", "lc_bwd_data_general", (1, 19, 21, 7, 5, 4, 131)), ("data", "lc_bwd_data_general", (33, 24, 38, 16, 6, 2, 96)),
          ("weights", "lc_bwd_weights_fast", (64, 11, 15, 16, 5, 2, 32)), ("weights", "lc_bwd_weights_fast", (92, 20, 14, 1, 8, 3, 192)),
          ("weights", "lc_bwd_weights_fast", (96, 11, 20, 14, 5, 3, 64)), ("weights", "lc_bwd_weights_fast", (80, 15, 15, 14, 5, 2, 96))]
OPS = {"forward": lc.LC_OP_FORWARD, "data": lc.LC_OP_BACKWARD_DATA, "weights": lc.LC_OP_BACKWARD_WEIGHTS}


# A single product: 2^-24 for the partial products that are left out, and what the matrix unit cuts off where it adds the other five
# to the first, at most a unit in the last place (2^-23) of a sum that may lie just below the power of two it is aligned to.
SINGLE = 2.0 ** -22


def bar(n):
    return 4.0 * max(n, 16) ** 0.5 * 2.0 ** -24


def run(op, shape, first, second):
    """The pass on its two operands, (x, w), (dy, w) or (x, dy), and the oracle's result."""
    g, G = wl.LCGeom(*shape), lc.geom(*shape)
    a, b = torch.from_numpy(first).cuda(), torch.from_numpy(second).cuda()
    if op == "forward":
        out = torch.full((g.B, g.LH, g.LW, g.F), float("nan"), device="cuda")
        lc.lc_forward(G, a, b, None, 1.0, out)
        ref = oracle.lc_forward(shape, first, second)
    elif op == "data":
        out = torch.full((g.B, g.H, g.W, g.C), float("nan"), device="cuda")
        lc.lc_backward_data(G, a, b, out)
        ref = oracle.lc_backward_data(shape, first, second)
    else:
        out = torch.full((g.LH, g.LW, g.K, g.F), float("nan"), device="cuda")
        lc.lc_backward_weights(G, a, b, 0.0, out)
        ref = oracle.lc_backward_weights(shape, first, second)
    return out.cpu().numpy().astype(np.float64), ref


def operands(op, g):
    x, w, y = (g.B, g.H, g.W, g.C), (g.LH, g.LW, g.K, g.F), (g.B, g.LH, g.LW, g.F)
    return {"forward": (x, w), "data": (y, w), "weights": (x, y)}[op]


def terms(op, g):
    return {"forward": g.K, "data": g.F * (-(-g.R // g.S)) ** 2, "weights": g.B}[op]


@pytest.mark.parametrize("scale", [2.0 ** -112, 2.0 ** -118, 2.0 ** -126, 2.0 ** -130], ids=["2^-112", "2^-118", "2^-126", "2^-130"])
@pytest.mark.parametrize("small", [0, 1], ids=["first", "second"])
@pytest.mark.parametrize("op,kernel,shape", LAYERS, ids=str)
def test_small_operands(op, kernel, shape, small, scale):
    """Every value of one operand in [1, 2) times the scale, of the other in [1, 2) times 2^100.  Tolerance as for the general kernels."""
    print(f"case split small {op} {shape} {small} {scale}", flush=True)
    g = wl.LCGeom(*shape)
    assert lc.plan_query(lc.geom(*shape), OPS[op], lc.LC_F32)[0]["kernel"] == kernel
    rng = np.random.default_rng(8)
    v = [(rng.uniform(1.0, 2.0, s) * rng.choice([-1.0, 1.0], s)).astype(np.float32) for s in operands(op, g)]
    v[small] *= np.float32(scale)
    v[1 - small] *= np.float32(2.0 ** 100)
    out, ref = run(op, shape, *v)
    assert rel_fro(out / scale, ref / scale) <= bar(terms(op, g))


@pytest.mark.parametrize("op,kernel,shape", LAYERS, ids=str)
def test_some_small_operands(op, kernel, shape):
    """One value in a thousand of one operand at 2^-126 and the rest of it zero, so that few outputs have anything else in them."""
    print(f"case split some small {op} {shape}", flush=True)
    g = wl.LCGeom(*shape)
    rng = np.random.default_rng(9)
    v = [(rng.uniform(1.0, 2.0, s) * rng.choice([-1.0, 1.0], s)).astype(np.float32) for s in operands(op, g)]
    v[0] *= (rng.random(v[0].shape) < 1e-3) * np.float32(2.0 ** -126)
    v[1] *= np.float32(2.0 ** 100)
    out, ref = run(op, shape, *v)
    assert rel_fro(out * 2.0 ** 126, ref * 2.0 ** 126) <= bar(terms(op, g))


@pytest.mark.parametrize("op,kernel,shape", LAYERS, ids=str)
def test_single_products(op, kernel, shape):
    """Sums with one product that is not zero (every term of an output but one meets a zero)."""
    print(f"case split single products {op} {shape}", flush=True)
    g = wl.LCGeom(*shape)
    rng = np.random.default_rng(10)
    first, second = operands(op, g)
    a, b = rng.standard_normal(first).astype(np.float32), rng.standard_normal(second).astype(np.float32)
    if op == "forward":                                       # one element of every filter
        keep = rng.integers(0, g.K, (g.LH, g.LW, 1, g.F))
        b *= np.arange(g.K)[None, None, :, None] == keep
    elif op == "data":                                        # one filter of every gradient vector, and one field in (R/S)^2
        keep = rng.integers(0, g.F, (g.B, g.LH, g.LW, 1))
        a *= np.arange(g.F)[None, None, None, :] == keep
        n = -(-g.R // g.S)
        far = (np.arange(g.LH)[:, None] % n == 0) & (np.arange(g.LW)[None, :] % n == 0)
        a *= far[None, :, :, None]
    else:                                                     # one image of every gradient
        keep = rng.integers(0, g.B, (1, g.LH, g.LW, g.F))
        b *= np.arange(g.B)[:, None, None, None] == keep
    out, ref = run(op, shape, a, b)
    err = np.abs(out - ref)[ref != 0] / np.abs(ref[ref != 0])
    print(f"largest relative error 2^{np.log2(err.max()):.2f}, mean 2^{np.log2(err.mean()):.2f}", flush=True)
    assert np.all(out[ref == 0] == 0) and err.max() <= SINGLE
