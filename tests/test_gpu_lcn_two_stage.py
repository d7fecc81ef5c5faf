"""The two-stage per-channel normalisation: the kernel that walks both stages at once, at the edges of its strips, segments,
work items and windows, and the sizes on either side of its rule, against the fp64 oracle.

Tolerance: a window sum of KS + KS terms, a difference that cancels against the mean and two products, each rounded to
2^-24; the differences x - mu of neighbouring values lose at most the ratio |x| / std of the inputs (below 4 here):
4 * 4 * sqrt(2 KS) * 2^-24, and four times that for the gradient, which does it twice."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

SHAPES = [
    # smaller than the window, one row, one column, one value
    ((1, 1, 1, 1), 3), ((2, 2, 3, 4), 9), ((3, 1, 40, 8), 5), ((3, 40, 1, 6), 7), ((1, 4, 4, 20), 5),
    # channels of one, two and four a work item, a last piece of a pixel that is partly filled, a whole odd pixel
    ((5, 9, 11, 3), 3), ((5, 9, 11, 7), 5), ((4, 13, 12, 10), 7), ((4, 13, 12, 10), 9), ((2, 19, 17, 130), 5), ((3, 23, 21, 24), 9),
    # strips side by side and segments that end inside the map, work items of four channels
    ((2, 31, 301, 5), 3), ((1, 17, 603, 2), 7), ((9, 41, 60, 32), 3), ((9, 41, 60, 32), 5), ((3, 130, 47, 48), 5), ((2, 7, 700, 64), 5),
    # beyond the sizes that keep two passes
    ((4, 120, 31, 144), 7), ((4, 120, 31, 144), 9), ((6, 150, 146, 64), 5), ((40, 70, 4, 128), 5),
]


@pytest.mark.parametrize("flags", [5, 7])
@pytest.mark.parametrize("shape,ks", SHAPES)
def test_two_stage_per_channel(shape, ks, flags):
    print(f"case two-stage {shape} {ks} flags {flags}", flush=True)
    tol = 16.0 * (2 * ks) ** 0.5 * 2.0 ** -24
    rng = np.random.default_rng(7)
    x = (1.0 + rng.random(shape)).astype(np.float32)
    dy = rng.standard_normal(shape).astype(np.float32)
    y0, mu0, rs0 = oracle.lcn_var_fwd(x, ks, wl.LCN_SIGMA, 1e-2, flags)
    xd = torch.from_numpy(x).cuda()
    y, mu, rs, dx = (torch.full(shape, float("nan"), device="cuda") for _ in range(4))
    lc.lcn_variant_fwd(xd, y, mu, rs, ks, wl.LCN_SIGMA, 1e-2, flags)
    for got, ref in ((mu, mu0), (rs, rs0)):
        assert rel_fro(got.cpu().numpy(), ref) <= tol
    # one value has nothing but its mean's rounding left
    if y0.size > 1 or flags & 2:
        assert rel_fro(y.cpu().numpy(), y0) <= tol
    ws = torch.full((lc.lcn_variant_workspace_bytes(shape, flags) // 4,), float("nan"), device="cuda")
    mu32, rs32 = mu0.astype(np.float32), rs0.astype(np.float32)
    lc.lcn_variant_bwd(xd, torch.from_numpy(mu32).cuda(), torch.from_numpy(rs32).cuda(), torch.from_numpy(dy).cuda(), dx, ks,
                       wl.LCN_SIGMA, flags, ws)
    dx0 = oracle.lcn_var_bwd(x, mu32, rs32, dy, ks, wl.LCN_SIGMA, flags)
    assert np.all(np.isfinite(dx.cpu().numpy()))
    err = np.linalg.norm(dx.cpu().numpy() - dx0) / max(np.linalg.norm(dx0), np.linalg.norm(rs0 * dy))
    assert err <= 4 * tol
