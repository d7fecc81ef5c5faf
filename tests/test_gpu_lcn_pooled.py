"""Normalisation with statistics pooled over the channels in tiles, one and two stages, against the fp64 oracle: lanes and
vectors per pixel, channels that are no multiple of a vector, workgroups of 256 to 1024 threads, halos wider than the map, and
the gradient that leaves dx / x to the pooling gradient.

Tolerance: sums of ks*ks*C terms, of which the one-stage variance is a difference of two, a few times their size; inputs
between 1 and 2 keep mean and deviation within a factor of four: 32 * sqrt(ks*ks) * 2^-24, four times that for gradients."""
import numpy as np
import pytest
import torch

import oracle
import paper_1502_03409_amd as lc
import workloads as wl
from conftest import rel_fro

pytestmark = pytest.mark.gpu

SHAPES = [((3, 9, 11, 1), 3), ((3, 9, 11, 2), 5), ((2, 17, 9, 3), 7), ((2, 17, 19, 4), 5), ((2, 17, 19, 5), 5), ((3, 12, 21, 7), 3),
          ((2, 40, 18, 8), 9), ((2, 30, 21, 9), 5), ((1, 33, 34, 12), 7), ((2, 14, 15, 18), 5), ((2, 14, 15, 20), 5), ((3, 25, 8, 31), 3),
          ((2, 21, 17, 72), 9), ((1, 12, 9, 97), 5), ((1, 34, 5, 384), 7), ((2, 10, 12, 203), 5), ((1, 5, 6, 1030), 3), ((1, 1, 1, 6), 5),
          ((2, 1, 50, 10), 9), ((2, 3, 3, 33), 15), ((70, 33, 35, 6), 5), ((30, 18, 40, 50), 3)]


@pytest.mark.parametrize("flags", [0, 2, 4, 6])
@pytest.mark.parametrize("shape,ks", SHAPES, ids=str)
def test_pooled_statistics(shape, ks, flags):
    print(f"case pooled statistics {shape} {ks} {flags}", flush=True)
    tol = 32.0 * ks * 2.0 ** -24
    rng = np.random.default_rng(5)
    x = (1.0 + rng.random(shape)).astype(np.float32)
    dy = rng.standard_normal(shape).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    y, dx = (torch.full(shape, float("nan"), device="cuda") for _ in range(2))
    mu, rs = (torch.full(shape[:3], float("nan"), device="cuda") for _ in range(2))
    lc.lcn_variant_fwd(xd, y, mu, rs, ks, wl.LCN_SIGMA, 1e-2, flags)
    y0, mu0, rs0 = oracle.lcn_var_fwd(x, ks, wl.LCN_SIGMA, 1e-2, flags)
    for got, ref in ((mu, mu0), (rs, rs0), (y, y0)):
        if np.linalg.norm(ref) > 1e-5 * ref.size ** 0.5:          # a single value leaves nothing but rounding
            assert rel_fro(got.cpu().numpy(), ref) <= tol
    ws = torch.full((max(lc.lcn_variant_workspace_bytes(shape, flags) // 4, 4),), float("nan"), device="cuda")
    mu32, rs32 = mu0.astype(np.float32), rs0.astype(np.float32)
    lc.lcn_variant_bwd(xd, torch.from_numpy(mu32).cuda(), torch.from_numpy(rs32).cuda(), torch.from_numpy(dy).cuda(), dx, ks,
                       wl.LCN_SIGMA, flags, ws)
    dx0 = oracle.lcn_var_bwd(x, mu32, rs32, dy, ks, wl.LCN_SIGMA, flags)
    got = dx.cpu().numpy()
    assert np.all(np.isfinite(got))
    assert np.linalg.norm(got - dx0) <= 4 * tol * max(np.linalg.norm(dx0), np.linalg.norm(rs0[..., None] * dy))


@pytest.mark.parametrize("flags", [0, 2, 4, 6])
@pytest.mark.parametrize("shape,ks", [((2, 9, 11, 1), 3), ((2, 9, 11, 6), 5), ((1, 20, 18, 20), 9)], ids=str)
def test_means_up_to_the_largest_float(shape, ks, flags):
    """Sums over the channels up to 0.9 of the largest float: the window means are finite (the variances are not)."""
    print(f"case large means {shape} {ks} {flags}", flush=True)
    x = torch.full(shape, 3.0e38 / shape[3], device="cuda")
    y = torch.empty(shape, device="cuda")
    mu, rs = (torch.full(shape[:3], float("nan"), device="cuda") for _ in range(2))
    lc.lcn_variant_fwd(x, y, mu, rs, ks, wl.LCN_SIGMA, 1e-2, flags)
    _, mu0, _ = oracle.lcn_var_fwd(x.cpu().numpy(), ks, wl.LCN_SIGMA, 1e-2, flags)
    assert rel_fro(mu.cpu().numpy(), mu0) <= 32.0 * ks * 2.0 ** -24


@pytest.mark.parametrize("shape", [(2, 20, 21, 12), (2, 20, 21, 24), (1, 15, 300, 8), (1, 12, 1100, 4), (2, 16, 15, 100)], ids=str)
def test_gradient_through_normalisation_and_pooling(shape):
    """lcn_l2pool_bwd where the tile kernel hands dp / p to the pooling gradient."""
    print(f"case dx over x {shape}", flush=True)
    rng = np.random.default_rng(6)
    x = (1.0 + rng.random(shape)).astype(np.float32)
    p = oracle.l2pool_fwd(x, 3, 1, wl.POOL_EPS).astype(np.float32)
    _, mu, rs = oracle.lcn_fwd(p, 5, wl.LCN_SIGMA, 1e-2)
    mu, rs = mu.astype(np.float32), rs.astype(np.float32)
    dn = rng.standard_normal(p.shape).astype(np.float32)
    dx0 = oracle.l2pool_bwd(x, p, oracle.lcn_bwd(p, mu, rs, dn, 5, wl.LCN_SIGMA), 3, 1)
    cuda = [torch.from_numpy(a).cuda() for a in (x, p, mu, rs, dn)]
    scratch, dx = torch.full(p.shape, float("nan"), device="cuda"), torch.full(shape, float("nan"), device="cuda")
    lc.lcn_l2pool_bwd(*cuda, scratch, dx, 3, 1, 5, wl.LCN_SIGMA)
    assert rel_fro(dx.cpu().numpy(), dx0) <= 4 * 32.0 * 5 * 2.0 ** -24
