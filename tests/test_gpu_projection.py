"""Row norms and rescaling behind the fused update of sae_step (Eq. 1's unit filters): lanes per filter, vectors that
cross a filter row or a field, filters fewer than a vector."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import check_sae_results, run_sae

pytestmark = pytest.mark.gpu

CASES = {
    # blocks of 64 patch elements per filter: 1, then 2 to 64 lanes per filter with remainders
    "one_lane": wl.LCGeom(B=6, H=14, W=17, C=3, R=5, S=3, F=10),
    "two_lanes": wl.LCGeom(B=5, H=25, W=25, C=3, R=15, S=5, F=20),
    "split_odd_filters": wl.LCGeom(B=4, H=26, W=20, C=16, R=18, S=1, F=27),
    "one_field_64_lanes": wl.LCGeom(B=8, H=62, W=62, C=24, R=62, S=1, F=6),
    # vectors across rows and fields, weights that are no multiple of four, fewer filters than a vector holds
    "cross_fields": wl.LCGeom(B=7, H=13, W=11, C=3, R=3, S=1, F=5),
    "tail": wl.LCGeom(B=3, H=9, W=9, C=1, R=3, S=1, F=7),
    "three_filters": wl.LCGeom(B=9, H=15, W=16, C=2, R=5, S=2, F=3),
    "one_filter": wl.LCGeom(B=9, H=15, W=16, C=2, R=5, S=2, F=1),
    # four vectors a lane, in one trip and (over 17 million weights) in several, which carry field and filter along
    "four_vectors_odd": wl.LCGeom(B=3, H=40, W=40, C=3, R=9, S=2, F=27),
    "four_vectors_whole": wl.LCGeom(B=3, H=40, W=40, C=3, R=9, S=2, F=20),
    "trips_odd": wl.LCGeom(B=2, H=100, W=100, C=3, R=10, S=2, F=27),
    "trips_whole": wl.LCGeom(B=2, H=100, W=100, C=3, R=10, S=2, F=28),
}


@pytest.mark.parametrize("name", list(CASES))
def test_projection_matches_oracle(name):
    g = CASES[name]
    print(f"case projection {name} geom {g}", flush=True)
    x, w, _ = wl.lc_inputs(g, "gaussian", seed=1)
    b = (0.05 * np.random.default_rng(3).standard_normal((g.H, g.W, g.C))).astype(np.float32)
    alpha, lam, eps_s, lr, flags = 0.9, wl.SAE_LAMBDA, wl.SAE_EPS, 1e-2, 3
    got = run_sae(g, x, w, b, alpha, lam, eps_s, lr, flags)
    ref = oracle.sae_step(g.as_tuple(), x, w, b, alpha, lam, eps_s, lr, flags)
    check_sae_results(name, got, ref, (w, b), alpha, flags)
