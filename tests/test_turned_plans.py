"""The kernels that turn their operands in LDS: their index arithmetic replayed on the CPU from the launch plans.  Every product
of the definition is formed exactly once, every address a lane forms (32-bit offsets included) is inside its tensor."""
import random

import numpy as np
import pytest

import paper_1502_03409_amd as lc
from paper_1502_03409_amd import binding as B


def cdiv(a, b):
    return -(-a // b)


def divide(n, d):
    """Divisor::over."""
    s = 0
    while (1 << s) < d:
        s += 1
    m = (1 << (31 + s)) // d + 1
    assert m < 2 ** 32
    return (n * m) >> (31 + s)


def test_division_by_a_product():
    r = random.Random(1)
    for d in [1, 2, 3, 5, 7, 9, 64, 65535, 65537, 2 ** 30, 2 ** 31 - 1] + [r.randrange(1, 2 ** 31) for _ in range(2000)]:
        for n in [0, 1, d - 1, d, d + 1, 2 * d - 1, 2 ** 31 - 1] + [r.randrange(2 ** 31) for _ in range(20)]:
            if 0 <= n < 2 ** 31:
                assert divide(n, d) == n // d, (n, d)


def geometries(n, seed, filters):
    r = random.Random(seed)
    while n:
        R, S, C = r.randint(1, 9), r.randint(1, 6), r.choice([1, 2, 3, 4, 5, 8, 16])
        H, W = R + r.randint(0, 24), R + r.randint(0, 30)
        n -= 1
        yield (r.choice([1, 2, 5, 16, 17, 37, 64, 70, 130]), H, W, C, R, S, r.choice(filters))


@pytest.mark.parametrize("seed", range(3))
def test_forward(seed):
    forms = {1: 0, 2: 0}
    large = [(65, 37, 34, 4, 11, 1, 8), (17, 36, 42, 5, 10, 1, 24), (49, 43, 41, 3, 12, 1, 40), (70, 75, 99, 3, 11, 3, 40), (130, 60, 41, 7, 9, 2, 129),
             (33, 39, 32, 5, 11, 3, 163), (64, 51, 60, 1, 17, 2, 104)]
    for geo in [*geometries(500, 10 + seed, [8, 16, 24, 40, 64, 104, 129, 130, 136, 163]), *large]:
        G = lc.geom(*geo)
        Bn, H, W, C, R, S, F = geo
        LH, LW, K = lc.geom_derive(G)
        RC, WC = R * C, W * C
        for dtype in (B.LC_F32, B.LC_BF16):
            p = lc.plan_query(G, B.LC_OP_FORWARD, dtype)[0]
            if p["kernel"] != "lc_forward_general" or p["tparam"][7] == 0:
                continue
            MT, NT, nfw, ES, rag, ks, tasks, form = p["tparam"][:8]
            NV, nvt, per, nbt, ntask = p["arg"][:5]
            forms[form] += 1
            GP, PF = (2, 1) if ES == 4 and MT * NT >= 6 else (1, 4)
            seen = np.zeros(K, dtype=int)
            back = 4 * NV - RC
            for sl in range(ks):
                vbeg, vend = sl * per, min((sl + 1) * per, nvt)
                ng = cdiv(max(vend - vbeg, 0), 4)
                if ng == 0:
                    continue
                steps = cdiv(ng, GP)
                for q in range(GP * (steps + PF)):            # groups loaded; those from ng on are never used
                    for k4 in range(4):
                        vi = vbeg + 4 * q + k4
                        if form == 2:
                            e = min(vi, nvt - 1)
                            assert vi < nvt + 32 - 4          # the next group's place is read as well
                        else:
                            last = vbeg + 4 * (ng - 1)
                            e = min(vbeg + 4 * q, last) + k4
                        row, v = divide(e, NV), e - divide(e, NV) * NV
                        sh = back if v == NV - 1 else 0
                        xo, wo = row * WC + 4 * v - sh, (row * RC + 4 * v - sh) * F
                        # the four elements lie in the field's rows and in its K x F matrix
                        assert 0 <= xo and xo + 4 <= (R - 1) * WC + RC and 0 <= wo and wo + 3 * F + F <= K * F
                        if q < ng and vi < vend:
                            seen[row * RC + 4 * v:row * RC + 4 * v - sh + 4] += 1   # (its first `sh` elements count as zero)
            assert (seen == 1).all(), (geo, p)
            # four filters a lane, ending at the last one, and the run a lane reads of them
            if NT <= 2 and F >= 4:
                for f0 in range(0, cdiv(F, 16 * NT) * 16 * NT, 16 * NT):
                    for n in range(16):
                        fl = min(f0 + NT * n, F - NT)
                        q = (fl - f0 + NT - 1) // 4
                        start = min(f0 + 4 * q, F - 4)
                        assert 0 <= q < 4 * NT and 0 <= start <= fl and fl + NT <= start + 4
            assert ntask == LH * LW * nbt and p["grid"][0] * tasks >= ntask and p["block"] == 64 * ks * nfw * tasks
    assert min(forms.values()) > 5, forms


@pytest.mark.parametrize("seed", range(3))
def test_backward_data(seed):
    turned = 0
    for geo in geometries(120, 40 + seed, [13, 16, 26, 32, 40, 48, 53, 64, 65, 80, 112, 127, 131]):
        G = lc.geom(*geo)
        Bn, H, W, C, R, S, F = geo
        LH, LW, K = lc.geom_derive(G)
        RC = R * C
        for dtype in (B.LC_F32, B.LC_BF16):
            p = lc.plan_query(G, B.LC_OP_BACKWARD_DATA, dtype)[0]
            if p["kernel"] != "lc_bwd_data_general" or p["tparam"][7] == 0:
                continue
            turned += 1
            MT, NT, ES, _, ks, tasks = p["tparam"][:6]
            PR, PC, cbc, _, nbt, ntask = p["arg"][:6]
            V, N = 16 // ES, PR * PC * C
            GW, FG = 4 * V, cdiv(F, 4 * V)
            mask = not (PR == S and PC == S and R % S == 0 and F % GW == 0)
            vals = np.arange(N)
            dr, rem = vals // (PC * C), vals % (PC * C)
            dc, c = rem // C, rem % C
            for rb in {0, cdiv(H, PR) // 2, cdiv(H, PR) - 1}:
                for cb in {0, cbc // 2, cbc - 1}:
                    r0, c0 = rb * PR, cb * PC
                    i_lo, i_hi = max(0, r0 - R + S) // S, min(LH - 1, (r0 + PR - 1) // S)
                    j_lo, j_hi = max(0, c0 - R + S) // S, min(LW - 1, (c0 + PC - 1) // S)
                    na, nap = i_hi - i_lo + 1, j_hi - j_lo + 1
                    ngt = na * nap * FG if na > 0 and nap > 0 else 0
                    per = cdiv(ngt, ks)
                    rr, cc = r0 + dr - i_lo * S, c0 + dc - j_lo * S
                    formed = {}
                    first = i_lo * LW + j_lo
                    for sl in range(ks):
                        for q in range(sl * per, sl * per + max(min(per, ngt - sl * per), 0)):
                            fi, fg = q // FG, q % FG
                            fa, fp = int((np.float32(fi) + np.float32(0.5)) * (np.float32(1) / np.float32(nap))), 0
                            assert fa == fi // nap
                            fp = fi - fa * nap
                            ra, ca = fa * S, fp * S
                            rf, cf = r0 - i_lo * S - ra, c0 - j_lo * S - ca
                            part = rf < 0 or rf + PR > R or cf < 0 or cf + PC > R
                            ok = (rr - ra >= 0) & (rr - ra < R) & (cc - ca >= 0) & (cc - ca < R)
                            assert part or ok.all()
                            assert mask or not part
                            boff = (fa * (LW * K - S * RC) + fp * (K - S * C)) * F + GW * fg
                            aoff = (fa * LW + fp) * F + GW * fg
                            for kl in range(4):
                                over = max(0, GW * (FG - 1) + V * kl - (F - V)) if F % GW and fg == FG - 1 else 0
                                skip = min(over, V)
                                # 32-bit offsets from the block's first field
                                a = aoff + V * kl - over
                                assert 0 <= a and first * F + a + V <= LH * LW * F
                                off = boff + (rr * RC + cc * C + c) * F + V * kl - over
                                off = np.where(ok, off, 0) if part else off
                                assert (off >= 0).all() and (off < 2 ** 31).all()
                                assert (first * K * F + off + V <= LH * LW * K * F).all()
                                if not mask:                  # scalar and lane parts one by one
                                    assert (V * kl + (rr * RC + cc * C + c) * F >= 0).all()
                                field = (i_lo + fa) * LW + j_lo + fp
                                k = (rr - ra) * RC + (cc - ca) * C + c
                                want = (field - first) * K * F + k * F + GW * fg + V * kl - over
                                assert (off[ok] == want[ok]).all()
                                for t in range(skip, V):
                                    key = (field, GW * fg + V * kl - over + t)
                                    formed[key] = formed.get(key, 0) + ok.astype(int)
                    for v in (0, N // 2, N - 1):
                        row, col = r0 + int(dr[v]), c0 + int(dc[v])
                        if row >= H or col >= W:
                            continue
                        cover = {(i * LW + j, f) for i in range(LH) for j in range(LW) for f in range(F)
                                 if 0 <= row - i * S < R and 0 <= col - j * S < R}
                        got = {key: int(n[v]) for key, n in formed.items() if n[v]}
                        assert set(got) == cover and all(n == 1 for n in got.values()), (geo, p, row, col)
    assert turned > 60


# layers whose direct form adds a pixel's sum in this many slices, and whose tiles here are not split into bf16 parts
@pytest.mark.parametrize("dtype,shape,slices", [(0, (3, 174, 21, 24, 4, 1, 64), 4), (0, (23, 34, 105, 16, 14, 1, 32), 8), (0, (20, 59, 36, 24, 5, 1, 16), 2),
                                                (0, (16, 25, 83, 32, 11, 1, 32), 8), (1, (16, 25, 83, 32, 11, 1, 32), 8), (1, (98, 73, 85, 3, 13, 8, 80), 2),
                                                (1, (128, 21, 81, 16, 4, 1, 64), 4), (1, (169, 45, 94, 3, 18, 3, 64), 8), (1, (64, 59, 63, 1, 9, 8, 128), 8)],
                         ids=str)
def test_backward_data_slices(dtype, shape, slices):
    """A sum that is formed in fewer slices than the direct form's is rounded more often in a row."""
    p = lc.plan_query(lc.geom(*shape), lc.LC_OP_BACKWARD_DATA, dtype)[0]
    assert (p["kernel"], p["tparam"][7]) == ("lc_bwd_data_general", 1)
    assert (dtype == 0 and p["tparam"][0] * p["tparam"][1] >= 3) or p["tparam"][4] >= slices


@pytest.mark.parametrize("shape,wide", [((70, 23, 24, 20, 8, 1, 128), True), ((70, 23, 22, 20, 8, 1, 128), False),
                                        ((128, 40, 40, 64, 4, 2, 128), False), ((64, 23, 24, 20, 8, 1, 128), False),
                                        ((70, 23, 24, 19, 8, 4, 128), False), ((70, 23, 24, 20, 8, 1, 64), False)], ids=str)
def test_long_patches_take_the_workgroup_tiles(shape, wide):
    """Patches of 1200 elements and a workgroup for every compute unit without slices: no workspace either way."""
    g = lc.geom(*shape)
    assert (lc.plan_query(g, lc.LC_OP_FORWARD, lc.LC_F32)[0]["kernel"] == "lc_forward_wide") == wide
    assert lc.workspace_bytes(g, lc.LC_OP_FORWARD, lc.LC_F32) == 0


@pytest.mark.parametrize("geo,dtype", [((64, 28, 142, 5, 20, 8, 223), 0), ((64, 28, 142, 5, 20, 8, 223), 1),
                                       ((64, 88, 28, 5, 16, 5, 382), 0)])
def test_large_layers_fill_the_compute_units(geo, dtype):
    """Layers of 131072 blocks and more: no tile whose workgroups leave a round of compute units more than a fifth empty where a
    smaller one does not (these had 160, 128 and 270 workgroups that a compute unit runs one by one)."""
    p = lc.plan_query(lc.geom(*geo), B.LC_OP_FORWARD, dtype)[0]
    n = p["grid"][0] * p["grid"][1]
    assert p["tparam"][7] and n / (256 * cdiv(n, 256)) >= 0.8, p


@pytest.mark.parametrize("geo,wide", [((130, 22, 69, 32, 14, 2, 128), False), ((133, 60, 52, 16, 12, 4, 128), False), ((200, 64, 31, 64, 6, 5, 256), False),
                                      ((160, 53, 59, 32, 10, 4, 128), False), ((256, 64, 64, 32, 8, 2, 128), True), ((80, 23, 22, 32, 7, 1, 512), True)])
def test_long_patches_in_padded_batches_and_rounds(geo, wide):
    """The workgroup-tiled kernel where its tiles of the batch and its rounds of workgroups are filled: just above either the general
    kernel is up to 1.4 times as fast."""
    assert (lc.plan_query(lc.geom(*geo), B.LC_OP_FORWARD, B.LC_F32)[0]["kernel"] == "lc_forward_wide") == wide


@pytest.mark.parametrize("geo,turned", [((16, 53, 22, 24, 17, 3, 313), False), ((4, 28, 25, 24, 15, 1, 64), False), ((16, 154, 23, 24, 20, 3, 96), False),
                                        ((4, 76, 158, 24, 16, 8, 64), False), ((32, 34, 24, 24, 16, 3, 256), False), ((96, 49, 106, 64, 16, 8, 24), True),
                                        ((96, 44, 21, 64, 16, 7, 160), True)])
def test_workgroups_of_sixteen_waves_beyond_a_round(geo, turned):
    """A third of a second round of workgroups that a compute unit runs one by one, where the direct form needs one round: the direct
    form.  More of a second round, or none: the turned one."""
    p = lc.plan_query(lc.geom(*geo), B.LC_OP_FORWARD, B.LC_F32)[0]
    assert p["kernel"] == "lc_forward_general" and bool(p["tparam"][7]) == turned, p
