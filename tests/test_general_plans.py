"""The general kernels (any geometry, operands straight from global memory): their index arithmetic replayed on the CPU
from the launch plans, against the contraction it stands for.  Every product of the definition is formed exactly once,
every address is inside its tensor, every output is stored."""
import random

import numpy as np
import pytest

import paper_1502_03409_amd as lc
from general_tiles import TILES
from paper_1502_03409_amd import binding as B


def cdiv(a, b):
    return -(-a // b)


def geometries(n, seed):
    r = random.Random(seed)
    out = []
    while len(out) < n:
        R, S, C = r.randint(1, 9), r.randint(1, 6), r.choice([1, 2, 3, 4, 5, 7, 16])
        H, W = R + r.randint(0, 9), R + r.randint(0, 12)
        F, Bn = r.choice([r.randint(1, 40), r.randint(1, 130), 16 * r.randint(1, 8)]), r.choice([1, 2, 5, 16, 17, 37, 64, 70, 130])
        out.append((Bn, H, W, C, R, S, F))
    return out


def forward_vectors(R, RC, NV, nvt, per, ks):
    """(slice, lane group kk, step) -> the vectors a wave loads: arrays of patch row, offset in the row, leading elements
    that count as zero; walked the way the kernel does."""
    back, dv, dr = 4 * NV - RC, 4 % NV, 4 // NV
    out = []
    for sl in range(ks):
        vbeg, vend = sl * per, min((sl + 1) * per, nvt)
        ng = cdiv(max(vend - vbeg, 0), 4)
        for kk in range(4):
            vi = vbeg + kk
            row, v = vi // NV, vi % NV
            for _ in range(ng):
                if vi < vend:
                    sh = back if v == NV - 1 else 0
                    out.append((sl, kk, row, 4 * v - sh, sh))
                else:
                    out.append((sl, kk, 0, 0, 4))
                vi, v, row = vi + 4, v + dv, row + dr
                if v >= NV:
                    v, row = v - NV, row + 1
    return out


@pytest.mark.parametrize("seed", range(4))
def test_general_forward_covers_every_product_once(seed):
    n_general = 0
    for geo in geometries(150, 10 + seed):
        G = lc.geom(*geo)
        Bn, H, W, C, R, S, F = geo
        LH, LW, K = lc.geom_derive(G)
        RC = R * C
        for dtype in (B.LC_F32, B.LC_BF16):
            plans = lc.plan_query(G, B.LC_OP_FORWARD, dtype)
            p = plans[0]
            if p["kernel"] != "lc_forward_general":
                assert p["kernel"] != "lc_forward_generic" or RC < 4, (geo, p)
                continue
            n_general += 1
            MT, NT, nfw, ES, rag, ks, tasks = p["tparam"][:7]
            NV, nvt, per, nbt, ntask = p["arg"][:5]
            assert NV == cdiv(RC, 4)
            # patch elements: each exactly once over slices, lane groups and steps; four elements inside the patch row
            seen = np.zeros(K, dtype=int)
            for _, _, row, off, skip in forward_vectors(R, RC, NV, nvt, per, ks):
                assert 0 <= row < R and 0 <= off and off + 4 <= RC
                seen[row * RC + off + skip:row * RC + off + 4] += 1
            assert (seen == 1).all(), (geo, p)
            # filters: runs of NT inside the filters, all of them reached by a wave that stores
            f = set()
            for f0 in range(0, p["grid"][1] * nfw * NT * 16, NT * 16):
                if f0 >= F:
                    continue
                for n in range(16):
                    fl = min(f0 + NT * n, F - NT)
                    assert 0 <= fl and fl + NT <= F
                    f.update(range(fl, fl + NT))
            assert f == set(range(F))
            # tasks: every field with every batch tile, images clamped into the batch
            assert ntask == LH * LW * nbt and nbt * 16 * MT >= Bn > (nbt - 1) * 16 * MT
            assert p["grid"][0] * tasks >= ntask and p["block"] == 64 * ks * nfw * tasks
    assert n_general > 100


@pytest.mark.parametrize("seed", range(4))
def test_general_backward_data_covers_every_product_once(seed):
    n_general = 0
    for geo in geometries(80, 50 + seed):
        G = lc.geom(*geo)
        Bn, H, W, C, R, S, F = geo
        LH, LW, K = lc.geom_derive(G)
        for dtype in (B.LC_F32, B.LC_BF16):
            plans = lc.plan_query(G, B.LC_OP_BACKWARD_DATA, dtype)
            p = plans[0]
            if p["kernel"] != "lc_bwd_data_general":
                short = R <= S and F <= 32                     # few products a value
                assert p["kernel"] != "lc_bwd_data_generic" or F < 4 or short, (geo, p)
                continue
            n_general += 1
            MT, NT, ES, mask, ks, tasks, VW = p["tparam"][:7]
            PR, PC, cbc, NVF, nbt, ntask = p["arg"][:6]
            N, cbr = PR * PC * C, cdiv(H, PR)
            assert ntask == cbr * cbc * nbt and p["grid"][0] * tasks >= ntask and p["grid"][1] * NT * 16 >= N
            vals = np.arange(N)
            dr, rem = vals // (PC * C), vals % (PC * C)
            dc, c = rem // C, rem % C
            # products formed per output value and field, summed over filters: [H, W, C] -> set of (field, filter) counts
            for rb in {0, cbr // 2, cbr - 1}:
                for cb in {0, cbc // 2, cbc - 1}:
                    r0, c0 = rb * PR, cb * PC
                    i_lo, i_hi = max(0, -(-(r0 - R + 1) // S)), min(LH - 1, (r0 + PR - 1) // S)
                    j_lo, j_hi = max(0, -(-(c0 - R + 1) // S)), min(LW - 1, (c0 + PC - 1) // S)
                    na, nap = i_hi - i_lo + 1, j_hi - j_lo + 1
                    nvt = na * nap * NVF if na > 0 and nap > 0 else 0
                    rr, cc = r0 + dr - i_lo * S, c0 + dc - j_lo * S
                    formed = {}
                    per = cdiv(cdiv(nvt, 4), ks) * 4 if nvt else 0
                    vec = [vi for sl in range(ks) for vi in range(sl * per, min((sl + 1) * per, nvt))]
                    assert vec == list(range(nvt))
                    for vi in vec:
                        fi, fv = vi // NVF, vi % NVF
                        assert int((np.float32(vi) + np.float32(0.5)) * np.float32(np.float32(1) / np.float32(NVF))) == fi
                        fa, fp = fi // nap, fi % nap
                        assert int((np.float32(fi) + np.float32(0.5)) * np.float32(np.float32(1) / np.float32(nap))) == fa
                        sh = (VW * NVF - F) if mask and fv == NVF - 1 else 0
                        fo = VW * fv - sh
                        assert 0 <= fo and fo + VW <= F
                        ok = (rr - fa * S >= 0) & (rr - fa * S < R) & (cc - fp * S >= 0) & (cc - fp * S < R)
                        if not mask:
                            assert ok.all()
                        k = (rr - fa * S) * R * C + (cc - fp * S) * C + c
                        # the kernel's offset from the block's first field, in elements
                        off = (fa * (LW * K - S * R * C) + fp * (K - S * C)) * F + fo + (rr * R * C + cc * C + c) * F
                        field = (i_lo + fa) * LW + j_lo + fp
                        want = (field - (i_lo * LW + j_lo)) * K * F + k * F + fo
                        assert (off[ok] == want[ok]).all() and (want[ok] >= 0).all()
                        for t in range(sh, VW):
                            key = (field, fo + t)
                            formed[key] = formed.get(key, 0) + ok.astype(int)
                    for v in (0, N // 2, N - 1):
                        row, col = r0 + int(dr[v]), c0 + int(dc[v])
                        if row >= H or col >= W:
                            continue
                        cover = {(i * LW + j, f) for i in range(LH) for j in range(LW) for f in range(F)
                                 if 0 <= row - i * S < R and 0 <= col - j * S < R}
                        got = {key: int(n[v]) for key, n in formed.items() if n[v]}
                        assert set(got) == cover and all(n == 1 for n in got.values()), (geo, p, row, col)
    assert n_general > 60


@pytest.mark.parametrize("seed", range(4))
def test_general_backward_weights_stores_every_element_once(seed):
    n_general = 0
    for geo in geometries(150, 90 + seed):
        G_ = lc.geom(*geo)
        Bn, H, W, C, R, S, F = geo
        LH, LW, K = lc.geom_derive(G_)
        RC = R * C
        plans = [(lc.plan_query(G_, B.LC_OP_BACKWARD_WEIGHTS, dtype)[0], False) for dtype in (B.LC_F32, B.LC_BF16)]
        plans += [(p, True) for p in lc.plan_query(G_, B.LC_OP_SAE_STEP) if p["kernel"].startswith("lc_bwd_weights")]
        for p, squares in plans:
            if p["kernel"] != "lc_bwd_weights_general":
                # the masked kernel: short patch rows, and small batches of some layers
                assert p["kernel"] != "lc_bwd_weights_generic" or RC < 4 or Bn <= 16, (geo, p)
                continue
            n_general += 1
            G, NT, ES = p["tparam"][:3]
            NV, nvt, kblocks, nfb, ntask = p["arg"][:5]
            assert ntask == LH * LW * kblocks * nfb and p["grid"][0] * 4 >= ntask and p["block"] == 256
            assert not squares or kblocks <= cdiv(K, 64)     # room for the partial sums of squares
            # patch elements: stored by exactly one vector, all four of a vector inside the patch row
            seen = np.zeros(K, dtype=int)
            for vi in range(kblocks * G * 16):
                if vi >= nvt:
                    continue
                assert int((np.float32(vi) + np.float32(0.5)) * np.float32(np.float32(1) / np.float32(NV))) == vi // NV
                row, v = vi // NV, vi % NV
                skip = 4 * NV - RC if v == NV - 1 else 0
                assert 0 <= 4 * v - skip and 4 * v - skip + 4 <= RC
                seen[row * RC + 4 * v:row * RC + 4 * v - skip + 4] += 1
            assert (seen == 1).all()
            # filters likewise
            seen = np.zeros(F, dtype=int)
            for f0 in range(0, nfb * NT * 16, NT * 16):
                for m in range(16):
                    fl = min(f0 + NT * m, F - NT)
                    shared = f0 + NT * m - fl
                    assert fl >= 0
                    if shared < NT:
                        seen[fl + shared:fl + NT] += 1
            assert (seen == 1).all()
            # images: each in one step, one or four per lane
            IM = 1 if ES == 4 else 4
            images = np.zeros(Bn, dtype=int)
            for st in range(cdiv(Bn, 4 * IM)):
                for kk in range(4):
                    left = Bn - (st * 4 * IM + IM * kk)
                    images[st * 4 * IM + IM * kk:st * 4 * IM + IM * kk + max(0, min(IM, left))] += 1
            assert (images == 1).all()
    assert n_general > 100


def test_derived_sizes_follow_the_geometry():
    """The binding remembers derived sizes by value: a geometry whose fields change, or an impossible one, is seen as it is."""
    G = lc.geom(2, 20, 20, 3, 5, 3, 8)
    assert lc.geom_derive(G) == (6, 6, 75)
    G.W, G.S = 29, 4
    assert lc.geom_derive(G) == (4, 7, 75)
    G.R = 21
    for _ in range(2):
        with pytest.raises(lc.LcError) as e:
            lc.geom_derive(G)
        assert e.value.code == B.LC_EINVAL


def test_strides_of_hundreds_of_pixels_plan_backward_data():
    """A cell of S x S x C values beyond what the general kernel's grid holds in blocks of its tile: such layers plan on a
    wider tile or on the masked kernel (S*S*C just below, at and beyond each tile's limit of 16*NT*65535 values)."""
    for geo in ((21, 72, 102, 7, 42, 784, 1263), (1902, 16, 39, 13, 16, 669, 884), (2, 9, 9, 1, 3, 1023, 40), (2, 9, 9, 1, 3, 1024, 40),
                (2, 9, 9, 1, 3, 1025, 40), (2, 9, 9, 2, 3, 1023, 37), (1, 9, 9, 4, 3, 1023, 41), (1, 9, 9, 4, 3, 1024, 41),
                (2, 9, 9, 1, 3, 2047, 40), (2, 9, 9, 1, 3, 2049, 40)):
        G = lc.geom(*geo)
        for dtype in (B.LC_F32, B.LC_BF16):
            p = lc.plan_query(G, B.LC_OP_BACKWARD_DATA, dtype)[0]
            cell = geo[5] ** 2 * geo[3]
            assert p["kernel"] == ("lc_bwd_data_general" if cell <= 64 * 65535 else "lc_bwd_data_generic"), (geo, p)
            assert p["grid"][1] <= 65535
        assert lc.plan_query(G, B.LC_OP_SAE_STEP)


def test_millions_of_filters_plan_forward():
    """Filter blocks beyond the second grid dimension of the general kernel: a wider tile, or the masked kernel."""
    for geo in ((5, 2, 2, 2, 2, 5, 16173454), (54, 1, 1, 33, 1, 13, 11130312), (2, 9, 9, 1, 9, 2, 9843871), (1, 2, 2, 4, 2, 1, 16 * 65535),
                (1, 2, 2, 4, 2, 1, 16 * 65535 + 1), (1, 2, 2, 4, 2, 1, 64 * 65535), (1, 2, 2, 4, 2, 1, 64 * 65535 + 1)):
        G = lc.geom(*geo)
        for dtype in (B.LC_F32, B.LC_BF16):
            p = lc.plan_query(G, B.LC_OP_FORWARD, dtype)[0]
            assert p["kernel"] == ("lc_forward_general" if geo[6] <= 64 * 65535 else "lc_forward_generic"), (geo, p)
            assert p["grid"][1] <= 65535


def test_layers_beyond_the_task_limit_plan_on_other_kernels():
    """More tasks than the general kernels number (2^30): not refused, but planned on the kernels that took them."""
    for op, geo in ((B.LC_OP_BACKWARD_WEIGHTS, (1, 200, 242, 64, 47, 1, 310)), (B.LC_OP_BACKWARD_WEIGHTS, (31, 2048, 49, 44, 35, 1, 3705)),
                    (B.LC_OP_FORWARD, (3735, 2515, 8804, 1, 5, 1, 11)), (B.LC_OP_FORWARD, (3826, 818, 32230, 1, 5, 1, 10)),
                    (B.LC_OP_BACKWARD_DATA, (4000, 5000, 7000, 1, 4, 1, 5))):
        for dtype in (B.LC_F32, B.LC_BF16):
            p = lc.plan_query(lc.geom(*geo), op, dtype)[0]
            assert all(0 < g <= 0x7fffffff for g in p["grid"]), (op, geo, p)


def test_tile_layers_reach_every_tile():
    """The layers that the GPU tests run tile by tile reach every instance of the general kernels: images per wave (MT),
    columns per wave (NT), operand type, ragged or whole vectors, vector width, and contractions whole and in slices."""
    ops = {"forward": B.LC_OP_FORWARD, "backward_data": B.LC_OP_BACKWARD_DATA, "backward_weights": B.LC_OP_BACKWARD_WEIGHTS}
    slices = {"forward": set(), "backward_data": set()}
    for (op, dtype), shapes in TILES.items():
        seen = set()
        for shape in shapes:
            (p,) = lc.plan_query(lc.geom(*shape), ops[op], B.LC_BF16 if dtype == "bf16" else B.LC_F32)
            assert p["kernel"].endswith("_general"), (op, dtype, shape, p)
            t = p["tparam"]
            seen.add((t[0], t[1], t[4]) if op == "forward" else (t[0], t[1], t[3], t[6]) if op == "backward_data" else t[1])
            if op != "backward_weights":
                slices[op].add(t[5] if op == "forward" else t[4])
        runs = (1, 2, 4) if dtype == "bf16" else (1, 2, 3, 4)
        if op == "forward":
            want = {(mt, nt, rag) for mt in (1, 2, 3, 4) for nt in runs for rag in (0, 1)}
        elif op == "backward_data":
            want = {(mt, nt, mask, vw) for mt in (1, 2, 3, 4) for nt in (1, 2, 3, 4) for mask in (0, 1) for vw in (4, 8)}
        else:
            want = set(runs)
        assert seen == want, (op, dtype, want - seen, seen - want)
    assert slices["forward"] == {1, 2, 4, 8, 16} and slices["backward_data"] == {1, 2, 4, 8}, slices


# (images, height, width, channels, field, stride, filters), kernel in fp32, kernel in bf16: layers on both sides of the lines
# between the weight gradient's general kernel and the two it displaces
WEIGHT_ROUTES = [
    # small batches: at most 32 filters, four images in bf16 and eight in fp32
    ((8, 106, 43, 64, 16, 6, 18), "generic", "general"), ((9, 106, 43, 64, 16, 6, 18), "general", "general"),
    ((4, 106, 43, 64, 16, 6, 18), "generic", "generic"), ((5, 23, 26, 5, 5, 3, 32), "generic", "general"),
    ((4, 23, 26, 5, 5, 3, 33), "general", "general"),
    # patches of 64 elements at most
    ((16, 64, 198, 1, 8, 2, 223), "generic", "general"), ((8, 64, 198, 1, 8, 2, 223), "generic", "generic"),
    ((17, 64, 198, 1, 8, 2, 223), "general", "general"), ((7, 64, 198, 65, 1, 2, 223), "generic", "generic"),
    # filters that pad blocks of 64 by more than a third
    ((7, 64, 198, 1, 4, 2, 95), "general", "general"), ((7, 64, 198, 1, 4, 2, 97), "generic", "generic"),
    ((7, 64, 198, 1, 4, 2, 80), "general", "general"),
    # tiles of patch elements partly filled, over 2^22 elements of gradient
    ((3, 55, 69, 1, 9, 1, 323), "generic", "generic"), ((3, 20, 20, 1, 9, 1, 323), "general", "general"),
    ((3, 55, 69, 1, 16, 1, 323), "general", "general"),
    # fp32, odd numbers of 16-filter tiles: rounds of the pipelined kernel's waves
    ((256, 24, 123, 2, 14, 4, 48), "fast", "bf16_rows"), ((256, 97, 25, 8, 7, 7, 144), "general", "bf16_rows"),
    ((192, 27, 62, 12, 11, 6, 80), "fast", "bf16_rows"), ((196, 27, 62, 12, 11, 6, 80), "general", "general"),
    ((128, 15, 24, 32, 4, 2, 80), "general", "bf16_rows"),
]


@pytest.mark.parametrize("geo,f32,bf16", WEIGHT_ROUTES, ids=str)
def test_weight_gradient_routes(geo, f32, bf16):
    for dtype, kernel in ((B.LC_F32, f32), (B.LC_BF16, bf16)):
        (p,) = lc.plan_query(lc.geom(*geo), B.LC_OP_BACKWARD_WEIGHTS, dtype)
        assert p["kernel"] == "lc_bwd_weights_" + kernel, (geo, dtype, p)
    # the training step accumulates: the general kernel
    step = [p["kernel"] for p in lc.plan_query(lc.geom(*geo), B.LC_OP_SAE_STEP) if p["kernel"].startswith("lc_bwd_weights")]
    assert step == ["lc_bwd_weights_general"], (geo, step)


# the same for backward data's general kernel and short contractions: filters, images, overlap, values a cell, tasks
DATA_ROUTES = [
    ((1, 197, 153, 48, 7, 7, 5), "generic", "generic"), ((17, 197, 153, 48, 7, 7, 5), "generic", "general"),
    ((64, 143, 165, 48, 3, 3, 31), "generic", "general"), ((65, 143, 165, 48, 3, 3, 31), "general", "general"),
    ((4, 143, 165, 48, 3, 3, 33), "general", "general"), ((4, 143, 165, 48, 4, 3, 9), "general", "general"),
    ((4, 143, 165, 28, 3, 3, 31), "general", "general"), ((4, 40, 50, 48, 3, 3, 31), "generic", "general"),
    ((4, 30, 40, 48, 3, 3, 31), "general", "general"), ((16, 150, 150, 64, 4, 4, 16), "generic", "generic"),
]


@pytest.mark.parametrize("geo,f32,bf16", DATA_ROUTES, ids=str)
def test_backward_data_routes(geo, f32, bf16):
    for dtype, kernel in ((B.LC_F32, f32), (B.LC_BF16, bf16)):
        (p,) = lc.plan_query(lc.geom(*geo), B.LC_OP_BACKWARD_DATA, dtype)
        assert p["kernel"] == "lc_bwd_data_" + kernel, (geo, dtype, p)
