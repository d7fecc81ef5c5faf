"""bf16 on strips of four fields: the forward pass (both batch tiles, every width of filter block, chunks of one short block to
eight, partly filled strips, batch tiles and last blocks) and the weight gradient, on a GPU against fp64."""
import pytest
import torch

import paper_1502_03409_amd as lc
from paper_1502_03409_amd import binding as Bd

pytestmark = pytest.mark.gpu

# (B, H, W, C, R, S, F), (images / 16, filters / 16 of a workgroup, blocks of 16 values in a chunk, staging slots)
LAYERS = [
    ((17, 30, 142, 4, 3, 1, 16), (2, 1, 1, 6)),       # rows of 12 values: one block, a quarter of it empty
    ((64, 48, 47, 4, 1, 1, 16), (4, 1, 1, 6)),        # fields of one pixel: rows of 4 values
    ((33, 40, 70, 4, 7, 1, 48), (4, 1, 2, 6)),        # one image past half a batch tile
    ((129, 21, 45, 16, 5, 1, 80), (4, 1, 5, 12)),     # one image past two batch tiles
    ((40, 60, 64, 4, 29, 1, 16), (4, 1, 8, 12)),      # rows of 116 values in one chunk
    ((65, 30, 29, 16, 8, 1, 16), (4, 1, 8, 12)),      # rows of 128 values
    ((65, 130, 104, 3, 20, 4, 32), (4, 2, 4, 6)),       # field offsets of 12 values
    ((40, 29, 35, 12, 9, 1, 96), (4, 2, 7, 12)),      # rows of 108
    ((64, 60, 61, 4, 29, 1, 64), (4, 1, 8, 12)),      # narrower blocks of filters keep a row of 116 whole
    ((30, 39, 40, 16, 8, 1, 64), (2, 4, 8, 6)),       # half a batch tile leaves room for both
    ((50, 45, 43, 4, 3, 1, 64), (4, 4, 1, 6)),
    ((130, 40, 33, 16, 11, 2, 128), (4, 4, 6, 12)),    # rows of 176 in chunks of 88
    ((32, 65, 66, 24, 9, 3, 96), (2, 2, 7, 12)),      # rows of 216 in chunks of 108
    ((99, 29, 80, 12, 7, 3, 96), (4, 2, 6, 12)),      # rows of 84 and rows of 496 in 124s with 32 filters in the LDS of two workgroups
    ((65, 43, 70, 16, 31, 1, 32), (4, 2, 8, 12)),
    ((65, 40, 70, 12, 9, 2, 64), (4, 4, 3, 12)),      # rows of 108 in thirds with 64 filters
    ((65, 2900, 2900, 4, 4, 14, 16), (4, 1, 1, 12)),  # offsets beyond 4 GB inside a batch tile
]


def _case(t):
    B, H, W, C, R, S, F = t
    LH, LW, K = (H - R) // S + 1, (W - R) // S + 1, R * R * C
    gen = torch.Generator(device="cuda").manual_seed(sum(t))
    x = torch.randn((B, H, W, C), generator=gen, device="cuda").bfloat16()
    w = torch.randn((LH, LW, K, F), generator=gen, device="cuda").bfloat16()
    bias = torch.randn((LH, LW, F), generator=gen, device="cuda")
    return (B, H, W, C, R, S, F, LH, LW, K), x, w, bias


def _reference(dims, x, w):
    """Sums of products and of their magnitudes in fp64, [B, LH, LW, F]."""
    B, _, _, _, R, S, F, LH, LW, K = dims
    y = torch.empty((2, B, LH, LW, F), dtype=torch.float64, device="cuda")
    for i in range(LH):
        p = x[:, i * S:i * S + R].double().unfold(2, R, S).permute(2, 0, 1, 4, 3).reshape(LW, B, K)
        y[0, :, i] = torch.bmm(p, w[i].double()).transpose(0, 1)
        y[1, :, i] = torch.bmm(p.abs(), w[i].double().abs()).transpose(0, 1)
    return y


@pytest.mark.parametrize("t,want", LAYERS, ids=["x".join(map(str, t)) for t, _ in LAYERS])
def test_against_fp64(t, want):
    dims, x, w, bias = _case(t)
    g = lc.geom(*t)
    plan = lc.plan_query(g, Bd.LC_OP_FORWARD, lc.LC_BF16)
    assert [p["kernel"] for p in plan] == ["lc_forward_bf16_staged"] and tuple(plan[0]["tparam"][:4]) == want
    y = torch.full((dims[0], dims[7], dims[8], dims[6]), float("nan"), device="cuda")
    lc.lc_forward(g, x, w, bias, 0.5, y, lc.LC_BF16)
    ref, mag = _reference(dims, x, w)
    # products of bf16 are exact in fp32; K additions, the scale and the bias round by 2^-24 of what they add up at most
    bound = (dims[9] + 2) * 2.0 ** -24 * (0.5 * mag + bias.double().abs())
    assert torch.all((y.double() - (0.5 * ref + bias.double())).abs() <= bound)


def test_blocks_of_filters_in_the_second_dimension():
    """2^24 workgroups and more: fields of four values, 65 blocks of 16 filters, against fp64 some field rows at a time."""
    t = (17, 258200, 1, 4, 1, 1, 1040)
    print(f"case strip grid.y {t}", flush=True)
    dims, x, w, bias = _case(t)
    g = lc.geom(*t)
    assert lc.plan_query(g, Bd.LC_OP_FORWARD, lc.LC_BF16)[0]["grid"] == (t[1], 65, 1)
    y = torch.full((t[0], t[1], 1, t[6]), float("nan"), device="cuda")
    lc.lc_forward(g, x, w, bias, 0.5, y, lc.LC_BF16)
    for i in range(0, t[1], 1 << 14):
        p, q, c = x[:, i:i + (1 << 14), 0].double().transpose(0, 1).contiguous(), w[i:i + (1 << 14), 0].double(), bias[i:i + (1 << 14)].double()
        ref, mag = 0.5 * torch.bmm(p, q) + c, 0.5 * torch.bmm(p.abs(), q.abs()) + c.abs()
        assert torch.all((y[:, i:i + (1 << 14), 0].transpose(0, 1).double() - ref).abs() <= 6 * 2.0 ** -24 * mag)


def test_pixels_outside_every_field_stay_out():
    """The last field of a row ends in a partly filled block whose lanes reach past it; the last strip has idle waves."""
    t = (64, 80, 64, 4, 3, 2, 32)                     # 31 fields end at pixel 63 of 64
    dims, x, w, _ = _case(t)
    end = (dims[8] - 1) * dims[5] + dims[4]
    assert end < t[2]
    g = lc.geom(*t)
    assert lc.plan_query(g, Bd.LC_OP_FORWARD, lc.LC_BF16)[0]["kernel"] == "lc_forward_bf16_staged"
    y, z = (torch.empty((dims[0], dims[7], dims[8], dims[6]), device="cuda") for _ in range(2))
    lc.lc_forward(g, x, w, None, 1.0, y, lc.LC_BF16)
    x[:, :, end:] = float("nan")
    lc.lc_forward(g, x, w, None, 1.0, z, lc.LC_BF16)
    assert torch.equal(y, z)


@pytest.mark.parametrize("t,chunk", [((17, 30, 142, 4, 3, 1, 16), 12), ((193, 62, 62, 8, 14, 3, 64), 56), ((65, 130, 104, 3, 20, 4, 32), 60)],
                         ids=["chunk12", "chunk56", "chunk60"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")], ids=["inf", "nan"])
def test_non_finite_pixels_stay_in_their_fields(t, chunk, value):
    """A pixel just right of a field reaches the fields that hold it and no other, whichever field of a strip that is."""
    print(f"case strip non-finite {t} {value}", flush=True)
    dims, x, w, _ = _case(t)
    B, _, _, _, R, S, F, LH, LW, _ = dims
    g = lc.geom(*t)
    plan = lc.plan_query(g, Bd.LC_OP_FORWARD, lc.LC_BF16)[0]
    assert plan["kernel"] == "lc_forward_bf16_staged" and plan["arg"][0] == chunk
    y, z = (torch.empty((B, LH, LW, F), device="cuda") for _ in range(2))
    lc.lc_forward(g, x, w, None, 1.0, y, lc.LC_BF16)
    holds = torch.zeros((B, LH, LW), dtype=torch.bool, device="cuda")
    for b, j in enumerate((0, 1, 2, 3, 6)):
        row, col = min(R, t[1] - 1) + b, j * S + R
        x[b, row, col] = value
        for i in range(LH):
            for k in range(LW):
                holds[b, i, k] = i * S <= row < i * S + R and k * S <= col < k * S + R
    lc.lc_forward(g, x, w, None, 1.0, z, lc.LC_BF16)
    assert 0 < int(holds.sum()) < holds.numel()
    assert torch.equal(z[~holds], y[~holds])
    assert not torch.isfinite(z[holds]).any()


# (B, H, W, C, R, S, F): one image, partly filled steps of 16, both sides of the streamed stores, blocks of 16 and 32 filters,
# rows of 45 to 64 values, strips of one to four fields
GRADIENTS = [(1, 22, 40, 4, 12, 1, 16), (17, 24, 41, 4, 15, 2, 32), (63, 31, 48, 3, 20, 4, 32), (64, 31, 48, 3, 20, 4, 96),
             (128, 4104, 4104, 1, 24, 24, 16), (128, 4104, 4104, 1, 24, 24, 32),      # offsets beyond 4 GB
             (32, 37, 44, 3, 20, 4, 32), (33, 37, 44, 3, 20, 4, 16),               # two and four steps of 16 images
             (127, 30, 45, 4, 13, 3, 48), (128, 40, 36, 4, 14, 1, 64), (65, 37, 40, 4, 16, 1, 32), (49, 37, 44, 3, 20, 4, 16)]


@pytest.mark.parametrize("t", GRADIENTS, ids=["x".join(map(str, t)) for t in GRADIENTS])
@pytest.mark.parametrize("beta", [0.0, 1.0])
def test_weight_gradient_against_fp64(t, beta):
    dims, x, dw0, _ = _case(t)
    B, _, _, _, R, S, F, LH, LW, K = dims
    g = lc.geom(*t)
    plan = lc.plan_query(g, Bd.LC_OP_BACKWARD_WEIGHTS, lc.LC_BF16)[0]
    assert plan["kernel"] == "lc_bwd_weights_bf16_strip" and plan["tparam"][3] == (2 if B <= 32 else 4 if B <= 64 else 8)
    dy = torch.randn((B, LH, LW, F), device="cuda").bfloat16()
    dw = dw0.float()
    if not beta:
        dw.fill_(float("nan"))
    lc.lc_backward_weights(g, x, dy, beta, dw, lc.LC_BF16)
    for i in range(LH):
        p = x[:, i * S:i * S + R].double().unfold(2, R, S).permute(2, 1, 4, 3, 0).reshape(LW, K, B)
        d = dy[:, i].double().transpose(0, 1).contiguous()
        ref, mag = torch.bmm(p, d) + beta * dw0[i].double(), torch.bmm(p.abs(), d.abs()) + beta * dw0[i].double().abs()
        assert torch.all((dw[i].double() - ref).abs() <= (B + 1) * 2.0 ** -24 * mag)


def test_infinities_of_the_last_image_stay_infinite():
    """The images that fill up a step of 16 count as zeros, not as copies of one that exists."""
    t = (33, 31, 48, 3, 20, 4, 32)
    dims, x, dw, _ = _case(t)
    x[-1, 5, 5, 0] = float("inf")
    dy = torch.ones((dims[0], dims[7], dims[8], dims[6]), device="cuda").bfloat16()
    out = torch.empty(dw.shape, device="cuda")
    lc.lc_backward_weights(lc.geom(*t), x, dy, 0.0, out, lc.LC_BF16)
    assert not torch.isnan(out).any() and torch.isinf(out).any()
