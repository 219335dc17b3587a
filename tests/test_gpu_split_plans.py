"""3x3 layers on every way of cutting the pixels into tiles - image by image, runs across images, patches that leave room for one
block per compute unit - with one tile to a block and several: the whole layer step against 64-bit values."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

from . import split_rules as R

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cout
SHAPES = [(80, 27, 27, 64, 64),    # image by image, several tiles to a block
          (16, 33, 33, 64, 128),   # one tile to a block, blocks in pairs
          (28, 32, 32, 64, 64),    # runs across images, one block per unit
          (20, 57, 57, 64, 64),    # large patches, several tiles to a block
          (30, 45, 45, 64, 64), (29, 55, 54, 64, 64),
          (130, 3, 40, 64, 64), (36, 22, 23, 32, 64), (15, 13, 60, 128, 64)]
IDS = ["x".join(map(str, s)) for s in SHAPES]


def f32(*size):
    return torch.full(size, float("nan"), device="cuda")


def raw(n):
    return torch.empty(max(16, int(n)), dtype=torch.uint8, device="cuda")


def conv64(a, w):
    """'Same' 3x3 convolution in 64 bits, a NHWC, w RSCK."""
    N, H, W, c = a.shape
    p, wd = torch.nn.functional.pad(a.double(), (0, 0, 1, 1, 1, 1)), w.double()
    y = torch.zeros(N * H * W, w.shape[3], dtype=torch.float64, device=a.device)
    for r in range(3):
        for q in range(3):
            y += p[:, r:r + H, q:q + W].reshape(-1, c) @ wd[r, q].contiguous()
    return y.view(N, H, W, -1)


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


@pytest.mark.parametrize("flags", [0, B.ABL_MATH_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_layer_step(s, flags):
    print("case layer step", s, flags, flush=True)
    N, H, W, ci, co = s
    s9, M, K = s + (3, 3, 1, 1), N * H * W, 4 if N % 2 else 8
    g = torch.Generator(device="cuda").manual_seed(9)

    def normal(*size):
        return torch.randn(*size, device="cuda", generator=g)

    x, w, dy = normal(N, H, W, ci), normal(3, 3, ci, co) * (2.0 / (9 * ci)) ** 0.5, normal(N, H, W, co)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, normal(ci) * 0.1
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    y = f32(N, H, W, co)
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, y, packed, stats, flags=flags)
    a3, a2t, p2 = f32(*x.shape), f32(*x.shape), raw(B.abl_packed_bytes(s9, K))
    B.abl_bn_relu_pack(x, M, ci, K, stats, a3, p2)
    assert torch.equal(packed, p2)
    rnd = (lambda t: t.bfloat16().float()) if flags else (lambda t: t)
    # one rounding of 2^-24 per 32 terms of a sum that is a random walk, two for the small products and the final sum; other bf16
    # kernels and the fp32 matrix cores round more often
    more = 3 if flags or not R.rows(s + (3,), 0) else 1
    assert rel(y, conv64(rnd(a3), rnd(w))) < more * 2.0 ** -24 * ((9 * ci / 32) ** 0.5 + 2)
    B.abl_unpack(packed, M, ci, K, stats, a2t)
    dx, dW, dg, db = f32(*x.shape), f32(*w.shape), f32(ci), f32(ci)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db, flags=flags)
    da3 = conv64(rnd(dy), rnd(w).flip(0, 1).transpose(2, 3).contiguous())
    da2 = torch.where(a2t > 0, da3, 0.0).view(M, ci)
    a1 = (a2t.double().view(M, ci) - beta.double()) / gamma.double()
    rstd = stats[: 28 * ci].view(torch.float32).view(7, ci)[2].double()
    rdb, rdg = da2.sum(0), (da2 * a1).sum(0)
    rdx = gamma.double() * rstd * (da2 - rdb / M - a1 * (rdg / M))
    more = 3 if flags or not R.rows(s + (3,), 1, False, True) else 1
    for got, ref in ((dx.view(M, ci), rdx), (dg, rdg), (db, rdb)):
        assert rel(got, ref) < more * 2.0 ** -24 * ((9 * co / 32) ** 0.5 + 5)   # (three more roundings in Eq. 8)
    at, dyr = torch.nn.functional.pad(a2t.clamp(min=0).double(), (0, 0, 1, 1, 1, 1)), rnd(dy).double().view(M, co)
    rdW = torch.stack([at[:, r:r + H, q:q + W].reshape(M, ci).t().contiguous() @ dyr for r in range(3) for q in range(3)])
    # (fp32 sums over M terms in random order, bf16 operands of the codes are rounded as well: 2^-9 of each)
    assert rel(dW.view(9, ci, co), rdW) < (2.0 ** -8 if flags else 2.0 ** -24 * ((M / 32) ** 0.5 + 5))
