"""1x1 gradients whose kernel splits the weights itself (few channels to contract): one phase of 64 channels and several, 64 and
128 channels per block, one tile to a block and more, 4- and 8-bit codes; few pixels and a long contraction; against 64-bit
values."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cout: the gradient contracts Cout channels
SHAPES = [(1, 110, 101, 64, 64), (1, 150, 150, 128, 64), (3, 141, 143, 192, 64), (2, 150, 151, 256, 64),
          (5, 117, 119, 256, 64), (2, 110, 103, 256, 128), (2, 150, 151, 512, 128),
          (26, 7, 7, 512, 2048), (15, 14, 13, 256, 1024)]   # two groups of waves
IDS = ["x".join(map(str, s)) for s in SHAPES]


def f32(*size):
    return torch.full(size, float("nan"), device="cuda")


def raw(n):
    return torch.empty(max(16, int(n)), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("flags", [0, B.ABL_MATH_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_backward(s, flags, K):
    print("case 1x1 gradient", s, K, flags, flush=True)
    N, H, W, ci, co = s
    s9, M = s + (1, 1, 1, 0), N * H * W
    g = torch.Generator(device="cuda").manual_seed(7)

    def normal(*size):
        return torch.randn(*size, device="cuda", generator=g)

    x, w, dy = normal(N, H, W, ci), normal(1, 1, ci, co) * (2.0 / ci) ** 0.5, normal(N, H, W, co)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, normal(ci) * 0.1
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    a3, a2t = f32(*x.shape), f32(*x.shape)
    B.abl_bn_stats(x, M, ci, gamma, beta, K, scratch, stats)
    B.abl_bn_relu_pack(x, M, ci, K, stats, a3, packed)
    B.abl_unpack(packed, M, ci, K, stats, a2t)
    dx, dW, dg, db = f32(*x.shape), f32(*w.shape), f32(ci), f32(ci)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db, flags=flags)
    d, v = (dy.bfloat16().float(), w.bfloat16().float()) if flags else (dy, w)
    da2 = torch.where(a2t.view(M, ci) > 0, d.double().view(M, co) @ v.double()[0, 0].t().contiguous(), 0.0)
    a1 = (a2t.double().view(M, ci) - beta.double()) / gamma.double()
    rstd = stats[: 28 * ci].view(torch.float32).view(7, ci)[2].double()
    rdb, rdg = da2.sum(0), (da2 * a1).sum(0)
    rdx = gamma.double() * rstd * (da2 - rdb / M - a1 * (rdg / M))
    # sqrt(co / 32) roundings of 2^-24 in the contraction and two for the small products and the final sum, three in Eq. 8; other
    # bf16 kernels round their sums more often
    tol = 2.0 ** -24 * ((co / 32) ** 0.5 + 5) * (3 if flags else 1)
    for got, ref in ((dx.view(M, ci), rdx), (dg, rdg), (db, rdb)):
        assert float((got.double() - ref).norm() / ref.norm()) < tol
    # element by element: no tile left out or written twice (roundings of the largest terms)
    assert float((dx.view(M, ci).double() - rdx).abs().max()) < 2.0 ** -20 * float(rdx.abs().max()) * (4 if flags else 1)


@pytest.mark.parametrize("flags", [0, B.ABL_MATH_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("s", [(26, 7, 7, 2048, 512), (26, 8, 8, 2048, 512), (15, 14, 13, 1024, 256)], ids=lambda s: "x".join(map(str, s)))
def test_forward(s, flags):
    print("case 1x1 forward", s, flush=True)
    N, H, W, ci, co = s
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn(N, H, W, ci, device="cuda", generator=g)
    w = torch.randn(1, 1, ci, co, device="cuda", generator=g) * (2.0 / ci) ** 0.5
    y = f32(N, H, W, co)
    B.abl_conv_fwd(s + (1, 1, 1, 0), x, w, None, y, flags=flags)
    a, v = (x.bfloat16().float(), w.bfloat16().float()) if flags else (x, w)
    ref = a.double().view(-1, ci) @ v.double()[0, 0]
    tol = 2.0 ** -24 * ((ci / 32) ** 0.5 + 2) * (3 if flags else 1)   # (as above)
    assert float((y.view(-1, co).double() - ref).norm() / ref.norm()) < tol
    assert float((y.view(-1, co).double() - ref).abs().max()) < 2.0 ** -20 * float(ref.abs().max()) * (4 if flags else 1)
