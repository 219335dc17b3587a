"""3x3 layers with 16 input and 16 output channels (csrc/conv_c16.hip): tiles of whole rows, one row to a tile, an image to a tile,
a last tile with fewer rows, quantizer offsets beyond one bf16; equal layers in a stack, whose Eq. 7-8 go along with the layer below."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

from .test_gpu_split_plans import conv64, f32, raw, rel

pytestmark = pytest.mark.gpu

C = 16
# N, H, W
SHAPES = [(1, 1, 1), (2, 5, 7), (8, 32, 32), (1, 3, 126), (3, 90, 9), (5, 33, 31), (37, 30, 34), (256, 16, 17), (128, 32, 32)]
IDS = ["x".join(map(str, s)) for s in SHAPES]


def draw(s, beta, seed=9):
    g = torch.Generator(device="cuda").manual_seed(seed)
    N, H, W = s

    def normal(*size):
        return torch.randn(*size, device="cuda", generator=g)

    gamma = torch.rand(C, device="cuda", generator=g) + 0.5
    gamma[3] = -gamma[3]
    return normal(N, H, W, C), normal(3, 3, C, C) / 12, gamma, beta + normal(C) * 0.1, normal(N, H, W, C)


def forward(s, K, x, w, gamma, beta):
    s9 = s + (C, C, 3, 3, 1, 1)
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    y = f32(*x.shape)
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, y, packed, stats)
    return s9, packed, stats, scratch, y


@pytest.mark.parametrize("K,beta", [(4, 0.0), (8, 0.0), (8, 0.3), (4, 45.0), (8, 45.0)])
@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_layer_step(s, K, beta):
    print("case 16-channel layer step", s, K, beta, flush=True)
    N, H, W = s
    M = N * H * W
    x, w, gamma, beta, dy = draw(s, beta)
    s9, packed, stats, scratch, y = forward(s, K, x, w, gamma, beta)
    a3, a2t, p2, y2 = f32(*x.shape), f32(*x.shape), raw(B.abl_packed_bytes(s9, K)), f32(*x.shape)
    B.abl_bn_relu_pack(x, M, C, K, stats, a3, p2)
    assert torch.equal(packed, p2)
    p2.fill_(7)
    B.abl_bn_conv_fwd(s9, K, x, stats, w, None, y2, p2)      # (the same kernel with the statistics given)
    assert torch.equal(packed, p2) and torch.equal(y, y2)
    # roundings of 2^-24: one per 32 of the 144 terms, the small products, their sum; of a value that may be a difference of
    # terms 45 / 0.5 times its size where beta is large
    worse = 1 if float(beta.abs().max()) < 1 else 20
    assert rel(y, conv64(a3, w)) < worse * 2.0 ** -24 * 5
    B.abl_unpack(packed, M, C, K, stats, a2t)
    dx, dW, dg, db = f32(*x.shape), f32(*w.shape), f32(C), f32(C)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db)
    da3 = conv64(dy, w.flip(0, 1).transpose(2, 3).contiguous())
    da2 = torch.where(a2t > 0, da3, 0.0).view(M, C)
    a1 = (a2t.double().view(M, C) - beta.double()) / gamma.double()
    rstd = stats[: 28 * C].view(torch.float32).view(7, C)[2].double()
    rdb, rdg = da2.sum(0), (da2 * a1).sum(0)
    rdx = gamma.double() * rstd * (da2 - rdb / M - a1 * (rdg / M))
    if M > 1:    # (one pixel: Eq. 8 is a difference of equal numbers)
        assert rel(dx.view(M, C), rdx) < worse * 2.0 ** -24 * 8
    # (A1 of a code and beta, both rounded: beta / gamma times the rounding of a value of the size of one)
    for got, ref in ((dg, rdg), (db, rdb)):
        assert rel(got, ref) < 10 * worse * 2.0 ** -24 * 8
    at, dyr = torch.nn.functional.pad(a2t.clamp(min=0).double(), (0, 0, 1, 1, 1, 1)), dy.double().view(M, C)
    rdW = torch.stack([at[:, r:r + H, q:q + W].reshape(M, C).t().contiguous() @ dyr for r in range(3) for q in range(3)])
    assert rel(dW.view(9, C, C), rdW) < worse * 2.0 ** -24 * ((M / 32) ** 0.5 + 5)


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("N,hw,count", [(2, 7, 2), (9, 33, 4), (24, 32, 6), (100, 33, 4)])   # (500 blocks a layer, two rounds of the chip)
def test_stack_equals_traced(N, hw, count, K):
    """Layers that share launches: every layer against 64-bit values on the gradient that the traced call says it received; the plain
    call's results are the traced one's bit for bit."""
    print("case 16-channel stack", N, hw, count, K, flush=True)
    s9, M = (N, hw, hw, C, C, 3, 3, 1, 1), N * hw * hw
    descs = []
    for i in range(count):
        _, w, gamma, beta, _ = draw((N, hw, hw), 0.0, 30 + i)
        descs.append(dict(shape=s9, W=w, gamma=gamma, beta=beta, packed=raw(B.abl_packed_bytes(s9, K)), stats=raw(B.abl_stats_bytes(s9)),
                          dW=f32(3, 3, C, C), dgamma=f32(C), dbeta=f32(C)))
    layers = B.make_layers(descs)
    n = M * C
    S, T = f32(B.abl_stack_buffer_bytes(layers) // 4), f32(B.abl_stack_buffer_bytes(layers) // 4)
    scratch = raw(B.abl_stack_scratch_bytes(layers, K))
    x, _, _, _, dy = draw((N, hw, hw), 0.0, 5)
    S[:n] = x.view(-1)
    B.abl_stack_forward(layers, K, 2, S, T, scratch)
    got, trace = [], [f32(N, hw, hw, C) for _ in descs]
    for wanted in (None, trace, [t if i % 3 == 1 else None for i, t in enumerate(trace)]):
        S[:n] = dy.view(-1)
        T.fill_(float("nan"))
        scratch.fill_(255)
        if wanted is None:
            B.abl_stack_backward(layers, K, 2, S, T, scratch)
        else:
            B.abl_stack_backward_traced(layers, K, 2, S, T, scratch, wanted)
        got.append([S[:n].clone()] + [t.clone() for d in descs for t in (d["dW"], d["dgamma"], d["dbeta"])])
        for d in descs:
            for t in (d["dW"], d["dgamma"], d["dbeta"]):
                t.fill_(float("nan"))
    for run in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], run))
    assert torch.equal(trace[-1], dy)
    for i, d in enumerate(descs):
        a2t, gamma, beta = f32(M, C), d["gamma"].double(), d["beta"].double()
        B.abl_unpack(d["packed"], M, C, K, d["stats"], a2t)
        a2t, dyr = a2t.double(), trace[i].double().view(M, C)
        da3 = conv64(trace[i], d["W"].flip(0, 1).transpose(2, 3).contiguous()).view(M, C)
        da2, a1 = torch.where(a2t > 0, da3, 0.0), (a2t - beta) / gamma
        rstd = d["stats"][: 28 * C].view(torch.float32).view(7, C)[2].double()
        rdb, rdg = da2.sum(0), (da2 * a1).sum(0)
        rdx = gamma * rstd * (da2 - rdb / M - a1 * (rdg / M))
        if i % 2 == 0:
            rdx = rdx + trace[i + 1].double().view(M, C)
        dW, dg, db = got[0][1 + 3 * i:4 + 3 * i]
        # (bounds of test_layer_step)
        assert rel((trace[i - 1] if i > 0 else got[0][0]).view(M, C), rdx) < 2.0 ** -24 * 8, i
        assert rel(dg, rdg) < 10 * 2.0 ** -24 * 8 and rel(db, rdb) < 10 * 2.0 ** -24 * 8, i
        at = torch.nn.functional.pad(a2t.clamp(min=0).view(N, hw, hw, C), (0, 0, 1, 1, 1, 1))
        rdW = torch.stack([at[:, r:r + hw, q:q + hw].reshape(M, C).t().contiguous() @ dyr for r in range(3) for q in range(3)])
        assert rel(dW.view(9, C, C), rdW) < 2.0 ** -24 * ((M / 32) ** 0.5 + 5), i


def test_values_the_split_cannot_carry():
    """Infinities, NaN, values whose parts leave the range and values below 2^-110 give what fp32 products and sums give."""
    s, K = (3, 12, 20), 4
    x, w, gamma, beta, dy = draw(s, 0.0)
    s9, packed, stats, scratch, _ = forward(s, K, x, w, gamma, beta)
    a2t = f32(*x.shape)
    B.abl_unpack(packed, x.numel() // C, C, K, stats, a2t)
    w = w.abs()
    for small in (False, True):
        dy = dy.abs()
        if small:
            dy *= 2.0 ** -118
        else:
            dy[0, 0, 0, 1] = float("inf")
            dy[2, 11, 19, 3] = float("nan")
            dy[1, 5, 5, 5] = 3e37
        da3, dW = f32(*x.shape), f32(3, 3, C, C)
        B.abl_conv_bwd_bn_reduce(s9, K, dy, w, packed, stats, scratch, da3, dW)
        # (zeros around the image take part, where they meet an infinity too)
        p, q = (torch.nn.functional.pad(t, (0, 0, 1, 1, 1, 1)) for t in (dy.double(), a2t.clamp(min=0).double()))
        wd = w.double().flip(0, 1)
        ref = sum((p[:, r:r + 12, c:c + 20, None, :] * wd[r, c]).sum(-1) for r in range(3) for c in range(3))
        refW = torch.stack([torch.stack([(q[:, r:r + 12, c:c + 20, :, None] * dy.double()[..., None, :]).sum((0, 1, 2)) for c in range(3)])
                            for r in range(3)])
        for got, want in ((da3, ref.float()), (dW, refW.float())):
            assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
            ok = torch.isfinite(want)
            # positive terms: each sum is accurate in itself (144 roundings one after the other where it is taken again in fp32)
            assert float(((got - want)[ok].abs() / want[ok].abs().clamp(min=1e-38)).max()) < 2.0 ** -24 * 720
