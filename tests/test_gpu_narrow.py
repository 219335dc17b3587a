"""Layers of few channels (csrc/conv_narrow.hip): patches of whole images and of single rows, a last tile that owns more rows than the
others, strides and paddings, channel counts in and off fours, quantizer offsets beyond one bf16 - the whole layer step against
64-bit values."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

from .test_gpu_split_plans import f32, raw, rel

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cout, R, stride, pad
SHAPES = [(128, 8, 8, 64, 64, 3, 1, 1),      # steps shared by two waves
          (2, 16, 16, 32, 32, 3, 1, 0),      # the last tile owns two rows more
          (5, 10, 9, 64, 96, 3, 1, 2),       # output larger than the input
          (50, 27, 21, 20, 36, 3, 1, 1),
          (40, 33, 32, 16, 32, 3, 2, 1),     # four classes of input pixels
          (9, 15, 14, 32, 64, 1, 2, 0),      # 1x1: other kernels
          (7, 12, 11, 50, 70, 5, 1, 2),      # channels not in fours: the pack pass in front, conv_ragged.hip's weight gradient
          (3, 11, 13, 12, 20, 5, 2, 1),
          (1, 6, 5, 4, 4, 3, 1, 1), (2, 3, 90, 8, 128, 3, 1, 1),                  # (the latter on other kernels)
          (9, 15, 14, 32, 64, (1, 3), 2, 0), (5, 14, 15, 20, 24, (3, 1), 2, 1),   # two classes without a tap; the others' weight gradient
          (28, 10, 8, 64, 64, 5, 1, 1), (3, 13, 16, 32, 64, 5, 2, 0),             # three tiles to a copy of dW
          (23, 10, 18, 15, 22, (5, 3), 1, 2), (7, 21, 24, 35, 32, 5, 1, 1)]       # dW in a launch of its own, channels not in fours
IDS = ["x".join(map(str, s)) for s in SHAPES]


def filters(s):
    return s[5] if isinstance(s[5], tuple) else (s[5], s[5])


def shape9(s):
    return s[:5] + filters(s) + s[6:]


def draw(s, beta, seed=3):
    N, H, W, ci, co, _, st, pad = s
    R, S = filters(s)
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*size):
        return torch.randn(*size, device="cuda", generator=g)

    gamma = torch.rand(ci, device="cuda", generator=g) + 0.5
    gamma[1] = -gamma[1]
    ho, wo = (H + 2 * pad - R) // st + 1, (W + 2 * pad - S) // st + 1
    return (normal(N, H, W, ci), normal(R, S, ci, co) * (2.0 / (R * S * ci)) ** 0.5, gamma, beta + normal(ci) * 0.1, normal(N, ho, wo, co))


def taps(s, ho, wo):
    (R, S), st = filters(s), s[6]
    for r in range(R):
        for q in range(S):
            yield r, q, slice(r, r + (ho - 1) * st + 1, st), slice(q, q + (wo - 1) * st + 1, st)


def gradients64(s, a3t, dy, w):
    """dA3 and dW in 64 bits."""
    N, H, W, ci, co, _, st, pad = s
    R, S = filters(s)
    ho, wo = dy.shape[1:3]
    p = torch.nn.functional.pad(a3t.double(), (0, 0, pad, pad, pad, pad))
    dp, dW, g, wd = torch.zeros_like(p), torch.zeros(R, S, ci, co, dtype=torch.float64, device="cuda"), dy.double().reshape(-1, co), w.double()
    for r, q, hs, ws in taps(s, ho, wo):
        piece = p[:, hs, ws]
        dW[r, q] = piece.reshape(-1, ci).t().contiguous() @ g
        dp[:, hs, ws] += (g @ wd[r, q].t().contiguous()).view(piece.shape)
    return dp[:, pad:pad + H, pad:pad + W], dW


# (2 t of the codes in one bf16; in two, both in LDS at a time or one after the other; in three)
@pytest.mark.parametrize("K,beta", [(4, 0.0), (8, 0.3), (4, 45.0), (8, 45.0), (8, 2000.0)])
@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_layer_step(s, K, beta):
    print("case layer of few channels", s, K, beta, flush=True)
    N, H, W, ci, co, _, st, pad = s
    R, S = filters(s)
    s9, M = shape9(s), N * H * W
    x, w, gamma, beta, dy = draw(s, beta)
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    y, skip = f32(*dy.shape), torch.randn_like(dy)
    B.abl_forward(s9, K, x, w, gamma, beta, skip, scratch, y, packed, stats)
    a3, a2t, p2, y2 = f32(*x.shape), f32(*x.shape), raw(B.abl_packed_bytes(s9, K)), f32(*dy.shape)
    B.abl_bn_relu_pack(x, M, ci, K, stats, a3, p2)
    B.abl_conv_fwd(s9, a3, w, skip, y2)
    assert torch.equal(packed, p2) and torch.equal(y, y2)    # (the same contraction, with and without the prologue)
    ref = skip.double()
    p = torch.nn.functional.pad(a3.double(), (0, 0, pad, pad, pad, pad))
    for r, q, hs, ws in taps(s, *dy.shape[1:3]):
        ref += (p[:, hs, ws].reshape(-1, ci) @ w[r, q].double()).view(ref.shape)
    # roundings of 2^-24: a random walk of one per 32 terms, the small products, the final sums; of terms that may be 45 / 0.5 times
    # their sum where beta is large
    top = float(beta.abs().max())
    worse = 1 if top < 1 else 20 if top < 50 else 900
    terms = 2.0 ** -24 * ((R * S * max(ci, co) / 32) ** 0.5 + 5)
    assert rel(y, ref) < worse * terms
    B.abl_unpack(packed, M, ci, K, stats, a2t)
    dx, dW, dg, db = f32(*x.shape), f32(*w.shape), f32(ci), f32(ci)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db)
    da3, rdW = gradients64(s, a2t.clamp(min=0), dy, w)
    da2 = torch.where(a2t > 0, da3, 0.0).view(M, ci)
    a1 = (a2t.double().view(M, ci) - beta.double()) / gamma.double()
    rstd = stats[: 28 * ci].view(torch.float32).view(7, ci)[2].double()
    rdb, rdg = da2.sum(0), (da2 * a1).sum(0)
    rdx = gamma.double() * rstd * (da2 - rdb / M - a1 * (rdg / M))
    for got, want in ((dx.view(M, ci), rdx), (dg, rdg), (db, rdb)):
        assert rel(got, want) < 10 * worse * terms
    assert rel(dW, rdW) < worse * 2.0 ** -24 * ((M / 32) ** 0.5 + 5)


# layers whose convolution with the prologue conv_split.hip has too
@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", [(64, 12, 12, 64, 64, 3, 1, 1), (27, 15, 15, 32, 128, 3, 1, 1), (68, 9, 9, 64, 128, 3, 1, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_stage_with_the_prologue_is_the_layers_kernel(s, K):
    """Where abl_forward_is_fused answers 1, abl_bn_conv_fwd runs what abl_forward runs: the same bits."""
    print("case layer of few channels, stage with the prologue", s, K, flush=True)
    s9, ci = shape9(s), s[3]
    x, w, gamma, beta, dy = draw(s, 0.1)
    assert B.abl_forward_is_fused(s9, K) == 1
    packed, stats, p2 = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_packed_bytes(s9, K))
    y, y2, skip = f32(*dy.shape), f32(*dy.shape), torch.randn_like(dy)
    B.abl_forward(s9, K, x, w, gamma, beta, skip, raw(B.abl_scratch_bytes(s9, K)), y, packed, stats)
    B.abl_bn_conv_fwd(s9, K, x, stats, w, skip, y2, p2)
    assert torch.equal(packed, p2) and torch.equal(y, y2)


# strided layers: dW beside the data gradient, by the kernels of other layers (own room for 12 copies and for one), 1x1
@pytest.mark.parametrize("s", [(40, 33, 32, 16, 32, 3, 2, 1), (32, 14, 14, 64, 32, 3, 2, 1), (2, 16, 16, 16, 16, 3, 2, 1), (64, 8, 8, 64, 64, 1, 2, 0)],
                         ids=lambda s: "x".join(map(str, s)))
def test_weight_gradient_over_the_weights(s):
    """dW over all of W and over a part of it: the data gradient reads W before."""
    print("case layer of few channels, dW over W", s, flush=True)
    N, H, W, ci, co, R, st, pad = s
    s9, K = (N, H, W, ci, co, R, R, st, pad), 4
    x, w, gamma, beta, dy = draw(s, 0.0)
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, f32(*dy.shape), packed, stats)
    want = [f32(*x.shape), f32(*w.shape), f32(ci), f32(ci)]
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, *want)
    n = w.numel()
    for at in (0, n // 2, n):   # (n: side by side)
        both = torch.empty(2 * n, device="cuda")
        both[:n] = w.view(-1)
        got = [f32(*x.shape), both[at:at + n].view(w.shape), f32(ci), f32(ci)]
        B.abl_backward(s9, K, packed, stats, dy, both[:n].view(w.shape), scratch, *got)
        # the same products in other tiles and copies: the bounds of test_layer_step, twice
        for a, b, tol in zip(got, want, (20, 2, 20, 20)):
            assert rel(a, b.double()) < tol * 2.0 ** -24 * ((max(R * R * max(ci, co), N * H * W) / 32) ** 0.5 + 5)
            assert at < n or torch.equal(a, b)


@pytest.mark.parametrize("s", [SHAPES[0], SHAPES[3], SHAPES[4], SHAPES[6]], ids=lambda s: "x".join(map(str, s)))
def test_values_the_split_cannot_carry(s):
    """An infinity and a NaN of dy reach the outputs that they reach in fp32 products, and no others."""
    print("case layer of few channels, not finite", s, flush=True)
    N, H, W, ci, co, R, st, pad = s
    s9, K = (N, H, W, ci, co, R, R, st, pad), 4
    x, w, gamma, beta, dy = draw(s, 0.0)
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, f32(*dy.shape), packed, stats)
    dx, dW, dg, db, da3, plain = f32(*x.shape), f32(*w.shape), f32(ci), f32(ci), f32(*x.shape), f32(*x.shape)
    B.abl_conv_dgrad(s9, dy, w, plain)
    at = (N // 2, dy.shape[1] - 1, 0)
    dy[at + (2,)] = float("inf")
    dy[0, 0, 0, 1] = float("nan")
    B.abl_conv_dgrad(s9, dy, w, da3)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db)
    hit = torch.zeros(N, H, W, dtype=torch.bool, device="cuda")
    for n, h, q in (at, (0, 0, 0)):
        h0, q0 = h * st - pad, q * st - pad
        hit[n, max(h0, 0):h0 + R, max(q0, 0):q0 + R] = True
    assert not bool(torch.isfinite(da3[hit]).any())
    assert float((da3 - plain)[~hit].abs().max()) <= 2.0 ** -19 * float(plain.abs().max())
    cols = torch.ones(co, dtype=torch.bool, device="cuda")
    cols[2] = cols[1] = False
    assert bool(torch.isfinite(dW[..., cols]).all()) and not bool(torch.isfinite(dW[R // 2, R // 2, :, 1:3]).all())
