"""Strided layers with at most 32 output channels at both sides of the rule that gives small grids tiles of 64 pixels
and larger ones tiles of 256: forward and data gradient against 64-bit values."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cout; 3x3, stride 2, padding 1.  Forward: 512 blocks of 256 x 32 outputs, 131072 pixels; data gradient:
# 192 blocks, 49152 pixels in four classes
SHAPES = [
    (127, 64, 64, 16, 32),    # forward below, data gradient far beyond
    (128, 64, 64, 16, 32),    # forward at 512 blocks
    (130, 63, 65, 32, 16),    # 32-channel chunks, odd sizes
    (47, 32, 32, 16, 16),     # data gradient below
    (48, 32, 32, 32, 32),     # data gradient at 192 blocks
    (9, 31, 33, 48, 16),
]


def tolerance(terms):
    # fp32 products and sums, rounded once per four terms at the magnitude of the running sum: a random walk
    return 2.0 ** -24 * ((terms / 4) ** 0.5 + 2)


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_strided_layers(s):
    print("case strided layer", s, flush=True)
    N, H, W, ci, co = s
    Ho, Wo = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    t = (N, H, W, ci, co, 3, 3, 2, 1)
    g = torch.Generator(device="cuda").manual_seed(9)
    x, dy = torch.randn(N, H, W, ci, device="cuda", generator=g), torch.randn(N, Ho, Wo, co, device="cuda", generator=g)
    w = torch.randn(3, 3, ci, co, device="cuda", generator=g)
    y, da = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    B.abl_conv_fwd(t, x, w, None, y)
    B.abl_conv_dgrad(t, dy, w, da)
    p = torch.nn.functional.pad(x.double(), (0, 0, 1, 2, 1, 2))
    y64, dp = torch.zeros(N * Ho * Wo, co, dtype=torch.float64, device="cuda"), torch.zeros_like(p)
    for r in range(3):
        for q in range(3):
            hs, ws = slice(r, r + 2 * Ho - 1, 2), slice(q, q + 2 * Wo - 1, 2)
            y64 += p[:, hs, ws].reshape(-1, ci) @ w[r, q].double()
            dp[:, hs, ws] += (dy.double().view(-1, co) @ w[r, q].double().t().contiguous()).view(N, Ho, Wo, ci)
    da64 = dp[:, 1:1 + H, 1:1 + W]
    assert float((y.view(-1, co) - y64).norm() / y64.norm()) < tolerance(9 * ci)
    assert float((da - da64).norm() / da64.norm()) < tolerance(9 * co)
