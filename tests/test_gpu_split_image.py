"""bf16 3x3 layers of 512 channels on images that fit the LDS: layer calls, whose weights come in parts, run the split kernel,
stage calls the image-resident one.  Same rounded operands, another order of fp32 sums."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

from . import split_rules as R
from .test_gpu_split_weights import draw, f32, raw, shape9

pytestmark = pytest.mark.gpu

# a grid of four-wave blocks, one round of images, runs of several images to a tile, more images than one row of sums each
SHAPES = [(40, 8, 8, 512, 512, 3), (28, 7, 7, 512, 512, 3), (14, 8, 8, 512, 512, 3), (30, 6, 6, 512, 512, 3), (520, 5, 6, 512, 64, 3)]


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_layer_against_image_kernel(s, K):
    print("case bf16 512 channels", s, K, flush=True)
    s9, C, M = shape9(s), s[3], s[0] * s[1] * s[2]
    x, w, gamma, beta, dy = draw(s, 17)
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    y = f32(*dy.shape)
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, y, packed, stats, flags=B.ABL_MATH_BF16)
    a3, p2, y2 = f32(*x.shape), raw(B.abl_packed_bytes(s9, K)), f32(*dy.shape)
    B.abl_bn_relu_pack(x, M, C, K, stats, a3, p2)
    B.abl_conv_fwd(s9, a3, w, None, y2, flags=B.ABL_MATH_BF16)
    assert torch.equal(packed, p2)
    # both sum exact products of the same operands in fp32: 9 C / 32 roundings each of at most 2^-24 of a partial sum (in 64
    # terms of the largest output)
    tol = 2.0 ** -19
    assert float((y - y2).abs().max()) < tol * float(y2.abs().max())
    dx, dw, dg, db = torch.empty_like(x), torch.empty_like(w), f32(C), f32(C)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dw, dg, db, flags=B.ABL_MATH_BF16)
    da3 = f32(*x.shape)
    B.abl_conv_dgrad(s9, dy, w, da3, flags=B.ABL_MATH_BF16)
    mine = scratch[:4 * x.numel()].view(torch.float32).view(x.shape)   # dA3 stays at the start of the workspace
    assert float((mine - da3).abs().max()) < tol * float(da3.abs().max())
    dx2, dg2, db2 = torch.empty_like(x), f32(C), f32(C)
    B.abl_bn_bwd(packed, stats, mine.clone(), M, C, K, raw(B.abl_bn_scratch_bytes(M, C)), dx2, dg2, db2)
    # (from the very same dA3: sums in 64 bits in another order, then a rounding or two of fp32)
    for got, want in ((dx, dx2), (dg, dg2), (db, db2)):
        assert float((got - want).abs().max()) <= 2.0 ** -20 * float(want.abs().max())


@pytest.mark.parametrize("s", [(108, 3, 3, 512, 64, 3), (74, 4, 5, 512, 128, 3)], ids=lambda s: "x".join(map(str, s)))
def test_one_round_of_small_images(s):
    """Forward on images of a tile or two, one round of the compute units: the image kernel in layer calls too."""
    print("case bf16 512 channels, small images", s, flush=True)
    K, s9, C, M = 4, shape9(s), s[3], s[0] * s[1] * s[2]
    x, w, gamma, beta, dy = draw(s, 18)
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    y, y2, a3 = f32(*dy.shape), f32(*dy.shape), f32(*x.shape)
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, y, packed, stats, flags=B.ABL_MATH_BF16)
    B.abl_bn_relu_pack(x, M, C, K, stats, a3, raw(B.abl_packed_bytes(s9, K)))
    B.abl_conv_fwd(s9, a3, w, None, y2, flags=B.ABL_MATH_BF16)
    assert torch.equal(y, y2)


def test_rule():
    """What the stage calls take is what it was."""
    assert not R.beats_image(SHAPES[0], 0) and not R.beats_image(SHAPES[0], 1)
