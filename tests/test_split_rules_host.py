"""Grids that the split convolutions choose, pinned where they were measured (no GPU)."""
import pytest

from . import split_rules as R


@pytest.mark.parametrize("s, want", [
    # image by image, two blocks per compute unit: 560 tiles in blocks of two, one tile each
    ((80, 27, 27, 128, 128, 3), 280), ((64, 27, 27, 128, 128, 3), 448), ((56, 29, 29, 128, 128, 3), 448),
    ((64, 33, 33, 64, 64, 3), 320), ((64, 40, 40, 64, 64, 3), 480), ((20, 22, 22, 256, 256, 3), 100),
    # runs across images, one block per unit: one round of them against more than a round's worth of pairs' first halves
    ((28, 32, 32, 64, 64, 3), 256), ((20, 26, 26, 128, 128, 3), 121),
    # patches beyond a pair's either way: fewer tiles, as many to a block as keep the units busy
    ((64, 55, 55, 64, 64, 3), 256), ((40, 57, 57, 64, 64, 3), 233),
    # patches within a pair's either way
    ((64, 14, 14, 256, 256, 3), 112), ((64, 56, 56, 64, 64, 3), 448), ((64, 28, 28, 128, 128, 3), 448)],
    ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_fused_forward(s, want):
    assert R.fused_rows(s) == want


@pytest.mark.parametrize("s, want", [((64, 55, 55, 64, 64, 3), 448), ((28, 55, 55, 64, 64, 3), 392), ((96, 57, 57, 64, 64, 3), 465),
                                     ((64, 56, 56, 64, 64, 3), 448)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_bf16_gradient(s, want):
    """With bf16 operands a large patch leaves room for two blocks per compute unit."""
    assert R.rows(s, 1, True, True) == want


@pytest.mark.parametrize("s, mode, want", [
    # gradients of several tiles per block: with 64 channels to contract, not with more
    ((80, 30, 30, 512, 128, 1), 1, 0), ((80, 28, 28, 512, 128, 1), 1, 0), ((40, 30, 30, 512, 128, 1), 1, 322),
    ((80, 56, 56, 256, 64, 1), 1, 249),
    # forward with 64 channels to contract: larger grids
    ((14, 56, 56, 64, 256, 1), 0, 0), ((16, 55, 55, 64, 256, 1), 0, 0), ((16, 56, 56, 64, 256, 1), 0, 448),
    ((28, 28, 28, 128, 512, 1), 0, 196)],
    ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_bf16_1x1(s, mode, want):
    assert R.rows(s, mode, True, mode == 1) == want


@pytest.mark.parametrize("s, bf16, want", [
    ((128, 8, 8, 64, 64, 3), False, False), ((24, 28, 28, 64, 64, 3), False, False), ((40, 28, 28, 64, 64, 3), True, True),
    ((64, 56, 56, 64, 64, 3), False, True), ((64, 14, 14, 256, 256, 3), False, True), ((40, 7, 7, 512, 512, 3), True, True),
    ((14, 55, 55, 64, 256, 1), False, False), ((64, 55, 55, 64, 256, 1), False, True), ((14, 28, 28, 128, 512, 1), False, False),
    ((26, 28, 28, 128, 512, 1), False, True), ((40, 14, 14, 1024, 256, 1), False, False), ((40, 14, 14, 256, 1024, 1), False, True),
    ((34, 56, 56, 64, 256, 1), True, False), ((34, 14, 14, 256, 1024, 1), True, False), ((64, 14, 14, 256, 1024, 1), True, True),
    ((52, 15, 15, 1024, 256, 1), True, True)],
    ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_a_launch_of_its_own_to_split_weights(s, bf16, want):
    assert R.parts_pay(s, 1, bf16, own_launch=True) == want
    assert R.parts_pay(s, 1, bf16)   # in the launch of the layer above they all are split


@pytest.mark.parametrize("s, want", [((12, 55, 55, 64, 256, 1), False), ((14, 56, 56, 64, 256, 1), False), ((16, 56, 56, 64, 256, 1), True),
                                     ((12, 28, 28, 128, 512, 1), True), ((12, 8, 8, 64, 64, 3), True)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_weights_of_a_forward(s, want):
    assert R.parts_pay(s, 0) == want and R.parts_pay(s, 0, True) == want


@pytest.mark.parametrize("s, fwd, bwd", [
    ((64, 7, 7, 256, 256, 3), False, False), ((52, 7, 7, 256, 256, 3), False, False), ((80, 7, 7, 256, 256, 3), True, True),
    ((128, 7, 7, 128, 128, 3), False, False), ((40, 8, 8, 256, 256, 3), False, True), ((64, 10, 10, 256, 256, 3), False, True),
    ((64, 12, 12, 128, 128, 3), True, True), ((40, 7, 7, 512, 512, 3), True, True), ((64, 14, 14, 256, 256, 3), True, True)],
    ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_small_images_with_bf16_operands(s, fwd, bwd):
    assert (R.beats_image(s, 0), R.beats_image(s, 1)) == (fwd, bwd)
