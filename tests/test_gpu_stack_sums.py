"""Stacks of layers whose convolution adds up the statistics' sums of its input itself and leaves those of its output for the next
layer (csrc/conv_c16.hip, csrc/conv_narrow.hip): the rows that are read and those that are written lie apart, also where the grid is
more than the chip takes at a time and the first blocks end before the last begin.  Every layer of a traced forward on its own input."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

from .test_gpu_narrow import draw, taps
from .test_gpu_split_plans import f32, raw, rel

pytestmark = pytest.mark.gpu


def equal(N, H, W, c, count=4):
    return [(N, H, W, c, c, 3, 1, 1)] * count


# 512, 500, 300 and 256 blocks a layer; pairs of layers in place; then rows that go from kernel to kernel through every kind of layer: few channels,
# strided, with the weights split beside the second pass (64 -> 64 @14x14), 16 channels behind those
STACKS = {"16ch 32x32 N256": (equal(256, 32, 32, 16), 2), "16ch 33x33 N100": (equal(100, 33, 33, 16), 2),
          "24ch 5x5 10x10 N300": ([(300, 10, 10, 24, 24, 5, 1, 2)] * 5, 0),
          "32ch 16x16 N128": (equal(128, 16, 16, 32), 2), "16ch 32x32 N256, in place": (equal(256, 32, 32, 16, 6), 3),
          "mixed": ([(80, 28, 28, 64, 32, 3, 1, 1), (80, 28, 28, 32, 64, 3, 2, 1)] + equal(80, 14, 14, 64, 3) +
                    [(80, 14, 14, 64, 16, 3, 1, 1)] + equal(80, 14, 14, 16, 3) + [(80, 14, 14, 16, 32, 3, 2, 1)], 0)}


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("name", STACKS)
def test_forward_layer_by_layer(name, K):
    print("case stack sums", name, K, flush=True)
    shapes, every = STACKS[name]
    descs, xs = [], []
    for i, s in enumerate(shapes):
        N, H, W, ci, co, R, st, pad = s
        s9 = (N, H, W, ci, co, R, R, st, pad)
        x, w, gamma, beta, dy = draw(s, 0.0, 50 + i)
        descs.append(dict(shape=s9, W=w, gamma=gamma, beta=beta, packed=raw(B.abl_packed_bytes(s9, K)), stats=raw(B.abl_stats_bytes(s9)),
                          dW=f32(*w.shape), dgamma=f32(ci), dbeta=f32(ci)))
        xs.append(x if i == 0 else torch.empty_like(x))
    y_shape = dy.shape
    layers = B.make_layers(descs)
    nb = B.abl_stack_buffer_bytes(layers) // 4
    S, T, scratch = f32(nb), f32(nb), raw(B.abl_stack_scratch_bytes(layers, K))
    x0 = xs[0].clone()
    runs = []
    for traced in (True, False):
        S[:x0.numel()] = x0.view(-1)
        T.fill_(float("nan"))
        scratch.fill_(255)
        if traced:
            B.abl_stack_forward_traced(layers, K, every, S, T, scratch, xs)
        else:
            B.abl_stack_forward(layers, K, every, S, T, scratch)
        runs.append([S[:dy.numel()].view(y_shape).clone()] + [d[k].clone() for d in descs for k in ("packed", "stats")])
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    for i, (s, d) in enumerate(zip(shapes, descs)):
        N, H, W, ci, co, R, st, pad = s
        M, x, y = N * H * W, xs[i], xs[i + 1] if i + 1 < len(shapes) else runs[0][0]
        stats, a3, packed = raw(32 * ci), f32(*x.shape), raw(B.abl_packed_bytes(d["shape"], K))
        B.abl_bn_stats(x, M, ci, d["gamma"], d["beta"], K, raw(B.abl_bn_scratch_bytes(M, ci)), stats)
        mine, want = (t[:28 * ci].view(torch.float32).view(7, ci) for t in (d["stats"], stats))
        # sums of doubles in another order, then one rounding to fp32 (a mean beside the deviation)
        assert bool(((mine - want)[0].abs() <= 2.0 ** -22 * want[0].abs() + 1e-9 * want[1].sqrt()).all()), i
        assert bool(((mine - want)[1:].abs() <= 2.0 ** -22 * want[1:].abs()).all()), i
        B.abl_bn_relu_pack(x, M, ci, K, d["stats"], a3, packed)
        assert torch.equal(packed, d["packed"]), i
        ref = torch.zeros(y.shape, dtype=torch.float64, device="cuda")
        p = torch.nn.functional.pad(a3.double(), (0, 0, pad, pad, pad, pad))
        for r, q, hs, ws in taps(s, *y.shape[1:3]):
            ref += (p[:, hs, ws].reshape(-1, ci) @ d["W"][r, q].double()).view(ref.shape)
        if every and (i + 1) % every == 0:
            ref += xs[i + 1 - every].double()
        # as in test_gpu_narrow.py
        assert rel(y, ref) < 2.0 ** -24 * ((R * R * ci / 32) ** 0.5 + 5), i
