"""Weights split once per call: the layer and stack calls, whose convolutions read the parts from the workspace, against the
stage calls, which have no workspace and split in the kernel.  Same parts, same order of sums: the same bits, where the stage
takes the same grid."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

from . import split_rules as R

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cout, R: every kernel of the plan (blocks of four and eight waves, 64 and 128 channels), patches of more
# than 256 positions, several tiles to a block, one phase and an odd number of them
SHAPES = [(220, 7, 7, 64, 64, 3), (64, 14, 14, 192, 128, 3), (64, 14, 14, 128, 128, 3), (100, 12, 11, 32, 64, 3), (12, 57, 57, 64, 64, 3),
          (40, 28, 28, 128, 128, 3), (40, 56, 56, 64, 64, 3), (1, 110, 101, 64, 64, 1), (64, 14, 14, 1024, 256, 1),
          (2, 150, 151, 128, 256, 1), (9, 141, 143, 192, 64, 1), (40, 56, 56, 64, 256, 1)]
IDS = ["x".join(map(str, s)) for s in SHAPES]


def shape9(s):
    return s[:5] + (s[5], s[5], 1, (s[5] - 1) // 2)


def f32(*size):
    return torch.empty(*size, dtype=torch.float32, device="cuda")


def raw(n):
    return torch.empty(max(16, int(n)), dtype=torch.uint8, device="cuda")


def draw(s, seed):
    N, H, W, ci, co, R = s
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*size):
        return torch.randn(*size, device="cuda", generator=g)

    return (normal(N, H, W, ci), normal(R, R, ci, co) * (2.0 / (ci * R * R)) ** 0.5, torch.rand(ci, device="cuda", generator=g) + 0.5,
            normal(ci) * 0.1, normal(N, H, W, co))


@pytest.mark.parametrize("flags", [0, B.ABL_MATH_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_layer_equals_stages(s, flags):
    K, s9 = (8 if s[0] % 8 else 4), shape9(s)
    x, w, gamma, beta, dy = draw(s, 11)
    M, C = s[0] * s[1] * s[2], s[3]
    packed, stats, scratch = raw(B.abl_packed_bytes(s9, K)), raw(B.abl_stats_bytes(s9)), raw(B.abl_scratch_bytes(s9, K))
    n = max(x.numel(), dy.numel())
    buf = f32(n)   # output over input: the pack pass and the plain convolution
    buf[:x.numel()] = x.view(-1)
    y = buf[:dy.numel()].view(dy.shape)
    B.abl_forward(s9, K, buf[:x.numel()].view(x.shape), w, gamma, beta, None, scratch, y, packed, stats, flags=flags)
    a3, p2, y2 = f32(*x.shape), raw(B.abl_packed_bytes(s9, K)), f32(*dy.shape)
    B.abl_bn_relu_pack(x, M, C, K, stats, a3, p2)
    B.abl_conv_fwd(s9, a3, w, None, y2, flags=flags)
    assert torch.equal(packed, p2) and torch.equal(y, y2)
    dx, dw, dg, db = torch.empty_like(x), torch.empty_like(w), f32(C), f32(C)
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dw, dg, db, flags=flags)
    da3, dx2, dw2, dg2, db2 = f32(*x.shape), torch.empty_like(x), f32(*w.shape), f32(C), f32(C)
    B.abl_conv_dgrad(s9, dy, w, da3, flags=flags)
    # dA3 stays at the start of the workspace
    mine = scratch[:4 * x.numel()].view(torch.float32).view(x.shape)
    grids = [R.rows(s, 1, bool(flags), sums) for sums in (False, True)]
    stage_splits = grids[0] > 0 and not (flags and s[5] == 1 and s[4] < 1024)   # (shorter bf16 1x1 stages: another kernel)
    if grids[0] == grids[1] and stage_splits and not (flags and R.beats_image(s, 1) != (grids[0] > 0)):
        assert torch.equal(mine, da3)
    else:
        assert float((mine - da3).abs().max()) < 2.0 ** -19 * float(da3.abs().max())
    B.abl_conv_wgrad_packed(s9, K, packed, stats, dy, raw(B.abl_wgrad_scratch_bytes(s9)), dw2, flags=flags)
    B.abl_bn_bwd(packed, stats, da3, M, C, K, raw(B.abl_bn_scratch_bytes(M, C)), dx2, dg2, db2)
    # the sums of Eq. 7 are taken in another order and by another kernel, whose data gradient may be another one as well:
    # roundings of an fp32 accumulator per 32 terms (2e-6 for 2304 terms), bf16 operands the same but for their order
    # (dW: the same products, the pixels in other parts)
    for a, b in ((dx, dx2), (dw, dw2), (dg, dg2), (db, db2)):
        assert float((a.double() - b.double()).norm() / b.double().norm()) < 4e-6
    # no element left out or written twice: roundings of the largest
    for a, b in ((dx, dx2), (dw, dw2)):
        assert float((a - b).abs().max()) < 2.0 ** -19 * float(b.abs().max())


@pytest.mark.parametrize("flags", [0, B.ABL_MATH_BF16], ids=["fp32", "bf16"])
def test_stack_equals_layers(flags):
    """Layers of different sizes one after the other: the parts of the next layer's weights lie beyond both layers' buffers."""
    K, N, hw = 4, 24, 28
    chain = [(64, 512, 1), (512, 128, 1), (128, 128, 3), (128, 64, 1), (64, 64, 3)]
    shapes = [(N, hw, hw, ci, co, R) for ci, co, R in chain]
    descs, params = [], []
    for i, s in enumerate(shapes):
        _, w, gamma, beta, _ = draw(s, 20 + i)
        s9 = shape9(s)
        params.append((s9, w))
        descs.append(dict(shape=s9, W=w, gamma=gamma, beta=beta, packed=raw(B.abl_packed_bytes(s9, K)),
                          stats=raw(B.abl_stats_bytes(s9)), dW=torch.empty_like(w), dgamma=f32(s[3]), dbeta=f32(s[3])))
    layers = B.make_layers(descs)
    nb = B.abl_stack_buffer_bytes(layers) // 4
    S, T = f32(nb), f32(nb)
    scratch = raw(B.abl_stack_scratch_bytes(layers, K))
    x, dy = draw(shapes[0], 5)[0], draw(shapes[-1], 6)[4]
    S[:x.numel()] = x.view(-1)
    B.abl_stack_forward(layers, K, 0, S, T, scratch, flags=flags)
    S[:dy.numel()] = dy.view(-1)
    scratch.fill_(255)
    B.abl_stack_backward(layers, K, 0, S, T, scratch, flags=flags)
    d = dy
    for s, (s9, w), e in reversed(list(zip(shapes, params, descs))):
        dx, dw, dg, db = f32(*s[:4]), torch.empty_like(w), f32(s[3]), f32(s[3])
        B.abl_backward(s9, K, e["packed"], e["stats"], d, w, raw(B.abl_scratch_bytes(s9, K)), dx, dw, dg, db, flags=flags)
        assert torch.equal(dw, e["dW"].view(dw.shape)) and torch.equal(dg, e["dgamma"]) and torch.equal(db, e["dbeta"])
        d = dx
    assert torch.equal(d.view(-1), S[:x.numel()])


@pytest.mark.parametrize("flags", [0, B.ABL_MATH_BF16], ids=["fp32", "bf16"])
def test_dw_depends_on_the_layer_alone(flags):
    """A layer whose own room holds 85 copies of dW where 128 blocks would share its pixels: the same bits of dW wherever dx lies,
    added to or not, and in a stack with a shortcut and larger layers."""
    s, K, N = (64, 56, 56, 64, 64, 3), 4, 64 * 56 * 56 * 64
    s9 = shape9(s)
    x, w, gamma, beta, dy = draw(s, 31)

    def layer():
        return dict(shape=s9, W=w, gamma=gamma, beta=beta, packed=raw(B.abl_packed_bytes(s9, K)), stats=raw(B.abl_stats_bytes(s9)),
                    dW=f32(*w.shape), dgamma=f32(64), dbeta=f32(64))

    one = layer()
    scratch = raw(B.abl_scratch_bytes(s9, K))
    B.abl_forward(s9, K, x, w, gamma, beta, None, scratch, f32(*dy.shape), one["packed"], one["stats"], flags=flags)

    def backward(dy, dx, more=0):
        dw, dg, db = f32(*w.shape), f32(64), f32(64)
        scratch.fill_(255)
        B.abl_backward(s9, K, one["packed"], one["stats"], dy, w, scratch, dx, dw, dg, db, flags=flags | more)
        return dx, dw, dg, db

    dx, dw, dg, db = backward(dy, torch.full_like(x, float("nan")))
    stage = f32(*w.shape)
    B.abl_conv_wgrad_packed(s9, K, one["packed"], one["stats"], dy, raw(B.abl_wgrad_scratch_bytes(s9)), stage, flags=flags)
    assert float((dw.double() - stage.double()).norm() / stage.double().norm()) < 2e-6   # (sums over the pixels in other parts)
    for at in (0, N // 2):   # dx over all of dy and over half of it; dy is dead once both contractions have run
        both = torch.empty(2 * N, device="cuda")
        dy2 = both[at:at + N].view(dy.shape)
        dy2.copy_(dy)
        for a, b in zip(backward(dy2, both[:N].view(x.shape)), (dx, dw, dg, db)):
            assert torch.equal(a, b)
    over = w.clone()   # dW over the weights: written behind the data gradient, which reads them
    dx2, dg2, db2 = torch.empty_like(x), f32(64), f32(64)
    B.abl_backward(s9, K, one["packed"], one["stats"], dy, over, scratch, dx2, over, dg2, db2, flags=flags)
    assert torch.equal(dx2, dx) and torch.equal(dg2, dg)
    assert float((over.double() - stage.double()).norm() / stage.double().norm()) < 2e-6
    acc = backward(dy, torch.ones_like(x), B.ABL_ACCUM_DX)
    assert torch.equal(acc[0], 1.0 + dx) and all(torch.equal(a, b) for a, b in zip(acc[1:], (dw, dg, db)))

    # in stacks, pairs of layers with a shortcut: alone (the layer's own room) and below layers with a larger workspace
    for widths in ((), (64, 256, 64)):
        shapes = [s, s] + [(64, 56, 56, a, b, 1) for a, b in zip(widths, widths[1:])]
        descs = [layer(), layer()]
        for i, t in enumerate(shapes[2:]):
            _, tw, tg, tb, _ = draw(t, 40 + i)
            descs.append(dict(shape=shape9(t), W=tw, gamma=tg, beta=tb, packed=raw(B.abl_packed_bytes(shape9(t), K)),
                              stats=raw(B.abl_stats_bytes(shape9(t))), dW=f32(*tw.shape), dgamma=f32(t[3]), dbeta=f32(t[3])))
        layers = B.make_layers(descs)
        nb = B.abl_stack_buffer_bytes(layers) // 4
        S, T, ws = f32(nb), f32(nb), raw(B.abl_stack_scratch_bytes(layers, K))
        S[:N] = x.view(-1)
        B.abl_stack_forward(layers, K, 2, S, T, ws, flags=flags)
        S[:N] = dy.view(-1)
        ws.fill_(255)
        B.abl_stack_backward(layers, K, 2, S, T, ws, flags=flags)
        d = dy
        for pair in reversed(range(0, len(descs), 2)):
            skip = d
            for t, e in reversed(list(zip(shapes[pair:pair + 2], descs[pair:pair + 2]))):
                dx, dw, dg, db = f32(*t[:4]), f32(*e["W"].shape), f32(t[3]), f32(t[3])
                B.abl_backward(shape9(t), K, e["packed"], e["stats"], d, e["W"], raw(B.abl_scratch_bytes(shape9(t), K)), dx, dw, dg, db,
                               flags=flags)
                assert torch.equal(dw, e["dW"]) and torch.equal(dg, e["dgamma"]) and torch.equal(db, e["dbeta"])
                d = dx
            d = skip + d
        assert torch.equal(S[:N], d.view(-1))
