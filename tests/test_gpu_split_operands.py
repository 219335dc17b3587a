"""fp32 contractions whose operands are split into three bf16 parts, against 64-bit values, at the edges of their
tiles (runs of 112 pixels within an image, across images or of whole images; 64 or 128 output channels per block;
32-channel phases) and for values that the split cannot carry."""
import pytest
import torch

from paper_1901_07988_amd import binding as B

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cout, R
SHAPES = [
    (2100, 1, 1, 64, 64, 3),     # images of one pixel: 21 of them to a patch
    (220, 7, 7, 64, 64, 3),      # runs of whole images; two groups of waves
    (120, 14, 14, 64, 128, 3),   # runs across images; 128 channels per block forward, 64 backward
    (100, 12, 11, 32, 64, 3),    # one 32-channel phase; two images' borders in a patch
    (12, 57, 57, 64, 64, 3),     # a run of 112 pixels touches three rows
    (29, 28, 28, 64, 128, 3),    # seven runs of four rows to an image
    (40, 56, 56, 64, 64, 3),     # several tiles to a block
    (11, 13, 60, 128, 192, 3),
    (1, 110, 101, 64, 64, 1),    # 112 pixels to a tile, the last one short; two groups of waves
    (1, 150, 150, 64, 128, 1),
    (2, 150, 151, 128, 256, 1),  # more blocks than compute units
    (3, 141, 143, 192, 64, 1),   # several tiles to a block
]
IDS = ["x".join(map(str, s)) for s in SHAPES]
# layers whose gradient with the sums is not taken as a stage of its own (more than 512 tiles of the halo kernel)
STAGE_REFUSES = [(12, 57, 57, 64, 64, 3), (40, 56, 56, 64, 64, 3)]


def shape9(s):
    return s[:5] + (s[5], s[5], 1, (s[5] - 1) // 2)


def conv64(a, w):
    """'Same' stride-1 convolution in 64 bits, a NHWC, w RSCK."""
    R, pad = w.shape[0], (w.shape[0] - 1) // 2
    N, H, W, c = a.shape
    p, wd = torch.nn.functional.pad(a.double(), (0, 0, pad, pad, pad, pad)), w.double()
    y = torch.zeros(N * H * W, w.shape[3], dtype=torch.float64, device=a.device)
    for r in range(R):
        for q in range(R):
            y += p[:, r:r + H, q:q + W].reshape(-1, c) @ wd[r, q].contiguous()
    return y.view(N, H, W, -1)


def grad_weights(w):
    return w.flip(0, 1).transpose(2, 3).contiguous()


def tolerance(terms):
    # the large products are rounded once per 32 terms at the magnitude of the running sum, which is a random walk
    # for these inputs: sqrt(terms / 32) roundings of 2^-24, and two for the small products and the final sum
    return 2.0 ** -24 * ((terms / 32) ** 0.5 + 2)


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


def draw(s, seed=3):
    N, H, W, ci, co, R = s
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*size):
        return torch.randn(*size, device="cuda", generator=g)

    return normal(N, H, W, ci), normal(R, R, ci, co) * (2.0 / (ci * R * R)) ** 0.5, normal(N, H, W, co)


@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_forward_and_gradient(s):
    print("case split operands", s, flush=True)
    x, w, dy = draw(s)
    R, ci, co = s[5], s[3], s[4]
    y, da3, y2 = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan")), torch.empty_like(dy)
    B.abl_conv_fwd(shape9(s), x, w, None, y)
    B.abl_conv_dgrad(shape9(s), dy, w, da3)
    B.abl_conv_fwd(shape9(s), x, w, dy, y2)
    assert rel(y, conv64(x, w)) < tolerance(R * R * ci)
    if ci % 64 == 0:   # (other kernels compute gradients of 32 channels)
        assert rel(da3, conv64(dy, grad_weights(w))) < tolerance(R * R * co)
    assert torch.equal(y2, y + dy)   # the shortcut is one fp32 addition


@pytest.mark.parametrize("s", SHAPES, ids=IDS)
def test_bf16_operands(s):
    """ABL_MATH_BF16: each operand rounded to bf16 once, sums in fp32."""
    print("case bf16 operands", s, flush=True)
    x, w, dy = draw(s)
    R, ci, co = s[5], s[3], s[4]
    y, da3 = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    B.abl_conv_fwd(shape9(s), x, w, None, y, flags=B.ABL_MATH_BF16)
    B.abl_conv_dgrad(shape9(s), dy, w, da3, flags=B.ABL_MATH_BF16)
    xr, wr, dr = (t.bfloat16().float() for t in (x, w, dy))
    # (the other bf16 kernels and the fp32 ones round per 4 to 32 terms)
    assert rel(y, conv64(xr, wr)) < 3 * tolerance(R * R * ci)
    assert rel(da3, conv64(dr, grad_weights(wr))) < 3 * tolerance(R * R * co)


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", [s for s in SHAPES if s[3] % 64 == 0], ids=lambda s: "x".join(map(str, s)))
def test_sums_of_the_gradient(s, K):
    print("case split operands, sums", s, K, flush=True)
    x, w, dy = draw(s)
    N, H, W, ci, co, R = s
    M, s9 = N * H * W, shape9(s)
    g = torch.Generator(device="cuda").manual_seed(1)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, torch.randn(ci, device="cuda", generator=g) * 0.1
    stats = torch.empty(32 * ci, dtype=torch.uint8, device="cuda")
    packed = torch.empty(B.abl_packed_bytes(s9, K), dtype=torch.uint8, device="cuda")
    scratch = torch.empty(B.abl_scratch_bytes(s9, K), dtype=torch.uint8, device="cuda")
    a3, a2t, da3, plain = (torch.empty_like(x) for _ in range(4))
    B.abl_bn_stats(x, M, ci, gamma, beta, K, scratch, stats)
    B.abl_bn_relu_pack(x, M, ci, K, stats, a3, packed)
    B.abl_unpack(packed, M, ci, K, stats, a2t)
    B.abl_conv_dgrad(s9, dy, w, plain)
    da2 = torch.where(a2t > 0, plain, torch.zeros_like(plain)).double().view(M, ci)
    a1 = (a2t.double().view(M, ci) - beta.double()) / gamma.double()
    # sums in 64 bits; a2t is rounded to 32 bits here and not there
    bounds = [2.0 ** -23 * float(t.abs().sum(0).max()) for t in (da2, da2 * a1)]
    refs = [da2.sum(0), (da2 * a1).sum(0)]
    dx, dW, dg, db = torch.empty_like(x), torch.empty_like(w), torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")
    B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db)
    for got, ref, bound in zip((db, dg), refs, bounds):
        assert float((got.double() - ref).abs().max()) <= bound + 2.0 ** -24 * float(ref.abs().max())
    if s in STAGE_REFUSES:
        with pytest.raises(B.AblError) as e:
            B.abl_conv_dgrad_bn_reduce(s9, K, dy, w, packed, stats, scratch, da3)
        assert e.value.code == B.ABL_ERR_SHAPE
        return
    rows = B.abl_conv_dgrad_bn_reduce(s9, K, dy, w, packed, stats, scratch, da3)
    assert torch.equal(da3, plain)
    sums = scratch[: rows * 2 * ci * 8].view(torch.float64).view(rows, 2, ci).sum(0)
    for got, ref, bound in zip(sums, refs, bounds):
        assert float((got - ref).abs().max()) <= bound


@pytest.mark.parametrize("s", [SHAPES[2], SHAPES[5], SHAPES[9], SHAPES[10]], ids=lambda s: "x".join(map(str, s)))
def test_statistics_of_the_output(s):
    """The next layer's statistics from the sums that the convolution leaves."""
    print("case split operands, statistics", s, flush=True)
    x, w, _ = draw(s)
    N, H, W, ci, co, R = s
    first, second = shape9(s), (N, H, W, co, 64, 1, 1, 1, 0)
    w2 = torch.randn(1, 1, co, 64, device="cuda") * 0.1
    descs = []
    for sh, wt in ((first, w), (second, w2)):
        c = sh[3]
        f = torch.zeros
        descs.append(dict(shape=sh, W=wt, gamma=torch.ones(c, device="cuda"), beta=f(c, device="cuda"),
                          packed=torch.empty(B.abl_packed_bytes(sh, 4), dtype=torch.uint8, device="cuda"),
                          stats=torch.empty(32 * c, dtype=torch.uint8, device="cuda"), dW=f(wt.numel(), device="cuda"),
                          dgamma=f(c, device="cuda"), dbeta=f(c, device="cuda")))
    layers = B.make_layers(descs)
    nb = B.abl_stack_buffer_bytes(layers) // 4
    bs, bt = torch.zeros(nb, device="cuda"), torch.zeros(nb, device="cuda")
    bs[: x.numel()].copy_(x.view(-1))
    B.abl_stack_forward(layers, 4, 0, bs, bt, torch.empty(B.abl_stack_scratch_bytes(layers, 4), dtype=torch.uint8, device="cuda"))
    y = bt[: N * H * W * co].view(-1, co).double()   # the first layer writes the second buffer
    planes = descs[1]["stats"][: 28 * co].view(torch.float32).view(7, co).double()
    var = y.var(0, unbiased=False)
    assert float((planes[0] - y.mean(0)).abs().max()) <= 2.0 ** -23 * float(y.abs().mean(0).max())
    assert float(((planes[1] - var) / var).abs().max()) <= 2.0 ** -22


@pytest.mark.parametrize("s", [SHAPES[1], SHAPES[5], SHAPES[8], SHAPES[10]], ids=lambda s: "x".join(map(str, s)))
def test_values_the_split_cannot_carry(s):
    """Infinities, NaN and values that round to an infinite bf16 give what fp32 products and sums give."""
    print("case split operands, not finite", s, flush=True)
    x, w, _ = draw(s)
    x, w = x.abs() + 0.5, w.abs() + 0.01
    big = 3.4e38
    w[..., 1] = 2.0 ** -20          # keeps the largest values finite
    w[..., 2] = 0.0                 # infinity times zero
    x[0, 0, 0, 5] = float("inf")
    x[-1, -1, -1, 7] = float("nan")
    x[x.shape[0] // 2, x.shape[1] // 2, x.shape[2] // 2, 9] = big
    x[0, -1, 0, 11] = -float("inf")
    y = torch.empty(*x.shape[:3], s[4], device="cuda")
    B.abl_conv_fwd(shape9(s), x, w, None, y)
    ref = conv64(x, w).float()
    assert torch.equal(torch.isnan(y), torch.isnan(ref))
    assert torch.equal(torch.isinf(y), torch.isinf(ref))
    ok = torch.isfinite(ref)
    assert float(((y - ref)[ok].abs() / ref[ok].abs().clamp(min=1e-30)).max()) < 1e-5   # (positive terms: no cancellation)


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", [SHAPES[3], SHAPES[4], SHAPES[5], SHAPES[7], SHAPES[6]], ids=lambda s: "x".join(map(str, s)))
def test_forward_with_prologue(s, K):
    """abl_forward where the kernel normalises and packs while it stages: the codes are those of the separate pass bit
    for bit, the output is the separate pass's convolution up to the order of the sums."""
    print("case split operands, fused forward", s, K, flush=True)
    x, w, skip = draw(s)
    N, H, W, ci, co, R = s
    s9, M = shape9(s), N * H * W
    assert B.abl_forward_is_fused(s9, K)
    g = torch.Generator(device="cuda").manual_seed(2)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, torch.randn(ci, device="cuda", generator=g) * 0.1

    def raw(n):
        return torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")

    scratch = raw(B.abl_scratch_bytes(s9, K))
    y, packed, stats = torch.full_like(skip, float("nan")), raw(B.abl_packed_bytes(s9, K)), raw(32 * ci)
    B.abl_forward(s9, K, x, w, gamma, beta, skip, scratch, y, packed, stats)
    a3, packed2, stats2 = torch.empty_like(x), raw(B.abl_packed_bytes(s9, K)), raw(32 * ci)
    B.abl_bn_stats(x, M, ci, gamma, beta, K, scratch, stats2)
    B.abl_bn_relu_pack(x, M, ci, K, stats2, a3, packed2)
    assert torch.equal(stats, stats2) and torch.equal(packed, packed2)
    assert rel(y, conv64(a3, w) + skip.double()) < tolerance(R * R * ci)


SMALL = 2.0 ** -120   # products with values near 1 stay normal, two of the three bf16 parts of such a value do not


@pytest.mark.parametrize("tiny", ["values", "weights"])
@pytest.mark.parametrize("s", [SHAPES[1], SHAPES[5], SHAPES[8], SHAPES[10]], ids=lambda s: "x".join(map(str, s)))
def test_small_operands(s, tiny):
    """Operands far below 1 keep their 24 bits."""
    print("case split operands, small", s, tiny, flush=True)
    x, w, dy = draw(s)
    R, ci, co = s[5], s[3], s[4]
    if tiny == "values":
        x, dy = x * SMALL, dy * SMALL
    else:
        w = w * SMALL
    y, da3 = torch.empty_like(dy), torch.empty_like(x)
    B.abl_conv_fwd(shape9(s), x, w, None, y)
    B.abl_conv_dgrad(shape9(s), dy, w, da3)
    # (outputs are rounded to multiples of 2^-149: 2^-29 of their size)
    assert rel(y, conv64(x, w)) < tolerance(R * R * ci)
    assert rel(da3, conv64(dy, grad_weights(w))) < tolerance(R * R * co)
    if tiny == "weights" and R == 3 and B.abl_forward_is_fused(shape9(s), 4):
        stats = torch.empty(32 * ci, dtype=torch.uint8, device="cuda")
        packed = torch.empty(B.abl_packed_bytes(shape9(s), 4), dtype=torch.uint8, device="cuda")
        scratch = torch.empty(B.abl_scratch_bytes(shape9(s), 4), dtype=torch.uint8, device="cuda")
        ones, a3 = torch.ones(ci, device="cuda"), torch.empty_like(x)
        B.abl_forward(shape9(s), 4, x, w, ones, ones * 0, None, scratch, y, packed, stats)
        B.abl_bn_relu_pack(x, x.numel() // ci, ci, 4, stats, a3, packed)
        assert rel(y, conv64(a3, w)) < tolerance(R * R * ci)


def assert_same_kind(got, ref64):
    """NaN, infinities and finite values where the 64-bit values have them (positive terms: no cancellation)."""
    ref = ref64.float()
    edge = (ref64.abs() > 3.3e38) & (ref64.abs() < 3.5e38)   # (within a rounding of the largest value either way)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isinf(got)[~edge], torch.isinf(ref)[~edge])
    ok = torch.isfinite(ref) & ~edge
    assert float(((got - ref)[ok].abs() / ref[ok].abs().clamp(min=1e-30)).max()) < 1e-5


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", [SHAPES[1], SHAPES[5], SHAPES[8], SHAPES[10]], ids=lambda s: "x".join(map(str, s)))
def test_gradients_the_split_cannot_carry(s, K):
    """... in the data gradient (other indexing of the weights than the forward), and ahead of the sums of its epilogue."""
    print("case split operands, gradient not finite", s, K, flush=True)
    x, w, dy = draw(s)
    N, H, W, ci, co, R = s
    s9, M = shape9(s), N * H * W
    dy, w = dy.abs() + 0.5, w.abs() + 0.01
    w[:, :, 1] = 2.0 ** -20          # keeps the largest values finite
    w[:, :, 2] = 0.0                 # infinity times zero
    w[0, 0, 3, 6] = float("inf")
    dy[0, 0, 0, 5] = float("inf")
    dy[-1, -1, -1, 7] = float("nan")
    dy[N // 2, H // 2, W // 2, 9] = 3.4e38
    dy[0, -1, 0, 11] = -float("inf")
    da3 = torch.empty_like(x)
    B.abl_conv_dgrad(s9, dy, w, da3)
    assert_same_kind(da3, conv64(dy, grad_weights(w)))
    stats = torch.empty(32 * ci, dtype=torch.uint8, device="cuda")
    packed = torch.empty(B.abl_packed_bytes(s9, K), dtype=torch.uint8, device="cuda")
    scratch = torch.empty(B.abl_scratch_bytes(s9, K), dtype=torch.uint8, device="cuda")
    a3, a2t, ones = torch.empty_like(x), torch.empty_like(x), torch.ones(ci, device="cuda")
    B.abl_bn_stats(x, M, ci, ones, ones * 0.1, K, scratch, stats)
    B.abl_bn_relu_pack(x, M, ci, K, stats, a3, packed)
    B.abl_unpack(packed, M, ci, K, stats, a2t)
    dx, dW, dg, db = torch.empty_like(x), torch.empty_like(w), torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")

    def sums():
        B.abl_backward(s9, K, packed, stats, dy, w, scratch, dx, dW, dg, db)
        B.abl_conv_dgrad(s9, dy, w, da3)
        return torch.where(a2t > 0, da3, torch.zeros_like(da3)).double().view(M, ci).sum(0)

    ref = sums()
    assert torch.equal(torch.isnan(db), torch.isnan(ref)) and torch.equal(torch.isfinite(db), torch.isfinite(ref.float()))
    assert not bool(torch.isfinite(dg)[~torch.isfinite(ref)].any())
    # a value that rounds to an infinite bf16, times small weights: everything stays finite
    dy = torch.rand(dy.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4)) + 0.5
    dy[N // 2, H // 2, W // 2, 9] = 3.4e38
    w = w.clamp(max=1.0)
    w[..., 9] = 2.0 ** -20
    ref = sums()
    a1 = (a2t.double().view(M, ci) - 0.1)
    ref_g = (a1 * torch.where(a2t > 0, da3, torch.zeros_like(da3)).double().view(M, ci)).sum(0)
    for got, want in ((db, ref), (dg, ref_g)):
        assert bool(torch.isfinite(got).all())
        assert float((got - want).abs().max()) <= 1e-5 * float(want.abs().max())


@pytest.mark.parametrize("s", [SHAPES[4], SHAPES[5]], ids=lambda s: "x".join(map(str, s)))
def test_fused_forward_with_weights_the_split_cannot_carry(s):
    """... in the forward that normalises while it stages, which computes such outputs from x itself."""
    print("case split operands, fused forward not finite", s, flush=True)
    x, w, _ = draw(s)
    N, H, W, ci, co, R = s
    s9 = shape9(s)
    assert B.abl_forward_is_fused(s9, 4)
    w = w.abs() + 0.01
    w[0, 0, 3, 1] = float("inf")
    w[1, 2, 4, 2] = float("nan")
    w[2, 1, 5, 3] = 3.4e38
    w[1, 1, 6, 4] = -float("inf")
    g = torch.Generator(device="cuda").manual_seed(2)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, torch.rand(ci, device="cuda", generator=g) * 0.2
    stats = torch.empty(32 * ci, dtype=torch.uint8, device="cuda")
    packed = torch.empty(B.abl_packed_bytes(s9, 4), dtype=torch.uint8, device="cuda")
    scratch = torch.empty(B.abl_scratch_bytes(s9, 4), dtype=torch.uint8, device="cuda")
    y, a3 = torch.empty(N, H, W, co, device="cuda"), torch.empty_like(x)
    B.abl_forward(s9, 4, x, w, gamma, beta, None, scratch, y, packed, stats)
    B.abl_bn_relu_pack(x, N * H * W, ci, 4, stats, a3, packed)
    assert_same_kind(y, conv64(a3, w))


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", [SHAPES[3], SHAPES[4], SHAPES[5], SHAPES[7], SHAPES[6], (20, 28, 28, 64, 256, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_fused_stage_is_the_layers_kernel(s, K):
    """Where abl_forward_is_fused answers 1, abl_bn_conv_fwd runs what abl_forward runs: the same output, bit for bit."""
    print("case split operands, fused stage", s, K, flush=True)
    x, w, skip = draw(s)
    N, H, W, ci, co, R = s
    s9 = shape9(s)
    assert B.abl_forward_is_fused(s9, K)
    g = torch.Generator(device="cuda").manual_seed(2)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, torch.randn(ci, device="cuda", generator=g) * 0.1

    def raw(n):
        return torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")

    y, packed, stats = torch.empty_like(skip), raw(B.abl_packed_bytes(s9, K)), raw(32 * ci)
    B.abl_forward(s9, K, x, w, gamma, beta, skip, raw(B.abl_scratch_bytes(s9, K)), y, packed, stats)
    y2, packed2 = torch.empty_like(skip), raw(B.abl_packed_bytes(s9, K))
    B.abl_bn_conv_fwd(s9, K, x, stats, w, skip, y2, packed2)
    assert torch.equal(y, y2) and torch.equal(packed, packed2)


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("s", [SHAPES[1], (128, 8, 8, 64, 64, 3), (16, 14, 14, 256, 256, 3), (12, 20, 20, 64, 128, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_forward_with_the_pack_pass_in_front(s, K):
    """3x3 layers whose plain convolution runs on split operands and whose fused one would run on the halo kernel: the
    layer is the pack pass and the plain convolution, bit for bit; the fused stage still takes them."""
    print("case split operands, pass in front", s, K, flush=True)
    x, w, skip = draw(s)
    N, H, W, ci, co, R = s
    s9, M = shape9(s), N * H * W
    assert not B.abl_forward_is_fused(s9, K)
    assert B.abl_split_products(s9, K, "conv_fwd") == 6 and B.abl_split_products(s9, K, "bn_conv_fwd") == 0
    g = torch.Generator(device="cuda").manual_seed(2)
    gamma, beta = torch.rand(ci, device="cuda", generator=g) + 0.5, torch.randn(ci, device="cuda", generator=g) * 0.1

    def raw(n):
        return torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")

    y, packed, stats = torch.empty_like(skip), raw(B.abl_packed_bytes(s9, K)), raw(32 * ci)
    B.abl_forward(s9, K, x, w, gamma, beta, skip, raw(B.abl_scratch_bytes(s9, K)), y, packed, stats)
    a3, packed2, y2 = torch.empty_like(x), raw(B.abl_packed_bytes(s9, K)), torch.empty_like(skip)
    B.abl_bn_relu_pack(x, M, ci, K, stats, a3, packed2)
    B.abl_conv_fwd(s9, a3, w, skip, y2)
    assert torch.equal(packed, packed2) and torch.equal(y, y2)
    ref = conv64(a3, w) + skip.double()
    assert rel(y, ref) < tolerance(9 * ci)
    y3, packed3 = torch.empty_like(skip), raw(B.abl_packed_bytes(s9, K))
    B.abl_bn_conv_fwd(s9, K, x, stats, w, skip, y3, packed3)
    assert torch.equal(packed, packed3)
    # (fp32 matrix cores: rounded at every fourth term, twice that for sums of several partial ones)
    assert rel(y3, ref) < 2.0 ** -23 * ((9 * ci / 4) ** 0.5 + 2)


@pytest.mark.parametrize("s,stage,split", [
    ((20, 14, 14, 1024, 512, 1), "conv_fwd", True),     # 280 four-wave blocks: 140 of eight waves and 128 channels instead
    ((10, 29, 29, 256, 512, 1), "conv_dgrad", True),    # 304, its tiles of 128 pixels do not fit one round
    ((12, 13, 13, 1024, 1024, 1), "conv_dgrad", False), # 304, they do
    ((44, 14, 14, 256, 256, 1), "conv_fwd", True),      # 308, they do not: four waves
    ((20, 27, 27, 256, 128, 1), "conv_fwd", False),     # 262, they do
    ((18, 20, 20, 128, 512, 1), "conv_fwd", True),      # 260 blocks of 128 channels
    ((32, 16, 16, 64, 512, 1), "conv_fwd", False),      # 296 of 128 channels, 64 to contract
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_grids_a_little_over_a_round(s, stage, split):
    """1x1 layers on a little more four-wave blocks than compute units: the kernel that they take and its result."""
    print("case split operands, a little over a round", s, stage, flush=True)
    assert B.abl_split_products(shape9(s), 4, stage) == (6 if split else 0)
    x, w, dy = draw(s)
    if stage == "conv_fwd":
        out, ref, terms = torch.empty_like(dy), conv64(x, w), s[3]
        B.abl_conv_fwd(shape9(s), x, w, None, out)
    else:
        out, ref, terms = torch.empty_like(x), conv64(dy, grad_weights(w)), s[4]
        B.abl_conv_dgrad(shape9(s), dy, w, out)
    # (fp32 matrix cores: rounded at every fourth term, twice that for sums of several partial ones)
    assert rel(out, ref) < (tolerance(terms) if split else 2.0 ** -23 * ((terms / 4) ** 0.5 + 2))
