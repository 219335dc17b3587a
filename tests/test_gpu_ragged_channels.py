"""Layers whose channel counts are not multiples of 16 (the gathered-tile kernels) against the oracle, at the
edges of their tiles: 64 rows, 16 to 64 columns, 32-deep chunks of the flattened (tap, channel) index, 32-pixel
chunks and their shares in the weight gradient.  TOL: fp32 products, sums of at most N Ho Wo terms."""
import pytest

from paper_1901_07988_amd import synth
from paper_1901_07988_amd.synth import LayerShape

from tests.test_gpu_parity import TOL, oshape, rel, G  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    LayerShape(1, 1, 1, 1, 1, 1, 1, 1, 0),           # one of everything
    LayerShape(2, 8, 4, 3, 17),                      # 64 rows exactly; one column past a tile
    LayerShape(3, 5, 13, 7, 15),                     # 195 rows; 63 rows of dW
    LayerShape(2, 9, 9, 32, 20),                     # one of the two counts a multiple of 16
    LayerShape(2, 9, 9, 20, 48),
    LayerShape(4, 11, 7, 33, 31, 1, 1, 1, 0),        # 33 of a chunk of 32
    LayerShape(3, 10, 11, 12, 50, 3, 3, 2, 1),       # strided: taps that reach every other pixel
    LayerShape(2, 10, 11, 5, 65, 3, 3, 3, 0),        # two column tiles, no padding
    LayerShape(2, 9, 10, 9, 36, 5, 5, 1, 2),
    LayerShape(30, 21, 27, 20, 36),                  # several shares of the pixels
]


@pytest.mark.parametrize("K", [4, 8, 32])
@pytest.mark.parametrize("s", SHAPES, ids=lambda s: "x".join(map(str, s.as_tuple())))
def test_layer_with_any_channel_count(G, oracle, s, K):
    o = oracle
    print("case ragged layer", s.as_tuple(), K, flush=True)
    x, w, gamma, beta, dy = synth.draw_layer(s, 5, "normal", "random")
    run = G.LayerRun(s, K)
    y = run.forward(x, w, gamma, beta)
    y_ref, saved = o.layer_forward(x, w, gamma, beta, K, oshape(o, s))
    n = saved.store.size * saved.store.itemsize
    assert run.packed.cpu().numpy().tobytes()[:n] == saved.store.tobytes()
    ref = o.layer_backward(saved, dy, w)
    got = run.backward(dy, w)
    assert rel(y, y_ref) < TOL
    if s.M > 1:   # (one row: the normalized input and its gradient are zero up to rounding)
        for a, b in zip(got, ref):
            assert rel(a, b) < TOL
