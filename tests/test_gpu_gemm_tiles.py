"""The matrix products choose their tile by a rule on sizes.  Whatever the tile, an element is the same sum in the same
order, so the first rows of a product have the bits of the product of those rows -- at sizes that between them take every
tile of the rule, with ragged last tiles and one, two, three and seven slabs of K."""
import numpy as np
import pytest

import synth
from test_gpu_hooks import exact_and_scale, random_codes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def model():
    import paper_2510_23264_amd as P
    shape = synth.ModelShape(n_layers=1, n_heads=4, d_head=64, d_model=256, d_mlp=256, vocab=4096, n_ctx=16, act=1)
    gm = P.Model(shape, synth.make_weights(shape, 1, std=0.02), 8, 16, max_batch_edges=512)     # room for the products
    yield gm
    gm.close()


#                              tiles taken, in turn
@pytest.mark.parametrize("n,k,rows", [
    (500, 384, (24500, 16300, 8150, 2040, 33, 1)),      # 128 x 128, 256 x 128, 64 x 128, 64 x 64, 32 x 64 twice
    (60, 256, (65500, 8200, 4000, 1)),                  # 128 x 64, 64 x 64, 32 x 64 twice
    (257, 128, (24500, 2000, 70)),
    (130, 896, (3000, 300)),
    (960, 1536, (7500, 5100, 40))])                     # 128 x 128 (at K <= 1024 it would be 64 x 64), 64 x 128, 32 x 64
def test_every_tile_gives_the_same_bits(model, n, k, rows):
    rng = np.random.default_rng(n + k)
    a, w = random_codes(rng, rows[0], k), random_codes(rng, n, k)
    out = [model.gemm_codes(a[:m], w) for m in rows]
    for m, got in zip(rows[1:], out[1:]):
        assert np.array_equal(got.view(np.uint32), out[0][:m].view(np.uint32)), (m, n, k)
    ends = np.r_[0:40, rows[0] - 40:rows[0]]
    exact, mag = exact_and_scale(a[ends], w)
    assert (np.abs(out[0][ends] - exact) <= k * 2.0 ** -24 * mag).all()      # k additions of binary32
