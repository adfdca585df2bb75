"""The matrix products choose their tile by a rule on sizes.  Whatever the tile, an element is the same sum in the same
order, so the first rows of a product have the bits of the product of those rows -- at sizes that between them take every
tile of the rule, with ragged last tiles and one, two, three and seven slabs of K."""
import os
import sys
import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import synth
import tile_rules as T
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


# Plain problems of enough tiles take 256 x 256, whose tiles at the edges overlap their neighbours: by all rows but one (32513 = 127 * 256
# + 1), by one row and 32 columns, by one row and half the columns.  Smaller numbers of rows take other tiles.
@pytest.mark.parametrize("n,k,rows", [(512, 768, (32513, 8193, 300)), (480, 896, (30207, 2000, 1)), (640, 768, (21759, 9000, 77))])
def test_overlapping_tiles_give_the_same_bits(model, n, k, rows):
    takes = [T.exact_tile(1, m, n, k, wide=T.wide_ok(m, n, k, n)) == T.TILE_256x256 for m in rows]
    assert takes == [True, False, False] and T.tiles(1, rows[0], n, 256, 256) <= 256
    test_every_tile_gives_the_same_bits(model, n, k, rows)


@pytest.fixture(scope="module")
def roomy():
    import paper_2510_23264_amd as P
    shape = synth.ModelShape(n_layers=1, n_heads=4, d_head=64, d_model=256, d_mlp=256, vocab=4096, n_ctx=16, act=1)
    gm = P.Model(shape, synth.make_weights(shape, 1, std=0.02), 8, 16, max_batch_edges=2048)
    yield gm
    gm.close()


# From 257 such tiles on a workgroup takes several: the next one's slabs and scales are on their way during the epilogue, and with
# an odd number of slabs the stages swap roles from tile to tile.  Five and seven slabs, and two (a tile's scales arrive with the
# last of its slabs).
@pytest.mark.parametrize("n,k,rows", [(512, 640, (70000, 3000)), (480, 896, (65537, 8193)), (416, 256, (82811, 5000))])
def test_several_tiles_of_a_workgroup_give_the_same_bits(roomy, n, k, rows):
    takes = [T.exact_tile(1, m, n, k, wide=T.wide_ok(m, n, k, n)) == T.TILE_256x256 for m in rows]
    assert takes == [True, False] and T.tiles(1, rows[0], n, 256, 256) > 256
    test_every_tile_gives_the_same_bits(roomy, n, k, rows)


# The MLP's products of a full batch, their number of 256 x 256 tiles (0: other tiles) and slabs: without a residual (input) and with
# one (output), one tile a workgroup or several, even and odd numbers of slabs, codes and bfloat16, two slabs.
@pytest.mark.parametrize("d,m,batch,options,products", [
    (512, 1280, 224, dict(), ((530, 4), (0, 10))), (512, 1280, 224, dict(nonattn_bf16=True), ((530, 8), (212, 20))),
    (768, 1408, 400, dict(), ((1128, 6), (564, 11))), (768, 1344, 400, dict(nonattn_bf16=True), ((1128, 12), (564, 21))),
    (128, 768, 400, dict(nonattn_bf16=True), ((564, 2), (0, 12)))])
def test_scores_do_not_depend_on_the_tile_of_a_batch(d, m, batch, options, products):
    """The candidates' rows (position 0 is shared), with 24 and with one of them in other tiles."""
    import paper_2510_23264_amd as P
    B, S, V = 8, 16, 600
    b16 = bool(options)
    for n in (batch, 24, 1):
        rows = B + n * 120 if n > 1 else B * S
        for (cols, k, residual), (want, slabs) in zip(((m, d, False), (d, m, True)), products):
            k = -(-k * (1 + b16) // 128) * 128
            assert k == 128 * slabs
            takes = T.exact_tile(1, rows, cols, k, b16=b16, wide=T.wide_ok(rows, cols, k, cols), residual=residual) == T.TILE_256x256
            assert (T.tiles(1, rows, cols, 256, 256) if takes else 0) == (want if n == batch else 0)
    shape = synth.ModelShape(n_layers=2, n_heads=4, d_head=64, d_model=d, d_mlp=m, vocab=V, n_ctx=S, act=1)
    w = synth.make_weights(shape, 6, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(6)
    clean = rng.integers(0, V, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:6] = (clean[:, 1:6] + 1 + rng.integers(0, V - 1, (B, 5))) % V
    out = []
    for n in (batch, 24, 1):
        gm = P.Model(shape, w, B, S, max_batch_edges=n, **options)
        try:
            gm.clean_cache(clean, corrupt)
            r = 3 * 4
            before = gm.counters()[1]
            out.append(gm.eval_edges(r, np.resize(np.arange(P.n_upstream(gm.cfg, r), dtype=np.int32), batch)[:n]))
            assert gm.counters()[1] == before + 1
        finally:
            gm.close()
    for got in out:
        assert np.isfinite(got).all() and np.array_equal(got.view(np.uint32), out[0][:got.size].view(np.uint32))


@pytest.mark.parametrize("options", [dict(), dict(nonattn_bf16=True), dict(low_bits=16)])
def test_scores_across_the_tiles_of_one_and_two_bytes(options):
    """Scores by batch where the same layer's products take other tiles, in one-byte codes and in bfloat16: with 48, 24 and 1
    candidates the first MLP's input product has 5768, 2888 and 128 rows of 1280 columns (128 x 128, 64 x 128, 32 x 64; its output
    product 64 x 64 and 32 x 64), and the unembedding with the KL epilogue 384, 192 and 8 rows of 20001 (128 x 128, then
    64 x 128)."""
    import paper_2510_23264_amd as P
    B, S, V = 8, 16, 20001
    shape = synth.ModelShape(n_layers=2, n_heads=4, d_head=64, d_model=512, d_mlp=1280, vocab=V, n_ctx=S, act=1)
    w = synth.make_weights(shape, 5, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(5)
    clean = rng.integers(0, V, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:6] = (clean[:, 1:6] + 1 + rng.integers(0, V - 1, (B, 5))) % V      # position 0 is shared
    out = []
    for batch in (48, 24, 1):
        gm = P.Model(shape, w, B, S, max_batch_edges=batch, **options)
        try:
            gm.clean_cache(clean, corrupt)
            r = 3 * 4                                   # the first layer's MLP input: every row of it is a candidate's own
            senders = np.resize(np.arange(P.n_upstream(gm.cfg, r), dtype=np.int32), 48)[:batch]
            before = gm.counters()[1]
            out.append(gm.eval_edges(r, senders))
            assert gm.counters()[1] == before + 1
        finally:
            gm.close()
    for got in out:
        assert np.isfinite(got).all() and np.array_equal(got.view(np.uint32), out[0][:got.size].view(np.uint32))
