"""The fused output projection takes tiles of 32 rows where those of 128 would leave compute units idle.  Either way an
element is the same sum: a candidate scores the same bits alone and in batches whose layers take the other tile.

The receiver is the MLP input of the first of three layers.  Its candidates run the second layer in full, all rows and all
heads in one fused projection: 8 + n * 15 * 8 rows, position 0 being equal in both prompts of all eight pairs.  (A head's
input would be no use: the heads beside it are computed for one instance.  Nor the last layer: it has eight rows a candidate.)"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def takes_128_rows(rows, H, dh, d, options):
    """The rule of launch_oproj_x, by tiles of 128 x 64 and slabs of 128 bytes."""
    b16 = options.get("low_bits") == 16
    slabs = H * dh * (2 if b16 else 1) // 128
    limit = 256 if slabs < (4 if b16 else 8) else 192 if not b16 or slabs < 12 else 128
    return -(-rows // 128) * -(-d // 64) >= limit


#                          heads d_head d_model options, batches on either side of the rule's limit
@pytest.mark.parametrize("H,dh,d,options,batches", [
    (16, 64, 512, {}, (25, 24)), (2, 128, 704, {}, (25, 24)), (3, 128, 704, {}, (25, 24)), (4, 64, 448, dict(low_bits=4), (39, 38)),
    (4, 64, 448, dict(low_bits=16), (29, 28)), (6, 32, 640, dict(low_bits=16), (27, 26)), (14, 64, 512, dict(low_bits=16), (16, 15))])
def test_scores_by_batch(H, dh, d, options, batches):
    B, S = 8, 16
    large, small = batches
    assert takes_128_rows(B + large * (S - 1) * B, H, dh, d, options)
    assert not takes_128_rows(B + small * (S - 1) * B, H, dh, d, options) and not takes_128_rows(B * S, H, dh, d, options)
    same_scores(H, dh, d, options, (large, small, 1))


def takes_128_columns(rows, d):
    """The rule of launch_oproj_x for tiles of 128 x 128."""
    def rounds(bn):
        t = -(-rows // 128) * -(-d // bn) / 512
        return 0.5 * (-(-t // 1) + t)
    return 0.4 + 1.5 * rounds(128) <= rounds(64)


#                    whole tiles across; half a tile over; one head a slab; bfloat16 of 64 and of 128 bytes
@pytest.mark.parametrize("H,dh,d,options,large", [
    (8, 64, 512, {}, 128), (4, 64, 704, {}, 160), (3, 128, 704, {}, 160), (6, 32, 640, dict(low_bits=16), 176), (3, 64, 512, dict(low_bits=16), 128)])
def test_scores_by_batch_in_wide_tiles(H, dh, d, options, large):
    assert takes_128_columns(8 + large * 120, d) and not takes_128_columns(8 + 24 * 120, d)
    same_scores(H, dh, d, options, (large, 24, 1))


# The middle layer's first head and last one feed nobody: the projection leaves them out (their codes are what an earlier pass
# left) and adds the corrupted run's outputs in their place.
@pytest.mark.parametrize("H,dh,d,options,large", [
    (8, 64, 512, {}, 128), (3, 128, 704, {}, 160), (6, 32, 640, dict(low_bits=16), 176), (3, 64, 512, dict(low_bits=16), 128)])
def test_dead_heads_in_wide_tiles(H, dh, d, options, large):
    assert takes_128_columns(8 + large * 120, d) and not takes_128_columns(8 + 24 * 120, d)
    same_scores(H, dh, d, options, (large, 24, 1), dead=(0, H - 1))


def same_scores(H, dh, d, options, batches, dead=()):
    import paper_2510_23264_amd as P
    from oracle.graph import Graph
    B, S = 8, 16
    shape = synth.ModelShape(n_layers=3, n_heads=H, d_head=dh, d_model=d, d_mlp=256, vocab=300, n_ctx=S, act=1)
    w = synth.make_weights(shape, 5, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(5)
    clean = rng.integers(0, 300, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:6] = (clean[:, 1:6] + 1 + rng.integers(0, 299, (B, 5))) % 300
    g = Graph(3, H, True)
    removed = np.zeros((g.n_receivers, g.n_senders), bool)
    for h in dead:
        removed[list(g.receivers_downstream_of(g.head(1, h))), g.head(1, h)] = True
    out = []
    for batch in batches:
        gm = P.Model(shape, w, B, S, max_batch_edges=batch, **options)
        try:
            gm.clean_cache(clean, corrupt)
            if dead:
                gm.set_removed(g.removed_to_flat(removed).astype(np.uint8))
            r = 3 * H
            n = P.n_upstream(gm.cfg, r)
            senders = np.resize(np.arange(n, dtype=np.int32), batches[0])
            before = gm.counters()[1]
            out.append(gm.eval_edges(r, senders[:batch]))
            assert gm.counters()[1] == before + 1              # one device batch: the rows above
        finally:
            gm.close()
    for got in out:
        assert np.isfinite(got).all() and np.array_equal(got.view(np.uint32), out[0][:got.size].view(np.uint32))
