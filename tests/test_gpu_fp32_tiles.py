"""The fp32 products choose their tile by the number of tiles, and the output projections of a layer's fp32 heads are one
launch.  Whatever the tile, an element is the same sum in the same order: a candidate scores the same bits in batches that
take the smallest, the middle and the largest tile, and the scores are the oracle's.  An odd vocabulary takes the form that
loads single words of the unembedding, heads of 16 (four of them: K = 64 in, 16 out) the kernel for K not a multiple of 32."""
import os
import sys
import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import synth                                        # noqa: E402
import tile_rules as T                              # noqa: E402
from synth import ModelShape                        # noqa: E402
from oracle.acdc import Acdc, MODE_ALL_FP32         # noqa: E402
from oracle.model import Model as OModel            # noqa: E402
from test_gpu_modes import F32_ATOL, F32_RTOL       # noqa: E402

pytestmark = pytest.mark.gpu


#                          heads d_head d_model d_mlp vocab  removed
@pytest.mark.parametrize("H,dh,d,m,V,frac", [(8, 64, 512, 1024, 1031, 0.0), (8, 64, 512, 1024, 1028, 0.4), (3, 128, 320, 480, 515, 0.4),
                                             (4, 16, 64, 100, 67, 0.4), (5, 32, 192, 160, 300, 0.0)])
def test_fp32_scores_by_batch_and_against_the_oracle(H, dh, d, m, V, frac):
    import paper_2510_23264_amd as P
    B, S = 8, 16
    shape = ModelShape(n_layers=2, n_heads=H, d_head=dh, d_model=d, d_mlp=m, vocab=V, n_ctx=S, act=1)
    w = synth.make_weights(shape, 11, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(11)
    clean = rng.integers(0, V, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:5] = rng.integers(0, V, (B, 4))
    om = OModel(shape, w)
    g, oa = om.g, Acdc(om, clean, corrupt, MODE_ALL_FP32)
    r = g.headin(0, 1, 2)                            # a value input of the first layer: every later layer is recomputed
    r2 = g.headin(1, 0, 0)
    state = np.zeros(g.n_edges(), np.uint8)
    first = sum(g.n_upstream(q) for q in range(r2))
    state[first:] = rng.random(g.n_edges() - first) < frac
    out = []
    for batch in (40, 6, 1):
        gm = P.Model(shape, w, B, S, precision=P.ALL_FP32, max_batch_edges=batch)
        try:
            gm.clean_cache(clean, corrupt)
            a = gm.eval_edges(r, np.zeros(40, np.int32))
            gm.set_removed(state)
            n = g.n_upstream(r2)
            out.append(np.concatenate([a, gm.eval_edges(r2, np.resize(np.arange(n, dtype=np.int32), 40))]))
            n_up = n
        finally:
            gm.close()
    for got in out[1:]:
        assert np.array_equal(got.view(np.uint32), out[0].view(np.uint32))
    want = oa.kl_edge(r, 0)
    assert abs(out[0][0] - want) <= F32_ATOL + F32_RTOL * abs(want)
    if frac == 0.0:
        for u in range(n_up):
            want = oa.kl_edge(r2, u)
            assert abs(out[0][40 + u] - want) <= F32_ATOL + F32_RTOL * abs(want), u


# The MLP's products of the first layer: 68 candidates have 8168 rows, 20 have 2408, 1 has 128.  Slabs of 32: 10 and 32 of them
# (input, output), whole tiles of columns; 6 and 31, the last step of four not full, ragged columns and rows; 16 and 18 slabs of
# the input product in tiles of 128 x 128 (8168 rows), whole and ragged columns.
@pytest.mark.parametrize("H,dh,d,m", [(5, 64, 320, 1024), (6, 32, 192, 992), (8, 64, 512, 1024), (18, 32, 576, 992)])
def test_scores_in_large_tiles_and_in_steps_of_four_slabs(H, dh, d, m):
    import paper_2510_23264_amd as P
    B, S, V = 8, 16, 300
    large = [T.f32_tile(1, rows, m, d) == T.F32_128x128 for rows in (8 + 68 * 120, 8 + 20 * 120, 128)]
    assert large == [d >= 512, False, False]
    assert T.f32_tile(1, 128, d, m) in (T.F32_32x32_STEP4, T.F32_32x64_STEP4)
    shape = ModelShape(n_layers=2, n_heads=H, d_head=dh, d_model=d, d_mlp=m, vocab=V, n_ctx=S, act=1)
    w = synth.make_weights(shape, 13, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(13)
    clean = rng.integers(0, V, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:6] = (clean[:, 1:6] + 1 + rng.integers(0, V - 1, (B, 5))) % V      # position 0 is shared
    r = 3 * H                                        # the first layer's MLP input
    out = []
    for batch in (68, 20, 1):
        gm = P.Model(shape, w, B, S, precision=P.ALL_FP32, max_batch_edges=batch)
        try:
            gm.clean_cache(clean, corrupt)
            senders = np.resize(np.arange(P.n_upstream(gm.cfg, r), dtype=np.int32), 68)[:batch]
            before = gm.counters()[1]
            out.append(gm.eval_edges(r, senders))
            assert gm.counters()[1] == before + 1
        finally:
            gm.close()
    for got in out[1:]:
        assert np.array_equal(got.view(np.uint32), out[0][:got.size].view(np.uint32))
    om = OModel(shape, w)
    oa = Acdc(om, clean, corrupt, MODE_ALL_FP32)
    for u in (0, P.n_upstream(gm.cfg, r) - 1):
        want = oa.kl_edge(r, u)
        assert abs(out[0][u] - want) <= F32_ATOL + F32_RTOL * abs(want), u


# Receivers of the last layer no longer read some heads of the middle one: their outputs are wanted one by one, less the
# corrupted run's.  The middle layer's projections (N = d_model) take the three tiles by batch, with one slab a head and with two.
@pytest.mark.parametrize("H,dh,d,batches", [(8, 64, 512, (36, 12, 1)), (10, 32, 320, (60, 23, 1)), (4, 128, 448, (43, 14, 1))])
def test_second_outputs_of_heads_by_tile(H, dh, d, batches):
    import paper_2510_23264_amd as P
    B, S, V = 8, 16, 300
    tiles = [T.tiles(1, B + n * (S - 1) * B if n > 1 else B * S, d, 64, 64) for n in batches]
    assert tiles[0] >= 512 and 96 <= tiles[1] < 512 and tiles[2] < 96
    shape = ModelShape(n_layers=3, n_heads=H, d_head=dh, d_model=d, d_mlp=128, vocab=V, n_ctx=S, act=1)
    w = synth.make_weights(shape, 17, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(17)
    clean = rng.integers(0, V, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:6] = (clean[:, 1:6] + 1 + rng.integers(0, V - 1, (B, 5))) % V      # position 0 is shared
    om = OModel(shape, w)
    g, oa = om.g, Acdc(om, clean, corrupt, MODE_ALL_FP32)
    removed = g.empty_removed()
    for q in range(g.headin(2, 0, 0), g.n_receivers):
        removed[q, [g.head(1, h) for h in range(1, H)]] = rng.random(H - 1) < 0.4      # (head 0 keeps all its edges)
    r = 3 * H                                        # the first layer's MLP input
    n = g.n_upstream(r)
    out = []
    for batch in batches:
        gm = P.Model(shape, w, B, S, precision=P.ALL_FP32, max_batch_edges=batch)
        try:
            gm.clean_cache(clean, corrupt)
            gm.set_removed(g.removed_to_flat(removed).astype(np.uint8))
            before = gm.counters()[1]
            out.append(gm.eval_edges(r, np.resize(np.arange(n, dtype=np.int32), batches[0])[:batch]))
            assert gm.counters()[1] == before + 1    # one device batch: the rows above
        finally:
            gm.close()
    for got in out[1:]:
        assert np.array_equal(got.view(np.uint32), out[0][:got.size].view(np.uint32))
    assert np.array_equal(out[0][n:2 * n].view(np.uint32), out[0][:n].view(np.uint32))
    for u in (0, n - 1):
        want = oa.kl_edge(r, u, removed=removed)
        assert abs(out[0][u] - want) <= F32_ATOL + F32_RTOL * abs(want), u
