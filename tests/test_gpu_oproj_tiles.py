"""The fused output projection takes tiles of 32 rows where those of 128 would leave compute units idle.  Either way an
element is the same sum: a candidate scores the same bits alone and in a batch whose layers take the other tile."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


#                          heads d_head d_model options; up to 48 * 15 * 8 rows, 128-row tiles from 256 of them on
@pytest.mark.parametrize("H,dh,d,options", [(8, 64, 512, {}), (3, 128, 704, {}), (4, 64, 448, dict(low_bits=16)), (6, 32, 640, dict(low_bits=16)),
                                            (4, 64, 512, dict(low_bits=4))])
def test_scores_by_batch(H, dh, d, options):
    import paper_2510_23264_amd as P
    B, S = 8, 16
    shape = synth.ModelShape(n_layers=3, n_heads=H, d_head=dh, d_model=d, d_mlp=256, vocab=300, n_ctx=S, act=1)
    w = synth.make_weights(shape, 5, std=0.08, affine_std=0.1)
    rng = np.random.default_rng(5)
    clean = rng.integers(0, 300, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:6] = rng.integers(0, 300, (B, 5))
    out = []
    for batch in (48, 1):
        gm = P.Model(shape, w, B, S, max_batch_edges=batch, **options)
        try:
            gm.clean_cache(clean, corrupt)
            r = 3 * H + 1 + 1                          # an input of the second layer's first head
            n = P.n_upstream(gm.cfg, r)
            out.append(gm.eval_edges(r, np.resize(np.arange(n, dtype=np.int32), 48)))
        finally:
            gm.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))
