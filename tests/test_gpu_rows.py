"""The rows a pass computes: the last layer at the last position only, and -- for the candidates of a batch -- the rows
at which the two prompts cannot differ once for all of them.  Sizes at which that can go wrong: one layer (the first is
the last), one position, one sequence, tiles of 16 positions that end or begin with a shared row; prompts that differ
from the first position on, from the last but one, or nowhere."""
import os
import sys
import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import synth                                        # noqa: E402
from synth import ModelShape                        # noqa: E402
from oracle.acdc import Acdc, MODE_ALL_FP32         # noqa: E402
from oracle.model import Model as OModel, ALL       # noqa: E402
from test_gpu_modes import F32_ATOL, F32_RTOL, rnd_removed   # noqa: E402

pytestmark = pytest.mark.gpu

#       layers heads d_head d_mlp B  S  llama
SIZES = [(1, 3, 16, 96, 4, 7, 0), (1, 2, 64, 0, 3, 16, 0), (2, 2, 64, 132, 3, 17, 0), (2, 3, 32, 64, 1, 33, 0),
         (2, 2, 128, 96, 2, 5, 1), (2, 4, 64, 96, 5, 1, 0), (3, 2, 64, 68, 1, 70, 1)]
FIRST = {"start": lambda S, b: 0, "late": lambda S, b: max(0, S - 2), "mixed": lambda S, b: (5 * b + 3) % max(1, S - 1), "never": None}


def make(size, first, seed):
    L, H, dh, m, B, S, llama = size
    more = dict(norm=1, act=2, pos=1, norm_eps=1e-6) if llama else dict(act=1 if m else 0)
    shape = ModelShape(n_layers=L, n_heads=H, d_head=dh, d_model=128, d_mlp=m, vocab=211, n_ctx=S, **more)
    w = synth.make_weights(shape, seed, std=0.15, affine_std=0.1)
    rng = np.random.default_rng(seed)
    clean = rng.integers(0, shape.vocab, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    if FIRST[first]:
        for b in range(B):
            at = FIRST[first](S, b)
            corrupt[b, at] = (clean[b, at] + 1 + rng.integers(0, shape.vocab - 1)) % shape.vocab
            for s in range(at + 1, S - 1):
                if rng.random() < 0.3:
                    corrupt[b, s] = rng.integers(0, shape.vocab)
    return shape, w, clean, corrupt


@pytest.mark.parametrize("first", sorted(FIRST))
@pytest.mark.parametrize("size", SIZES)
def test_against_the_oracle(size, first):
    """Nothing quantised: every edge of the graph, on the whole graph and on a pruned one, to rounding."""
    import paper_2510_23264_amd as P
    shape, w, clean, corrupt = make(size, first, 3)
    gm = P.Model(shape, w, *clean.shape, precision=P.ALL_FP32, max_batch_edges=5)
    try:
        gm.clean_cache(clean, corrupt)
        om = OModel(shape, w)
        g, oa = om.g, Acdc(om, clean, corrupt, MODE_ALL_FP32)
        for frac in (0.0, 0.5):
            for r in range(g.n_receivers):
                R = rnd_removed(g, frac, 100 + r, r)
                gm.set_removed(g.removed_to_flat(R).astype(np.uint8))
                got = gm.eval_edges(r, np.arange(g.n_upstream(r), dtype=np.int32))
                want = np.array([oa.kl_edge(r, u, removed=R) for u in range(g.n_upstream(r))])
                assert (np.abs(got - want) <= F32_ATOL + F32_RTOL * np.abs(want)).all(), (size, first, frac, r)
        gm.set_removed(np.zeros(g.n_edges(), np.uint8))
        s = g.n_senders - 1
        a = gm.get_sender_output(1, s)
        b = om.forward(corrupt, ALL)[0][s].reshape(a.shape)
        assert np.abs(a - b).max() <= 1e-4 * np.abs(b).max()
    finally:
        gm.close()


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("options", [dict(), dict(precision=1), dict(low_bits=4), dict(nonattn_bf16=True), dict(split_qkv=False), dict(mma=0)])
def test_a_score_does_not_depend_on_its_batch(size, options):
    """Quantised modes: a candidate's bits are the same alone (where every row is its own) and at any place in a batch."""
    import paper_2510_23264_amd as P
    shape, w, clean, corrupt = make(size, "mixed", 4)
    out = []
    for batch in (1, 7):
        gm = P.Model(shape, w, *clean.shape, max_batch_edges=batch, **options)
        try:
            gm.clean_cache(clean, corrupt)
            res, rng = [], np.random.default_rng(1)
            for r in range(P.n_receivers(gm.cfg)):
                first = sum(P.n_upstream(gm.cfg, q) for q in range(r))
                state = (rng.random(gm.n_edges) < (0.5 if r % 2 else 0.0)).astype(np.uint8)
                state[:first] = 0
                gm.set_removed(state)
                n = P.n_upstream(gm.cfg, r)
                got = np.empty(n, np.float32)
                order = np.arange(n, dtype=np.int32) if batch == 1 else rng.permutation(n).astype(np.int32)
                got[order] = gm.eval_edges(r, order)
                res.append(got)
                res.append(np.float32([gm.eval_current(r)]))
                if batch == 1:
                    rng.permutation(n)
            out.append(np.concatenate(res))
        finally:
            gm.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32)), (size, options)


@pytest.mark.parametrize("d", [64, 256, 320, 768, 960, 1024, 1088, 1280, 2112, 2304])
def test_gathered_inputs_by_width_and_number_of_terms(d):
    """A receiver's input is the stream and a sum of terms, of which as many as a row's registers allow are loaded ahead once
    a group has that many: rows of every width the kernels distinguish, with the first 0 to 7 of the edges into every receiver
    from the third layer's second head on gone, against the oracle."""
    import paper_2510_23264_amd as P
    shape = ModelShape(n_layers=4, n_heads=3, d_head=16, d_model=d, d_mlp=0, vocab=61, n_ctx=6, act=0)
    w = synth.make_weights(shape, 9, std=1.2 / d ** 0.5, affine_std=0.1)
    rng = np.random.default_rng(d)
    clean = rng.integers(0, 61, (3, 6)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[:, 1:4] = (clean[:, 1:4] + 1 + rng.integers(0, 60, (3, 3))) % 61
    gm = P.Model(shape, w, 3, 6, precision=P.ALL_FP32, max_batch_edges=4)
    try:
        gm.clean_cache(clean, corrupt)
        om = OModel(shape, w)
        g, oa = om.g, Acdc(om, clean, corrupt, MODE_ALL_FP32)
        for gone in (0, 1, 2, 3, 4, 5, 7):
            r = g.headin(2, 1, 0)
            R = g.empty_removed()
            for q in range(r, g.n_receivers):
                R[q, :min(gone, g.n_upstream(q))] = True
            gm.set_removed(g.removed_to_flat(R).astype(np.uint8))
            senders = np.array([0, 3, 6], np.int32)
            got = gm.eval_edges(r, senders)
            want = np.array([oa.kl_edge(r, int(u), removed=R) for u in senders])
            assert (np.abs(got - want) <= F32_ATOL + F32_RTOL * np.abs(want)).all(), (d, gone)
    finally:
        gm.close()


@pytest.mark.parametrize("size", [(2, 2, 64, 132, 3, 17, 0), (3, 2, 64, 68, 2, 70, 1), (2, 3, 32, 64, 1, 33, 0)])
@pytest.mark.parametrize("options", [dict(), dict(precision=0), dict(nonattn_bf16=True)])
def test_one_handle_with_one_prompt_pair_after_another(size, options):
    """The order of a tile's rows belongs to the prompt pair: a handle that has seen other pairs, with other first changes, gives
    the bits of a fresh one -- scores, a circuit's logits and the cached outputs."""
    import paper_2510_23264_amd as P

    def everything(gm, clean, corrupt):
        gm.clean_cache(clean, corrupt)
        res, rng = [gm.get_sender_output(0, 1).ravel(), gm.get_sender_output(1, P.n_senders(gm.cfg) - 1).ravel(), gm.get_logits(1).ravel()], np.random.default_rng(2)
        for r in (P.n_receivers(gm.cfg) - 1, P.n_receivers(gm.cfg) // 2, 0):
            state = (rng.random(gm.n_edges) < 0.4).astype(np.uint8)
            state[:sum(P.n_upstream(gm.cfg, q) for q in range(r))] = 0
            gm.set_removed(state)
            res.append(gm.eval_edges(r, np.arange(P.n_upstream(gm.cfg, r), dtype=np.int32)))
        kl, logits = gm.eval_circuit(kept=(rng.random(gm.n_edges) < 0.5).astype(np.uint8), want_logits=True)
        return np.concatenate(res + [np.float32([kl]), np.asarray(logits, np.float32).ravel()])

    pairs = [make(size, first, seed)[2:] for first, seed in (("late", 5), ("start", 6), ("mixed", 7), ("never", 8), ("mixed", 9), ("late", 5))]
    shape, w = make(size, "late", 5)[:2]
    used = P.Model(shape, w, *pairs[0][0].shape, max_batch_edges=5, **options)
    try:
        for clean, corrupt in pairs:
            fresh = P.Model(shape, w, *clean.shape, max_batch_edges=5, **options)
            try:
                want, got = everything(fresh, clean, corrupt), everything(used, clean, corrupt)
            finally:
                fresh.close()
            assert np.isfinite(want).all() and np.array_equal(got.view(np.uint32), want.view(np.uint32))
    finally:
        used.close()
