"""pahq_get_sender_output hands out a cached tile, [sequence][position][d_model], whatever the order its rows are held in."""
import ctypes as C

import numpy as np
import pytest

import synth
from synth import ModelShape

pytestmark = pytest.mark.gpu


def _status(field):
    with open("/proc/self/status") as f:
        return next(int(line.split()[1]) for line in f if line.startswith(field + ":")) * 1024


def test_a_tile_needs_no_second_copy_on_the_host():
    """Straight into the caller's buffer: the call may not hold another tile of host memory (a failed allocation would end the
    process, the library being C to its callers).  The peak resident size shows one, once the present size has been
    raised to the peak of what ran before.  Prompts that differ from different positions on: the rows are permuted."""
    import paper_2510_23264_amd as P
    B, S, d = 128, 64, 1024                              # a tile of 32 MiB
    shape = ModelShape(n_layers=1, n_heads=2, d_head=16, d_model=d, d_mlp=0, vocab=97, n_ctx=S, act=0)
    w = synth.make_weights(shape, 3, std=0.05, affine_std=0.1)
    rng = np.random.default_rng(3)
    clean = rng.integers(0, 97, (B, S)).astype(np.int32)
    corrupt = clean.copy()
    corrupt[np.arange(B), rng.integers(0, S - 1, B)] = rng.integers(0, 97, B)
    gm = P.Model(shape, w, B, S, max_batch_edges=1)
    try:
        gm.clean_cache(clean, corrupt)
        out = np.zeros((B, S, d), np.float32)
        ptr = out.ctypes.data_as(C.POINTER(C.c_float))
        assert P.lib().pahq_get_sender_output(gm.h, 0, 0, ptr) == 0        # staging of the runtime is set up
        out.fill(-1.0)
        ballast = np.ones(max(0, _status("VmHWM") - _status("VmRSS")) // 8 + (1 << 17))
        before = _status("VmHWM")
        assert before - _status("VmRSS") < out.nbytes // 8
        assert P.lib().pahq_get_sender_output(gm.h, 0, 0, ptr) == 0
        assert _status("VmHWM") - before < out.nbytes // 2
        assert ballast[-1] == 1.0
        want = w["W_E"][clean] + w["W_pos"][None, :S]
        assert np.array_equal(out, want)
    finally:
        gm.close()
