"""The tile rules of the matrix products, on the CPU: csrc/tile_rules.h compiled by itself, against the copy the GPU tests
use and against what its comments state."""
import os
import random
import shutil
import subprocess
import sys

import pytest

sys.path.insert(0, os.path.dirname(__file__))
import tile_rules as T                              # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "tile_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-I" + os.path.join(ROOT, "paper_2510_23264_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "tile_rules.cpp"), "-o", exe], check=True)

    def run(rule, launches):
        text = "".join(rule + " " + " ".join(map(str, q)) + "\n" for q in launches)
        out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()
        assert len(out) == len(launches)
        return [int(v) for v in out]
    return run


def log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def test_the_copy_of_the_fp32_rule_agrees(pick):
    rng = random.Random(3)
    launches = [(log_int(rng, 1, 36), log_int(rng, 1, 150000), log_int(rng, 1, 6000), 32 * log_int(rng, 1, 350)) for _ in range(20000)]
    got = pick("f32", launches)
    assert got == [T.f32_tile(*q) for q in launches]
    assert set(got) == set(range(6))


def test_short_sums_take_no_large_tile_and_no_step_that_is_mostly_empty(pick):
    # one head's output projection of 64 columns over a full batch (two slabs), and a toy's queries, keys and values
    assert pick("f32", [(1, 102400, 768, 64), (1, 102400, 768, 128), (1, 24576, 1024, 256)]) == [T.F32_64x64] * 3
    assert pick("f32", [(3, 128, 16, 64), (1, 128, 64, 32), (3, 1600, 64, 64), (1, 512, 512, 192)]) == [T.F32_32x32] * 4
    # and where they are long, they do
    assert pick("f32", [(1, 16384, 512, 2048), (1, 15616, 512, 2048), (1, 4096, 2048, 512)]) == [T.F32_128x128] * 3
    assert pick("f32", [(3, 256, 128, 4096), (1, 512, 512, 128)]) == [T.F32_32x32_STEP4] * 2
    assert pick("f32", [(3, 1184, 128, 4096)]) == [T.F32_32x64_STEP4]


def test_the_copy_of_the_exact_rule_agrees(pick):
    rng = random.Random(4)
    launches = []
    for _ in range(30000):
        kl = rng.random() < 0.2
        wide = not kl and rng.random() < 0.7
        launches.append((log_int(rng, 1, 3) if not wide else 1, log_int(rng, 1 if not wide else 256, 150000), log_int(rng, 1 if not wide else 256, 12000),
                         128 * log_int(rng, 2 if wide else 1, 90), int(rng.random() < 0.5), int(kl), int(wide), int(not kl and rng.random() < 0.5)))
    got = pick("exact", launches)
    assert got == [T.exact_tile(*q) for q in launches]
    assert set(got) == set(range(7))


def test_a_residual_behind_short_rows_keeps_the_smaller_tiles(pick):
    #            codes: 30 us in tiles of 64 x 128, 38 in 256 x 256; 97 / 110; 147 / 165.   bfloat16: 46 / 57, 48 / 57, 55 / 60
    slower = [(1, 2144, 6560, 512, 0), (1, 98571, 416, 384, 0), (1, 107172, 576, 640, 0), (1, 2564, 11104, 256, 1), (1, 51637, 448, 640, 1), (1, 12679, 1664, 1024, 1)]
    assert T.TILE_256x256 not in pick("exact", [q + (0, 1, 1) for q in slower])
    # the MLP outputs of a full batch take them, as plain products of these sizes do
    faster = [(1, 102400, 768, 3072, 0), (1, 40818, 5760, 3456, 0), (1, 72143, 4256, 2048, 0), (1, 20531, 6208, 384, 1), (1, 101434, 768, 768, 1)]
    assert set(pick("exact", [q + (0, 1, 1) for q in faster])) == {T.TILE_256x256}
    assert pick("exact", [(1, 107172, 576, 640, 0, 0, 1, 0)]) == [T.TILE_256x256]
