"""Registers and LDS of the built kernels, read from the code objects' own notes: they decide how many waves a compute unit
holds, and a change that costs some of them can be a fifth or two of a large launch's time while every result stays the same."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJECTS = os.path.join(ROOT, "paper_2510_23264_amd", "_build")
LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(registers, bytes of LDS) by source file, kernel and template arguments."""
    def read(source):
        path = os.path.join(OBJECTS, source + ".o")
        if not os.path.exists(path) or not os.path.exists(LLVM + "llvm-readelf"):
            pytest.skip("no object files or no tools to read them")
        d = tmp_path_factory.mktemp(source)
        fat, code = str(d / "fat"), str(d / "code")
        subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, path, str(d / "copy.o")], check=True)
        subprocess.run([LLVM + "clang-offload-bundler", "--type=o", "--unbundle", "--input=" + fat, "--output=" + code,
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", code], stdout=subprocess.PIPE, text=True, check=True).stdout
        out = {}
        for block in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+_ZN4pahq\d+(\w+?_k)I([Lib\dE]+)EE?v", block)
            if name:
                arguments = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", name.group(2) + "E"))
                number = lambda key: int(re.search(r"\." + key + r":\s+(\d+)", block).group(1))      # noqa: E731
                out[(name.group(1),) + arguments] = number("vgpr_count"), number("group_segment_fixed_size")
        assert out
        return out
    return read


# waves per SIMD that the kernels had before the values were requested early: tiles of 16 positions, d_head, rotated
@pytest.mark.parametrize("st,dh,rope,waves", [(4, 32, 1, 2), (4, 32, 0, 3), (4, 16, 1, 3), (4, 16, 0, 3), (2, 16, 1, 6), (2, 32, 0, 5), (2, 64, 0, 4),
                                              (1, 32, 1, 8), (1, 64, 1, 5), (3, 32, 0, 4)])
def test_early_values_cost_no_waves(kernels, st, dh, rope, waves):
    kinds = [v for k, v in kernels("attn_kl").items() if k[:4] == ("attention_mfma_k", st, dh, rope)]
    assert kinds
    for registers, _ in kinds:
        assert 512 // (-(-registers // 8) * 8) >= waves, registers


def test_head_projections_of_32_rows_fit_four_times(kernels):
    found = {k: v for k, v in kernels("gemm").items() if k[:2] == ("gemm_f32_heads_k", 1)}
    assert len(found) == 2
    for _, lds in found.values():
        assert 4 * lds <= 160 * 1024, lds
