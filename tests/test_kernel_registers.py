"""Registers of the built attention kernels, read from the code object's own notes: a wave's registers decide how many waves a
SIMD holds, and a change that costs one of two or three is a fifth to two fifths of a large launch's time while every result
stays the same."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJECT = os.path.join(ROOT, "paper_2510_23264_amd", "_build", "attn_kl.o")
LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """Registers by (tiles of 16 positions, d_head, rotated, kind of output)."""
    if not os.path.exists(OBJECT) or not os.path.exists(LLVM + "llvm-readelf"):
        pytest.skip("no object files or no tools to read them")
    d = tmp_path_factory.mktemp("regs")
    fat, code = str(d / "fat"), str(d / "code")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, OBJECT, str(d / "copy.o")], check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--type=o", "--unbundle", "--input=" + fat, "--output=" + code,
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([LLVM + "llvm-readelf", "--notes", code], stdout=subprocess.PIPE, text=True, check=True).stdout
    out = {}
    for block in notes.split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+_ZN4pahq16attention_mfma_kILi(\d+)ELi(\d+)ELb(\d)ELi(\d)E", block)
        if name:
            out[tuple(map(int, name.groups()))] = int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1))
    return out


# waves per SIMD that the kernels had before the values were requested early
@pytest.mark.parametrize("st,dh,rope,waves", [(4, 32, 1, 2), (4, 32, 0, 3), (4, 16, 1, 3), (4, 16, 0, 3), (2, 16, 1, 6), (2, 32, 0, 5), (2, 64, 0, 4),
                                              (1, 32, 1, 8), (1, 64, 1, 5), (3, 32, 0, 4)])
def test_early_values_cost_no_waves(registers, st, dh, rope, waves):
    kinds = [v for k, v in registers.items() if k[:3] == (st, dh, rope)]
    assert kinds
    for v in kinds:
        assert 512 // (-(-v // 8) * 8) >= waves, v
