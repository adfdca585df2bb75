"""The traffic figures bench.py takes from profiles/ are of the kernels that are built: summaries list kernels of today's sources
only, every kernel of a launch class is known to belong to it, and a summary that does not fit a run is not used."""
import glob
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench                                         # noqa: E402

KEY = "cfg3 batch=128 mma=1 precision=pahq"


def _kernels():
    """name -> number of template parameters, of every kernel in the sources."""
    out = {}
    for f in glob.glob(os.path.join(ROOT, "paper_2510_23264_amd", "csrc", "*.hip")):
        text = open(f).read()
        for m in re.finditer(r"(template <([^>]*)>\s*)?(?:static )?__global__ (?:__launch_bounds__\((?:[^()]|\([^()]*\))*\) )?void\s+(\w+)\(", text):
            out[m.group(3)] = len(m.group(2).split(",")) if m.group(2) else 0
    return out


def test_summaries_list_the_kernels_that_are_built():
    kernels = _kernels()
    assert {"gemm_p_k", "gemm_s_k", "build_inputs_k", "oproj_x_k", "noalloc_row_k"} <= set(kernels)
    for f in glob.glob(os.path.join(ROOT, "profiles", "*.txt")):
        seen = re.findall(r"^pahq::(\w+)(<[^>]*>)?\s", open(f).read(), re.M)
        assert seen or "by_launch_size" in f
        for name, args in seen:
            assert name in kernels and (args.count(",") + 1 if args else 0) == kernels[name], (f, name + args)


def test_kernels_of_a_class_are_known():
    known = {k.replace("pahq::", "") for ks in bench.KERNELS_OF_CLASS.values() for k in ks}
    kernels = _kernels()
    assert known <= set(kernels)
    assert {k for k in kernels if re.match(r"gemm_|oproj_|attention_|build_inputs|hidden_quant|patch_", k)} <= known


def test_a_summary_of_other_launches_is_not_used():
    line = next(x for x in open(os.path.join(ROOT, "profiles", bench.PROFILE_FILES["all_edges"])) if x.startswith("# classes of one pass"))
    launches, bytes_per_launch = bench.json.loads(line.split(":", 1)[1])["gemm_fp8"]
    per_pass = {"launches": launches, "bytes": launches * bytes_per_launch}
    got = bench.traffic_from_profile("all_edges", "gemm_fp8", KEY, per_pass)
    assert got is not None and got > 0.5 * bytes_per_launch
    for other in (dict(per_pass, launches=launches // 2), dict(per_pass, bytes=1.7 * per_pass["bytes"])):
        assert bench.traffic_from_profile("all_edges", "gemm_fp8", KEY, other) is None
    assert bench.traffic_from_profile("all_edges", "gemm_fp8", "cfg2 batch=8 mma=1 precision=pahq", per_pass) is None
