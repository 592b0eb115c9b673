"""The committed counter summaries that bench.py quotes belong to kernels of the built library."""
import glob
import os
import re

import pytest

import bench

PROFILES = sorted(glob.glob(os.path.join(bench.ROOT, "profiles", "hbm_traffic_*.txt")))
LIB = os.path.join(bench.ROOT, "paper_2509_24248_amd", "libspecexit.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="libspecexit.so not built")
@pytest.mark.parametrize("path", PROFILES, ids=os.path.basename)
def test_traffic_summaries_name_kernels_that_exist(path):
    key, shape = re.match(r"hbm_traffic_(.*?_(?:gemm|split))_(.*).txt", os.path.basename(path)).groups()
    assert bench.stored_traffic(key, shape) > 0


def test_traffic_of_a_kernel_that_is_gone_is_not_quoted(tmp_path):
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"..\0_ZN2sx1aE\0_ZN2sx1bE.kd\0..")
    for symbols, want in ((["_ZN2sx1aE"], 7), (["_ZN2sx1aE", "_ZN2sx1cE"], None), (["_ZN2sx1bE"], None), ([], None)):
        (tmp_path / "hbm_traffic_head_gemm_x.txt").write_text("HBM traffic of ...\n" + "".join(f"symbol {s}\n" for s in symbols) + "bytes_per_launch 7\n")
        assert bench.stored_traffic("head_gemm", "x", str(tmp_path), str(lib)) == want
    assert bench.stored_traffic("head_gemm", "y", str(tmp_path), str(lib)) is None


@pytest.mark.skipif(not os.path.exists(LIB), reason="libspecexit.so not built")
def test_traffic_of_a_kernel_that_was_rewritten_is_not_quoted(tmp_path):
    with open(LIB, "rb") as fh:
        digests = bench.kernel_digests(fh.read())
    assert len(digests) > 100 and len(set(digests.values())) > 100
    a, b = sorted(s for s in digests if "k_attn_ring" in s)[:2]
    right, other = digests[a], digests[b]
    for lines, want in (([a, right], 7), ([a, other], None), ([a, None], None), ([a, right, b, other], 7), ([a, other, b, right], None)):
        text = "".join(f"symbol {s}\n" + (f"code {d}\n" if d else "") for s, d in zip(lines[::2], lines[1::2]))
        (tmp_path / "hbm_traffic_split_x.txt").write_text(text + "bytes_per_launch 7\n")
        assert bench.stored_traffic("split", "x", str(tmp_path), same_code=True) == want
        assert bench.stored_traffic("split", "x", str(tmp_path)) == 7
