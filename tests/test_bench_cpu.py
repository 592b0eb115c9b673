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
