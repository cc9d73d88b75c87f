"""The direct-to-LDS loader's addresses for ragged panels of all sizes up to the 4 GiB limit, computed
on the host by the kernels' own functions (loader_addresses.cpp): no GPU, no panel."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the ROCm compiler")
def test_every_request_reads_its_granule_or_lies_out_of_range(tmp_path):
    exe = str(tmp_path / "loader_addresses")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2105_14500_amd", "csrc"), os.path.join(ROOT, "tests", "loader_addresses.cpp"),
                    "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "requests" in r.stdout, r.stdout[-2000:]
