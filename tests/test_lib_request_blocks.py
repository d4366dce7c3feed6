"""The number of block table entries of one request, checked on the CPU.

A bind adds up what its prefix needs of every group's block table; that sum
decides where the tables are read back to and how many blocks the finishing
kernel visits.  ``tests/c_abi/request_blocks_check.hip`` includes the
library's own header and checks the sum in 64 bits and its limit.  Host code
only: it runs without a GPU.
"""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "c_abi", "request_blocks_check.hip")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_block_table_entries_are_summed_in_64_bits(tmp_path):
    exe = str(tmp_path / "request_blocks_check")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-x", "hip",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_2608_17826_amd/csrc",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", SRC, "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:]
