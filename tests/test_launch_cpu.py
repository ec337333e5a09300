"""Launch geometry at the largest sizes the entry points take (tests/launch_check.cpp, built here with
the host compiler; no GPU), and that no launch casts an uncapped count of points, chains or projections
to a grid."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2606_04895_amd", "csrc")


def test_grids_fit_the_largest_sizes(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "launch_check")
    r = subprocess.run([cxx, "-O1", "-std=c++17", os.path.join(HERE, "launch_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout


def test_point_and_chain_kernels_launch_capped_grids():
    """One wave per point (plain_eval_kernel) and 1024 threads per 64 chains (ess_chain_stats_kernel)
    reach 2^32 work items at sizes that fit in memory: the batch is split on the host, the chain
    blocks are strided over."""
    src = open(os.path.join(CSRC, "kernels_aux.hip")).read()
    body = re.search(r"hipError_t launch_plain_eval\(.*?\n}\n", src, re.S).group(0)
    assert "capped_blocks((n - c + np - 1) / np, 64)" in body and "c += k.st.N" in body
    body = re.search(r"hipError_t launch_ess_chain_stats\(.*?\n}\n", src, re.S).group(0)
    assert "capped_blocks((N + 63) / 64, 64 * kStatWaves)" in body
    body = re.search(r"void ess_chain_stats_kernel\(.*?\n}\n", src, re.S).group(0)
    assert "cb += gridDim.x" in body
