"""CPU test of the tree's memory management: tests/native/tree_memory.cpp,
compiled with the library's own headers (host code only) and run.
"""
import os
import subprocess

import pytest

from paper_1309_3783_amd import build as hipbuild

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("native") / "tree_memory")
    subprocess.run([hipbuild.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-g",
                    os.path.join(HERE, "native", "tree_memory.cpp"), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    return r.returncode, r.stdout + r.stderr


@pytest.mark.parametrize("check", ["scratch_follows_the_memory", "reduction_table_needs_its_block",
                                   "optional_blocks_refuse_nothing"])
def test_tree_memory(output, check):
    rc, out = output
    assert f"ok {check}\n" in out, (rc, out)
