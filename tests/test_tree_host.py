"""The host-side definitions of the hierarchical summation (tests/tree_host_driver.cpp): record layout, coefficient
order, Hilbert index, and the expansion at the nearest place each order is taken, against direct float64
sums."""
import os
import subprocess

import paper_1601_05904_amd.build as build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tree_definitions(tmp_path):
    exe = str(tmp_path / "tree_host")
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I" + build.CSRC,
                        "-I" + os.path.join(build.ROOT, "include"), "-o", exe,
                        os.path.join(HERE, "tree_host_driver.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
