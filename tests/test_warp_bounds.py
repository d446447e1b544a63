"""The displacement nodes a warped brick keeps (csrc/warp_bounds.h), on the CPU:
tests/warp_bounds_driver.cpp looks up the outermost samples.
"""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_30166_amd", "csrc")


def test_nodes_hold_every_lookup(tmp_path):
    exe = str(tmp_path / "warp_bounds")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-D__host__=",
                           "-D__device__=", "-I" + CSRC,
                           os.path.join(HERE, "warp_bounds_driver.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
