"""The order in which workgroups take their work (csrc/launch_order.h), on the
CPU: tests/launch_order_driver.cpp walks whole launches.
"""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_30166_amd", "csrc")


def test_every_workgroup_order(tmp_path):
    exe = str(tmp_path / "launch_order")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I" + CSRC,
                           os.path.join(HERE, "launch_order_driver.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
