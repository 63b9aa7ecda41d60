"""The index arithmetic of the point lists that several workgroups write in
order, compiled for the host (ordered_lists.cpp): complete lists come in
order, and no part writes past its list when a predecessor's count is missing
or another launch's."""
import os
import subprocess

from paper_2105_05600_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_ordered_lists(tmp_path):
    exe = str(tmp_path / "ordered_lists")
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I",
                    os.path.join(build.HERE, "csrc"), os.path.join(HERE, "ordered_lists.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
