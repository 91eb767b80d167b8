"""The labelling's union-find walks under every order of their memory accesses: the library's own
header compiled for the host, each thread a fibre that stops before an access, all orders of two
and three threads on small trees walked one by one."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_every_order_of_the_walks_ends_at_the_roots(tmp_path):
    exe = str(tmp_path / "union_orders")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_1708_01608_amd", "csrc"),
                    os.path.join(HERE, "interleave", "union_orders.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "0 cases wrong" in r.stdout
