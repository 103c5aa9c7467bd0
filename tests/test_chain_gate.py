"""The order of block chains of different streams, on the CPU (chain_gate_host.cpp runs csrc/chain_gate.hpp
against a fake device): which launches wait for which chains, with large and small ones, a
launch that fails, a context that goes away, and a second thread that comes between one launch's
look around and its enqueue."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2502_20762_amd", "csrc")


def test_order_of_chains(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "chain_gate_host")
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, os.path.join(HERE, "chain_gate_host.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
