"""The block chains' protocol on the CPU (chain_sync_host.cpp runs csrc/chain_sync.hpp on threads): every
launch ends with the right result whether or not the device has room for all of its
workgroups, alone or with a second chain that takes part of the room, over progress words that
wrap.  Where all have room no launch is sealed."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2502_20762_amd", "csrc")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("chain") / "chain_sync_host")
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, os.path.join(HERE, "chain_sync_host.cpp"), "-o", exe],
                   check=True)
    return exe


# places, tiles of two contexts, polls for the rest (< 0: seal at once)
@pytest.mark.parametrize("places,n,other,limit,sealed", [
    (24, 24, 0, 1 << 26, False),   # room for all: the chain goes on
    (40, 16, 24, 1 << 26, False),
    (24, 1, 0, 1 << 26, False),    # one tile has no neighbours
    (10, 24, 0, 200, True),        # never room for all
    (1, 6, 0, 50, True),
    (24, 16, 16, 300, None),       # two chains that fit alone: each may hold a part of the room
    (24, 24, 0, -1, True),         # sealed at once, some before others have started
])
def test_every_launch_ends_right(host, places, n, other, limit, sealed):
    r = subprocess.run([host, str(places), str(n), str(other), str(limit)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stdout + r.stderr
    if sealed is not None:
        assert (int(r.stdout.split()[1]) > 0) == sealed
