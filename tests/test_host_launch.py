"""How a QMC launch's blocks are dealt out (csrc/xcd_map.h), built for the host by g++: every slot of the item list once,
and every part of the list spread over all XCDs, since a launch that chain lengths share lists its long chains first."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_15195_amd", "csrc")
XCDS, STRIPE = 8, 32


def _build(name, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / name)
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, os.path.join(ROOT, "tests", "host_sanitize", name + ".cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-500:]
    return exe


def test_blocks_cover_the_slots_and_spread_every_part_over_the_xcds(tmp_path):
    exe = _build("xcd_map_check", tmp_path)
    sizes = [1, 7, 8, 9, 31, 32, 33, 255, 256, 257, 511, 513, 4000, 4096, 6001, 24000]
    out = subprocess.run([exe], input="\n".join(map(str, sizes)), capture_output=True, text=True, timeout=60).stdout
    for n, line in zip(sizes, out.splitlines()):
        slot = np.array(line.split(), dtype=np.int64)
        assert np.array_equal(np.sort(slot), np.arange(n)), n
        xcd = np.empty(n, dtype=np.int64)
        xcd[slot] = np.arange(n) % XCDS                 # block b runs on XCD b mod 8
        share = np.cumsum(xcd[:, None] == np.arange(XCDS), axis=0)
        # of the first t slots every XCD has t / 8, give or take a stripe
        even = (np.arange(n) + 1)[:, None] / XCDS
        assert np.abs(share - even).max() <= STRIPE, n
