"""How a QMC launch's blocks are dealt out (csrc/xcd_map.h), built for the host by g++: every slot of the item list once;
every part of the list spread over all XCDs, since a launch that chain lengths share lists its long chains first; and one
contiguous part of it per XCD for a launch of equal items."""
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
    cases = [(n, even) for n in sizes for even in (0, 1)]
    out = subprocess.run([exe], input="\n".join(f"{n} {e}" for n, e in cases), capture_output=True, text=True,
                         timeout=60).stdout
    for (n, even), line in zip(cases, out.splitlines()):
        slot = np.array(line.split(), dtype=np.int64)
        assert np.array_equal(np.sort(slot), np.arange(n)), n
        if even:
            assert all(np.array_equal(np.diff(slot[x::XCDS]), np.ones(max(0, len(slot[x::XCDS]) - 1))) for x in range(XCDS))
            continue
        xcd = np.empty(n, dtype=np.int64)
        xcd[slot] = np.arange(n) % XCDS                 # block b runs on XCD b mod 8
        share = np.cumsum(xcd[:, None] == np.arange(XCDS), axis=0)
        # of the first t slots every XCD has t / 8, give or take a stripe
        assert np.abs(share - (np.arange(n) + 1)[:, None] / XCDS).max() <= STRIPE, n
