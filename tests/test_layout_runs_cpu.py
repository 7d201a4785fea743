"""Which wave of the layout's rank kernel ranks which entries, from the functions that its
launch and the kernel use (tests/host/layout_runs_test.cpp, built by hipcc for the host only):
every entry has exactly one wave, in the tile that counted it, also where the rounds of a run
do not divide the tile's.
"""
import os
import subprocess

import pytest

from paper_2609_40093_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASES = [(300000, 160),    # 98 tiles of 3 rounds, 2 runs of 2 rounds
         (294912, 512),    # 9 rounds, 5 runs of 2
         (20481, 130), (131075, 256), (262144, 256), (480000, 300), (72000, 2047), (1048576, 256), (1, 1),
         (65536, 1), (1 << 22, 2048)]


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("runs") / "layout_runs_test")
    cmd = [cc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O2", "-I", build.INCLUDE, "-I", build.CSRC,
           os.path.join(ROOT, "tests", "host", "layout_runs_test.cpp"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return out


@pytest.mark.parametrize("entries,experts", CASES)
def test_every_entry_has_one_wave(binary, entries, experts):
    res = subprocess.run([binary, str(entries), str(experts)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
