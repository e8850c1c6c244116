"""Mapping the pages of an export's output arrays beside the sort
(csrc/pp_pages.hpp) leaves their contents alone, so a failed export has not
touched its caller's arrays, and leaves the copies no pages to fault in."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pages_bin(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("pages") / "pages_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread",
                           f"-I{os.path.join(ROOT, 'paper_2512_12094_amd', 'csrc')}",
                           "-o", out, os.path.join(ROOT, "tests", "pages_check.cpp")])
    return out


@pytest.mark.parametrize("nbytes", [1, 4096, (1 << 20) + 5, (2 << 20) + 4095, 33_000_001])
def test_pages_are_mapped_and_unchanged(pages_bin, nbytes):
    res = subprocess.run([pages_bin, str(nbytes)], capture_output=True, text=True, check=True)
    changed, faults = map(int, res.stdout.split())
    assert changed == 0
    if nbytes >= 2 << 20:                      # smaller arrays are left to the copies
        assert faults < nbytes // 4096 // 8
