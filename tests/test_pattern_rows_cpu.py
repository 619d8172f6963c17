"""Which matrices may have row patterns, on the CPU (the rule is built as host
code from the kernels' own header: a matrix next to the int32 limit needs more
memory than a test has).  A wave of the pattern products computes the end of
its tile and rows of the next pass, at most 256 rows plus 256 plus 64 past a
row of the matrix, in 32 bits: no matrix with patterns may let these pass
2^31 - 1, where an index would wrap round and read before the arrays."""
import os
import subprocess

import pytest

from paper_1711_10622_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILE, PASS, WAVE = 256, 256, 64


@pytest.fixture(scope="module")
def may_have_patterns(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rows") / "pattern_rows_driver")
    cmd = [build.hipcc(), "--cuda-host-only", "-O1", "-std=c++17", f"-I{build.CSRC}", f"-I{build.INCLUDE}", "-x", "hip",
           os.path.join(ROOT, "tests", "pattern_rows_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return lambda n: subprocess.run([exe, str(n)], capture_output=True, text=True, check=True).stdout == "1\n"


@pytest.mark.parametrize("below", [0, 1, 63, 64, 127, 255, 256, 319, 320, 511, 575, 576, 1023, 1024, 1025, 4096])
def test_indexes_stay_in_int32(may_have_patterns, below):
    n = 2 ** 31 - 1 - below
    if may_have_patterns(n):
        assert n + TILE + PASS + WAVE < 2 ** 31
    else:
        assert below < 2048  # the range given up is a few tiles


def test_ordinary_sizes(may_have_patterns):
    assert [may_have_patterns(n) for n in (0, 16383, 16384, 2 ** 21, 12582912, 10 ** 9)] == [False, False, True, True,
                                                                                              True, True]
