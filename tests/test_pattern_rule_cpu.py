"""Which products read row patterns, on the CPU (the dispatch rule built as host
code).  Grids whose lines are short against the rows of a wave were measured
slower from patterns than from codes (lines of 28 rows, m = 16, 380,800 rows:
34.7 -> 38.3 us; omega pass of 2.2M rows, binary32 m = 12, lines of 20 rows:
0.71 times as fast) and must stay on codes; those measured faster must keep
patterns.  A grid line gives runs of a third of its rows."""
import os
import subprocess

import pytest

from paper_1711_10622_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def reads_patterns(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rule") / "pattern_rule_driver")
    cmd = [build.hipcc(), "--cuda-host-only", "-O0", "-std=c++17", f"-I{build.CSRC}", f"-I{build.INCLUDE}", "-x", "hip",
           os.path.join(ROOT, "tests", "pattern_rule_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(size, m, n, line, product=1):
        r = subprocess.run([exe, str(size), str(m), str(n), str(line // 3), str(product)], capture_output=True,
                           text=True, check=True)
        return r.stdout == "1\n"
    return ask


@pytest.mark.parametrize("size,m,n,line", [
    (8, 1, 400000, 28), (8, 4, 400000, 40), (8, 5, 110592, 48), (8, 5, 1600000, 56), (8, 7, 49152, 48),
    (8, 9, 389851, 77), (8, 11, 1600000, 80), (8, 13, 294912, 96), (8, 13, 524288, 128), (8, 15, 819200, 128),
    (8, 16, 44460, 13), (8, 16, 380800, 28), (4, 5, 1600000, 40), (4, 7, 1600000, 28), (4, 16, 400000, 13),
    (8, 4, 12582912, 256), (8, 16, 3145728, 256)])
def test_slower_from_patterns(reads_patterns, size, m, n, line):
    assert not reads_patterns(size, m, n, line)


@pytest.mark.parametrize("size,m,n,line", [
    (8, 1, 1600000, 56), (8, 1, 12582912, 256), (8, 2, 938091, 131), (8, 4, 524288, 128), (8, 5, 400000, 80),
    (8, 7, 938091, 131), (8, 9, 524288, 128), (8, 10, 128000, 80), (8, 16, 90000, 300), (8, 16, 400000, 80),
    (4, 1, 400000, 6), (4, 4, 1600000, 13), (4, 8, 400000, 20), (4, 8, 524288, 128), (4, 13, 294912, 96),
    (4, 16, 400000, 56)])
def test_faster_from_patterns(reads_patterns, size, m, n, line):
    assert reads_patterns(size, m, n, line)


@pytest.mark.parametrize("size,m,n,line,pays", [
    (8, 1, 2200000, 13, False), (8, 2, 2200000, 28, True), (8, 4, 2200000, 40, False), (8, 16, 2200000, 20, False),
    (8, 16, 12582912, 256, True), (8, 8, 524288, 128, False), (4, 4, 2200000, 6, True), (4, 8, 2200000, 56, False),
    (4, 12, 2200000, 80, False), (4, 16, 12582912, 256, True)])
def test_omega_pass(reads_patterns, size, m, n, line, pays):
    assert reads_patterns(size, m, n, line, 2) == pays
